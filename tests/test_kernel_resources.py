"""What the compiler gave the kernels, read from the code objects' metadata in the built library, and what it is told about inline
assembly (no GPU needed)."""
import glob
import os
import re

import pytest

from helpers import built_package


def scratch_per_kernel(path):
    """Kernel name -> bytes of scratch per lane: in the metadata the two stand next to each other, as MessagePack."""
    entry = rb"\.name(?:[\xa0-\xbf]|\xd9.|\xda..)([\x20-\x7e]+?)\xbb\.private_segment_fixed_size(\xcc.|\xcd..|\xce....|[\x00-\x7f])"
    with open(path, "rb") as f:
        found = re.findall(entry, f.read(), re.S)
    return {name.decode(): int.from_bytes(v[1:] if len(v) > 1 else v, "big") for name, v in found}


@pytest.fixture(scope="module")
def scratch():
    return scratch_per_kernel(built_package().binding.LIB_PATH)


def test_readout_kernels_use_no_scratch(scratch):
    readouts = {name: n for name, n in scratch.items() if any(k in name for k in ("fwd_bf16_kernel", "fwd_f32_kernel", "fwd_f32_halves_kernel"))}
    # bf16: two head dimensions, three tile splits, with and without the fused map; fp32: two kernels, two head dimensions
    assert len(readouts) == 12 + 2 + 2, sorted(scratch)
    assert not any(readouts.values()), {name: n for name, n in readouts.items() if n}


def test_no_walk_kernel_that_nothing_launches(scratch):
    walks = [name for name in scratch if "gdn_walk" in name]
    # four wavefronts at D = 64 and eight at D = 128, each with one run of blocks and with several
    assert len(walks) == 4 and not any("gdn_walk_kernelILi128E" in name for name in walks), walks


def test_assembly_that_writes_m0_says_so_or_hands_it_back():
    csrc = os.path.join(os.path.dirname(built_package().binding.LIB_PATH), "csrc")
    statements = [a for path in sorted(glob.glob(os.path.join(csrc, "*"))) for a in re.findall(r"asm volatile\((.*?)\);", open(path).read(), re.S)]
    writing = [a for a in statements if "s_mov_b32 m0," in a]
    assert len(writing) >= 2
    for a in writing:          # as an output: the compiler does not honour "m0" in a list of clobbers
        assert '"={m0}"' in a or re.search(r'"s_mov_b32 (%\d), m0\\n.*s_mov_b32 m0, \1"', a, re.S), a
