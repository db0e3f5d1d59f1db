"""What the compiler gave the kernels, read from the code objects' metadata in the built library (no GPU needed)."""
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
    readouts = {name: n for name, n in scratch.items() if "fwd_bf16_kernel" in name or "fwd_f32_kernel" in name}
    # bf16: two head dimensions, three tile splits, with and without the fused map; fp32: two head dimensions
    assert len(readouts) == 12 + 2, sorted(scratch)
    assert not any(readouts.values()), {name: n for name, n in readouts.items() if n}
