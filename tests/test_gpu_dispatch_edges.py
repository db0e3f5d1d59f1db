"""GPU parity at the sizes where a kernel's tiles, splits and dispatch rules change over, against the CPU oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from helpers import TOL_F32, rel_err, rel_err_per_head, to_np
from test_gpu_parity import dev, gpu_commit, gpu_fwd, lib  # noqa: F401  (lib is the fixture)

pytestmark = pytest.mark.gpu


# fp32: 32-row workgroups whose four wavefronts take every fourth block of 32 keys (fewer than four blocks, a ragged
# last one, more than one round), groups of 16 tokens over eight wavefronts in the commit, 32- and 64-wide state blocks
# (64-wide from 64 heads at D = 128, 256 at D = 64).
@pytest.mark.parametrize("B,H,Lq,Lkv,D", [
    (1, 2, 1, 1, 64), (1, 2, 31, 31, 128), (2, 1, 33, 33, 64), (1, 3, 64, 127, 128), (1, 1, 129, 129, 128), (1, 2, 40, 161, 64),
    (2, 32, 17, 17, 128), (4, 64, 33, 33, 64), (1, 2, 300, 300, 128)])
def test_fp32_tiles_and_key_groups(lib, oracle, B, H, Lq, Lkv, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["tiny"], name=f"f32_{B}_{H}_{Lq}_{Lkv}_{D}", B=B, H=H, L=Lq, D=D, qkv_scale=1.0)
    q, _, _, g = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, D), tag) for tag in (1, 2))
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, None, None)), oracle.fwd(to_np(q), to_np(k), to_np(v)))
    assert e <= TOL_F32, f"softmax: {e:.3e}"
    if Lq != Lkv:
        return
    S = W.normal(6, w, (B, H, D, D), 3, io_dtype="f32")
    S64 = to_np(S).astype(np.float64)
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, S, g)), oracle.fwd(to_np(q), to_np(k), to_np(v), S64, to_np(g)))
    assert e <= TOL_F32, f"readout: {e:.3e}"
    _, _, gate = W.clean_inputs(w, 0)
    S_dev = dev(S).clone()
    gpu_commit(lib, k, v, gate, S_dev)
    e = rel_err_per_head(to_np(S_dev), oracle.commit(to_np(k), to_np(v), to_np(gate), S64))
    assert e <= TOL_F32, f"commit: {e:.3e}"
