"""GPU parity at the sizes where a kernel's tiles, splits and dispatch rules change over, against the CPU oracle."""
import dataclasses
import json
import re

import numpy as np
import pytest
import torch

import workloads as W
from helpers import TOL_BF16_OUT, TOL_F32, TOL_STATE, rel_err, rel_err_per_head, to_np
from test_gpu_parity import dev, gpu_commit, gpu_fwd, lib  # noqa: F401  (lib is the fixture)

pytestmark = pytest.mark.gpu


# fp32: workgroups of 32 query rows, or of 16 for what is left beyond a multiple of the CUs (all tiles, some, none; a last tile
# with rows for one of its halves or for both), whose four wavefronts take every fourth block of 32 keys (fewer than four
# blocks, a ragged last one, more than one round), groups of 16 tokens over eight wavefronts in the commit, 32- and 64-wide state blocks
# (64-wide from 64 heads at D = 128, 256 at D = 64).
@pytest.mark.parametrize("B,H,Lq,Lkv,D", [
    (1, 2, 1, 1, 64), (1, 2, 31, 31, 128), (2, 1, 33, 33, 64), (1, 3, 64, 127, 128), (1, 1, 129, 129, 128), (1, 2, 40, 161, 64),
    (2, 32, 17, 17, 128), (4, 64, 33, 33, 64), (1, 2, 300, 300, 128),
    (1, 43, 200, 200, 64), (1, 43, 208, 208, 128), (3, 48, 49, 49, 128), (4, 32, 64, 70, 128), (2, 43, 64, 70, 64)])
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


# Keys masked by logits of -inf: a wavefront whose first key blocks are all masked still merges what it has, or nothing.
@pytest.mark.parametrize("dtype,B,H,Lq,Lkv,D,lo,hi", [
    ("f32", 1, 2, 40, 300, 64, 0, 140), ("f32", 1, 2, 40, 200, 128, 32, 64), ("f32", 1, 1, 33, 300, 128, 10, 300),
    ("bf16", 1, 2, 40, 128, 128, 32, 64), ("bf16", 1, 2, 130, 128, 64, 0, 64), ("bf16", 1, 2, 40, 64, 128, 32, 64),
    ("bf16", 17, 16, 40, 100, 64, 0, 40)])
def test_readout_keys_masked_by_infinite_logits(lib, oracle, dtype, B, H, Lq, Lkv, D, lo, hi):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["tiny" if dtype == "f32" else "ragged_small"], name=f"inf_{dtype}_{B}_{H}_{Lq}_{Lkv}_{D}",
                            B=B, H=H, L=Lq, D=D, qkv_scale=1.0)
    q, _, _, _ = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, D), tag) for tag in (1, 2))
    q[..., 0] = 1.0
    k[:, lo:hi, :, 0] = -float("inf")
    seen = [j for j in range(Lkv) if not lo <= j < hi]
    ref = oracle.fwd(to_np(q), to_np(k[:, seen].contiguous()), to_np(v[:, seen].contiguous()))
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, None, None)), ref)
    assert e <= (TOL_F32 if dtype == "f32" else TOL_BF16_OUT), f"{e:.3e}"


# Readout: half tiles of 128 rows with two key groups while they fit one round (more than 128 rows and two or more key
# tiles, a last tile with keys for one or both groups), whole tiles of 256 rows beyond or with fewer rows or keys, and whole
# tiles followed by half tiles when the last round would be at most half full (272 and 544 tiles; a last half tile with and
# without rows).  At D = 64 whole tiles are of four wavefronts with 64 rows each from 257 tiles on (rows for one of a wavefront's
# two blocks, for some of the wavefronts; one key tile).
@pytest.mark.parametrize("B,H,Lq,Lkv,D", [
    (1, 2, 40, 32, 128), (1, 2, 40, 33, 128), (2, 1, 128, 64, 64), (1, 3, 129, 65, 128), (1, 2, 256, 97, 64), (1, 2, 300, 128, 128),
    (1, 2, 130, 161, 128), (2, 2, 385, 385, 64), (1, 2, 200, 200, 128), (8, 17, 150, 150, 64), (17, 16, 40, 40, 64), (17, 16, 200, 200, 64),
    (17, 16, 300, 70, 64), (17, 16, 130, 40, 128), (3, 43, 290, 290, 128), (17, 16, 1, 64, 64), (17, 16, 65, 65, 64), (17, 16, 193, 193, 64),
    (43, 6, 257, 129, 64), (65, 4, 129, 20, 64)])
def test_readout_tile_splits(lib, oracle, B, H, Lq, Lkv, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"split_{B}_{H}_{Lq}_{Lkv}_{D}", B=B, H=H, L=Lq, D=D)
    q, _, _, g = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, D), tag) for tag in (1, 2))
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, None, None)), oracle.fwd(to_np(q), to_np(k), to_np(v)))
    assert e <= TOL_BF16_OUT, f"softmax: {e:.3e}"
    # logits far above the first block's maximum: the running maximum has to be raised later on
    k2 = k.clone()
    k2[:, Lkv // 2:] *= 16
    e = rel_err(to_np(gpu_fwd(lib, q, k2, v, None, None)), oracle.fwd(to_np(q), to_np(k2), to_np(v)))
    assert e <= TOL_BF16_OUT, f"late maximum: {e:.3e}"
    if Lq != Lkv:
        return
    S = W.normal(6, w, (B, H, D, D), 3, io_dtype="f32") * 0.2
    S64 = to_np(S).astype(np.float64)
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, S, g)), oracle.fwd(to_np(q), to_np(k), to_np(v), S64, to_np(g)))
    assert e <= TOL_BF16_OUT, f"readout: {e:.3e}"
    # the fused query map against the two calls it stands for
    Wq, _, _ = W.feature_weights(w)
    cs, sn = W.rope_tables(w)
    ql, out, ref = (torch.empty_like(q, device="cuda") for _ in range(3))
    lib.arl2_feature_map(dev(q), dev(Wq), dev(cs), dev(sn), ql)
    lib.arl2_hybrid_attn_fwd_ex(dev(q), dev(k), dev(v), ql, dev(S), dev(g), ref)
    lib.arl2_hybrid_attn_fwd_fm(dev(q), dev(k), dev(v), dev(q), dev(Wq), dev(cs), dev(sn), dev(S), dev(g), out)
    torch.cuda.synchronize()
    # both round the mapped query to bf16 on fp32 sums in different orders: one ulp of an entry, then of the output
    assert rel_err(to_np(out), to_np(ref)) <= 2.0 ** -7


# Whole tiles: the ring of four key tiles (fewer tiles than stages, one more, a ragged last tile of one key or one short of
# full), with rows of one head (the smallest row distance) and of several, and wavefronts without query rows.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,H,Lq,Lkv", [
    (1, 1, 100, 1), (1, 1, 100, 63), (1, 1, 33, 64), (2, 1, 100, 65), (1, 1, 100, 128), (1, 2, 100, 129), (1, 1, 128, 193), (1, 3, 70, 256),
    (1, 1, 100, 257), (1, 1, 1, 320), (2, 2, 100, 383), (65, 4, 200, 321)])
def test_readout_key_ring(lib, oracle, B, H, Lq, Lkv, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"ring_{B}_{H}_{Lq}_{Lkv}_{D}", B=B, H=H, L=Lq, D=D)
    q, _, _, _ = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, D), tag) for tag in (1, 2))
    e = rel_err(to_np(gpu_fwd(lib, q, k, v, None, None)), oracle.fwd(to_np(q), to_np(k), to_np(v)))
    assert e <= TOL_BF16_OUT, f"{e:.3e}"


# Whole tiles at D = 64 take their LDS at launch, one size per form: also in a captured graph, several replays between other work.
@pytest.mark.parametrize("B,H,L", [(2, 30, 600), (3, 43, 600)])
def test_readout_in_a_graph_with_lds_of_the_launch(lib, B, H, L):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"graph_{B}_{H}_{L}", B=B, H=H, L=L, D=64)
    q, k, v, _ = (dev(x) for x in W.pass_inputs(w, 0, 0))
    out, ref = torch.zeros_like(q), torch.empty_like(q)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        lib.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lib.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    for i in range(3):
        q.mul_(0.5)
        out.zero_()
        lib.arl2_hybrid_attn_fwd(q, k, v, None, None, ref)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), i


# Delta rule: tiles of 64 (D = 128) or 128 (D = 64) tokens shared by two or four token groups, one split per CU as far as
# heads, tiles and the workspace allow (one tile, a ragged tile of one group, several rounds of the load ring, more heads
# than CUs).
@pytest.mark.parametrize("B,H,L,D", [
    (1, 2, 1, 128), (1, 2, 33, 64), (2, 3, 64, 128), (1, 3, 65, 128), (1, 2, 128, 64), (1, 2, 129, 64), (2, 24, 321, 128),
    (3, 86, 300, 64), (13, 20, 260, 128)])
def test_delta_tiles_and_splits(lib, oracle, B, H, L, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"delta_{B}_{H}_{L}_{D}", B=B, H=H, L=L, D=D)
    k, v, gate = W.clean_inputs(w, 0)
    beta = W.uniform(2, w, (B, H), 0.2, 1.0, 0, 0, 97) / (1.0 + (L / D) ** 0.5) ** 2
    S = W.normal(6, w, (B, H, D, D), 3, io_dtype="f32")
    S_dev = dev(S).clone()
    ws = lib.alloc_workspace(B, H, L, D, torch.bfloat16)
    lib.arl2_state_commit_delta(dev(k), dev(v), dev(gate), dev(beta), S_dev, ws)
    torch.cuda.synchronize()
    ref = oracle.commit_delta(to_np(k), to_np(v), to_np(gate), to_np(beta), to_np(S).astype(np.float64))
    e = rel_err_per_head(to_np(S_dev), ref)
    assert e <= TOL_STATE, f"{e:.3e}"


# Token-sequential delta rule where the triangular solve of a 64-token block matters most: keys of a block nearly alike,
# learning rates up to one, gates of zero and one inside 16-token blocks, one token to several blocks and runs.
@pytest.mark.parametrize("B,H,L,D", [(1, 2, 1, 128), (1, 3, 17, 64), (2, 2, 64, 128), (1, 2, 81, 64), (1, 5, 300, 128), (2, 3, 600, 64)])
def test_gdn_blocks_of_similar_keys(lib, oracle, B, H, L, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"gdn_alike_{B}_{H}_{L}_{D}", B=B, H=H, L=L, D=D)
    k, v, _ = W.clean_inputs(w, 0)
    k = (0.1 * k.float() + k[:, :1].float()).to(torch.bfloat16)
    alpha, beta = W.uniform(2, w, (B, L, H), 0.9, 1.0, 0, 0, 98), W.uniform(2, w, (B, L, H), 0.5, 1.0, 0, 0, 99)
    alpha[:, 3::37], alpha[:, 5::41], beta[:, 7::29], beta[:, 9::31] = 0.0, 1.0, 0.0, 1.0
    S = W.normal(6, w, (B, H, D, D), 3, io_dtype="f32")
    S_dev = dev(S).clone()
    ws = torch.empty(lib.arl2_gdn_workspace_bytes(B, H, L, D), dtype=torch.uint8, device="cuda")
    lib.arl2_state_commit_gdn(dev(k), dev(v), dev(alpha), dev(beta), S_dev, ws)
    torch.cuda.synchronize()
    ref = oracle.commit_gdn(to_np(k), to_np(v), to_np(alpha), to_np(beta), to_np(S).astype(np.float64))
    e = rel_err_per_head(to_np(S_dev), ref)
    print(f"gdn similar keys {B}x{H}x{L}x{D}: {e:.2e}")
    assert e <= TOL_STATE, f"{e:.3e}"


# Dense gate projection: 128 x 128 tiles with four stages (fewer hidden steps than stages, ragged tokens and outputs, rows
# of g that do not start aligned), with two stages beyond one tile per CU, 256 x 256 tiles once they need fewer rounds
# (odd step counts, outputs that end inside a tile).
@pytest.mark.parametrize("B,L,H,D,mode,gdt", [
    (1, 1, 1, 64, "element", "f32"), (2, 65, 33, 64, "head", "f32"), (1, 129, 39, 64, "head", "bf16"), (1, 200, 5, 64, "element", "bf16"),
    (3, 127, 3, 128, "element", "f32"), (1, 33000, 1, 64, "element", "f32"), (3, 11001, 35, 64, "head", "bf16"),
    (1, 33000, 2, 128, "element", "bf16"), (2, 16500, 3, 64, "element", "f32")])
def test_gate_dense_tiles(lib, B, L, H, D, mode, gdt):  # noqa: F811
    gen = torch.Generator().manual_seed(B * L + H)
    n = H if mode == "head" else H * D
    x = torch.randn((B, L, H * D), generator=gen).to(torch.bfloat16)
    Wg = (torch.randn((n, H * D), generator=gen) / (H * D) ** 0.5).to(torch.bfloat16)
    shape = (B, L, H) if mode == "head" else (B, L, H, D)
    pad = 64                                              # guard values behind the gate: rows past the end are not stored
    buf = torch.full((B * L * n + pad,), 7.0, dtype=torch.bfloat16 if gdt == "bf16" else torch.float32, device="cuda")
    g = buf[:B * L * n].view(shape)
    lib.arl2_gate_proj(dev(x), dev(Wg), g)
    torch.cuda.synchronize()
    ref = torch.sigmoid(x.reshape(B * L, -1).double() @ Wg.double().T).reshape(shape)
    # sigmoid changes by at most a quarter of the fp32 sum's error; a bf16 gate adds half an ulp below one
    err = (g.cpu().double() - ref).abs().max().item()
    assert err <= (2.0 ** -9 + 2e-6 if gdt == "bf16" else 2e-6), f"{err:.3e}"
    assert bool((buf[B * L * n:] == 7.0).all())


# Where the readout's tile split changes over: two key tiles (65 keys) where halving makes more workgroups; ten (D = 128) or
# eight (D = 64) where it does not, 32 at D = 128 on more than three quarters of the CUs; tails of ragged tiles with few
# and with many rows.  `split` is the form of the kernel: 0 whole tiles, 1 halves, 2 whole ones, then halves.
@pytest.mark.parametrize("B,H,Lq,Lkv,D,split", [
    (1, 2, 130, 64, 128, 0), (1, 2, 130, 65, 128, 1), (2, 3, 200, 64, 64, 0), (2, 3, 200, 65, 64, 1), (2, 12, 64, 64, 128, 0),
    (1, 2, 100, 639, 128, 0), (1, 2, 100, 640, 128, 1), (1, 3, 33, 511, 64, 0), (1, 3, 33, 512, 64, 1), (2, 12, 128, 128, 64, 0),
    (14, 14, 20, 2047, 128, 0), (14, 14, 20, 2048, 128, 1), (17, 16, 128, 128, 128, 0), (17, 16, 20, 512, 64, 2), (17, 16, 300, 70, 64, 0),
    (17, 16, 400, 70, 64, 2)])
def test_readout_takes_the_faster_tile_split(lib, oracle, B, H, Lq, Lkv, D, split):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"line_{B}_{H}_{Lq}_{Lkv}_{D}", B=B, H=H, L=Lq, D=D)
    q, _, _, _ = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, D), tag) for tag in (1, 2))
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        out = gpu_fwd(lib, q, k, v, None, None)
    kernels = [e.key for e in prof.key_averages() if "fwd_bf16_kernel" in e.key]
    assert len(kernels) == 1 and re.search(rf"<{D}, [^,]*\){split}, false>", kernels[0]), kernels
    e = rel_err(to_np(out), oracle.fwd(to_np(q), to_np(k), to_np(v)))
    assert e <= TOL_BF16_OUT, f"{e:.3e}"


# D = 64, where a whole tile's four wavefronts have 64 rows each and a small one's 32: eight wavefronts up to 256 tiles of 256
# rows; beyond, small tiles for up to 128 rows (from 65 rows on, with fewer than eight key tiles, or with more than 448 tiles)
# and for one key tile (up to 1024 tiles); halves behind whole tiles where the last ones have up to 128 rows (up to 512 tiles).
@pytest.mark.parametrize("B,H,Lq,Lkv,split,threads,workgroups", [
    (16, 16, 200, 70, 0, 512, 256), (1, 257, 200, 70, 2, 256, 258), (16, 25, 200, 70, 0, 256, 400),
    (1, 257, 128, 128, 2, 256, 257), (16, 25, 128, 640, 2, 256, 400), (16, 25, 1, 1, 2, 256, 400), (16, 25, 64, 511, 2, 256, 400),
    (16, 25, 64, 512, 0, 256, 400), (16, 25, 65, 512, 2, 256, 400), (32, 14, 20, 512, 0, 256, 448), (1, 449, 20, 512, 2, 256, 449),
    (16, 25, 129, 64, 2, 256, 800), (16, 25, 129, 65, 0, 256, 400), (1, 256, 1000, 33, 2, 256, 2048), (41, 5, 1100, 64, 0, 256, 1025),
    (17, 8, 257, 257, 2, 256, 288), (24, 8, 384, 200, 2, 256, 512), (25, 8, 384, 200, 0, 256, 400)])
def test_readout_small_tiles(lib, oracle, tmp_path, B, H, Lq, Lkv, split, threads, workgroups):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"small_{B}_{H}_{Lq}_{Lkv}", B=B, H=H, L=Lq, D=64)
    q, _, _, _ = W.pass_inputs(w, 0, 0)
    k, v = (W.normal(5, w, (B, Lkv, H, 64), tag) for tag in (1, 2))
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        out = gpu_fwd(lib, q, k, v, None, None)
    prof.export_chrome_trace(str(tmp_path / "trace.json"))
    kernels = [e for e in json.loads((tmp_path / "trace.json").read_text())["traceEvents"] if "fwd_bf16_kernel" in e.get("name", "") and "grid" in e.get("args", {})]
    assert len(kernels) == 1 and re.search(rf"<64, [^,]*\){split}, false>", kernels[0]["name"]), kernels
    assert kernels[0]["args"]["block"][0] == threads and kernels[0]["args"]["grid"][0] == workgroups, kernels
    e = rel_err(to_np(out), oracle.fwd(to_np(q), to_np(k), to_np(v)))
    assert e <= TOL_BF16_OUT, f"{e:.3e}"


# fp32 readout: root mean square error over that of the result.  With `D` products in one chain a rounding random walk gives
# the linear branch about 2^-24 / sqrt(3) * 0.72 * sqrt(D / 2) (the first two bounds lie below that: 2.0e-7 and 1.4e-7); with
# logits of +-20 the products of queries and keys decide, where a kernel with 16 partial sums per row has 7.8e-7.
@pytest.mark.parametrize("D,scale,state,bound", [(128, 0.125, 4.0, 1.8e-7), (64, 0.125, 4.0, 1.35e-7), (128, 2.0, 0.1, 7.8e-7), (64, 2.0, 0.1, 7.8e-7)])
def test_fp32_readout_error(lib, oracle, D, scale, state, bound):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["tiny"], name=f"f32_err_{D}_{scale}", B=1, H=4, L=500, D=D, qkv_scale=scale)
    q, k, v, g = W.pass_inputs(w, 0, 0)
    S = W.normal(6, dataclasses.replace(w, qkv_scale=state), (1, 4, D, D), 3, io_dtype="f32")
    ref = oracle.fwd(to_np(q), to_np(k), to_np(v), to_np(S).astype(np.float64), to_np(g))
    e = np.linalg.norm(to_np(gpu_fwd(lib, q, k, v, S, g)) - ref) / np.linalg.norm(ref)
    print(f"fp32 readout D={D} scale {scale}: {e:.3e}")
    assert e <= bound, f"{e:.3e}"


# Gates of every granularity and type, the linear branch's own query and the fused map, in each form of the readout: halves
# (two key groups that finish a share of the features each), whole tiles, whole ones and then halves, small tiles of D = 64; both
# head dimensions.
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,H,L", [(1, 2, 130), (8, 17, 150), (17, 16, 200), (16, 17, 100)])
def test_readout_gates_in_every_tile_split(lib, oracle, B, H, L, D):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"gates_{B}_{H}_{L}_{D}", B=B, H=H, L=L, D=D)
    q, k, v, _ = W.pass_inputs(w, 0, 0)
    q_lin = W.normal(7, w, (B, L, H, D), 1)
    S = W.normal(6, w, (B, H, D, D), 3, io_dtype="f32") * 0.2
    S64 = to_np(S).astype(np.float64)
    for shape, dtype in (((B, L), torch.bfloat16), ((B, L, H), torch.bfloat16), ((B, L, H, D), torch.float32), ((B, L, H, D), torch.bfloat16)):
        g = W.uniform(8, w, shape, 0.0, 1.0, len(shape)).to(dtype)
        e = rel_err(to_np(gpu_fwd(lib, q, k, v, S, g)), oracle.fwd(to_np(q), to_np(k), to_np(v), S64, to_np(g)))
        assert e <= TOL_BF16_OUT, f"gate {shape} {dtype}: {e:.3e}"
    g = W.uniform(8, w, (B, L, H), 0.0, 1.0, 9)
    out = torch.empty_like(q, device="cuda")
    lib.arl2_hybrid_attn_fwd_ex(dev(q), dev(k), dev(v), dev(q_lin), dev(S), dev(g), out)
    torch.cuda.synchronize()
    e = rel_err(to_np(out), oracle.fwd(to_np(q), to_np(k), to_np(v), S64, to_np(g), q_lin=to_np(q_lin)))
    assert e <= TOL_BF16_OUT, f"own query: {e:.3e}"
    Wq, _, _ = W.feature_weights(w)
    cs, sn = W.rope_tables(w)
    lib.arl2_hybrid_attn_fwd_fm(dev(q), dev(k), dev(v), dev(q_lin), dev(Wq), dev(cs), dev(sn), dev(S), dev(g), out)
    torch.cuda.synchronize()
    mapped = torch.from_numpy(oracle.feature_map(to_np(q_lin), to_np(Wq), to_np(cs), to_np(sn))).to(torch.bfloat16)   # as the kernel rounds it
    e = rel_err(to_np(out), oracle.fwd(to_np(q), to_np(k), to_np(v), S64, to_np(g), q_lin=to_np(mapped)))
    assert e <= TOL_BF16_OUT, f"fused map: {e:.3e}"


# State commits: the values (plain rule) enter as a truncated bf16 part and the rounded rest, which leaves at most 2^-16 of each
# product, the corrections (delta rule) as two rounded parts, which leaves 2^-18.  The state that the delta rule multiplies enters as three: with two its error is the same for every token and
# adds up, to what the oracle shows for a state rounded to two parts.
@pytest.mark.parametrize("D,L", [(128, 3000), (64, 1500)])
def test_commits_keep_their_split_precision(lib, oracle, D, L):  # noqa: F811
    w = dataclasses.replace(W.WORKLOADS["ragged_small"], name=f"split_precision_{D}_{L}", B=1, H=3, L=L, D=D)
    k, v, gate = W.clean_inputs(w, 0)
    S = W.normal(6, w, (1, 3, D, D), 3, io_dtype="f32")
    S64 = to_np(S).astype(np.float64)
    S_dev = dev(S).clone()
    gpu_commit(lib, k, v, gate, S_dev)
    ref = oracle.commit(to_np(k), to_np(v), to_np(gate), S64)
    e = np.linalg.norm(to_np(S_dev) - ref) / np.linalg.norm(ref)
    assert e <= 2.0 ** -16, f"plain: {e:.3e}"

    beta = torch.full((1, 3), 0.5 * D / L)
    v = 0.1 * v                                           # the products of the keys with the state decide
    S_dev = dev(S).clone()
    lib.arl2_state_commit_delta(dev(k), dev(v), dev(gate), dev(beta), S_dev, lib.alloc_workspace(1, 3, L, D, torch.bfloat16))
    torch.cuda.synchronize()
    ref = oracle.commit_delta(to_np(k), to_np(v), to_np(gate), to_np(beta), S64)
    hi = S.to(torch.bfloat16).float()
    two = (hi + (S - hi).to(torch.bfloat16).float()).double().numpy()
    two = oracle.commit_delta(to_np(k), to_np(v), 0.0 * to_np(gate), to_np(beta), two) + to_np(gate)[..., None, None] * S64
    e, e_two = (np.linalg.norm(x - ref) / np.linalg.norm(ref) for x in (to_np(S_dev), two))
    print(f"delta rule D={D} L={L}: {e:.3e}, with a state of two parts at least {e_two:.3e}")
    assert e <= min(2.0 ** -18, 0.7 * e_two), f"{e:.3e}, two parts {e_two:.3e}"
