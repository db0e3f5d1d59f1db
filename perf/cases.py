"""The work that a user of this package has it do, as measurable cases.

A case is one pass of a user's loop over the package's entry points: the chunk step of a hybrid layer (read-only
denoising passes, then the commit), the same step with the learned maps and the gate projection on the path, the
clean pass alone under one of the delta rules, the pass of a layer that keeps softmax over its key/value cache,
and the element-wise gate.  Sizes are those of workloads/ and bench.py (12 heads x 128, a latent frame of
30 x 52 = 1560 tokens, a chunk of three frames) and generic ones around them.

    listed()          the cases that are always measured
    draw(rng)         one more case from the ranges that the listed ones stand for
    prepare(case, s)  what the user's program holds before the call, on the GPU, from the seed alone
    run(state)        one pass
    work(case)        bytes and operations that the pass cannot do without
    tolerance(case)   how far another correct implementation at the same precision may be
"""
import math

import torch

import paper_2605_16579_amd as A

KINDS = ("step", "mapped_step", "clean", "cache", "element_gate")


def listed():
    return [
        # The smallest step there is: the fp32 configuration that is checked in full on a CPU.  Launches and latency.
        dict(name="tiny_f32", kind="step", B=1, H=2, D=64, L=64, dtype="f32", passes=2, gate="head", gate_dtype="f32"),
        # fp32 throughout at one latent frame: a layer compared with, or run without, reduced precision.
        dict(name="frame_f32", kind="step", B=1, H=12, D=128, L=1560, dtype="f32", passes=4, gate="head", gate_dtype="f32"),
        # A reduced layer with a ragged token count, two streams: tests, small models, previews at low resolution.
        dict(name="small_ragged", kind="step", B=2, H=3, D=128, L=328, dtype="bf16", passes=2, gate="head", gate_dtype="bf16"),
        # Chunks of one latent frame (frame-by-frame generation): four denoising passes and the commit.
        dict(name="frame", kind="step", B=1, H=12, D=128, L=1560, dtype="bf16", passes=4, gate="head", gate_dtype="f32"),
        # The usual step: one layer, chunks of three latent frames.
        dict(name="chunk", kind="step", B=1, H=12, D=128, L=4680, dtype="bf16", passes=4, gate="head", gate_dtype="f32"),
        # The same for eight streams at once: serving several videos.
        dict(name="chunk_streams", kind="step", B=8, H=12, D=128, L=4680, dtype="bf16", passes=4, gate="head", gate_dtype="f32"),
        # 64-wide heads, an odd token count, the scalar gate of the gate ablation stored in bf16.
        dict(name="narrow_heads", kind="step", B=3, H=24, D=64, L=999, dtype="bf16", passes=2, gate="token", gate_dtype="bf16"),
        # The step as a trained layer runs it: gate projected from the hidden state, query, key and value maps fused in.
        dict(name="chunk_mapped", kind="mapped_step", B=1, H=12, D=128, L=4680, passes=4),
        # Clean pass of the token-sequential gated delta rule on keys and values that pass through the learned maps.
        dict(name="clean_gdn", kind="clean", rule="gdn", maps=True, B=1, H=12, D=128, L=4680),
        # Clean pass of the frame-level delta rule for a few streams.
        dict(name="clean_delta", kind="clean", rule="delta", maps=False, B=4, H=12, D=128, L=1560),
        # A layer that keeps softmax: one chunk of queries over the cache of a whole 21-frame video.
        dict(name="cache", kind="cache", B=1, H=12, D=128, L=4680, Lkv=32760),
        # The element-wise gate of the gate ablation: its dense projection, and the pass that reads it.
        dict(name="element_gate", kind="element_gate", B=1, H=12, D=128, L=4680, gate_dtype="f32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Token counts are spread over their logarithm; a drawn case asks for less work than the largest listed one."""
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(("step", "step", "step", "mapped_step", "clean", "clean", "cache", "element_gate"))
        c = dict(kind=kind, B=rng.choice((1, 1, 2, 3, 4, 8)), H=rng.choice((2, 3, 5, 8, 12, 16, 24)), D=rng.choice((64, 128, 128)))
        if kind == "step":
            c["dtype"] = rng.choice(("bf16", "bf16", "bf16", "f32"))
            c["L"] = _log_int(rng, 64, 6240 if c["dtype"] == "bf16" else 1560)
            c["passes"] = rng.choice((2, 4))
            c["gate"] = rng.choice(("head", "head", "token"))
            c["gate_dtype"] = "f32" if c["dtype"] == "f32" else rng.choice(("f32", "bf16"))
        elif kind == "mapped_step":
            c["L"], c["passes"] = _log_int(rng, 200, 6240), rng.choice((2, 4))
        elif kind == "clean":
            c["L"], c["rule"], c["maps"] = _log_int(rng, 100, 6240), rng.choice(("plain", "delta", "gdn")), rng.random() < 0.5
        elif kind == "cache":
            c["L"] = _log_int(rng, 200, 4680)
            c["Lkv"] = c["L"] * rng.randint(1, 7)
        else:
            c["L"], c["gate_dtype"] = _log_int(rng, 200, 4680), rng.choice(("f32", "bf16"))
        if _cost(c) <= most and _elements(c) <= 2 ** 29:
            return c


def _cost(case):
    """Work in bf16 matrix operations: an fp32 one counts 16 times, a byte about 300."""
    w = work(case)
    return w["flops"] * (16 if case.get("dtype") == "f32" else 1) + 300 * w["bytes"]


def _elements(case):
    return case["B"] * max(case["L"], case.get("Lkv", 0)) * case["H"] * case["D"] * case.get("passes", 1)


def _shape(case):
    return case["B"], case["H"], case["D"], case["L"]


def _io(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


class _Draws:
    """Random tensors on the GPU from one seed."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(int(seed))

    def normal(self, shape, std=1.0, dtype=torch.float32):
        return (torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32) * std).to(dtype)

    def uniform(self, shape, lo, hi, dtype=torch.float32):
        return (torch.rand(shape, generator=self.g, device="cuda", dtype=torch.float32) * (hi - lo) + lo).to(dtype)

    def feature_weights(self, H, D):
        """A learned per-head map adapted from the pretrained representation: identity plus noise."""
        eye = torch.eye(D, device="cuda")[None]
        return (eye + self.normal((H, D, D), 0.5 / math.sqrt(D))).to(torch.bfloat16)


def _rope(L, D):
    """Rotary tables [L][D/2] over (latent frame, row, column) of a 30 x 52 grid of tokens."""
    l = torch.arange(L, device="cuda")
    pos = torch.stack([l // 1560, (l // 52) % 30, l % 52], dim=1).double()
    half = D // 2
    n = half // 3
    ang = torch.cat([pos[:, a:a + 1] * (10000.0 ** (-torch.arange(m, device="cuda").double() / m))[None]
                     for a, m in enumerate((half - 2 * n, n, n))], dim=1)
    return ang.cos().float().contiguous(), ang.sin().float().contiguous()


def _gate_shape(case):
    B, H, D, L = _shape(case)
    return {"head": (B, L, H), "token": (B, L), "element": (B, L, H, D)}[case["gate"]]


def prepare(case, seed):
    B, H, D, L = _shape(case)
    kind, io, d = case["kind"], _io(case), _Draws(seed)
    rows = (B, L, H, D)
    s = dict(case=case)
    if kind == "cache":
        kv = (B, case["Lkv"], H, D)
        s.update(q=d.normal(rows, 1.0, io), k=d.normal(kv, 1.0, io), v=d.normal(kv, 1.0, io))
        s["out"] = torch.empty_like(s["q"])
        return s

    # Normalised keys of L random tokens per chunk, several chunks old: the state's scale under each rule.
    std = {"plain": 2.5 * math.sqrt(L / D), "delta": 0.3, "gdn": 1.0}[case.get("rule", "plain")]
    s["S"] = d.normal((B, H, D, D), std)
    if kind in ("step", "mapped_step"):
        # q, k, v of every denoising pass, then k, v of the clean pass; rows scaled by 1/8 in the fp32 configuration
        std = 0.125 if io == torch.float32 else 1.0
        s["passes"] = [[d.normal(rows, std, io) for _ in range(3)] for _ in range(case["passes"])]
        s["clean"] = [d.normal(rows, std, io) for _ in range(2)]
        s["out"] = [torch.empty(rows, dtype=io, device="cuda") for _ in range(case["passes"])]
        s["forget"] = d.uniform((B, H), 0.9, 0.999)
        s["ws"] = A.alloc_workspace(B, H, L, D, io)
    if kind == "step":
        gdt = torch.bfloat16 if case["gate_dtype"] == "bf16" else torch.float32
        s["g"] = [d.uniform(_gate_shape(case), 0.45, 0.55, gdt) for _ in range(case["passes"])]
    elif kind == "mapped_step":
        s["x"] = [d.normal((B, L, H * D), 1.0, io) for _ in range(case["passes"])]
        s["xq"] = [d.normal(rows, 1.0, io) for _ in range(case["passes"])]
        s["g"] = [torch.empty((B, L, H), device="cuda") for _ in range(case["passes"])]
        s["Wg"] = d.normal((H, H * D), 0.1 / math.sqrt(H * D), io)
        s["Wq"], s["Wk"], s["Wv"] = (d.feature_weights(H, D) for _ in range(3))
        s["rope"] = _rope(L, D)
    elif kind == "clean":
        s["k"], s["v"] = d.normal(rows, 1.0, io), d.normal(rows, 1.0, io)
        if case["maps"]:
            s["Wk"], s["Wv"], s["rope"] = d.feature_weights(H, D), d.feature_weights(H, D), _rope(L, D)
            s["yk"], s["yv"] = torch.empty_like(s["k"]), torch.empty_like(s["v"])
        if case["rule"] == "gdn":
            s["alpha"] = d.uniform((B, 1, H), 0.9, 0.999) ** (d.uniform((B, L, H), 0.0, 2.0) / L)
            s["beta"] = d.uniform((B, L, H), 0.05, 0.95)
            s["ws"] = torch.empty(max(16, A.arl2_gdn_workspace_bytes(B, H, L, D)), dtype=torch.uint8, device="cuda")
        else:
            s["forget"] = d.uniform((B, H), 0.9, 0.999)
            # learning rates below the contraction bound of a frame-level update, 2 / (largest eigenvalue of K'^T K')
            s["beta"] = d.uniform((B, H), 0.2, 1.0) / (1.0 + math.sqrt(L / D)) ** 2
            s["ws"] = A.alloc_workspace(B, H, L, D, io)
    else:
        s["x"] = d.normal((B, L, H * D), 1.0, io)
        s["Wg"] = d.normal((H * D, H * D), 0.1 / math.sqrt(H * D), io)
        s["g"] = torch.empty(rows, dtype=torch.bfloat16 if case["gate_dtype"] == "bf16" else torch.float32, device="cuda")
        s["q"], s["k"], s["v"] = (d.normal(rows, 1.0, io) for _ in range(3))
        s["out"] = torch.empty_like(s["q"])
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "step":
        for (q, k, v), g, out in zip(s["passes"], s["g"], s["out"]):
            A.arl2_hybrid_attn_fwd(q, k, v, s["S"], g, out)
        A.arl2_state_commit(*s["clean"], s["forget"], s["S"], s["ws"])
        return s["out"] + [s["S"]]
    if kind == "mapped_step":
        for (q, k, v), x, xq, g, out in zip(s["passes"], s["x"], s["xq"], s["g"], s["out"]):
            A.arl2_gate_proj(x, s["Wg"], g)
            A.arl2_hybrid_attn_fwd_fm(q, k, v, xq, s["Wq"], *s["rope"], s["S"], g, out)
        xk, xv = s["clean"]
        A.arl2_state_commit_fm(xk, s["Wk"], *s["rope"], xv, s["Wv"], s["forget"], s["S"], s["ws"])
        return s["g"] + s["out"] + [s["S"]]
    if kind == "clean":
        k, v, rule, mapped = s["k"], s["v"], s["case"]["rule"], []
        if s["case"]["maps"]:
            A.arl2_feature_map(k, s["Wk"], *s["rope"], s["yk"])
            A.arl2_feature_map(v, s["Wv"], None, None, s["yv"])
            k, v = mapped = [s["yk"], s["yv"]]
        if rule == "gdn":
            A.arl2_state_commit_gdn(k, v, s["alpha"], s["beta"], s["S"], s["ws"])
        elif rule == "delta":
            A.arl2_state_commit_delta(k, v, s["forget"], s["beta"], s["S"], s["ws"])
        else:
            A.arl2_state_commit(k, v, s["forget"], s["S"], s["ws"])
        return mapped + [s["S"]]
    if kind == "cache":
        A.arl2_hybrid_attn_fwd(s["q"], s["k"], s["v"], None, None, s["out"])
        return s["out"]
    A.arl2_gate_proj(s["x"], s["Wg"], s["g"])
    A.arl2_hybrid_attn_fwd(s["q"], s["k"], s["v"], s["S"], s["g"], s["out"])
    return [s["g"], s["out"]]


def work(case):
    B, H, D, L = _shape(case)
    kind = case["kind"]
    io = 4 if case.get("dtype") == "f32" else 2
    rows, state, head_maps = B * L * H * D, B * H * D * D * 4, H * D * D * 2
    tables = 2 * L * (D // 2) * 4
    flops_inter = 2 * rows * D                      # readout of the state, the commit's contraction, one feature map
    flops_pass = 4 * rows * case.get("Lkv", L) + (flops_inter if kind != "cache" else 0)
    if kind == "cache":
        return {"bytes": 2 * rows * io + 2 * B * case["Lkv"] * H * D * io, "flops": flops_pass}
    if kind == "step":
        g = math.prod(_gate_shape(case)) * (2 if case["gate_dtype"] == "bf16" else 4)
        return {"bytes": case["passes"] * (4 * rows * io + state + g) + 2 * rows * io + 2 * state + 4 * B * H,
                "flops": case["passes"] * flops_pass + flops_inter}
    if kind == "mapped_step":
        # per pass: x, q, k, v, xq in, g and out written; then the clean projections, the state in and out
        one = 6 * rows * 2 + B * L * H * 4 + state + H * H * D * 2 + head_maps + tables
        return {"bytes": case["passes"] * one + 2 * rows * 2 + 2 * head_maps + tables + 2 * state + 4 * B * H,
                "flops": case["passes"] * (flops_pass + flops_inter + 2 * rows * H) + 3 * flops_inter}
    if kind == "clean":
        maps = (2 * rows * 2 + 2 * head_maps + tables) if case["maps"] else 0
        gates = 2 * B * L * H * 4 if case["rule"] == "gdn" else 2 * B * H * 4
        # the contraction, and for the delta rules the products of the keys with the state (or among themselves)
        return {"bytes": 2 * rows * 2 + 2 * state + gates + maps,
                "flops": flops_inter * ((2 if case["maps"] else 0) + (1 if case["rule"] == "plain" else 2))}
    dm, gb = H * D, 2 if case["gate_dtype"] == "bf16" else 4
    return {"bytes": 5 * rows * 2 + dm * dm * 2 + 2 * rows * gb + state, "flops": flops_pass + 2 * rows * dm}


def tolerance(case):
    # About four times the distance measured against 64-bit arithmetic on the same stored inputs.
    if case.get("dtype") == "f32":                  # outputs 2e-7 (largest 1.7e-6), state 5e-8
        return {"rel": 1e-6, "max": 1e-5}
    if case["kind"] == "clean" and not case["maps"]:
        if case["rule"] == "gdn":                   # 7e-6 (4e-5): L dependent updates on operands split into bf16 pairs
            return {"rel": 3e-5, "max": 2e-4}
        return {"rel": 8e-6, "max": 4e-5}           # 2e-6 (8e-6)
    if case["kind"] == "cache":                     # 2.4e-3 (1e-2): bf16 weights and outputs, no state to dominate them
        return {"rel": 1e-2, "max": 4e-2}
    return {"rel": 7e-3, "max": 3e-2}               # bf16 outputs: 1.7e-3 (7e-3 where a mapped row is rounded in between)
