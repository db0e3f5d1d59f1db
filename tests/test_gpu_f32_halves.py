"""The fp32 readout on sums of two halves: the sizes where its tiles, blocks and dispatch can go wrong, and the values that two halves do not
stand for, against float64 on the GPU."""
import pytest
import torch

import paper_2605_16579_amd as A

pytestmark = pytest.mark.gpu

# Relative 2-norm error: rounding the operands to 23 bits and the fp32 sums give 1e-7 to 2.5e-7 for logits of a few units.
TOL = 6e-7


def draw(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda")


def exact(q, k, v, S=None, g=None, q_lin=None):
    """[B, L, H, D] tensors; g broadcasts against the output."""
    q, k, v = (x.double().transpose(1, 2) for x in (q, k, v))
    o = torch.softmax((q @ k.transpose(-1, -2).contiguous()) * q.shape[-1] ** -0.5, -1) @ v
    if S is not None:
        x = q if q_lin is None else q_lin.double().transpose(1, 2)
        inter = (x / torch.sqrt((x * x).sum(-1, keepdim=True) + 1e-6)) @ S.double()
        o = o + (inter if g is None else inter * g.double().transpose(1, 2))
    return o.transpose(1, 2)


def error(got, ref):
    assert torch.isfinite(got).all()
    return float((got.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("B,H,Lq,Lkv,D", [
    (1, 130, 33, 1, 128), (1, 70, 64, 31, 64), (1, 140, 40, 33, 64), (1, 66, 100, 129, 128),     # one block, key groups without one
    (1, 50, 70, 520, 128), (2, 3, 40, 700, 128), (2, 3, 40, 740, 128), (1, 2, 40, 2050, 64), (1, 2, 40, 4100, 64), (1, 60, 257, 384, 64),    # last rows and keys of a tile
    (3, 8, 1000, 128, 128), (1, 12, 1560, 97, 128), (2, 136, 64, 64, 64)])                         # whole tiles, halved last ones
def test_softmax(B, H, Lq, Lkv, D):
    q, k, v = draw(1, B, Lq, H, D), draw(2, B, Lkv, H, D), draw(3, B, Lkv, H, D)
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    e = error(out, exact(q, k, v))
    assert e <= TOL, f"{e:.2e}"


@pytest.mark.parametrize("D", [64, 128])
def test_one_key_is_copied(D):
    q, k, v = draw(1, 1, 256, 40, D), draw(2, 1, 1, 40, D), draw(3, 1, 1, 40, D)
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    assert torch.equal(out, v.expand_as(out))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Lkv", [33, 64, 128, 700])
@pytest.mark.parametrize("kind", ["usual", "large logits", "very large logits", "one direction", "larger keys later"])
def test_no_less_exact_than_fp32_products(kind, Lkv, D):
    """Against the kernel on fp32 products, which serves launches of up to 32 rows."""
    B, H, Lq = 1, 40, 256
    q, k, v = draw(1, B, Lq, H, D), draw(2, B, Lkv, H, D), draw(3, B, Lkv, H, D)
    if kind == "large logits":
        q *= 4
    elif kind == "very large logits":
        q *= 24
    elif kind == "one direction":                                                # logits of 23 and 45
        q, k = 0.3 * q + 2, 0.3 * k + 2
    elif kind == "larger keys later":
        k[:, 100:] *= 40
        q *= 40 ** -0.5
    ref, out, one = exact(q, k, v), torch.full_like(q, float("nan")), torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    for r in range(0, Lq, 32):
        part = torch.empty_like(q[:, r:r + 32].contiguous())
        A.arl2_hybrid_attn_fwd(q[:, r:r + 32].contiguous(), k, v, None, None, part)
        one[:, r:r + 32] = part
    assert not torch.equal(out, one)
    assert error(out, ref) <= 1.03 * error(one, ref), f"{error(out, ref):.2e} {error(one, ref):.2e}"


@pytest.mark.parametrize("B,H,L,D,gate,own", [
    (1, 130, 40, 128, "head", False), (2, 40, 100, 64, "token", True), (1, 66, 130, 128, "element", True), (1, 12, 700, 64, "element", False),
    (1, 3, 700, 128, None, True)])
def test_state_gates_and_own_query(B, H, L, D, gate, own):
    q, k, v, x = (draw(i, B, L, H, D) for i in range(4))
    S = draw(5, B, H, D, D) * torch.logspace(-3, 3, D, device="cuda")            # columns of every size
    shape = {"head": (B, L, H), "token": (B, L), "element": (B, L, H, D)}.get(gate)
    g = None if gate is None else torch.rand(shape, device="cuda")
    out = torch.full_like(q, float("nan"))
    if own:
        A.arl2_hybrid_attn_fwd_ex(q, k, v, x, S, g, out)
    else:
        A.arl2_hybrid_attn_fwd(q, k, v, S, g, out)
    wide = None if g is None else {"head": lambda: g[..., None], "token": lambda: g[..., None, None], "element": lambda: g}[gate]()
    ref = exact(q, k, v, S, wide, x if own else None)
    for c in range(0, D, 16):                                                     # (a norm over all columns would only see the largest)
        e = error(out[..., c:c + 16], ref[..., c:c + 16])
        assert e <= TOL, f"columns {c}: {e:.2e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("own", [True, False])
@pytest.mark.parametrize("kind", ["one feature", "large beside small", "zero state", "zero columns and rows", "zero queries"])
def test_state_entries_of_every_size(kind, own, D):
    """Every output by itself is as exact as the sizes of the products that it sums allow."""
    B, H, L = 1, 40, 420
    q, k, v, x, S = draw(0, B, L, H, D), draw(1, B, L, H, D), draw(2, B, L, H, D), draw(3, B, L, H, D), draw(4, B, H, D, D)
    v[..., ::2] = 0                              # every second output is the state's alone
    if kind == "one feature":                    # queries that only see entries far below the others of their columns
        S[:, :, 1] *= torch.logspace(-20, 0, D, device="cuda")
        x[..., :1], x[..., 2:] = 0, 0
    elif kind == "large beside small":
        x[..., 3] *= 1e7
        S[:, :, 3] *= 1e-7
    elif kind == "zero state":
        S.zero_()
    elif kind == "zero columns and rows":
        S[..., D // 4:D // 2], S[:, :, 5:9] = 0, 0
    else:
        x[:, 7:100] = 0
    out = torch.full_like(q, float("nan"))
    if own:
        A.arl2_hybrid_attn_fwd_ex(q, k, v, x, S, None, out)
    else:
        q = x * 1e-7 if kind == "large beside small" else x                       # (ordinary logits)
        k[..., 3] *= 1e-3 if kind == "large beside small" else 1
        A.arl2_hybrid_attn_fwd(q, k, v, S, None, out)
        x = q
    ref, size = exact(q, k, v, S, None, x), exact(q, k, v.abs(), S.abs(), None, x.abs())
    assert ((out.double() - ref).abs() <= 2 ** -20 * size).all(), f"{((out.double() - ref).abs() / size.clamp(min=1e-300)).max():.2e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kind", ["small", "large", "outlier first", "outlier later", "large logits", "zero values", "zero then small"])
def test_values_of_every_size(kind, D):
    B, H, L = 1, 40, 400
    q, k, v = (draw(i, B, L, H, D) for i in range(3))
    if kind == "small":
        q, k, v = q * 1e-18, k * 1e18, v * 1e-30
    elif kind == "large":
        q, k, v = q * 1e15, k * 1e-15, v * 1e30
    elif kind == "outlier first":                # a value far above the others at a key that has 1e-8 of the largest weight
        q[..., 0] = 2 * D ** 0.5
        k[:, :, :, 0] = 0
        k[:, 3, :, 0] = -9
        v[:, 3] *= 1e6
    elif kind == "outlier later":
        q[..., 0] = 2 * D ** 0.5
        k[:, :, :, 0] = 0
        k[:, 300, :, 0] = -9
        v[:, 300] *= 1e7
    elif kind == "large logits":
        q = q * 20
    elif kind == "zero values":
        v = torch.zeros_like(v)
    else:
        k[:, :200] = 0
        v[:, :200] = 0
        v *= 1e-5
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    ref = exact(q, k, v)
    if kind == "zero values":
        assert (out == 0).all()
        return
    rows = (out.double() - ref).norm(dim=-1) / ref.norm(dim=-1)                   # every row by itself
    # A logit is a sum in some eight steps that round by 2^-24 of what it has reached, three of that as they come by chance or 2^-22.4 of the
    # largest; a row is off by up to twice what its logits are, and by a few roundings of its own sums.
    largest = (q.double().transpose(1, 2) @ k.double().permute(0, 2, 3, 1).contiguous()).abs().amax(-1).transpose(1, 2) * D ** -0.5
    assert (rows <= 2 ** -22 * (4 + largest)).all(), f"{float((rows / (4 + largest)).max() * 2 ** 22):.2f}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [100, 400, 700])
@pytest.mark.parametrize("kind", ["logspace", "every second", "constant and noise", "small later", "small then nothing", "zero", "near the smallest", "one outlier"])
def test_value_features_of_every_size(kind, L, D):
    """The features of V are outputs of their own: each by itself is as exact as where they are of one size."""
    B, H = 1, 40
    q, k, v = (draw(i, B, L, H, D) for i in range(3))
    if kind == "logspace":
        v = v * torch.logspace(-10, 3, D, device="cuda")
    elif kind == "every second":
        v[..., 1::2] *= 1e-8
    elif kind == "constant and noise":
        v *= 1e-8
        v[..., 3] = 1.0
    elif kind == "small later":                 # and nearly all that queries look at
        v[:, 128:, :, 5] *= 1e-7
        k[..., 0], q[..., 0] = 0.0, 2 * D ** 0.5
        k[:, :128 if L > 128 else 0, :, 0] = -9.0
    elif kind == "small then nothing":
        v[..., 5] *= 1e-7
        v[:, 40:, :, 5] = 0
    elif kind == "zero":                         # narrower values in wider rows
        v[..., D // 2:] = 0
    elif kind == "one outlier":
        v[:, 3, :, 5] = 300
    else:
        v *= 1e-37
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    ref = exact(q, k, v)
    if kind == "zero":
        assert (out[..., D // 2:] == 0).all()
        out, ref = out[..., :D // 2], ref[..., :D // 2]
    e = float(((out.double() - ref).norm(dim=1) / ref.norm(dim=1)).max())         # the worst feature of a head, over its rows
    assert e <= 2 * TOL, f"{e:.2e}"


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("size", [1.0, 1e6, 1e9, 1e11])
@pytest.mark.parametrize("later", [True, False])
def test_first_keys_zero(size, later, D):
    """The first 128 keys, from which the scale is taken, say nothing about the others: logits are ordinary whatever the sizes of q and k."""
    B, H, Lq, Lkv = 1, 40, 400, 401
    q, k, v = draw(0, B, Lq, H, D) * size, draw(1, B, Lkv, H, D) / size, draw(2, B, Lkv, H, D)
    k[:, :128 if later else Lkv] = 0
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    e = error(out, exact(q, k, v))
    assert e <= TOL, f"{e:.2e}"


@pytest.mark.parametrize("D", [64, 128])
def test_infinities_and_nan(D):
    B, H, L = 1, 40, 300
    q, k, v = (draw(i, B, L, H, D) for i in range(3))
    q[..., 0] = 1.0
    k[:, 10:50, :, 0] = -float("inf")            # masked keys
    out = torch.full_like(q, float("nan"))
    A.arl2_hybrid_attn_fwd(q, k, v, None, None, out)
    keep = [j for j in range(L) if not 10 <= j < 50]
    e = error(out, exact(q, k[:, keep], v[:, keep]))
    assert e <= TOL, f"{e:.2e}"
    k[:, 10:50, :, 0] = 0.0
    v[0, 7, 3, 5], v[0, 9, 3, 6], v[0, 200, 4, 8], S = float("inf"), float("nan"), -float("inf"), draw(9, B, H, D, D)
    S[0, 6, 2, 9], S[0, 6, 3, 10] = float("inf"), float("nan")
    A.arl2_hybrid_attn_fwd(q, k, v, S, None, out)
    ref = exact(q, k, v, S)
    assert torch.equal(torch.isnan(out), torch.isnan(ref))
    assert torch.equal(torch.isinf(out), torch.isinf(ref)) and torch.equal(out[torch.isinf(out)].double(), ref[torch.isinf(ref)])
    ok = torch.isfinite(ref)
    assert float((out.double()[ok] - ref[ok]).norm() / ref[ok].norm()) <= TOL
