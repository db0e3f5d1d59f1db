"""The binding's two ways into the C ABI, the compiled one for plain calls and the checked one behind it, accept, refuse and
compute the same."""
import inspect

import pytest
import torch

import paper_2605_16579_amd as A
from helpers import built_package
from paper_2605_16579_amd import binding


@pytest.fixture(autouse=True, scope="module")
def built():
    built_package().load_library()
    assert binding._host_call is not binding._no_host_call


class Checked(torch.Tensor):
    """A tensor that is no plain torch.Tensor: every call with it goes through the checked path."""


def calls(dev, D, dtype=torch.bfloat16):
    """name -> (call, tensors, those that are written)."""
    g = torch.Generator().manual_seed(D)
    B, L, H = 2, 70, 3

    def t(*shape, dt=dtype, scale=1.0):
        return (torch.rand(shape, generator=g) * scale).to(dt).to(dev)

    rows, f32 = (B, L, H, D), torch.float32
    q, k, v, out, S = t(*rows), t(*rows), t(*rows), t(*rows), t(B, H, D, D, dt=f32)
    W, cs, sn = t(H, D, D), t(L, D // 2, dt=f32), t(L, D // 2, dt=f32)
    gate, al, be = t(B, H, dt=f32), t(B, L, H, dt=f32), t(B, L, H, dt=f32)
    ws = torch.empty(max(A.arl2_workspace_bytes(B, H, L, D, dtype), A.arl2_gdn_workspace_bytes(B, H, L, D)), dtype=torch.uint8, device=dev)
    c = {
        "fwd": (A.arl2_hybrid_attn_fwd, [q, k, v, S, t(B, L, H, dt=f32), out], [5]),
        "fwd softmax": (A.arl2_hybrid_attn_fwd, [q, t(B, 40, H, D), t(B, 40, H, D), None, None, out], [5]),
        "commit": (A.arl2_state_commit, [k, v, gate, S, ws], [3]),
    }
    if dtype == torch.bfloat16:
        c.update({
            "fwd token gate": (A.arl2_hybrid_attn_fwd, [q, k, v, S, t(B, L), out], [5]),
            "fwd element gate": (A.arl2_hybrid_attn_fwd, [q, k, v, S, t(*rows), out], [5]),
            "fwd_ex": (A.arl2_hybrid_attn_fwd_ex, [q, k, v, t(*rows), S, None, out], [6]),
            "fwd_fm": (A.arl2_hybrid_attn_fwd_fm, [q, k, v, t(*rows), W, cs, sn, S, t(B, L, H, dt=f32), out], [9]),
            "feature_map": (A.arl2_feature_map, [q, W, cs, sn, out], [4]),
            "feature_map plain": (A.arl2_feature_map, [q, W, None, None, out], [4]),
            "commit_static": (A.arl2_state_commit_static, [k, v, gate, S], [3]),
            "commit_fm": (A.arl2_state_commit_fm, [k, W, cs, sn, v, t(H, D, D), gate, S, ws], [7]),
            "commit_delta": (A.arl2_state_commit_delta, [k, v, gate, t(B, H, dt=f32, scale=0.01), S, ws], [4]),
            "commit_gdn": (A.arl2_state_commit_gdn, [k, v, al, be, S, ws], [4]),
        })
    return c


def wrong(ts):
    """Every tensor of a call in turn on the host, transposed, of another type, of another shape (a workspace may be of any)."""
    for i, t in enumerate(ts):
        if t is None:
            continue
        bads = [t.cpu()]
        if t.dtype != torch.uint8:
            bads += [t.transpose(0, 1), t.double(), t[None], t[..., 1:].contiguous()]
        for bad in bads:
            yield i, ts[:i] + [bad] + ts[i + 1:]


def outcome(fn, ts, **kw):
    try:
        fn(*ts, **kw)
        return None
    except Exception as e:      # noqa: BLE001  (both ways have to raise the same)
        return type(e), str(e)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_plain_and_checked_calls_agree_about_none(dtype):
    for name, (fn, ts, _) in calls("cuda", 64, dtype).items():
        for i in range(1, len(ts)):
            args = ts[:i] + [None] + ts[i + 1:]
            assert outcome(fn, args) == outcome(fn, [args[0].as_subclass(Checked)] + args[1:]), (name, i)
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D", [64, 128])
def test_plain_and_checked_calls_agree(D, dtype, monkeypatch):
    seen, host_call = [], binding._host_call

    def recorded(*args):
        seen.append(host_call(*args))
        return seen[-1]

    monkeypatch.setattr(binding, "_host_call", recorded)
    for name, (fn, ts, written) in calls("cuda", D, dtype).items():
        start = [ts[i].clone() for i in written]

        def results(args, status, **kw):
            for i, x in zip(written, start):
                ts[i].copy_(x)
            seen.clear()
            assert outcome(fn, args, **kw) is None, name
            assert seen == [status], name              # the compiled way was taken, or left
            torch.cuda.synchronize()
            return [ts[i].clone() for i in written]

        checked = [ts[0].as_subclass(Checked)] + ts[1:]
        scales = {key: x for key, x in (("sm_scale", 0.3), ("l2_eps", 0.5)) if key in inspect.signature(fn).parameters}
        for kw in ({}, {"stream": torch.cuda.current_stream().cuda_stream}, scales):
            plain = results(ts, 0, **kw)
            assert all(torch.equal(a, b) for a, b in zip(plain, results(checked, None, **kw))), name
            assert all(not torch.equal(a, b) for a, b in zip(plain, start)), name
            if kw is not scales:
                usual = plain
            elif kw:
                assert all(not torch.equal(a, b) for a, b in zip(plain, usual)), name
        for i, bad in wrong(ts):
            got = outcome(fn, bad)
            assert got is not None, (name, i)
            if i > 0:
                assert got == outcome(fn, [bad[0].as_subclass(Checked)] + bad[1:]), (name, i)


def test_plain_calls_leave_everything_else_to_the_checked_path():
    A.load_library()
    addr = binding._addr["arl2_hybrid_attn_fwd"]
    q = torch.zeros((1, 8, 2, 64), dtype=torch.bfloat16)
    for args in ((b"qkkSgq", 0.0, 0.0, 0, None, q, q, q, None, None, q), (b"qkkSgq", 0.0, 0.0, 0, None, q, q, q, None, None),
                 (b"qkkSgq", "x", 0.0, 0, None, q, q, q, None, None, q), (b"qkkSgq", 0.0, 0.0, None, None, q, q, q, None, None, q),
                 (b"qkkSgq", 0.0, 0.0, 0, None, None, None, None, None, None, None), (b"qkkSgq", 0.0, 0.0, 0, None, 1, 2, 3, 4, 5, 6),
                 (b"", 0.0, 0.0, 0, None), ("qkkSgq", 0.0, 0.0, 0, None, q, q, q, None, None, q)):
        assert binding._host_call(addr, *args) is None, args
    with pytest.raises(ValueError):
        A.arl2_hybrid_attn_fwd(q, q, q, None, None, q)


def test_without_the_compiled_module_every_call_is_marshalled_in_python(monkeypatch, tmp_path):
    broken = tmp_path / "broken.so"
    broken.write_bytes(b"no shared object")
    q = torch.zeros((1, 8, 2, 64), dtype=torch.bfloat16)
    for name, value, why in (("HOST_PATH", str(tmp_path / "missing.so"), "missing"), ("HOST_PATH", str(broken), "broken"),
                             ("HOST_FOR", "Python 2.7, torch 0.1", "this is Python 2.7")):
        with monkeypatch.context() as m:
            m.setattr(binding, "_lib", None)
            m.setattr(binding, "_host_call", None)
            m.setattr(binding, name, value)
            with pytest.warns(RuntimeWarning, match=why):
                lib = A.load_library()
            assert binding._host_call is binding._no_host_call
            assert A.arl2_version() == lib.arl2_version() >= 100
            with pytest.raises(ValueError, match="q must live in device memory"):
                A.arl2_hybrid_attn_fwd(q, q, q, None, None, q)
