"""The native call path of the Python binding against its general path: the same
results, the same refusals, and the general path wherever a call is out of the
ordinary."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2406_14909_amd import moa as M
from paper_2406_14909_amd import search

pytestmark = pytest.mark.gpu


def _state(dt="bf16", b=2, n=150, hq=4, hkv=2, d=64):
    plan = M.moa_plan(hq, hkv, d, 4, n, dt, [30.0, 100.0], [0.0, 0.0])
    gen = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(plan.torch_dtype)
    return plan, draw(b, n, hq, d), draw(b, n, hkv, d), draw(b, n, hkv, d)


def _whole_path(stream, dt):
    """Every entry point once; stream None takes the native path, a stream the general one."""
    plan, q, k, v = _state(dt)
    b, n = q.shape[:2]
    out = [M.moa_prefill(plan, q, k, v, stream=stream)]
    kc, vc, pc = M.new_cache(plan, b)
    ws = M.new_workspace(plan, b)
    M.moa_kv_append(plan, kc, vc, pc, k, v, 0, stream=stream)
    last = [x[:, -1:].contiguous() for x in (k, v)]
    M.moa_kv_append(plan, kc, vc, pc, *last, n, stream=stream)
    qd = q[:, -1].contiguous()
    out += [kc.clone(), vc.clone(), pc.clone(), M.moa_decode(plan, qd, kc, vc, n, ws, stream=stream)]
    out.append(M.moa_decode_noalloc(plan, qd, kc, vc, n, torch.empty_like(qd), stream=stream))
    at = torch.tensor([n + 1, -1], dtype=torch.int32, device="cuda")
    M.moa_kv_append_ragged(plan, kc, vc, pc, *last, at, stream=stream)
    out += [kc, vc, pc, M.moa_decode_ragged(plan, qd, kc, vc, at, ws, o=torch.zeros_like(qd), stream=stream)]
    if dt == "bf16":
        e = M.moa_influence(q, k, v, q.flip(1).contiguous(), stream=stream)
        out += [e, *M.moa_rule_loss(e, n, 4, *search.candidate_rules(), stream=stream)]
    return out


@pytest.mark.parametrize("dt", ["bf16", "f32"])
def test_native_path_equals_general_path(dt):
    print("[case] binding", dt, flush=True)
    for a, b in zip(_whole_path(None, dt), _whole_path(torch.cuda.current_stream(), dt)):
        assert a.dtype == b.dtype and torch.equal(a, b)


def test_native_path_takes_ordinary_calls_and_leaves_the_others():
    print("[case] binding routes", flush=True)
    plan, q, k, v = _state()
    native = lambda *a: M._fast.prefill(plan._bound, *a)
    o = torch.empty_like(q)
    assert native(q, k, v, o) is o and native(q, k, v, None).shape == q.shape
    odd = [(q[:, :-1], k, v, None), (q, k.float(), v, None), (q, k, v.cpu(), None), (q, k, v, o[:1]),
           (q.transpose(0, 1).contiguous().transpose(0, 1), k, v, None), (q.reshape(-1), k, v, None), (None, k, v, None)]
    for a in odd:
        assert native(*a) is None
    with torch.device("cpu"):                      # an active torch function mode
        assert native(q, k, v, o) is None
        M.moa_prefill(plan, q, k, v, o)
    assert torch.vmap(lambda x: x * (native(x, k, v, None) is None))(q[None]).equal(q[None])
    with pytest.raises(M.MoaError, match="expected dtype"):
        M.moa_prefill(plan, q, k.float(), v)
    with pytest.raises(M.MoaError, match="overlaps"):
        M.moa_prefill(plan, q, k, v, q)
    kc, vc, pc = M.new_cache(plan, 2)
    M.moa_kv_append(plan, kc, vc, pc, k, v, np.int64(0))        # any integer is a position
    with pytest.raises(M.MoaError, match="start_pos"):
        M.moa_kv_append(plan, kc, vc, pc, k, v, -1)
    with pytest.raises(M.MoaError, match="workspace"):
        M.moa_decode(plan, q[:, 0].contiguous(), kc, vc, 10, torch.empty(256, dtype=torch.uint8, device="cuda"))
    e = torch.zeros((2, 3, 3), device="cuda")
    assert M.moa_rule_loss(e, 150, 4, [1.0, 2.0], [0.0, 0.0])[0].shape == (2, 2)     # lists, as before
    with pytest.raises(M.MoaError, match="1-D"):
        M.moa_rule_loss(e, 150, 4, np.zeros(2), np.zeros(3))
    bound = plan._bound
    plan.free()
    assert bound is not None and plan._bound is None and M._fast.prefill(plan._bound, q, k, v, o) is None


def test_native_path_runs_on_the_current_stream():
    print("[case] binding stream", flush=True)
    plan, q, k, v = _state()
    ref = M.moa_prefill(plan, q, k, v)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        o = M.moa_prefill(plan, q, k, v)
        side.synchronize()
        with torch.cuda.graph(g, stream=side):     # captured, so it ran on this stream
            p = M.moa_prefill(plan, q, k, v)
    p.zero_()
    torch.cuda.synchronize()
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(o, ref) and torch.equal(p, ref)


def _calls(dt="bf16"):
    """name -> (its capsule, ordinary arguments of the native function, positions of the tensors in them)."""
    plan, q, k, v = _state(dt)
    b, n = q.shape[:2]
    kc, vc, pc = M.new_cache(plan, b)
    M.moa_kv_append(plan, kc, vc, pc, k, v, 0)
    kn, vn, qd = k[:, -1:].contiguous(), v[:, -1:].contiguous(), q[:, -1].contiguous()
    at = torch.tensor([n, n], dtype=torch.int32, device="cuda")
    ws = M.new_workspace(plan, b)
    alpha, beta = search.candidate_rules()
    e = q[0, :9, 0, :2].t().float().reshape(2, 3, 3).contiguous()
    return {
        "moa_prefill": (plan, [q, k, v, torch.zeros_like(q)], (0, 1, 2, 3)),
        "moa_kv_append": (plan, [kc, vc, pc, kn, vn, n], (0, 1, 2, 3, 4)),
        "moa_kv_append_ragged": (plan, [kc, vc, pc, kn, vn, at], (0, 1, 2, 3, 4, 5)),
        "moa_decode": (plan, [qd, kc, vc, n, ws, torch.zeros_like(qd)], (0, 1, 2, 4, 5)),
        "moa_decode_noalloc": (plan, [qd, kc, vc, n, torch.zeros_like(qd)], (0, 1, 2, 4)),
        "moa_decode_ragged": (plan, [qd, kc, vc, at, ws, torch.zeros_like(qd)], (0, 1, 2, 3, 4, 5)),
        "moa_influence": (None, [q, k, v, q.flip(1).contiguous(), torch.zeros((4, 3, 3), device="cuda"), 0.0], (0, 1, 2, 3, 4)),
        "moa_rule_loss": (None, [e, 150, 4, np.asarray(alpha), np.asarray(beta), 0], (0,)),
    }


NATIVE = ["moa_prefill", "moa_kv_append", "moa_decode", "moa_decode_noalloc", "moa_kv_append_ragged",
          "moa_decode_ragged", "moa_influence", "moa_rule_loss"]


def _native(name, plan, args):
    return getattr(M._fast, name[4:])(M._bound if plan is None else plan._bound, *args)


def _public(name, plan, args, **kw):
    return getattr(M, name)(*([] if plan is None else [plan]), *args, **kw)


def _snapshot(args):
    return [a.clone() for a in args if torch.is_tensor(a)]


@pytest.mark.parametrize("name", NATIVE)
def test_every_native_function_makes_the_ordinary_call(name):
    print("[case] binding native", name, flush=True)
    plan, args, tensors = _calls()[name]
    plan2, args2, _ = _calls()[name]                     # the same inputs, for the general path
    done = _native(name, plan, args)
    assert done is not None and ("append" not in name or done is True)
    ref = _public(name, plan2, args2, stream=torch.cuda.current_stream())
    if name == "moa_rule_loss":
        assert all(torch.equal(x, y) for x, y in zip(done, ref))
    else:
        outs = args[:3] if "append" in name else [args[tensors[-1]]]
        refs = args2[:3] if "append" in name else [ref]
        assert all(torch.equal(x, y) for x, y in zip(outs, refs)) and any(x.any() for x in outs)


@pytest.mark.parametrize("name", NATIVE)
def test_every_native_function_leaves_odd_arguments(name):
    """Another shape, type, device or stride of any tensor: None, and nothing written."""
    print("[case] binding odd", name, flush=True)
    plan, args, tensors = _calls()[name]
    for i in tensors:
        t = args[i]
        workspace = t.dtype == torch.uint8               # any contiguous type and length: the library looks at its bytes
        odd = [None, t.cpu(), torch.stack((t, t), -1)[..., 0]]
        if not workspace:
            odd += [t.unsqueeze(0), t.long() if t.dtype == torch.int32 else t.double()]
            odd += [torch.cat((t, t), 1 if name == "moa_rule_loss" else 0)]          # of a profile any number of heads
        for x in odd:
            if x is None and i == len(args) - 1 and not name.endswith(("append", "ragged", "noalloc")):
                continue                                 # no output given: an ordinary call
            if x is None and name in ("moa_decode_ragged", "moa_influence") and i == tensors[-1]:
                continue
            bad = list(args)
            bad[i] = x
            before = _snapshot(args)
            assert _native(name, plan, bad) is None, (i, x if x is None else (x.shape, x.dtype, x.stride()))
            assert all(torch.equal(a, b) for a, b in zip(before, _snapshot(args)))
    assert _native(name, plan, args[:-1]) is None


@pytest.mark.parametrize("name", NATIVE)
def test_a_failed_launch_raises_and_is_not_repeated(name):
    """The library's status reaches the caller, once: neither a second call nor a
    silent success where the second one passes."""
    print("[case] binding status", name, flush=True)
    plan, args, _ = _calls()[name]
    seen = []

    @ctypes.CFUNCTYPE(ctypes.c_int)                      # looks at no argument
    def fails():
        seen.append(1)
        return M.MOA_ERR_HIP

    table = list(M._table)
    table[M._NATIVE.index(name)] = ctypes.cast(fails, ctypes.c_void_p).value
    layer = (0,) * 5 if plan is None else (plan.handle.value, plan.num_q_heads, plan.num_kv_heads, plan.head_dim,
                                           plan.cache_rows)
    bound = M._fast.bind(tuple(table), *layer, True, M._check)
    before = _snapshot(args)
    with pytest.MonkeyPatch.context() as mp:
        mp.setattr(*((M, "_bound") if plan is None else (plan, "_bound")), bound)
        with pytest.raises(M.MoaError) as e:
            _public(name, plan, args)
    assert e.value.status == M.MOA_ERR_HIP and len(seen) == 1
    assert all(torch.equal(a, b) for a, b in zip(before, _snapshot(args)))
