"""Prefill at the edges of its kernels' size classes and tiles, against fp64
attention in plain torch: bf16 work-groups of 64 and 128 rows with one and two
key groups; fp32 with 1, 2 and 4 waves per row block, 32 and 64 rows per wave,
with and without a die per (KV head, sequence) pair; lengths around whole
tiles."""
import math

import pytest
import torch

from paper_2406_14909_amd import moa as M

pytestmark = pytest.mark.gpu


def _reference(q, k, v, windows, s, block):
    b, n, hq, d = q.shape
    group = hq // len(windows)
    i = torch.arange(n, device=q.device)
    o = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    for g, w in enumerate(windows):
        first = (i // 64 - -(-w // 64) + 1) * 64 if block else i - w + 1
        seen = (i[None] <= i[:, None]) & ((i[None] < s) | (i[None] >= first[:, None]))
        for m in range(b):
            kt, vv = k[m, :, g].double().t().contiguous(), v[m, :, g].double()
            for h in range(g * group, (g + 1) * group):
                p = (q[m, :, h].double() @ kt / math.sqrt(d)).masked_fill_(~seen, -math.inf)
                o[m, :, h] = torch.softmax(p, 1) @ vv
    return o


def _run(dt, b, hq, hkv, d, n, s, flags, windows):
    print("[case] prefill sizes", dt, b, hq, hkv, d, n, s, flags, flush=True)
    plan = M.moa_plan(hq, hkv, d, s, 1 << 20, dt, [float(w) for w in windows], [0.0] * hkv, flags=flags)
    gen = torch.Generator(device="cuda").manual_seed(n + hq)
    draw = lambda h: torch.randn((b, n, h, d), generator=gen, device="cuda").to(plan.torch_dtype)
    q, k, v = draw(hq), draw(hkv), draw(hkv)
    o = torch.full_like(q, float("nan"))
    M.moa_prefill(plan, q, k, v, o)
    ref = _reference(q, k, v, windows, s, bool(flags & M.MOA_BLOCK_BAND))
    # the bars of the fp32 and bf16 paths elsewhere; outputs over 1 also carry half an ulp of bf16
    tol = 1e-5 if dt == "f32" else 1e-2 + 2.0 ** -8 * ref.abs()
    err = (o.double() - ref).abs()
    assert bool((err <= tol).all()), err.max().item()


@pytest.mark.parametrize("b,hq,hkv,d,n,s,flags", [
    (1, 4, 4, 64, 1, 0, 0), (1, 4, 2, 64, 31, 3, 0), (1, 4, 4, 64, 32, 0, 0), (2, 4, 1, 64, 33, 40, 0),
    (1, 4, 4, 128, 63, 0, 0), (1, 4, 2, 128, 65, 64, 0), (1, 2, 2, 128, 127, 1, M.MOA_BLOCK_BAND),
    (1, 8, 8, 64, 1501, 4, 0), (1, 32, 8, 64, 1000, 64, M.MOA_BLOCK_BAND),
    (5, 28, 7, 64, 130, 4, 0),              # 35 pairs over 8 dies
    (8, 16, 16, 64, 877, 4, 0),             # 3,584 blocks: 64 rows per wave, 2 waves per block
    (9, 32, 4, 64, 401, 64, 0),             # the same with 8 query heads per KV head, 36 pairs
    (2, 16, 8, 128, 800, 4, 0),             # 800 blocks of head_dim 128: 2 waves per block
    (5, 16, 16, 128, 1000, 70, 0),          # 2,560: one
])
def test_prefill_f32_sizes(b, hq, hkv, d, n, s, flags):
    windows = [1 + (97 * g * g + 13 * g) % max(1, n) for g in range(hkv)]
    windows[-1] = n
    _run("f32", b, hq, hkv, d, n, s, flags, windows)


@pytest.mark.parametrize("b,hq,hkv,n,s,flags,w", [
    # tiles shared through LDS: last tiles of 1, 63 and 64 keys, and rows that end inside one
    (1, 64, 8, 2497, 4, 0, 2497), (1, 64, 8, 2559, 64, M.MOA_BLOCK_BAND, 700), (1, 64, 8, 1408, 0, 0, 1408),
    (1, 32, 8, 3520, 70, 0, 600), (1, 8, 8, 8065, 1, 0, 900),
    # 64 rows per wave, 2 waves per block
    (1, 32, 32, 1023, 4, 0, 65), (1, 32, 8, 3520, 70, 0, 64),
])
def test_prefill_f32_head_dim_64_long(b, hq, hkv, n, s, flags, w):
    _run("f32", b, hq, hkv, 64, n, s, flags, [max(1, w - 5 * g) for g in range(hkv)])


def test_prefill_f32_window_of_one_key_is_exact():
    """Every path returns v bit for bit where a query sees one key."""
    for b, h, d, n in ((1, 2, 64, 99), (8, 16, 64, 877), (1, 4, 128, 99), (2, 16, 128, 805), (5, 16, 128, 1000),
                       (1, 20, 64, 5001)):
        print("[case] prefill one key", b, h, d, n, flush=True)
        plan = M.moa_plan(h, h, d, 0, n, "f32", [1.0] * h, [0.0] * h)
        gen = torch.Generator(device="cuda").manual_seed(n)
        q, k, v = (torch.randn((b, n, h, d), generator=gen, device="cuda") for _ in range(3))
        assert torch.equal(M.moa_prefill(plan, q, k, v), v)


@pytest.mark.parametrize("b,hq,hkv,d,n,s,flags", [
    # 64 rows, two key groups (from three tiles of 64 keys on)
    (1, 4, 4, 128, 129, 0, 0), (1, 4, 2, 128, 130, 3, 0), (1, 8, 1, 128, 191, 64, M.MOA_BLOCK_BAND),
    (1, 32, 32, 128, 512, 4, 0), (1, 4, 4, 64, 129, 0, 0), (1, 16, 4, 64, 2047, 70, 0), (3, 16, 8, 64, 640, 0, 0),
    # one more work-group than fits, and too short a chain: 128 rows, one key group
    (1, 4, 4, 128, 128, 0, 0), (3, 32, 8, 128, 200, 64, 0),
    # 128 rows, two key groups
    (1, 32, 32, 128, 513, 0, 0), (1, 32, 8, 128, 1024, 64, M.MOA_BLOCK_BAND), (1, 16, 2, 128, 3001, 1, 0),
    (4, 16, 16, 64, 1000, 4, 0), (1, 16, 16, 64, 4033, 64, 0),
    # few (KV head, sequence) pairs, whose work-groups share a die: 128 rows and one key group, or, with long or few
    # chains, as above
    (1, 8, 1, 128, 1024, 4, 0), (1, 16, 2, 128, 777, 64, 0), (1, 8, 1, 64, 1024, 4, 0), (1, 8, 1, 64, 4096, 4, 0),
    (1, 16, 2, 64, 3000, 64, 0), (1, 4, 4, 128, 193, 0, 0), (1, 4, 1, 128, 1500, 4, 0),
    # two work-groups of 128 rows per compute unit and more
    (2, 32, 32, 128, 1025, 4, 0), (5, 16, 4, 64, 1000, 0, M.MOA_BLOCK_BAND),
])
@pytest.mark.parametrize("narrow", [False, True])
def test_prefill_bf16_sizes(b, hq, hkv, d, n, s, flags, narrow):
    windows = [1 + (97 * g * g + 13 * g) % max(1, n // 8 if narrow else n) for g in range(hkv)]
    if not narrow:
        windows[-1] = n
    _run("bf16", b, hq, hkv, d, n, s, flags, windows)
