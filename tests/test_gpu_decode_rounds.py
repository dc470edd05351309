"""Decode where the work split can go wrong: caches of a whole number of rounds
of the kernels' key loops (64, 128 or 256 keys), one key more or less, many
partials per cache, pieces of one round and of many, for every kind of kernel,
with one position for the batch and with a position per sequence; against fp64
attention over the caches' filled slots in plain torch."""
import math

import pytest
import torch

from paper_2406_14909_amd import moa as M

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, Hq, Hkv, D, batch, sinks, windows, position
    ("bf16", 4, 4, 128, 1, 0, (127, 128, 129, 8191), 9000),
    ("bf16", 4, 4, 64, 2, 1, (255, 256, 254, 1), 3000),
    ("f32", 4, 4, 128, 1, 0, (63, 64, 65, 4100), 4500),
    ("f32", 4, 2, 64, 3, 2, (126, 1000), 999),
    ("bf16", 8, 2, 128, 1, 0, (8193, 1), 20000),          # 65 rounds: two per worker
    ("bf16", 16, 2, 128, 3, 4, (124, 16500), 16383),
    ("bf16", 4, 2, 64, 1, 64, (64, 65), 127),
    ("bf16", 32, 32, 128, 16, 0, tuple(range(4000, 4320, 10)), 5000),   # pieces of many rounds
    ("bf16", 32, 4, 64, 24, 3, (5000, 3, 1021, 2045), 7000),
    ("bf16", 16, 8, 128, 4, 0, (3072,) * 7 + (3073,), 5000),            # a little over a round per slot: two each
    ("bf16", 64, 8, 128, 8, 4, (4090, 4093) * 4, 5000),                 # over two: rounds dealt
    ("bf16", 64, 8, 128, 8, 4, (4090,) * 8, 5000),                      # equal numbers of keys
    ("bf16", 8, 1, 128, 1, 0, (32769,), 40000),                         # 129 partials for the merge
    ("bf16", 2, 2, 64, 2, 5, (66000, 33000), 70000),                    # 130 and fewer
    ("f32", 4, 2, 64, 1, 0, (33000, 9000), 40000),
]


def _reference(q, kc, vc, offset, fills, group):
    b, hq, d = q.shape
    o = torch.zeros_like(q, dtype=torch.float64)
    for i in range(b):
        for g in range(hq // group):
            n = fills[i][g]
            if n == 0:
                continue
            rows = slice(int(offset[g]), int(offset[g]) + n)
            k, v = kc[i, rows].double(), vc[i, rows].double()
            p = torch.softmax(q[i, g * group:(g + 1) * group].double() @ k.t().contiguous() / math.sqrt(d), 1)
            o[i, g * group:(g + 1) * group] = p @ v
    return o


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-hq{c[1]}-hkv{c[2]}-d{c[3]}-B{c[4]}-pos{c[7]}")
def test_decode_at_round_edges(case):
    dt, hq, hkv, d, b, s, windows, pos = case
    print("[case] decode rounds", case, flush=True)
    plan = M.moa_plan(hq, hkv, d, s, 1 << 20, dt, [float(w) for w in windows], [0.0] * hkv)
    gen = torch.Generator(device="cuda").manual_seed(pos)
    draw = lambda *shape: torch.randn(shape, generator=gen, device="cuda").to(plan.torch_dtype)
    q, kc, vc = draw(b, hq, d), draw(b, plan.cache_rows, d), draw(b, plan.cache_rows, d)
    ws = M.new_workspace(plan, b).fill_(255)                      # NaN patterns: nothing unwritten may count
    cap = plan.capacity.tolist()
    # bf16: half an ulp of the stored output (2^-9 of it) and of each weight (2^-9 of sums of |v| <= 5);
    # fp32: as the library's fp32 bar elsewhere
    tol = 1e-5 if dt == "f32" else 1e-2
    o = M.moa_decode(plan, q, kc, vc, pos, ws)
    ref = _reference(q, kc, vc, plan.offset, [[min(pos + 1, c) for c in cap]] * b, hq // hkv)
    assert (o.double() - ref).abs().max().item() <= tol * max(1.0, ref.abs().max().item())
    positions = [(pos * (2 * i + 1)) // (2 * b) for i in range(b)]
    positions[0] = pos
    if b > 2:
        positions[1] = -1
    o = torch.zeros_like(q)
    M.moa_decode_ragged(plan, q, kc, vc, torch.tensor(positions, dtype=torch.int32, device="cuda"), ws, o=o)
    ref = _reference(q, kc, vc, plan.offset, [[min(p + 1, c) for c in cap] for p in positions], hq // hkv)
    assert (o.double() - ref).abs().max().item() <= tol * max(1.0, ref.abs().max().item())
