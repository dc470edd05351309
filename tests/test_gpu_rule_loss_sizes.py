"""The rule-loss table at the edges of its kernel's size classes (64, 128, 256,
512 and 1024 block rows), with whole and cut last block rows, sink edges inside
and past the profile, and windows around whole blocks, against pair counts
taken row by row in plain torch."""
import numpy as np
import pytest
import torch

from paper_2406_14909_amd import moa as M

pytestmark = pytest.mark.gpu


def _expected(e, n, s, window, block):
    """sum over blocks of (hidden pairs of the block) * e, per head, in fp64."""
    nb = e.shape[1]
    i = torch.arange(n, device=e.device)
    first = (i // 64 - -(-window // 64) + 1) * 64 if block else i - window + 1
    end = torch.minimum(first.clamp(min=0), i + 1)
    start = torch.arange(nb, device=e.device) * 64
    out = torch.zeros(e.shape[0], dtype=torch.float64, device=e.device)
    for b in range(nb):
        rows = end[b * 64:(b + 1) * 64]
        count = (rows[:, None].minimum(start + 64) - start.clamp(min=s)).clamp(min=0).sum(0)
        out += e[:, b].double() @ count.double()
    return out


@pytest.mark.parametrize("n,s,flags", [
    (1, 0, 0), (63, 4, 0), (65, 64, 0), (4096, 64, 0), (4097, 70, 0), (8192, 100, 0), (8193, 64, M.MOA_BLOCK_BAND),
    (16384, 1, 0), (16385, 16300, 0), (32768, 64, 0), (32769, 127, M.MOA_BLOCK_BAND), (65536, 63, 0), (65475, 64, 0),
    (200, 500, 0),
])
def test_rule_loss_at_size_class_edges(n, s, flags):
    print("[case] rule loss", n, s, flags, flush=True)
    nb = -(-n // 64)
    gen = torch.Generator(device="cuda").manual_seed(n)
    e = torch.randn((2, nb, nb), generator=gen, device="cuda")   # the upper triangle is never read
    windows = sorted({min(max(w, 1), n) for w in (1, 2, 63, 64, 65, 66, 127, 128, 129, n // 2, n - 64, n - 1, n)})
    dl, dens = M.moa_rule_loss(e, n, s, np.array(windows, dtype=np.float64), np.zeros(len(windows)), flags)
    low = torch.tril(e)
    for r, w in enumerate(windows):
        ref = _expected(low, n, s, w, bool(flags & M.MOA_BLOCK_BAND))
        # sums of at most nb^2 / 2 fp64 terms of up to 4096 |e| <= 4096 * 6: their roundings stay below
        # 2^-53 * nb * (sum of the terms' sizes) <= 2^-53 * 1024 * 4096 * 4 * nb^2 / 2
        assert torch.all((dl[:, r] - ref).abs() <= 1e-12 * 4096 * nb * nb), (w, dl[:, r], ref)
        assert dens[r].item() == min(s + w, n) / n
