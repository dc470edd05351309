"""The influence kernel's alternation of tile stages: every parity of a pass's
tile count, of a wave's own share of it and of the item's number, with row
tiles whose last waves have no rows.  Same oracle and bound as the parity
cases."""
import numpy as np
import pytest
import torch

from oracle import influence_oracle as io
from paper_2406_14909_amd import moa as M
from tests.test_gpu_influence import _check, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bsz,n", [(2, 31), (3, 97), (2, 161), (3, 225), (4, 321), (1, 415)])
def test_influence_stage_parities(bsz, n, d):
    hq, hkv = 2, 1
    print("[case] influence stages", bsz, n, d, flush=True)
    q, k, v, do = _inputs(bsz, n, hq, hkv, d, 700 + n)
    got = M.moa_influence(q, k, v, do).cpu().numpy()
    torch.cuda.synchronize()
    e = io.influence_ref(io.causal_probabilities(q, k), io.grad_wrt_probabilities(v, do, hq))
    _check(got, io.block_average_ref(e), io.block_average_ref(np.abs(e)), f"B={bsz} n={n} d={d}")
