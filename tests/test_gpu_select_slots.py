"""Sorted selection at the edges of its row sizes, bit for bit.

The kernel is compiled for rows of up to 256, 512, 1024, 2048 and 4096 blocks,
skips groups of 512 candidates past a row's end, and sorts rows of at most 128
candidates whole.  Each length sits on one side of such a line; budgets put R
(listed candidates, or the m + 1 of sigma) at 128 and just past it, and past
192, where the pre-filter ends.  Scores are tie-heavy, hold both zeros and
infinities; the oracle selects from the same tensor.
"""
import numpy as np
import pytest

import oracle
import paper_2607_07724_amd as ugbs

from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [3, 64, 66, 130, 131, 256, 257, 512, 513, 1024, 1025, 2049])
@pytest.mark.parametrize("k,rho", [(3, 1), (5, 2), (65, 2), (66, 2), (129, 1), (97, 2), (98, 2), (194, 1), (130, 2)])
def test_row_sizes(T, k, rho):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(5000 + T + k)
    H = 2 if T <= 513 else 1
    S = g.standard_normal((1, H, T, T)).astype(np.float32)
    S = np.where(g.random(S.shape) < 0.5, np.round(S * 4) / 4, S).astype(np.float32)
    S[g.random(S.shape) < 0.01] = -0.0
    S[g.random(S.shape) < 0.002] = -np.inf
    p = ugbs.Problem.make(1, H, 1, 64 * T, 64, k, 0.1, rho=rho)
    Q = torch.zeros((1, H, 64 * T, 64), dtype=torch.bfloat16, device="cuda")
    meta = torch.zeros((1, 1, T, 64, 1), dtype=torch.bfloat16, device="cuda")
    idx = torch.full((1, H, T, p.W), -7, dtype=torch.int32, device="cuda")
    sig = torch.full((1, H, T), float("nan"), dtype=torch.float32, device="cuda")
    only = torch.full_like(sig, float("nan"))
    ugbs.ugbs_score_select(p, Q, meta, idx, sig, scores_in=dev(S))
    ugbs.ugbs_score_select(p, Q, meta, None, only, scores_in=dev(S))
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        ridx, rsig = oracle.select(S, k, rho=rho)
    assert np.array_equal(host(idx), ridx)
    # infinities at the cut give NaN (inf - inf) on both sides
    assert np.array_equal(host(sig), rsig, equal_nan=True)
    assert np.array_equal(host(only), rsig, equal_nan=True)
