"""The route at the edges of its search and of its row copy, bit for bit.

Tile counts around a wave's 64 keys, the 1024 up to which one wave searches
(and the workgroup's threads), twice that, and the largest accepted; sigmas
with heavy ties (the quantile search ends early only on distinct ones), all
equal, and zero; rows of four-slot accesses and not, lists whose pointers are
not 16-byte aligned, in place and out of place.
"""
import numpy as np
import pytest

import oracle
import paper_2607_07724_amd as ugbs

from gpu_helpers import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,rho", [(1, 3, 2), (5, 3, 1), (63, 4, 2), (64, 5, 2), (65, 4, 3), (66, 33, 2), (513, 64, 2),
                                     (1024, 6, 4), (1025, 5, 3), (2048, 9, 2), (2049, 33, 2), (4096, 4, 2)])
@pytest.mark.parametrize("kind", ["distinct", "ties", "equal"])
def test_route_rows(T, k, rho, kind):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(6000 + T)
    B, H = (2, 3) if T <= 1025 else (1, 2)
    sig = g.random((B, H, T)).astype(np.float32)
    if kind == "ties":
        sig = (np.round(sig * 3) / 4).astype(np.float32)
    elif kind == "equal":
        sig = np.zeros_like(sig)
    idx = g.integers(0, T + 1, (B, H, T, rho * k)).astype(np.int32)
    n = idx.size
    for q in (0.0, 0.07, 0.5, 1.0):
        p = ugbs.Problem.make(B, H, 1, 64 * T, 64, k, q, rho=rho)
        rkv, rsb, rtau, rtrig = oracle.route(sig, idx, k, q, rho=rho)
        for shift in (0, 1):            # ints before the list: its alignment
            for in_place in (False, True):
                src = torch.empty(n + 4, dtype=torch.int32, device="cuda")[shift:shift + n].view(idx.shape)
                src.copy_(dev(idx))
                out = src if in_place else torch.full((n + 4,), -9, dtype=torch.int32,
                                                      device="cuda")[shift:shift + n].view(idx.shape)
                ws = torch.empty((max(256, ugbs.ugbs_workspace_bytes(p)),), dtype=torch.uint8, device="cuda")
                sb = torch.empty((B, T), dtype=torch.float32, device="cuda")
                tau = torch.empty((B,), dtype=torch.float32, device="cuda")
                trig = torch.empty((B, T), dtype=torch.uint8, device="cuda")
                ugbs.ugbs_route(p, dev(sig), src, out, ws, sb, tau, trig)
                torch.cuda.synchronize()
                assert np.array_equal(host(out), rkv), (q, shift, in_place)
                assert np.array_equal(host(sb), rsb) and np.array_equal(host(tau), rtau)
                assert np.array_equal(host(trig), rtrig)
