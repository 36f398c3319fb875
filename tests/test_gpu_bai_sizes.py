"""Diagnostics at the sizes where their kernels change form: rows on both
sides of 512 and 1024 blocks, ranks on both sides of a group of eight, a
partial group of heads, and head statistics over many tied tiles and over
NaN records."""
import numpy as np
import pytest

import paper_2607_07724_amd as ugbs
from oracle import bai
from paper_2607_07724_amd import synth
from gpu_helpers import dev
from test_gpu_bai import check_tiles, compare_heads, gpu_heads, gpu_tiles

pytestmark = pytest.mark.gpu


def tile_scores(H, T, seed):
    g = np.random.default_rng(seed)
    S = g.standard_normal((1, H, T, T), dtype=np.float32)
    blk = np.arange(T)
    S[:, :, ~((blk[None, :] >= 1) & (blk[None, :] < blk[:, None]))] = -np.inf
    return S


@pytest.mark.parametrize("H,T,k", [(5, 40, 9), (4, 40, 10), (3, 40, 11), (1, 512, 4), (1, 513, 33),
                                   (2, 1024, 5), (1, 1025, 10)])
def test_tiles_at_row_and_group_sizes(H, T, k):
    S = tile_scores(H, T, 100 * T + k)
    tau32 = np.full((1, H), 0.2, np.float32)
    z = synth.mc_normals(7, 70, T)
    p = ugbs.Problem.make(1, H, 1, 64 * T, 64, k, 0.3)
    check_tiles(gpu_tiles(p, S, tau32, z)[1], S, k, tau32, z)      # bit for bit


@pytest.mark.parametrize("T", [1, 63, 64, 65, 511, 513, 1025, 2048])
@pytest.mark.parametrize("q", [0.0, 0.1, 1.0])
def test_heads_with_tied_tiles(T, q):
    """Records on a coarse grid: many equal sigmas, spacings and failure
    differences, decided by tile order; some tiles not valid."""
    g = np.random.default_rng(T)
    H, k, n_s = 2, 4, 16
    rec = np.zeros((1, H, T), np.dtype(ugbs.BAI_TILE_FIELDS))
    grid = lambda n: (g.integers(0, n, (1, H, T)) / np.float32(n)).astype(np.float32)
    rec["g"], rec["sigma"], rec["delta2"] = grid(8), grid(5), grid(6) + np.float32(0.125)
    rec["r"] = grid(64) + np.float32(0.5)
    rec["G"] = rec["g"] + np.float32(1)
    rec["fail_k"] = g.integers(0, n_s + 1, (1, H, T))
    rec["fail_rk"] = g.integers(0, 4, (1, H, T))
    rec["valid"] = g.random((1, H, T)) < 0.9
    tau32 = np.full((1, H), 0.3, np.float32)
    p = ugbs.Problem.make(1, H, 1, 64 * T, 64, k, q)
    hd = gpu_heads(p, dev(rec.view(np.uint8).reshape(-1)), tau32, n_s)
    gaps = {f: rec[f] for f in ("g", "G", "r", "sigma", "delta2")}
    gaps["valid"] = rec["valid"].astype(bool)
    compare_heads(hd, bai.head_stats(gaps, rec["fail_k"], rec["fail_rk"], tau32, q, k, n_s))


@pytest.mark.parametrize("T", [40, 90])
def test_heads_with_nan_records(T):
    """NaN spacings and sigmas (infinite scores) rank above every number; the
    tiles of NaN sigmas count among the routed ones besides the nq first."""
    g = np.random.default_rng(50 + T)
    n_s, q, nq = 16, 0.3, int(np.ceil(0.3 * T))
    rec = np.zeros((1, 1, T), np.dtype(ugbs.BAI_TILE_FIELDS))
    for f in ("g", "G", "r", "sigma", "delta2"):
        rec[f] = g.random((1, 1, T)).astype(np.float32) + np.float32(0.5)
    rec["sigma"][0, 0, [3, T // 2, T - 1]] = np.nan
    rec["delta2"][0, 0, ::4] = np.nan
    rec["fail_k"] = g.integers(0, n_s + 1, (1, 1, T))
    rec["valid"] = 1
    p = ugbs.Problem.make(1, 1, 1, 64 * T, 64, 4, q)
    hd = gpu_heads(p, dev(rec.view(np.uint8).reshape(-1)), np.full((1, 1), 0.3, np.float32), n_s)
    sig, d2, d = (rec[f][0, 0] for f in ("sigma", "delta2", "fail_k"))
    order = np.argsort(sig, kind="stable")             # NaN last
    assert hd["sigma_q"][0, 0] == np.float64(sig[order[nq - 1]])
    assert hd["delta2_p05"][0, 0] == np.float64(np.sort(d2)[int(0.05 * (T - 1))])
    assert hd["delta2_p50"][0, 0] == np.float64(np.sort(d2)[int(0.5 * (T - 1))])
    top, routed = int(np.sort(d)[::-1][:nq].sum()), int(d[order[:nq]].sum() + d[np.isnan(sig)].sum())
    assert hd["mc_regret"][0, 0] == (top / n_s - routed / n_s) / T
