"""Lists of more than 766 blocks and bitmaps of more than 2558, at the lengths
where d 128 changes kernel; sampled units against the fp64 oracle, and the
in-kernel selection against the lists."""
import numpy as np
import pytest

import oracle
import paper_2607_07724_amd as ugbs

from gpu_helpers import attention_error, dev, dev_bf16, host_bits
from test_gpu_attend_waves import inputs, lists

pytestmark = pytest.mark.gpu
ATOL_MAX, ATOL_RMS = 2e-2, 2e-3


def sampled(g, H, T, n):
    tiles = [0, 1, T - 1, T - 2] + [int(x) for x in g.integers(0, T, n - 4)]
    return np.array([(0, int(g.integers(0, H)), t) for t in tiles], np.int32)


def check(O, Q, K, V, kv, units, T):
    got = host_bits(O)
    got = np.stack([got[b, h, 64 * t:64 * t + 64] for b, h, t in units])
    ref = oracle.attend(Q, K, V, kv_idx=np.stack([kv[b, h, t] for b, h, t in units]), units=units)
    mx, rms = attention_error(got, ref)
    assert mx <= ATOL_MAX and rms <= ATOL_RMS


@pytest.mark.parametrize("d,T,W", [(128, 1100, 900), (128, 1407, 1000), (128, 1408, 1000), (64, 1408, 1000), (256, 900, 800)])
def test_wide_lists(d, T, W):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(5100 + d + T)
    Q, K, V = inputs(g, 1, 2, 1, 64 * T, d)
    kv = lists(g, 1, 2, T, W)
    p = ugbs.Problem.make(1, 2, 1, 64 * T, d, 3, 0.0, ugbs.QUEST)
    O = torch.full((1, 2, 64 * T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ugbs.ugbs_attend(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(kv), O)
    torch.cuda.synchronize()
    assert not torch.isnan(O).any()
    check(O, Q, K, V, kv, sampled(g, 2, T, 20), T)


@pytest.mark.parametrize("d", [64, 128, 256])
def test_bitmap_of_many_blocks(d):
    torch = pytest.importorskip("torch")
    T = 2600
    g = np.random.default_rng(5200 + d)
    Q, K, V = inputs(g, 1, 1, 1, 64 * T, d)
    p = ugbs.Problem.make(1, 1, 1, 64 * T, d, 3, 0.0)
    on = (g.random((1, 1, T, 32 * ugbs.bitmap_words(p))) < 0.3).astype(np.uint8)
    bits = np.packbits(on, axis=-1, bitorder="little").view(np.int32)
    O = torch.full((1, 1, 64 * T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ugbs.ugbs_attend_bitmap(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(bits), O)
    torch.cuda.synchronize()
    assert not torch.isnan(O).any()
    kv = np.where(on[..., :T], np.arange(T, dtype=np.int32), T).astype(np.int32)
    check(O, Q, K, V, kv, sampled(g, 1, T, 12), T)


@pytest.mark.parametrize("T,k,backbone", [(1407, 8, ugbs.KMEAN), (1408, 8, ugbs.KMEAN), (1408, 300, ugbs.QUEST),
                                          (2100, 8, ugbs.KMEAN), (2100, 200, ugbs.QUEST)])
def test_selection_in_the_kernel_gives_the_lists_bits(T, k, backbone):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(5300 + T + k)
    Q, K, V = (dev_bf16(x) for x in inputs(g, 1, 2, 1, 64 * T, 128))
    p = ugbs.Problem.make(1, 2, 1, 64 * T, 128, k, 0.3, backbone)
    bufs, O1, O2 = ugbs.Buffers(p), torch.empty_like(Q), torch.empty_like(Q)
    ugbs.prefill(p, Q, K, V, O1, bufs)
    ugbs.prefill_fused(p, Q, K, V, O2, bufs)
    torch.cuda.synchronize()
    assert np.array_equal(host_bits(O1), host_bits(O2))
