"""Attention with the keys of a unit split over two or four waves (d 64, 128).

Four waves take over when the units are few (d 128: 512 and fewer, d 64: 768)
and when there are a few rounds of units with long chains; for bitmaps up to
1024 units of 96 and more blocks (d 64: 7680).  Lists of at most four blocks take
the kernel whose waves split the rows, up to 1024 units.  The parametrised
shapes lie on both sides of those lines.  The lists are where the split can go wrong: single blocks (waves
without an entry), the diagonal alone (a wave whose keys are all masked for
half of the rows), rows without the diagonal, odd and even counts, empty
rows (O = 0), widths past one 64-entry read.  A large logit scale makes the
running maxima of the waves move and differ.  Checked on every row against
the fp64 oracle; the in-kernel selection must give the lists path's bits.
"""
import numpy as np
import pytest

import oracle
import paper_2607_07724_amd as ugbs
from paper_2607_07724_amd import synth

from gpu_helpers import attention_error, bf16_to_f64, dev, dev_bf16, host_bits

pytestmark = pytest.mark.gpu
ATOL_MAX, ATOL_RMS = 2e-2, 2e-3


def lists(g, B, H, T, W):
    """Rows of 0..W distinct blocks of 0..t: none, the diagonal alone, one
    other block, or a random subset with or without the diagonal."""
    kv = np.full((B, H, T, W), T, np.int32)
    for idx in np.ndindex(B, H, T):
        t = idx[2]
        kind = int(g.integers(0, 5))
        if kind == 0:
            row = [t]
        elif kind == 1:
            row = [int(g.integers(0, t + 1))]
        elif kind == 2 and g.random() < 0.3:
            row = []
        else:
            row = list(g.permutation(t + 1)[:int(g.integers(1, W + 1))])
        kv[idx][:len(row)] = row
    return kv


def inputs(g, B, H, Hkv, N, d):
    return [synth.bf16_bits(g.standard_normal((B, h, N, d), dtype=np.float32)) for h in (H, Hkv, Hkv)]


@pytest.mark.parametrize("scale", [0.0, 0.9])
@pytest.mark.parametrize("d,B,H,Hkv,T,W", [(64, 1, 4, 2, 9, 4), (64, 1, 4, 2, 9, 8), (64, 1, 3, 3, 70, 67), (64, 1, 32, 8, 129, 7),
                                           (128, 1, 4, 2, 9, 4), (128, 1, 4, 2, 9, 8), (128, 2, 2, 1, 70, 67), (128, 1, 16, 4, 129, 7)])
def test_lists_of_every_kind(d, B, H, Hkv, T, W, scale):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(4100 + d + T + W)
    Q, K, V = inputs(g, B, H, Hkv, 64 * T, d)
    kv = lists(g, B, H, T, W)
    p = ugbs.Problem.make(B, H, Hkv, 64 * T, d, 3, 0.0, scale=scale)
    O = torch.full((B, H, 64 * T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ugbs.ugbs_attend(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(kv), O)
    torch.cuda.synchronize()
    ref = oracle.attend(Q, K, V, kv_idx=kv, scale=scale if scale else None)
    mx, rms = attention_error(host_bits(O), ref)
    assert mx <= ATOL_MAX and rms <= ATOL_RMS
    empty = np.repeat((kv == T).all(-1), 64, axis=-1)
    assert np.all(bf16_to_f64(host_bits(O))[empty] == 0)


@pytest.mark.parametrize("d,H,Hkv,T", [(64, 4, 2, 40), (64, 28, 4, 150), (128, 4, 2, 40), (128, 14, 2, 150)])
@pytest.mark.parametrize("k", [5, 90])
def test_selection_in_the_kernel_gives_the_lists_bits(d, H, Hkv, T, k):
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(4200 + d + T)
    Q, K, V = (dev_bf16(x) for x in inputs(g, 1, H, Hkv, 64 * T, d))
    p = ugbs.Problem.make(1, H, Hkv, 64 * T, d, k, 0.3, ugbs.QUEST, rho=3)
    bufs, O1, O2 = ugbs.Buffers(p), torch.empty_like(Q), torch.empty_like(Q)
    ugbs.prefill(p, Q, K, V, O1, bufs)
    ugbs.prefill_fused(p, Q, K, V, O2, bufs)
    torch.cuda.synchronize()
    assert np.array_equal(host_bits(O1), host_bits(O2))


@pytest.mark.parametrize("d,H,Hkv,T,W", [(64, 4, 2, 9, 4), (64, 4, 2, 9, 8), (64, 32, 8, 129, 7), (128, 4, 2, 9, 4),
                                           (128, 4, 2, 9, 8), (128, 16, 4, 129, 7), (256, 4, 2, 9, 8)])
def test_scores_that_overflow(d, H, Hkv, T, W):
    """Positive queries against keys of -3e38 or 3e38: scores of -inf, whose
    weight is 0 beside any finite score, or +inf, which makes the row NaN.
    Every second half block is -inf, so one wave of each pair sees nothing else,
    every third block is -inf whole, and one block is +inf."""
    torch = pytest.importorskip("torch")
    g = np.random.default_rng(4400 + d + T)
    Q, K, V = (synth.bf16_bits(np.abs(g.standard_normal((1, h, 64 * T, d), dtype=np.float32))) for h in (H, Hkv, Hkv))
    low, high = synth.bf16_bits(np.array([-3e38, 3e38], np.float32))
    kb = K.reshape(1, Hkv, T, 64, d)
    kb[:, :, :, 32:] = low
    kb[:, :, 2::3] = low
    kv = lists(g, 1, H, T, W)
    kv[..., 0] = 0                                     # a block with finite scores in every row
    kv[..., 1:][kv[..., 1:] == 0] = T
    p = ugbs.Problem.make(1, H, Hkv, 64 * T, d, 3, 0.0)

    def run():
        O = torch.empty((1, H, 64 * T, d), dtype=torch.bfloat16, device="cuda")
        ugbs.ugbs_attend(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(kv), O)
        torch.cuda.synchronize()
        return host_bits(O)
    O = run()
    mx, rms = attention_error(O, oracle.attend(Q, K, V, kv_idx=kv))
    assert mx <= ATOL_MAX and rms <= ATOL_RMS
    kb[:, :, 4, 63] = high                             # the last key of block 4
    hit = np.repeat((kv == 4).any(-1), 64, axis=-1)
    hit.reshape(1, H, T, 64)[:, :, 4, :63] = False     # rows before it don't see it
    O2 = run()
    assert np.isnan(bf16_to_f64(O2)[hit]).all() and np.array_equal(O2[~hit], O[~hit])


@pytest.mark.parametrize("d", [64, 128])
def test_bitmaps_on_both_sides_of_the_line(d):
    torch = pytest.importorskip("torch")
    for H, Hkv, T in ((2, 1, 33), (28, 4, 150 if d == 128 else 280)):     # four waves, two waves
        g = np.random.default_rng(4300 + d + T)
        Q, K, V = inputs(g, 1, H, Hkv, 64 * T, d)
        kv = lists(g, 1, H, T, 9)
        p = ugbs.Problem.make(1, H, Hkv, 64 * T, d, 3, 0.0)
        on = np.zeros((1, H, T, 32 * ugbs.bitmap_words(p) + 1), np.uint8)
        np.put_along_axis(on, np.where(kv == T, on.shape[-1] - 1, kv), 1, axis=-1)
        bits = np.packbits(on[..., :-1], axis=-1, bitorder="little").view(np.int32)
        O = torch.full((1, H, 64 * T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ugbs.ugbs_attend_bitmap(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(bits), O)
        torch.cuda.synchronize()
        mx, rms = attention_error(host_bits(O), oracle.attend(Q, K, V, kv_idx=kv))
        assert mx <= ATOL_MAX and rms <= ATOL_RMS
