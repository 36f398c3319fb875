"""Every unit of the attention is computed whatever the tile count.

The workgroup -> (batch, head, tile) order pads the grid when the tiles do
not divide over the XCDs, turns around above 64 tiles and falls back to a
plain order below; each parametrised length sits on one side of those lines.
O starts as NaN, so a unit that no workgroup takes shows; the rows are
checked against the fp64 oracle over the same short random lists.
"""
import numpy as np
import pytest

import oracle
import paper_2607_07724_amd as ugbs
from paper_2607_07724_amd import synth

from gpu_helpers import attention_error, dev, dev_bf16, host_bits

pytestmark = pytest.mark.gpu
ATOL_MAX, ATOL_RMS = 2e-2, 2e-3


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("T,B,H,Hkv", [(1, 1, 4, 2), (7, 1, 3, 3), (17, 2, 2, 1), (63, 1, 4, 2), (64, 1, 4, 2),
                                       (65, 1, 3, 1), (66, 1, 4, 2), (67, 2, 7, 1), (129, 1, 3, 3), (131, 1, 4, 2)])
def test_every_unit_is_attended(T, B, H, Hkv, d):
    torch = pytest.importorskip("torch")
    W = 5
    g = np.random.default_rng(900 + T + d)
    Q = synth.bf16_bits(g.standard_normal((B, H, 64 * T, d), dtype=np.float32))
    K = synth.bf16_bits(g.standard_normal((B, Hkv, 64 * T, d), dtype=np.float32))
    V = synth.bf16_bits(g.standard_normal((B, Hkv, 64 * T, d), dtype=np.float32))
    kv = synth.random_kv_idx(T, B, H, T, W)
    p = ugbs.Problem.make(B, H, Hkv, 64 * T, d, 3, 0.0)
    O = torch.full((B, H, 64 * T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ugbs.ugbs_attend(p, dev_bf16(Q), dev_bf16(K), dev_bf16(V), dev(kv), O)
    torch.cuda.synchronize()
    mx, rms = attention_error(host_bits(O), oracle.attend(Q, K, V, kv_idx=kv))
    assert mx <= ATOL_MAX and rms <= ATOL_RMS
