"""Score workgroups that span tiles, and waves that own two units.

A score workgroup takes four (long rows: eight) consecutive units of a kv
head, so with few query heads per kv head it spans several tiles, and the last
one is partial where the count doesn't divide.  On small integers every sum
is exact, so the tile scores must equal the vector-ALU form's bit for bit, and
the packed-row selection must equal the full-tensor one.
"""
import pytest

import paper_2607_07724_amd as ugbs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,H,Hkv,T", [(64, 1, 3, 3, 67), (128, 2, 1, 1, 33), (128, 1, 6, 3, 65), (256, 1, 2, 1, 35),
                                         (128, 1, 5, 1, 3), (128, 1, 16, 16, 1025), (128, 1, 21, 3, 1027),
                                         (128, 1, 16, 4, 1023)])
def test_units_across_tiles(d, B, H, Hkv, T):
    torch = pytest.importorskip("torch")
    g = torch.Generator(device="cuda").manual_seed(7000 + T + d)

    def ints(h):
        return torch.randint(-4, 5, (B, h, 64 * T, d), generator=g, device="cuda").to(torch.bfloat16)

    Q, K = ints(H), ints(Hkv)
    p = ugbs.Problem.make(B, H, Hkv, 64 * T, d, 6, 0.1, ugbs.QUEST)
    meta = torch.empty((B, Hkv, T, d, 2), dtype=torch.bfloat16, device="cuda")
    ugbs.ugbs_block_meta(p, K, meta)
    want, got = (torch.full((B, H, T, T), float("nan"), device="cuda") for _ in range(2))
    idx, sig = torch.empty((B, H, T, p.W), dtype=torch.int32, device="cuda"), torch.empty((B, H, T), device="cuda")
    idx2, sig2 = torch.empty_like(idx), torch.empty_like(sig)
    ws = torch.empty((max(256, ugbs.ugbs_workspace_bytes(p)),), dtype=torch.uint8, device="cuda")
    ugbs.ugbs_quest_scores_valu(p, Q, meta, want)
    ugbs.ugbs_score_select(p, Q, meta, idx, sig, scores_out=got)
    ugbs.ugbs_score_select(p, Q, meta, idx2, sig2, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(want, got)
    assert torch.equal(idx, idx2) and torch.equal(sig, sig2)
