"""The launches the library makes, recorded on the CPU (launch_probe.py): which
attention kernel a call takes, and what its LDS leaves resident."""
import pytest

import paper_2607_07724_amd as ugbs
from launch_probe import launches, static_lds, workgroups_per_cu

make = ugbs.Problem.make


def waves_per_cu(x):
    return workgroups_per_cu(x) * x["block"] // 64


@pytest.mark.parametrize("d", [64, 128, 256])
def test_lists_of_every_length_leave_the_simds_full(d):
    """Two waves per SIMD (three at d 64, which its registers allow) whatever
    the list's length: entries of 16 bits, at most one per block.  (The coupled
    kernel at d 128 holds three units of two waves where a list has more than
    3836 entries.)"""
    calls = []
    for NB in (64, 767, 1024, 1407, 1408, 2048, 2559, 4096):
        p = make(1, 8, 2, 64 * NB, d, 64, 0.1, ugbs.QUEST)
        calls += [("attend", p, W) for W in (1, 128, 766, 767, 1024, 4096)] + [("attend_bitmap", p)]
    for st, xs in launches(calls):
        assert st == 0 and len(xs) == 1
        x = xs[0]
        coupled = x["kernel"].startswith("attend_kernel<128") and x["dynamic"] > 2 * 3836
        assert waves_per_cu(x) >= (12 if d == 64 else 6 if coupled else 8), x
        assert x["dynamic"] <= 2 * 4096


def test_long_walks_at_d128_keep_their_waves_coupled():
    def kernel(NB, backbone, k, W=None, H=28, Hkv=4):
        p = make(1, H, Hkv, 64 * NB, 128, k, 0.1, backbone)
        return launches([("attend", p, W or 2 * k)])[0][1][0]["kernel"]
    for NB in (1408, 2048, 4096):                     # every visible block listed
        assert kernel(NB, ugbs.QUEST, 64, NB) == "attend_kernel<128, 0>"
    assert kernel(2048, ugbs.KMEAN, 64) == "attend_kernel<128, 0>"
    assert kernel(2048, ugbs.QUEST, 256) == "attend_kernel<128, 0>"
    for NB, backbone, k in ((1407, ugbs.KMEAN, 64), (1024, ugbs.KMEAN, 500), (2048, ugbs.QUEST, 64), (4096, ugbs.QUEST, 64)):
        assert kernel(NB, backbone, k).startswith("attend_keys_kernel<128, 0,")


def test_lists_and_selection_take_the_same_kernel():
    """The two entry points agree bit for bit, so they have to split a unit's
    work alike: same kernel, same block, same LDS for the list."""
    probs = [make(B, H, Hkv, 64 * NB, d, k, q, bb, rho=rho)
             for B, H, Hkv in ((1, 4, 1), (1, 28, 4), (2, 8, 2)) for NB in (4, 16, 100, 700, 1407, 1408, 2049, 4096)
             for d in (64, 128, 256) for k, q, bb, rho in ((3, 0.0, ugbs.QUEST, 2), (4, 0.25, ugbs.KMEAN, 2), (64, 0.1, ugbs.QUEST, 2),
                                                            (400, 0.4, ugbs.QUEST, 4))]
    a = launches([("attend", p, p.W) for p in probs])
    b = launches([("attend_select", p) for p in probs])
    for p, (_, (x,)), (_, (y,)) in zip(probs, a, b):
        form = lambda z: z["kernel"].replace(", 0", ", m").replace(", 1", ", m").replace(", 3", ", m")
        assert form(x) == form(y), p
        assert (x["block"], x["grid"], x["dynamic"]) == (y["block"], y["grid"], y["dynamic"]), p
        assert static_lds()[x["kernel"]] == static_lds()[y["kernel"]], p


def test_bitmaps_take_two_waves_where_units_are_many():
    def waves(B, H, Hkv, NB, d):
        x = launches([("attend_bitmap", make(B, H, Hkv, 64 * NB, d, 16, 0.1))])[0][1][0]
        return x["block"] // 64
    assert waves(1, 32, 8, 100, 128) == waves(1, 28, 4, 512, 128) == waves(1, 28, 4, 512, 64) == 2
    assert waves(1, 8, 2, 128, 128) == waves(1, 32, 8, 80, 128) == waves(1, 32, 8, 200, 64) == 4
    for NB in (1532, 1533):          # the list of a two-wave unit reaches a quarter of a CU's LDS
        assert waves(1, 32, 8, NB, 128) == (2 if NB == 1532 else 4)
    assert all(waves(1, 32, 8, NB, 64) == 2 for NB in (512, 4096))


def test_diagnostics_of_wide_budgets_fit_the_lds():
    """Budgets beyond a row's candidates give records that are not valid; the
    launch still has to fit a workgroup's LDS, whatever k and rho."""
    probs = [make(1, 4, 1, 64 * NB, 64, k, 0.1, rho=rho)
             for NB in (40, 512, 1025, 2048) for k, rho in ((4, 2), (766, 4), (767, 4), (3066, 1), (1533, 2), (4096, 1), (512, 8))]
    for p, (st, xs) in zip(probs, launches([("bai_tiles", p, 16) for p in probs])):
        assert st == 0 and len(xs) == 1
        assert static_lds()[xs[0]["kernel"]] + xs[0]["dynamic"] <= 160 * 1024, p


def test_a_refused_lds_limit_is_reported():
    """Kernels with 64 KiB of static LDS need their dynamic limit raised; the
    call fails, without a launch, where the runtime refuses that."""
    p256, p128 = make(1, 4, 1, 64 * 300, 256, 16, 0.1), make(1, 4, 1, 64 * 100, 128, 16, 0.1)
    calls = [(fn, p, p.W if fn == "attend" else 0, True) for p in (p256, p128)
             for fn in ("attend", "attend_select", "attend_bitmap")]
    for st, xs in launches(calls):
        assert (st, xs) == (8, [])


def test_waves_per_unit_of_lists():
    """(kernel, waves) around the lines of the choice: few short lists on the
    coupled kernel, four waves for few units or chains that expansion makes long."""
    def form(d, H, Hkv, NB, k, q, rho=2):
        x = launches([("attend", make(1, H, Hkv, 64 * NB, d, k, q, rho=rho), rho * k)])[0][1][0]
        return ("keys" if "keys" in x["kernel"] else "coupled", x["block"] // 64)
    for d in (64, 128):
        assert form(d, 4, 1, 16, 3, 0.4, 1) == form(d, 4, 1, 16, 3, 0.0) == form(d, 32, 8, 32, 4, 0.1, 1) == ("coupled", 2)
        assert form(d, 4, 1, 16, 3, 0.1) == form(d, 4, 1, 16, 5, 0.0, 1) == ("keys", 4)
        assert form(d, 32, 8, 33, 3, 0.0, 1) == ("keys", 2)
        assert form(d, 32, 8, 32, 24, 0.1, 1) == ("keys", 2)         # no chain longer than the others
        assert form(d, 32, 8, 32, 24, 0.1) == ("keys", 4)
    assert form(64, 4, 1, 160, 3, 0.4) == ("keys", 2) and form(64, 4, 1, 160, 4, 0.4) == ("keys", 4)
    assert form(128, 32, 8, 64, 16, 0.1) == ("keys", 2) and form(128, 32, 16, 64, 16, 0.1) == ("keys", 4)
    assert form(128, 3, 3, 300, 8, 0.1, 4) == ("keys", 4)
