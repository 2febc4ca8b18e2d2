"""GPU tests of the default pruning mode, which takes the relation-factorised kernel where that is the shorter way: the same
records as with pruning on, whichever way a call goes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

AUTO, ON = 0, 2


def _case(seed, N, R, d, rows, sigma, dtype):
    import torch
    g = np.random.default_rng(seed)
    k = max(2, N // rows)
    cent = g.standard_normal((k, d))
    lab = g.integers(0, k, N)
    E = cent[lab] + sigma * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    return (torch.from_numpy(E.astype(np.float32)).cuda().to(tt).contiguous(),
            torch.from_numpy(Rv.astype(np.float32)).cuda().to(tt).contiguous())


def _records(prune, dtype, E, Rv, p, delta, cap, r_range=None):
    import paper_2307_12059_amd as kgc
    j = kgc.Join(dtype=dtype, prune=prune)
    try:
        got = j.join(E, Rv, p, delta, cap) if r_range is None else j.join(E, Rv, p, delta, cap, r_range=r_range)
    finally:
        j.close()
    assert got["code"] == 0
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o]], 1), got["dist"][o], got["stats"]


# way: the kernel the call must end on with the default mode (100 = factorised, straight or after grouping; None: a pruned one).
# Edges of the rules: the fewest rows and relations, a call one relation below; clusters that group well (straight by size, or not:
# too many hits asked for), clusters too small to group, one broad group; L1 with a short list, and with a sample that rules
# the list out; d past the factorised kernel
@pytest.mark.parametrize("N,R,d,p,rows,sigma,dtype,cap,way", [
    (256, 24, 20, 2, 32, 0.1, "f32", 1 << 16, 100), (256, 23, 20, 2, 32, 0.1, "f32", 1 << 16, None),
    (3001, 2, 33, 2, 60, 0.1, "bf16", 1 << 16, 100), (2000, 8, 32, 2, 100, 0.1, "f32", 1 << 16, 100),
    (2000, 300, 32, 2, 100, 0.1, "f32", 1 << 22, None), (9000, 900, 40, 2, 10, 0.1, "f32", 1 << 16, 100),
    (4110, 47, 121, 2, 42, 0.7, "f32", 1 << 20, 100), (600, 40, 603, 2, 30, 0.1, "f32", 1 << 16, None),
    (1500, 30, 40, 1, 12, 0.05, "f32", 1 << 16, 100), (1500, 30, 300, 1, 60, 0.15, "bf16", 1 << 20, None)])
def test_default_mode_returns_what_pruning_returns(N, R, d, p, rows, sigma, dtype, cap, way):
    E, Rv = _case(N + R + d, N, R, d, rows, sigma, dtype)
    # about a quarter of the aligned pairs (L2), a few per cent (L1)
    delta = float(np.float32(sigma * (np.sqrt(2.0 * d) - 0.7) if p == 2 else sigma * 1.128 * d * 0.9))
    a, da, st = _records(AUTO, dtype, E, Rv, p, delta, cap)
    b, db, _ = _records(ON, dtype, E, Rv, p, delta, max(cap, 1 << 22))
    assert (st["join_variant"] == 100) == (way == 100)
    assert a.shape[0] > 0
    np.testing.assert_array_equal(a, b)
    np.testing.assert_allclose(da, db, rtol=2.0 ** -23, atol=0)       # one rounding to float32 of either side's double


def test_default_mode_over_a_range_of_relations_and_with_a_list_that_grows(monkeypatch):
    E, Rv = _case(5, 2000, 20, 32, 100, 0.1, "f32")
    delta = float(np.float32(0.1 * np.sqrt(64.0) * 0.9))
    want, _, _ = _records(ON, "f32", E, Rv, 2, delta, 1 << 18)
    want = want[(want[:, 0] >= 3) & (want[:, 0] < 15)]
    monkeypatch.setenv("KGC_EXACT_LIST_CAP", "3")
    got, _, st = _records(AUTO, "f32", E, Rv, 2, delta, 1 << 18, r_range=(3, 15))
    assert st["join_variant"] == 100
    np.testing.assert_array_equal(got, want)
    # a list that cannot be had: back to the pruned kernels
    monkeypatch.setenv("KGC_PAIR_LIST_LIMIT", "1")
    got, _, st = _records(AUTO, "f32", E, Rv, 2, delta, 1 << 18, r_range=(3, 15))
    assert st["join_variant"] == 14
    np.testing.assert_array_equal(got, want)


# One cluster pair per relation with most of its pairs within delta: the list of pairs is the longer way.  A call that only counts (a
# sample tells), one with room for a few of them (the list outgrows what the room announced), one with room for all
@pytest.mark.parametrize("cap", [0, 1000, 1 << 23])
def test_calls_with_many_hits_go_over_the_groups_whatever_their_room(cap):
    import paper_2307_12059_amd as kgc
    E, Rv = _case(9, 6400, 46, 64, 400, 0.1, "f32")
    delta = float(np.float32(0.1 * np.sqrt(128.0) * 1.1))
    res = []
    for prune in (ON, AUTO):
        j = kgc.Join(prune=prune)
        try:
            got = [j.join(E, Rv, 2, delta, cap, fetch=False) for _ in range(2)][1]
        finally:
            j.close()
        res.append(got["count"])
        assert got["code"] == (1 if cap < got["count"] else 0) and got["stats"]["join_variant"] == 14
    assert res[0] == res[1] > 1 << 21


def test_counting_calls_with_few_hits_stay_on_the_factorised_kernel():
    import paper_2307_12059_amd as kgc
    E, Rv = _case(2, 2000, 8, 32, 100, 0.1, "f32")
    delta = float(np.float32(0.1 * np.sqrt(64.0) * 0.9))
    want = _records(ON, "f32", E, Rv, 2, delta, 1 << 18)[0].shape[0]
    j = kgc.Join(prune=AUTO)
    try:
        got = j.join(E, Rv, 2, delta, 0, fetch=False)
    finally:
        j.close()
    assert got["code"] == 1 and got["count"] == want > 0 and got["stats"]["join_variant"] == 100


def test_few_rows_without_a_group_do_not_send_a_large_join_to_the_factorised_kernel():
    """Clusters of 25 rows, a hundredth of which form no group: contracting every pair of 60,000 rows at d = 300 takes far longer than the
    pruned kernels spend on those few."""
    import paper_2307_12059_amd as kgc
    g = np.random.default_rng(8)
    N, R, d, k = 60_000, 6, 300, 2_400
    import torch
    cent = g.standard_normal((k, d)).astype(np.float32)
    lone = 800
    E = np.concatenate([np.repeat(cent, 25, axis=0)[:N - lone] + 0.1 * g.standard_normal((N - lone, d)).astype(np.float32),
                        g.standard_normal((lone, d)).astype(np.float32)])[g.permutation(N)].astype(np.float32)
    src = g.integers(0, k, R)
    Rv = (cent[(src + 1) % k] - cent[src]).astype(np.float32)
    E, Rv = torch.from_numpy(E).cuda(), torch.from_numpy(Rv).cuda()
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d) * 0.98))
    recs = []
    for prune in (AUTO, ON):
        j = kgc.Join(prune=prune)
        try:
            got = j.join(E, Rv, 2, delta, 1 << 18)
        finally:
            j.close()
        assert got["code"] == 0 and got["stats"]["join_variant"] != 100 and got["stats"]["groups"] > 1000, got["stats"]
        o = np.lexsort((got["t"], got["h"], got["r"]))
        recs.append(np.stack([got["r"][o], got["h"][o], got["t"][o]], 1))
    assert recs[0].shape[0] > 100
    np.testing.assert_array_equal(recs[0], recs[1])
