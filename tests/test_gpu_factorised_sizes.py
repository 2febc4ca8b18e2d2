"""GPU tests of the relation-factorised L2 join where joins take it by themselves: the same records, bit for bit, as the
kernels that contract every relation on its own (the exact stage decides both in double from the caller's rows)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PRUNE_OFF, PRUNE_ON = 1, 2


def _case(seed, N, R, d, k, sigma, dtype):
    import torch
    g = np.random.default_rng(seed)
    cent = g.standard_normal((k, d))
    lab = g.integers(0, k, N)
    E = cent[lab] + sigma * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    return (torch.from_numpy(E.astype(np.float32)).cuda().to(tt).contiguous(),
            torch.from_numpy(Rv.astype(np.float32)).cuda().to(tt).contiguous())


def _records(j, E, Rv, delta, cap):
    got = j.join(E, Rv, 2, delta, cap)
    assert got["code"] == 0, got["code"]
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1), got["stats"]


# d at the edges of the K slices and of the two tile shapes (256 head rows up to d = 282, 128 up to 602), N that fills
# its last tile with one row, or all but one, relations in one, several and not-whole groups of 64
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,R,d", [(1025, 385, 10), (1537, 200, 26), (2047, 97, 58), (1001, 700, 122), (4097, 25, 282),
                                   (1281, 260, 283), (2049, 129, 314), (3000, 64, 602), (15000, 8, 100)])
def test_matches_the_per_relation_kernels(N, R, d, dtype):
    import paper_2307_12059_amd as kgc
    sigma = 0.1
    E, Rv = _case(N + R + d, N, R, d, 9, sigma, dtype)
    delta = float(np.float32(sigma * np.sqrt(2.0 * d) * 0.97))
    cap = 1 << 23
    a = kgc.Join(dtype=dtype, prune=PRUNE_OFF)
    b = kgc.Join(dtype=dtype, prune=PRUNE_OFF, tile_cfg=18 if d <= 282 else 17)
    try:
        got, st = _records(a, E, Rv, delta, cap)
        want, st2 = _records(b, E, Rv, delta, cap)
    finally:
        a.close()
        b.close()
    assert st["join_variant"] == 100 and st2["join_variant"] == (18 if d <= 282 else 17)
    assert want.shape[0] > 1000
    assert got.shape == want.shape
    np.testing.assert_array_equal(got[:, :3], want[:, :3])
    # one distance, summed in double in the same order by both: the same float
    np.testing.assert_array_equal(got[:, 3], want[:, 3])


def test_list_of_pairs_grows(monkeypatch):
    import paper_2307_12059_amd as kgc
    E, Rv = _case(7, 1025, 400, 40, 9, 0.1, "f32")
    delta = float(np.float32(0.1 * np.sqrt(80.0)))
    a = kgc.Join(prune=PRUNE_OFF)
    monkeypatch.setenv("KGC_EXACT_LIST_CAP", "3")
    b = kgc.Join(prune=PRUNE_OFF)
    try:
        want, _ = _records(a, E, Rv, delta, 1 << 23)
        for _ in range(2):
            got, st = _records(b, E, Rv, delta, 1 << 23)
            assert st["join_variant"] == 100
            np.testing.assert_array_equal(got, want)
    finally:
        a.close()
        b.close()


def test_every_pair_passes_and_far_translations():
    """Thresholds that decide nothing (all pairs are hits: more than the list may hold), and relations far longer than
    the embeddings, whose products lose the small distances in float32: both are left to the exact stage."""
    import paper_2307_12059_amd as kgc
    E, Rv = _case(8, 1100, 400, 24, 5, 0.1, "f32")
    j = kgc.Join(prune=PRUNE_OFF)
    k = kgc.Join(prune=PRUNE_OFF, tile_cfg=18)
    try:
        got = j.join(E, Rv, 2, 1e3, 16)
        assert got["count"] == 1100 * 1100 * 400
        far, _ = _records(j, E, Rv * 300.0, 2.0, 1 << 20)
        want, _ = _records(k, E, Rv * 300.0, 2.0, 1 << 20)
        np.testing.assert_array_equal(far, want)
        E2 = E.clone()
        E2[:550] -= 1000.0
        R2 = Rv + 1000.0
        far, st = _records(j, E2, R2, 0.4, 1 << 22)
        want, _ = _records(k, E2, R2, 0.4, 1 << 22)
        assert want.shape[0] > 100
        np.testing.assert_array_equal(far, want)
    finally:
        j.close()
        k.close()


# relations that do not fill the last eight rows of the per-relation tables, entities whose squared norms leave float32's
# range: every filter value is a NaN or an infinity, all pairs go to the exact stage, and none of a relation that is not there
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("r_range", [None, (3, 20)])
def test_norms_past_float32_stay_with_the_relations_of_the_call(r_range, dtype):
    import torch
    import paper_2307_12059_amd as kgc
    g = np.random.default_rng(3)
    N, R, d, k = 1000, 17 if r_range is None else 25, 32, 20
    lab = g.integers(0, k, N)
    E = 1e19 * g.standard_normal((k, d))[lab]
    Rv = 1e19 * g.standard_normal((R, d))
    Rv[::2] = 0.0
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    Et, Rt = (torch.from_numpy(x.astype(np.float32)).cuda().to(tt).contiguous() for x in (E, Rv))
    lo, hi = r_range or (0, R)
    assert (hi - lo) % 8 != 0
    j = kgc.Join(dtype=dtype, prune=PRUNE_OFF)
    try:
        got = j.join(Et, Rt, 2, 1.0, 1 << 20, r_range=r_range)
    finally:
        j.close()
    assert got["code"] == 0 and got["stats"]["join_variant"] == 100
    assert got["r"].min() >= lo and got["r"].max() < hi
    h, t = np.nonzero(lab[:, None] == lab[None, :])                # two rows are the same or some 1e19 apart
    r = np.arange(lo + lo % 2, hi, 2)
    want = ((r[:, None] * N + h) * N + t).ravel()
    np.testing.assert_array_equal(np.sort((got["r"].astype(np.int64) * N + got["h"]) * N + got["t"]), np.sort(want))
    assert not got["dist"].any()


# the filter's margin comes from each row's own rounding: neither relations much longer than delta nor one entity far longer
# than the others may fill the list of pairs (the per-relation kernel's candidates are the measure)
@pytest.mark.parametrize("N,R,d,delta,long_row", [(1000, 16, 32, 0.5, 1.0), (4000, 40, 100, 5.2, 1.0), (4000, 40, 100, 5.2, 30.0)])
def test_candidates_do_not_grow_with_the_longest_row_or_relation(N, R, d, delta, long_row):
    import paper_2307_12059_amd as kgc
    E, Rv = _case(11, N, R, d, 20, 0.1 if d == 32 else 0.7, "f32")
    E[7] *= long_row
    a = kgc.Join(prune=PRUNE_OFF)
    b = kgc.Join(prune=PRUNE_OFF, tile_cfg=18)
    try:
        got, st = _records(a, E, Rv, delta, 1 << 20)
        want, st2 = _records(b, E, Rv, delta, 1 << 20)
    finally:
        a.close()
        b.close()
    assert st["join_variant"] == 100 and st2["join_variant"] == 18
    np.testing.assert_array_equal(got, want)
    assert st["candidates"] <= 2 * st2["candidates"] + N // 4, (st["candidates"], st2["candidates"])


# Row order: one tile of pivots and one row more than it, two tiles, the most (sixteen); both tile shapes and norms; rows
# that the caller has in order already, or backwards; one relation
@pytest.mark.parametrize("N,R,d,p,dtype,rows", [(256, 9, 20, 2, "f32", "random"), (257, 3, 100, 2, "bf16", "random"),
                                                (4100, 7, 33, 2, "f32", "sorted"), (4095, 6, 64, 1, "f32", "random"),
                                                (33000, 1, 40, 2, "bf16", "random"), (9001, 8, 290, 2, "bf16", "backwards")])
def test_row_order_leaves_the_result_alone(N, R, d, p, dtype, rows, monkeypatch):
    import paper_2307_12059_amd as kgc
    import torch
    E, Rv = _case(N + d, N, R, d, 9 if N < 1000 else 200, 0.1, dtype)
    if rows != "random":
        E = E[torch.argsort(E[:, 0].float(), descending=rows == "backwards")].contiguous()
    delta = float(np.float32(0.1 * (np.sqrt(2.0 * d) * 0.95 if p == 2 else 1.08 * d)))
    out = []
    for order in ("0", "1"):
        monkeypatch.setenv("KGC_ROW_ORDER", order)
        j = kgc.Join(dtype=dtype, prune=PRUNE_OFF, factorised=p == 2 and d <= 282)
        try:
            got = j.join(E, Rv, p, delta, 1 << 23)
        finally:
            j.close()
        assert got["code"] == 0 and got["stats"]["join_variant"] == 100
        o = np.lexsort((got["t"], got["h"], got["r"]))
        out.append(np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1))
    assert out[0].shape[0] > 100
    np.testing.assert_array_equal(out[0], out[1])


# The line from which dense L2 joins take this kernel by themselves: N R = 15,000 with two K slices and more, eight relations with one
# (d <= 26); calls on either side of it give the same records
@pytest.mark.parametrize("N,R,d,taken", [(1000, 15, 64, True), (999, 15, 64, False), (7500, 2, 27, True), (7500, 2, 26, False),
                                         (2200, 7, 26, False), (2200, 8, 26, True), (256, 60, 33, True), (255, 70, 33, False)])
def test_line_of_the_dense_dispatch(N, R, d, taken):
    import paper_2307_12059_amd as kgc
    E, Rv = _case(N + d, N, R, d, max(3, N // 40), 0.1, "f32")
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d) * 0.95))
    recs = []
    for tile in (0, 18):
        j = kgc.Join(prune=PRUNE_OFF, tile_cfg=tile)
        try:
            got = j.join(E, Rv, 2, delta, 1 << 20)
        finally:
            j.close()
        assert got["code"] == 0 and got["stats"]["join_variant"] == (100 if taken and not tile else 18)
        o = np.lexsort((got["t"], got["h"], got["r"]))
        recs.append(np.stack([got["r"][o], got["h"][o], got["t"][o]], 1))
    assert recs[0].shape[0] > 30
    np.testing.assert_array_equal(recs[0], recs[1])
