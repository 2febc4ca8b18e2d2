"""GPU tests of pruned L2 joins that hand rows to the relation-factorised kernel: the rows without a group (the packed
region behind the groups) and joins whose rows form one group.  The records are those of the dense per-relation kernels,
bit for bit where the distance is summed in the same order and to a rounding of float32 elsewhere."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PRUNE_OFF, PRUNE_ON = 1, 2


def _torch(x, dtype):
    import torch
    return torch.from_numpy(x.astype(np.float32)).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16).contiguous()


def _records(E, Rv, delta, cap, dtype, **cfg):
    import paper_2307_12059_amd as kgc
    j = kgc.Join(dtype=dtype, **cfg)
    try:
        out = []
        for _ in range(2):                     # the second call finds the handle's buffers in place
            got = j.join(E, Rv, 2, delta, cap)
            assert got["code"] == 0
            o = np.lexsort((got["t"], got["h"], got["r"]))
            out.append((np.stack([got["r"][o], got["h"][o], got["t"][o]], 1), got["dist"][o]))
        np.testing.assert_array_equal(out[0][0], out[1][0])
        return out[0][0], out[0][1], got["stats"]
    finally:
        j.close()


def _same(a, b):
    assert a[0].shape == b[0].shape
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_allclose(a[1], b[1], rtol=2.0 ** -22, atol=1e-30)


# clusters of 40 rows and rows far from everything, in random order; the latter fill, with the padding, a region whose
# first slot is no whole tile.  Relations lead from cluster to cluster, from a lone row to a lone row, and between the two
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_lone,n_big,R,d", [(1400, 37, 560, 20), (1281, 40, 650, 100), (1500, 41, 480, 250), (1300, 38, 600, 283),
                                              (1537, 130, 430, 64), (1290, 36, 610, 602)])
def test_rows_without_a_group(n_lone, n_big, R, d, dtype):
    g = np.random.default_rng(n_lone + d)
    cent = g.standard_normal((n_big, d))
    E = np.concatenate([np.repeat(cent, 40, 0) + 0.1 * g.standard_normal((40 * n_big, d)), g.standard_normal((n_lone, d))])
    N = E.shape[0]
    E = E[g.permutation(N)]
    h, t = g.integers(0, N, R), g.integers(0, N, R)
    Rv = E[t] - E[h] + 0.03 * g.standard_normal((R, d))
    Et, Rt = _torch(E, dtype), _torch(Rv, dtype)
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d)))
    got = _records(Et, Rt, delta, 1 << 20, dtype, prune=PRUNE_ON)
    want = _records(Et, Rt, delta, 1 << 20, dtype, prune=PRUNE_OFF, tile_cfg=18 if d <= 282 else 17)
    assert want[0].shape[0] > R and got[2]["groups"] >= n_big and got[2]["tiles_pruned"] > 0
    _same(got, want)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,R,d", [(1000, 16, 33), (2311, 37, 130), (1100, 20, 512)])
def test_one_group(N, R, d, dtype):
    g = np.random.default_rng(N)
    E = g.standard_normal((N, d))
    Rv = 0.5 * g.standard_normal((R, d))
    Et, Rt = _torch(E, dtype), _torch(Rv, dtype)
    delta = float(np.float32(np.sqrt(2.25 * d) - 2.2))
    got = _records(Et, Rt, delta, 1 << 22, dtype, prune=PRUNE_ON)
    want = _records(Et, Rt, delta, 1 << 22, dtype, prune=PRUNE_OFF, tile_cfg=18 if d <= 282 else 17)
    assert got[2]["join_variant"] == 100 and got[2]["groups"] >= 1 and want[0].shape[0] > 100
    _same(got, want)


def test_list_of_pairs_grows(monkeypatch):
    """The list of the region's pairs, and the list of the other tiles' blocks, are both too short at first."""
    g = np.random.default_rng(5)
    cent = g.standard_normal((30, 40))
    lone = g.standard_normal((1300, 40))
    E = np.concatenate([np.repeat(cent, 50, 0) + 0.1 * g.standard_normal((1500, 40)), lone])
    Rv = np.concatenate([lone[1:601] - lone[:600], cent[1:] - cent[:-1]])
    Et, Rt = _torch(E, "f32"), _torch(Rv, "f32")
    want = _records(Et, Rt, 1.0, 1 << 20, "f32", prune=PRUNE_OFF, tile_cfg=18)
    monkeypatch.setenv("KGC_EXACT_LIST_CAP", "3")
    got = _records(Et, Rt, 1.0, 1 << 20, "f32", prune=PRUNE_ON)
    assert want[0].shape[0] > 10000
    _same(got, want)


# the barrier-free kernel over tile lists (taken by itself from 262,144 entities on, here by its number): its candidates go
# through a list that is long enough, or that has to grow; few rows with long tile lists are walked in parts
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap", [None, "3"])
@pytest.mark.parametrize("N,R,d,k", [(1500, 6, 40, 9), (9000, 3, 100, 2), (5000, 4, 250, 40)])
def test_barrier_free_kernel_lists_its_candidates(N, R, d, k, cap, dtype, monkeypatch):
    g = np.random.default_rng(N + k)
    cent = g.standard_normal((k, d))
    E = cent[g.integers(0, k, N)] + 0.1 * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    Et, Rt = _torch(E, dtype), _torch(Rv, dtype)
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d) * 0.9))
    want = _records(Et, Rt, delta, 1 << 23, dtype, prune=PRUNE_OFF, tile_cfg=18)
    if cap:
        monkeypatch.setenv("KGC_EXACT_LIST_CAP", cap)
    got = _records(Et, Rt, delta, 1 << 23, dtype, prune=PRUNE_ON, tile_cfg=15)
    assert got[2]["join_variant"] == 15 and want[0].shape[0] > 50
    _same(got, want)


def _lone_rows(seed, n_lone, n_big, R, d, dtype):
    g = np.random.default_rng(seed)
    cent = g.standard_normal((n_big, d))
    E = np.concatenate([np.repeat(cent, 40, 0) + 0.1 * g.standard_normal((40 * n_big, d)), g.standard_normal((n_lone, d))])
    N = E.shape[0]
    E = E[g.permutation(N)]
    h, t = g.integers(0, N, R), g.integers(0, N, R)
    return _torch(E, dtype), _torch(E[t] - E[h] + 0.03 * g.standard_normal((R, d)), dtype)


# a workspace of one relation's operands: the part runs in batches of a few relations (R is no multiple of eight), the other
# tiles one relation at a time, and the list is emptied in between
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("extra", [0, 40, 400])
def test_rows_without_a_group_in_relation_batches(extra, dtype):
    n_lone, n_big, R, d = 1400, 37, 557, 20
    Et, Rt = _lone_rows(41, n_lone, n_big, R, d, dtype)
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d)))
    # two operands of 1,400 to 1,536 slots in one K slice of 64 bytes a slot, and the tables of `extra` relations
    ws = 2 * 64 * 1536 + extra * (4 * 1536 + 40 * 24)
    want = _records(Et, Rt, delta, 1 << 20, dtype, prune=PRUNE_ON)
    got = _records(Et, Rt, delta, 1 << 20, dtype, prune=PRUNE_ON, workspace_bytes=ws)
    assert want[2]["relation_batches"] == 1 and got[2]["relation_batches"] > 40 and want[0].shape[0] > R
    _same(got, want)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cap", [None, "3"])
def test_barrier_free_kernel_in_relation_batches(cap, dtype, monkeypatch):
    g = np.random.default_rng(17)
    N, R, d, k = 2500, 7, 40, 9
    cent = g.standard_normal((k, d))
    E = cent[g.integers(0, k, N)] + 0.1 * g.standard_normal((N, d))
    Rv = np.roll(cent, -1, 0)[:R] - cent[:R] + 0.02 * g.standard_normal((R, d))
    Et, Rt = _torch(E, dtype), _torch(Rv, dtype)
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d) * 0.9))
    want = _records(Et, Rt, delta, 1 << 23, dtype, prune=PRUNE_ON, tile_cfg=15)
    if cap:
        monkeypatch.setenv("KGC_EXACT_LIST_CAP", cap)
    got = _records(Et, Rt, delta, 1 << 23, dtype, prune=PRUNE_ON, tile_cfg=15, workspace_bytes=1)
    assert want[2]["relation_batches"] == 1 and got[2]["relation_batches"] == R and want[0].shape[0] > 50
    _same(got, want)


def test_the_part_keeps_to_the_workspace():
    """What a join with a part holds more than the same join without one (its kernel asked for by number) is the list of
    pairs: operands and tables share the memory of the batches."""
    import torch
    import paper_2307_12059_amd as kgc
    Et, Rt = _lone_rows(43, 12000, 40, 1000, 64, "f32")
    out = torch.empty((1 << 20, 4), dtype=torch.int32, device="cuda")
    held = {}
    for tile in (14, 0):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        j = kgc.Join(prune=PRUNE_ON, tile_cfg=tile, workspace_bytes=32 << 20)
        got = j.join(Et, Rt, 2, 1.0, 1 << 20, out=out, fetch=False)
        held[tile] = (before - torch.cuda.mem_get_info()[0], got["count"])
        j.close()
    assert held[0][1] == held[14][1] > 1000
    # the tables alone would be 1,000 x 12,000 x 4.6 bytes
    assert held[0][0] <= held[14][0] + (16 << 20) + (8 << 20), held


# the largest unit of the two-level bound test on both sides of the size up to which one wave summarises a unit, beside
# units of one micro-tile; both norms
@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("rows", [32, 4 * 32, 4 * 32 + 1, 33 * 32 + 1])
def test_summaries_of_large_units(rows, p):
    import paper_2307_12059_amd as kgc
    g = np.random.default_rng(rows)
    d, k = 70, 40
    cent = g.standard_normal((k, d))
    lab = np.concatenate([np.zeros(rows, int), np.repeat(np.arange(1, k), 30), np.arange(1, k)])
    E = (cent[lab] + 0.1 * g.standard_normal((lab.size, d)))[g.permutation(lab.size)]
    Rv = np.roll(cent, -1, 0)[[0, 5, k - 1]] - cent[[0, 5, k - 1]] + 0.02 * g.standard_normal((3, d))
    Et, Rt = _torch(E, "f32"), _torch(Rv, "f32")
    delta = float(np.float32(0.1 * np.sqrt(2.0 * d) * 0.95 if p == 2 else 0.1 * np.sqrt(2.0) * d * 0.75))
    out = []
    for prune in (PRUNE_ON, PRUNE_OFF):
        j = kgc.Join(prune=prune)
        try:
            got = j.join(Et, Rt, p, delta, 1 << 20)
        finally:
            j.close()
        assert got["code"] == 0
        o = np.lexsort((got["t"], got["h"], got["r"]))
        out.append((np.stack([got["r"][o], got["h"][o], got["t"][o]], 1), got["dist"][o]))
        if prune == PRUNE_ON:
            assert got["stats"]["tiles_pruned"] > 0
    assert out[0][0].shape[0] > 200
    _same(out[0], out[1])
