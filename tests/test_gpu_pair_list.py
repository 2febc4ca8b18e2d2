"""GPU tests of the list of pairs that the factorised kernel and the pruned barrier-free kernel hand to the exact stage: a list
that is too short grows, one that cannot be had is done without, and in both cases the records are the same."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PRUNE_OFF, PRUNE_ON = 1, 2


def _clusters(seed, N, R, d, k, lone=0):
    import torch
    g = np.random.default_rng(seed)
    cent = g.standard_normal((k, d))
    E = np.concatenate([cent[g.integers(0, k, N - lone)] + 0.1 * g.standard_normal((N - lone, d)), g.standard_normal((lone, d))])
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    return tuple(torch.from_numpy(x.astype(np.float32)).cuda() for x in (E, Rv))


def _call(j, E, Rv, p, delta):
    got = j.join(E, Rv, p, delta, 1 << 21)
    assert got["code"] == 0, got["code"]
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o]], 1), got["dist"][o], got["stats"]["join_variant"]


# path, join options, inputs, join_variant with and without the list (the pruned join of the rows without a group keeps its
# kernel either way)
CASES = {
    "dense_l2": (dict(prune=PRUNE_OFF), 2, (1500, 40, 40, 30), 1.0, (100, 18)),
    "dense_l1": (dict(prune=PRUNE_OFF), 1, (4000, 9, 64, 60), 6.5, (100, 0)),
    "lone_rows": (dict(prune=PRUNE_ON), 2, (2800, 600, 40, 30, 1400), 1.0, (14, 14)),
    "one_group": (dict(prune=PRUNE_ON, group_radius=100.0), 2, (1500, 40, 40, 30), 1.0, (100, 14)),
    "tile_lists": (dict(prune=PRUNE_ON, tile_cfg=15), 2, (3000, 6, 40, 30), 1.0, (15, 15)),
}


# room for the first length but not for a longer one (three pairs are too few for every case), and for none at all
@pytest.mark.parametrize("limit", ["60", "1"])
@pytest.mark.parametrize("name", list(CASES))
def test_list_that_cannot_be_had(name, limit, monkeypatch):
    import paper_2307_12059_amd as kgc
    cfg, p, shape, delta, variants = CASES[name]
    E, Rv = _clusters(len(name), *shape)
    a = kgc.Join(**cfg)
    monkeypatch.setenv("KGC_EXACT_LIST_CAP", "3")
    grows = kgc.Join(**cfg)
    monkeypatch.setenv("KGC_PAIR_LIST_LIMIT", limit)
    b = kgc.Join(**cfg)
    try:
        want = _call(a, E, Rv, p, delta)
        assert want[2] == variants[0] and want[0].shape[0] > 300
        for j, variant in ((grows, variants[0]), (grows, variants[0]), (b, variants[1]), (b, variants[1])):
            got = _call(j, E, Rv, p, delta)
            np.testing.assert_array_equal(got[0], want[0])
            np.testing.assert_allclose(got[1], want[1], rtol=2.0 ** -22, atol=1e-30)
            assert got[2] == variant
    finally:
        for j in (a, grows, b):
            j.close()


def test_block_by_block_join_keeps_its_row_order_without_the_list(monkeypatch):
    """kgc_join_blocks reuses the grouped order of its first unit; a list that cannot be had must not make a new one."""
    import paper_2307_12059_amd as kgc
    E, Rv = _clusters(3, 3000, 6, 40, 30)
    a = kgc.Join(prune=PRUNE_ON, tile_cfg=15)
    monkeypatch.setenv("KGC_PAIR_LIST_LIMIT", "1")
    b = kgc.Join(prune=PRUNE_ON, tile_cfg=15)
    try:
        want = _call(a, E, Rv, 2, 1.0)[0]
        parts, cursor = [], None
        while True:
            got = b.join_blocks(E, Rv, 2, 1.0, 1 << 20, 512, 2, cursor)
            cursor = got["cursor"]
            parts.append(np.stack([got["r"], got["h"], got["t"]], 1))
            if got["code"] == 0:
                break
            assert got["count"] > 0
        got = np.concatenate(parts)
    finally:
        a.close()
        b.close()
    np.testing.assert_array_equal(got[np.lexsort((got[:, 2], got[:, 1], got[:, 0]))], want)
