"""GPU tests of the two lists of a pruned L1 join by 32 x 32 blocks, through all three entry points: lists that are too short grow, a
list that cannot be had is done without, more blocks than the list may hold leave the batch to whole tiles; the records are the same
each time, and the statistics say which way a call went (exact_blocks: blocks that were summed one by one, 0 with whole tiles)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OFF, ON = 1, 2
ENVS = ("KGC_EXACT_LIST_CAP", "KGC_PAIR_LIST_LIMIT", "KGC_BLOCK_LIST_LIMIT", "KGC_BLOCK_LIST_MAX")


def _call(kind, d=24, N=1600, R=5):
    """(join handle) -> sorted records and statistics of one call over clusters of 25 rows"""
    import torch
    g = np.random.default_rng(len(kind))
    k = N // 25
    cent = g.standard_normal((k, d))
    E = cent[g.integers(0, k, N)] + 0.1 * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    W = [np.eye(d) + 0.03 / np.sqrt(d) * g.standard_normal((R, d, d)) for _ in range(2)]
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda()
    delta, cap = float(np.float32(0.1 * 1.128 * d * 0.85)), 1 << 20
    A = E[None] + Rv[:, None]
    args = {"join": (dev(E), dev(Rv)), "ab_shared": (dev(A), dev(E)), "ab": (dev(A), dev(E[None] @ W[1].transpose(0, 2, 1))),
            "se": (dev(E), dev(W[0]), dev(W[1]))}[kind]

    def run(j):
        fn = {"join": j.join, "se": j.join_se}.get(kind, j.join_ab)
        got = fn(*args, 1, delta, cap)
        assert got["code"] == 0
        o = np.lexsort((got["t"], got["h"], got["r"]))
        return np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1), got["stats"]
    return run


# the environment of the handle, and whether blocks are summed one by one
@pytest.mark.parametrize("kind", ["join", "ab_shared", "ab", "se"])
@pytest.mark.parametrize("env,by_blocks", [({}, True), ({"KGC_EXACT_LIST_CAP": "3"}, True),                       # both lists grow
                                           ({"KGC_PAIR_LIST_LIMIT": "1"}, False),                                 # no list of pairs ...
                                           ({"KGC_EXACT_LIST_CAP": "3", "KGC_PAIR_LIST_LIMIT": "60"}, False),     # ... or none of the length it needs
                                           ({"KGC_BLOCK_LIST_LIMIT": "1"}, False),                                # the same of the blocks
                                           ({"KGC_EXACT_LIST_CAP": "3", "KGC_BLOCK_LIST_LIMIT": "60"}, False),
                                           ({"KGC_BLOCK_LIST_MAX": "3"}, False)])                                 # more blocks than may be listed
def test_lists_of_pruned_l1_joins(kind, env, by_blocks, monkeypatch):
    import paper_2307_12059_amd as kgc
    run = _call(kind)
    ref = kgc.Join(prune=OFF, tile_cfg=17 if kind == "join" else 0)
    for e in ENVS:
        monkeypatch.delenv(e, raising=False)
    for e, v in env.items():
        monkeypatch.setenv(e, v)
    j = kgc.Join(prune=ON)
    try:
        want = run(ref)[0]
        assert want.shape[0] > 300
        for _ in range(2):                                 # (the second call starts with what the first has left on the handle)
            got, st = run(j)
            np.testing.assert_array_equal(got, want)
            assert (st["exact_blocks"] > 0) == by_blocks, st["exact_blocks"]
    finally:
        ref.close()
        j.close()


# Clusters of a dozen rows form no groups: micro-tiles of strangers, all of whose blocks are within reach.  Few rows of tiles (each dealt
# to several waves) and many; a batch small enough for blocks whatever they are
@pytest.mark.parametrize("N,R,d,by_blocks", [(6000, 6, 20, False), (3000, 120, 33, False), (700, 20, 16, True)])
def test_batches_whose_blocks_are_mostly_within_reach(N, R, d, by_blocks):
    import paper_2307_12059_amd as kgc
    import torch
    g = np.random.default_rng(N)
    k = N // 12
    cent = g.standard_normal((k, d))
    src = g.integers(0, k, R)
    E = torch.from_numpy((cent[g.integers(0, k, N)] + 0.1 * g.standard_normal((N, d))).astype(np.float32)).cuda()
    Rv = torch.from_numpy((cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src]).astype(np.float32)).cuda()
    delta = float(np.float32(0.1 * 1.128 * d))
    out = []
    for cfg in (dict(prune=OFF, tile_cfg=17), dict(prune=ON)):
        j = kgc.Join(**cfg)
        try:
            got = j.join(E, Rv, 1, delta, 1 << 20)
        finally:
            j.close()
        assert got["code"] == 0
        o = np.lexsort((got["t"], got["h"], got["r"]))
        out.append(np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1))
    assert out[0].shape[0] > 50 and (got["stats"]["exact_blocks"] > 0) == by_blocks, got["stats"]
    np.testing.assert_array_equal(out[1], out[0])


def test_a_call_of_many_tiles_goes_by_blocks():
    """16 blocks a tile times all its tiles is more than 32 bits count: the call goes by blocks all the same, batch by batch.  Its
    first and last relations are compared with the dense kernel."""
    import paper_2307_12059_amd as kgc
    import torch
    g = np.random.default_rng(3)
    N, R, d, k = 60_000, 1_300, 8, 2_000
    cent = 4.0 * g.standard_normal((k, d))
    E = torch.from_numpy((cent[g.permutation(np.repeat(np.arange(k), N // k))] + 0.03 * g.standard_normal((N, d))).astype(np.float32)).cuda()
    src = g.integers(0, k, R)
    Rv = torch.from_numpy((cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src]).astype(np.float32)).cuda()
    delta = float(np.float32(0.3))
    recs = []
    for cfg, ranges in ((dict(prune=ON), [None]), (dict(prune=OFF, tile_cfg=17), [(0, 3), (R - 3, R)])):
        j = kgc.Join(**cfg)
        try:
            parts = []
            for rr in ranges:
                got = j.join(E, Rv, 1, delta, 1 << 22, r_range=rr)
                assert got["code"] == 0
                parts.append(np.stack([got["r"], got["h"], got["t"], got["dist"].view(np.int32)], 1))
                if rr is None:
                    assert got["stats"]["tiles_total"] * 16 > 4e9 and got["stats"]["exact_blocks"] > 0, str(got["stats"])
        finally:
            j.close()
        x = np.concatenate(parts)
        x = x[(x[:, 0] < 3) | (x[:, 0] >= R - 3)]
        recs.append(x[np.lexsort((x[:, 2], x[:, 1], x[:, 0]))])
    assert recs[1].shape[0] > 100
    np.testing.assert_array_equal(recs[0], recs[1])
