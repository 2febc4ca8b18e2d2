"""GPU tests of the relation-factorised join over rows that hold a NaN or an infinity: the pairs of the other rows come out as
without them, none of their own is a hit, and none is listed for the exact stage."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

AUTO, OFF, ON = 0, 1, 2


def _case(seed, N, R, d, k, sigma, lone=0):
    g = np.random.default_rng(seed)
    cent = g.standard_normal((k, d))
    E = np.concatenate([cent[g.integers(0, k, N - lone)] + sigma * g.standard_normal((N - lone, d)), g.standard_normal((lone, d))])
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    return E.astype(np.float32), Rv.astype(np.float32)


def _join(E, Rv, p, delta, dtype, prune):
    import paper_2307_12059_amd as kgc
    import torch
    dev = lambda x: torch.from_numpy(x).cuda().to(torch.float32 if dtype == "f32" else torch.bfloat16).contiguous()
    j = kgc.Join(dtype=dtype, prune=prune)
    try:
        got = j.join(dev(E), dev(Rv), p, delta, 1 << 21)
    finally:
        j.close()
    assert got["code"] == 0
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1), got["stats"]


# without and with the row order (a bad row is its first pivot, too), both tile shapes, both norms and types, straight by the default mode
@pytest.mark.parametrize("N,R,d,p,dtype,prune,rows,sigma", [
    (400, 40, 20, 2, "f32", OFF, 50, 0.1), (2000, 60, 40, 2, "bf16", OFF, 50, 0.1), (3000, 40, 300, 2, "f32", OFF, 50, 0.1),
    (4000, 30, 64, 1, "f32", OFF, 50, 0.1), (2000, 8, 32, 2, "f32", AUTO, 50, 0.1), (1500, 30, 40, 1, "bf16", AUTO, 12, 0.05)])
def test_rows_that_are_no_numbers_cost_no_pairs(N, R, d, p, dtype, prune, rows, sigma):
    E, Rv = _case(N + d, N, R, d, N // rows, sigma)
    delta = float(np.float32(sigma * (np.sqrt(2.0 * d) * 0.95 if p == 2 else 1.05 * d)))
    want, st = _join(E, Rv, p, delta, dtype, prune)
    assert st["join_variant"] == 100 and want.shape[0] > 100
    bad = E.copy()
    gone = {0: np.nan, 7: np.inf, N // 2: -np.inf, N - 1: -np.nan}
    for i, (row, v) in enumerate(gone.items()):
        bad[row, (i * d) // 4] = v
    bad[N // 2, d - 1] = np.inf
    got, st2 = _join(bad, Rv, p, delta, dtype, prune)
    keep = ~np.isin(want[:, 1], list(gone)) & ~np.isin(want[:, 2], list(gone))
    assert st2["join_variant"] == 100
    np.testing.assert_array_equal(got, want[keep])
    assert st2["candidates"] <= st["candidates"], (st["candidates"], st2["candidates"])


def test_rows_that_are_no_numbers_in_the_part_without_groups():
    E, Rv = _case(11, 2800, 600, 40, 30, 0.1, lone=1400)
    want, st = _join(E, Rv, 2, 1.0, "f32", ON)
    E[2000, 3] = np.nan
    got, st2 = _join(E, Rv, 2, 1.0, "f32", ON)
    keep = (want[:, 1] != 2000) & (want[:, 2] != 2000)
    np.testing.assert_array_equal(got, want[keep])
