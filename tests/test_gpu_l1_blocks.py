"""GPU tests of pruned L1 joins by pairs of micro-tiles: the same records, bit for bit, as the dense L1 kernel (both score in double
from the caller's rows), with lists that are too short at first, and without a list."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OFF, ON = 1, 2


def _case(seed, N, R, d, rows, dtype):
    import torch
    g = np.random.default_rng(seed)
    k = max(2, N // rows)
    cent = g.standard_normal((k, d))
    E = cent[g.integers(0, k, N)] + 0.1 * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    return (torch.from_numpy(E.astype(np.float32)).cuda().to(tt).contiguous(),
            torch.from_numpy(Rv.astype(np.float32)).cuda().to(tt).contiguous())


def _records(E, Rv, delta, dtype, **cfg):
    import paper_2307_12059_amd as kgc
    j = kgc.Join(dtype=dtype, **cfg)
    try:
        got = j.join(E, Rv, 1, delta, 1 << 22)
    finally:
        j.close()
    assert got["code"] == 0
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1), got["stats"]["exact_blocks"]


# clusters of a micro-tile or less, of several (whole tiles survive), few and many blocks (either side of the line where a
# batch goes back to whole tiles), d at the edges of the 16-dimension slices and odd, rows that start on no vector boundary
@pytest.mark.parametrize("N,R,d,rows,dtype,by_blocks", [(700, 9, 16, 30, "f32", True), (1500, 40, 17, 33, "bf16", True),
                                                        (3000, 20, 100, 200, "f32", True), (4000, 300, 12, 300, "f32", False),
                                                        (2600, 7, 33, 20, "f32", True), (900, 5, 250, 60, "bf16", True)])
def test_blocks_match_the_dense_kernel(N, R, d, rows, dtype, by_blocks, monkeypatch):
    E, Rv = _case(N + d, N, R, d, rows, dtype)
    delta = float(np.float32(0.1 * np.sqrt(2.0) * (0.798 * d - (1.3 if d == 12 else 0.5) * np.sqrt(d))))      # (fewer hits of 27 M aligned pairs)
    want = _records(E, Rv, delta, dtype, prune=OFF, tile_cfg=17)[0]
    assert want.shape[0] > 100
    got, blocks = _records(E, Rv, delta, dtype, prune=ON)
    np.testing.assert_array_equal(got, want)
    assert (blocks > 0) == by_blocks
    monkeypatch.setenv("KGC_EXACT_LIST_CAP", "3")          # both lists grow
    got, grown = _records(E, Rv, delta, dtype, prune=ON)
    np.testing.assert_array_equal(got, want)
    assert (grown > 3) == by_blocks
    monkeypatch.setenv("KGC_PAIR_LIST_LIMIT", "1")         # no list of pairs: whole tiles, scored in place
    got, none = _records(E, Rv, delta, dtype, prune=ON)
    np.testing.assert_array_equal(got, want)
    assert none == 0
