"""GPU test: no pruned join loses a pair to the rounding of the coordinates h + r.  Every row of a cluster is the same, its elements
+-12,288, and relations are 5e-4 in every dimension, a little more than half a unit in the last place there: a bound summed in
float32 sees about twice the distance, 64 * 5e-4 (L1) or 8 * 5e-4 (L2)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

AUTO, OFF, ON = 0, 1, 2


# one group of ten micro-tiles (unit bound, refined), groups of two, groups of one (flat bound), and a tile that holds several groups
@pytest.mark.parametrize("p", [1, 2])
@pytest.mark.parametrize("clusters,rows,dtype", [(1, 300, "f32"), (40, 40, "f32"), (30, 20, "f32"), (90, 9, "f32"), (3, 200, "bf16")])
def test_no_pair_is_lost_far_from_the_origin(p, clusters, rows, dtype):
    import paper_2307_12059_amd as kgc
    import torch
    g = np.random.default_rng(clusters)
    d, R = 64, 2
    sign = np.where(g.random((clusters, d)) < 0.5, -1.0, 1.0)
    lab = g.permutation(np.repeat(np.arange(clusters), rows))
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    E = torch.from_numpy((12288.0 * sign[lab]).astype(np.float32)).cuda().to(tt).contiguous()
    Rv = torch.full((R, d), 5e-4, device="cuda").to(tt).contiguous()
    exact = 5e-4 * (64.0 if p == 1 else 8.0)
    for prune in (OFF, ON, AUTO):
        j = kgc.Join(dtype=dtype, prune=prune)
        try:
            got = j.join(E, Rv, p, float(np.float32(1.2 * exact)), 1 << 20)
        finally:
            j.close()
        assert got["code"] == 0
        assert got["count"] == clusters * rows * rows * R, (prune, got["count"])
        assert (lab[got["h"]] == lab[got["t"]]).all()
        np.testing.assert_allclose(got["dist"], exact, rtol=2e-3)       # (bfloat16: 4.997e-4)
