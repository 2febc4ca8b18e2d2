"""GPU tests of the L1 joins: the dense one that takes the relation-factorised kernel first (||x||_2 <= ||x||_1), and the
L1 kernel that leaves a tile's dimensions out once they decide nothing, against the double-precision oracle."""
import numpy as np
import pytest

import oracle
import workloads
from tests import parity

pytestmark = pytest.mark.gpu

PRUNE_OFF, PRUNE_ON = 1, 2


def _case(seed, N, R, d, k, sigma, dtype):
    g = np.random.default_rng(seed)
    cent = g.standard_normal((k, d))
    E = cent[g.integers(0, k, N)] + sigma * g.standard_normal((N, d))
    src = g.integers(0, k, R)
    Rv = cent[(src + 1 + g.integers(0, k - 1, R)) % k] - cent[src] + 0.02 * g.standard_normal((R, d))
    E, Rv = E.astype(np.float32), Rv.astype(np.float32)
    if dtype == "bf16":
        E = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(E)).reshape(E.shape)
        Rv = workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(Rv)).reshape(Rv.shape)
    return E, Rv


def _join(E, Rv, delta, cap, dtype, **cfg):
    import torch
    import paper_2307_12059_amd as kgc
    tt = torch.float32 if dtype == "f32" else torch.bfloat16
    j = kgc.Join(dtype=dtype, **cfg)
    try:
        return j.join(torch.from_numpy(E).cuda().to(tt).contiguous(), torch.from_numpy(Rv).cuda().to(tt).contiguous(), 1, delta, cap)
    finally:
        j.close()


# d around the 16-dimension slices, N around the 128-row tiles; broad clusters (nothing ends early), narrow ones (most
# tiles end after a slice or two, with few and with many pairs of a wave left)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("prune", [PRUNE_OFF, PRUNE_ON])
@pytest.mark.parametrize("N,R,d,k,sigma", [(1, 1, 1, 2, 0.1), (127, 3, 15, 4, 0.1), (129, 2, 16, 40, 0.3), (257, 3, 17, 60, 0.1),
                                           (700, 3, 100, 200, 0.1), (640, 2, 130, 8, 0.1), (300, 2, 33, 5, 0.8)])
def test_kernel_matches_the_oracle(N, R, d, k, sigma, prune, dtype):
    E, Rv = _case(N + d, N, R, d, k, sigma, dtype)
    for q in (0.25, 0.9):
        delta = float(np.float32(sigma * np.sqrt(2.0) * 0.8 * d * (0.6 + 0.5 * q)))
        ref = oracle.join(E, Rv, 1, delta, mode="brute")
        got = _join(E, Rv, delta, max(1024, 2 * ref["count"]), dtype, prune=prune)
        assert got["code"] == 0
        rep = parity.compare(got, ref, E, Rv, 1, delta, N)
        assert rep["only_gpu_in_band"] == 0 and rep["only_oracle_in_band"] == 0


def _records(got):
    assert got["code"] == 0
    o = np.lexsort((got["t"], got["h"], got["r"]))
    return np.stack([got["r"][o], got["h"][o], got["t"][o], got["dist"][o].view(np.int32)], 1)


# the dense join on the factorised kernel (join_variant 100) and, where L2 within delta rules too little out, on the L1
# kernel after all (0): the same records as the L1 kernel's.  d on both sides of the tile shapes' limit (282) and past
# the last (602)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,R,d,sigma,variant", [(5000, 9, 32, 0.1, 100), (1300, 70, 100, 0.1, 100), (3001, 3, 283, 0.05, 100),
                                                 (3500, 10, 65, 0.8, 0), (1100, 12, 300, 0.5, 0), (1500, 3, 603, 0.05, 0)])
def test_dense_takes_the_factorised_kernel_first(N, R, d, sigma, variant, dtype):
    E, Rv = _case(N + R, N, R, d, 60, sigma, dtype)      # (aligned pairs: one in 3,600, fewer than a list may hold)
    delta = float(np.float32(sigma * np.sqrt(2.0) * (0.798 * d - 0.603 * np.sqrt(d))))      # a sixth of the aligned pairs
    cap = 1 << 22
    a = _join(E, Rv, delta, cap, dtype, prune=PRUNE_OFF)
    b = _join(E, Rv, delta, cap, dtype, prune=PRUNE_OFF, tile_cfg=17)
    assert a["stats"]["join_variant"] == variant and b["stats"]["join_variant"] == 0
    assert b["count"] > 20
    want = _records(b)
    np.testing.assert_array_equal(_records(a), want)
    picks = np.random.default_rng(1).choice(want.shape[0], 20)
    r, h, t = want[picks, 0], want[picks, 1], want[picks, 2]
    ref = np.abs((E[h].astype(np.float64) + Rv[r]) - E[t]).sum(1)
    np.testing.assert_allclose(want[picks, 3].view(np.float32), ref, rtol=2.0 ** -23)      # a rounding to float32


# the line below which few rows under many relations stay with the L1 kernel
@pytest.mark.parametrize("N,variant", [(999, 0), (1000, 100)])
def test_few_rows_stay_with_the_l1_kernel(N, variant):
    E, Rv = _case(N, N, 400, 32, 120, 0.05, "f32")
    delta = float(np.float32(0.05 * np.sqrt(2.0) * 0.798 * 32))
    got = _join(E, Rv, delta, 1 << 22, "f32", prune=PRUNE_OFF)
    want = _join(E, Rv, delta, 1 << 22, "f32", prune=PRUNE_OFF, tile_cfg=17)
    assert got["stats"]["join_variant"] == variant and want["stats"]["join_variant"] == 0
    assert want["count"] > 1000
    np.testing.assert_array_equal(_records(got), _records(want))
