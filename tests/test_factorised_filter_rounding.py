"""The float32 arithmetic of the relation-factorised filter (k_stage_operands, k_fact_dot with fact_params, and level 3 of
k_join_l2_fact in csrc/kgc_kernels.h) against the definition in double.

The filter keeps (h, r, t) when G + 2 r.h~ <= limr + 2 r.t~, with rows rounded to bfloat16, G = ||h~ - t~||^2 less the rows'
rounding slacks, and limr = delta^2 + (bounds of the float32 sums) - ||r||^2.  Rounding may only ever keep more: no triple
within delta may be dropped, however long r is against delta.  The test re-states the kernels' operations in numpy float32
on triples a hair inside delta, and checks that some are dropped once the slacks are left out (so that it can fail)."""
import numpy as np
import pytest

import workloads

F = np.float32


def _bf16(x):
    return workloads.bf16_bits_to_f32(workloads.f32_to_bf16_bits(np.asarray(x, np.float32))).reshape(np.shape(x))


def _sum32(x):
    s = F(0)
    for v in x.astype(np.float32):
        s = F(s + v)
    return s


def _staged(x, delta, slack):
    b = _bf16(x)
    sq, er = _sum32(b * b), _sum32((x - b) * (x - b))
    e = F(F(np.sqrt(er)) * F(1.001) + F(1.2e-7) * F(np.sqrt(sq)))
    nrm = F(sq - F(F(2) * F(delta) * e + F(2) * e * e) * F(1.0001)) if slack else sq
    return b, sq, nrm


def _keeps(h, r, t, delta, max_sq, slack=True):
    d = h.size
    hb, hsq, hn = _staged(h, delta, slack)
    tb, tsq, tn = _staged(t, delta, slack)
    G = F(F(F(hn) + F(tn)) + _sum32(hb * (F(-2) * tb)))
    uh, ut, rn = _sum32(r * hb), _sum32(r * tb), _sum32(r * r)
    ma = mb = F(max(hsq, tsq, max_sq))
    na = nb = F(np.sqrt(ma)) * F(1.01)
    kp = (d + 6 + 31) // 32 * 32
    eacc = F(kp + 16) * F(1.2e-7) * F(2) * (ma + mb)
    eu = F(4) * F(d + 12) * F(6e-8) * (F(np.sqrt(rn)) * F(1.0001)) * (na + nb) + F(2e-6) * (rn + ma + mb)
    thr = F((F(delta) * F(delta) + eacc + eu) * (F(1) + F(1e-6)))
    limr = F(thr - rn)
    return bool(F(G + F(2) * uh) <= F(limr + F(2) * ut))


@pytest.mark.parametrize("d", [10, 100, 602])
def test_no_triple_within_delta_is_dropped(d):
    g = np.random.default_rng(d)
    trials = dropped_without_slack = 0
    for length in (0.0, 1.0, 10.0, 100.0):               # of r against the entities
        for delta in (0.02, 0.3, 3.0):
            for _ in range(30 if d < 600 else 8):
                h = g.standard_normal(d).astype(np.float32)
                r = (length * g.standard_normal(d)).astype(np.float32)
                # x along the sum of the two rows' rounding moves as far as t's can be known before t is: the worst side
                x = (h.astype(np.float64) - _bf16(h)) + 1e-3 * g.standard_normal(d) / 256
                x *= -delta * (1.0 - 1e-7) / np.linalg.norm(x)
                t = (h.astype(np.float64) + r - x).astype(np.float32)
                if np.linalg.norm(h.astype(np.float64) + r - t) > delta:      # rounding t to float32 pushed it out
                    continue
                trials += 1
                assert _keeps(h, r, t, delta, 0.0), (d, length, delta)
                dropped_without_slack += not _keeps(h, r, t, delta, 0.0, slack=False)
    assert trials > 20 and dropped_without_slack > 0


def test_the_length_of_the_relation_does_not_widen_the_filter():
    """Pairs at 1.2 delta of a relation 16 times as long as delta: a margin that holds ||r|| keeps them all."""
    g = np.random.default_rng(1)
    d, delta, kept = 32, 0.5, 0
    for _ in range(200):
        h = g.standard_normal(d).astype(np.float32)
        r = g.standard_normal(d)
        r = (r * (16 * delta / np.linalg.norm(r))).astype(np.float32)
        x = g.standard_normal(d)
        t = (h.astype(np.float64) + r - 1.2 * delta * x / np.linalg.norm(x)).astype(np.float32)
        kept += _keeps(h, r, t, delta, 60.0)
    assert kept == 0
