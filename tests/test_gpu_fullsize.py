"""Full-size parity on the benchmark workloads, in the launch configuration bench.py times.

The oracle cannot brute-force 3e11 .. 1e15 triples inside a test, so these checks use what holds at any size:
  (1) no false positives: every emitted triple is re-scored by the oracle, one by one, and must qualify
      (outside the 1e-4 * delta band) with the reported distance;
  (2) recall on a sample: the join restricted to a subset of entities and relations equals the full result
      filtered to that subset (restriction invariant), so a brute-force oracle run on a seeded
      cluster-aligned subsample -- whole clusters and the relations that link them, so hits exist -- is
      compared with the filtered GPU output, set against set;
  (3) each triple at most once; count == number of records; pruning on and off give the same set;
  (4) where tests/golden/oracle_counts.json holds the full oracle result (written by oracle/make_counts.py with
      the early-abandon mode, which is pinned to brute force): the whole GPU set, with the listed boundary-band
      triples removed, must hash to the stored digest -- bit-exact equality of the full-size result sets.
"""
import hashlib
import json
import os

import numpy as np
import pytest

import oracle
import workloads
from tests import parity

pytestmark = pytest.mark.gpu

COUNTS = os.path.join(os.path.dirname(__file__), "golden", "oracle_counts.json")


def _stored_count(name):
    if not os.path.exists(COUNTS):
        return None
    with open(COUNTS) as f:
        return json.load(f).get(name)


def _gpu_join(wl, prune, cap, tile_cfg=0):
    import torch

    import paper_2307_12059_amd as kgc
    spec = wl.spec
    if spec.storage == "bf16":
        E = torch.from_numpy(wl.E_bits.view(np.int16)).cuda().view(torch.bfloat16)
        Rv = torch.from_numpy(wl.Rv_bits.view(np.int16)).cuda().view(torch.bfloat16)
    else:
        E = torch.from_numpy(wl.E).cuda(); Rv = torch.from_numpy(wl.Rv).cuda()
    j = kgc.Join(dtype=spec.storage, prune=prune, tile_cfg=tile_cfg)
    try:
        return j.join(E, Rv, spec.p, wl.delta, cap)
    finally:
        j.close()


def _fullsize_checks(name, n_rel, max_entities, modes):
    import paper_2307_12059_amd as kgc
    wl = workloads.generate(name)
    spec = wl.spec
    N = spec.N
    cap = int(6 * spec.selectivity * spec.n_triples) + 4096
    results = {}
    for mode in modes:
        # dense: the kernel that scores every relation's pairs, by number (any number keeps an L1 join on the L1 kernel);
        # factorised: what a join with pruning off takes by itself at these sizes
        prune = {"dense": kgc.KGC_PRUNE_OFF, "prune": kgc.KGC_PRUNE_ON, "factorised": kgc.KGC_PRUNE_OFF}[mode]
        print(f"[{name}] running GPU join, mode={mode}", flush=True)
        got = _gpu_join(wl, prune, cap, tile_cfg=18 if mode == "dense" else 0)
        if mode != "prune":
            assert got["stats"]["join_variant"] == (100 if mode == "factorised" else 18 if spec.p == 2 else 0)
        assert got["code"] == 0, f"overflow: count {got['count']} > cap {cap}"
        key = (got["r"].astype(np.int64) * N + got["h"]) * N + got["t"]
        assert np.unique(key).size == key.size == got["count"]
        # (1) every emitted triple, re-scored by the oracle
        dref = oracle.dist_triples(wl.E, wl.Rv, spec.p, got["h"], got["r"], got["t"])
        band = np.abs(dref - wl.delta) <= parity.BAND * wl.delta
        assert np.all((dref <= wl.delta) | band), "GPU emitted a triple the oracle rejects"
        np.testing.assert_allclose(got["dist"], dref, rtol=parity.DIST_RTOL, atol=parity.DIST_ATOL)
        results[mode] = (got, np.sort(key), int(band.sum()))
        print(f"[{name}] mode={mode}: {got['count']} triples, {int(band.sum())} in the band, stats {got['stats']}", flush=True)
    # (3) modes agree
    keys = [v[1] for v in results.values()]
    for k in keys[1:]:
        assert np.array_equal(keys[0], k), "pruned and dense runs returned different sets"
    got = next(iter(results.values()))[0]
    # (2) recall on a cluster-aligned subsample, brute force
    ent, rel = workloads.cluster_aligned_subsample(wl, n_rel, max_entities, spec.seed + 900)
    sub = oracle.join(wl.E[ent], wl.Rv[rel], spec.p, wl.delta, mode="brute")
    ref = {"h": ent[sub["h"]], "r": rel[sub["r"]], "t": ent[sub["t"]], "dist": sub["dist"]}
    m = np.isin(got["h"], ent) & np.isin(got["t"], ent) & np.isin(got["r"], rel)
    gsub = {k: got[k][m] for k in ("h", "r", "t", "dist")}
    rep = parity.compare(gsub, ref, wl.E, wl.Rv, spec.p, wl.delta, N)
    print(f"[{name}] subsample {ent.size} entities x {rel.size} relations: {rep}", flush=True)
    assert rep["oracle_count"] > 0, "vacuous subsample"
    # (4) stored full result: exact set equality outside the band
    stored = _stored_count(name)
    if stored is not None:
        band = {(r * N + h) * N + t for r, h, t in stored["band"]}
        keys = next(iter(results.values()))[1]
        keep = np.array([k not in band for k in keys.tolist()], dtype=bool) if band else np.ones(keys.size, bool)
        dig = hashlib.sha256(np.sort(keys[keep]).astype("<i8").tobytes()).hexdigest()
        assert dig == stored["digest_no_band"], "full-size GPU set differs from the oracle set outside the band"
        assert abs(got["count"] - stored["count"]) <= len(band)
        print(f"[{name}] full set equals the oracle set: {stored['count']} triples, {len(band)} in the band", flush=True)
    else:
        print(f"[{name}] no stored full oracle result: full-set equality not checked (subsample recall only)", flush=True)
    return results


def test_c2_mid_l2_fullsize():
    _fullsize_checks("c2_mid_l2", n_rel=12, max_entities=3000, modes=["dense", "prune", "factorised"])


def test_c3_l1_fullsize():
    _fullsize_checks("c3_l1", n_rel=6, max_entities=3000, modes=["dense", "prune", "factorised"])


def test_c4_large_l2_fullsize():
    # dense here is the 2e12-triple launch the matrix pipes' figure is quoted on (0.65 s)
    _fullsize_checks("c4_large_l2", n_rel=12, max_entities=3000, modes=["prune", "dense", "factorised"])


def test_c5_scale_l2_fullsize():
    # 10^15 triples: pruned mode only; recall is verified on the subsample only, precision on every emitted triple
    _fullsize_checks("c5_scale_l2", n_rel=10, max_entities=5000, modes=["prune"])


@pytest.mark.parametrize("name", ["c2_mid_l2", "c4_large_l2"])
def test_top1_fullsize(name):
    """Top-1 at full size: it must be the smallest distance of the (oracle-verified) join result at the stored
    threshold, which is known to be non-empty, and its triple must attain it in the oracle's arithmetic."""
    import time

    import torch

    import paper_2307_12059_amd as kgc
    wl = workloads.generate(name)
    spec = wl.spec
    if spec.storage == "bf16":
        E = torch.from_numpy(wl.E_bits.view(np.int16)).cuda().view(torch.bfloat16)
        Rv = torch.from_numpy(wl.Rv_bits.view(np.int16)).cuda().view(torch.bfloat16)
    else:
        E = torch.from_numpy(wl.E).cuda(); Rv = torch.from_numpy(wl.Rv).cuda()
    j = kgc.Join(dtype=spec.storage, prune=kgc.KGC_PRUNE_ON)
    try:
        full = j.join(E, Rv, spec.p, wl.delta, int(6 * spec.selectivity * spec.n_triples) + 4096)
        for excl in (False, True):
            t0 = time.perf_counter()
            got = j.top1(E, Rv, spec.p, excl)
            ms = (time.perf_counter() - t0) * 1e3
            m = (full["h"] != full["t"]) if excl else np.ones(full["h"].size, bool)
            assert m.any()
            dref = oracle.dist_triples(wl.E, wl.Rv, spec.p, full["h"][m], full["r"][m], full["t"][m])
            best = float(dref.min())
            dg = oracle.dist_triples(wl.E, wl.Rv, spec.p, [got["h"]], [got["r"]], [got["t"]])[0]
            print(f"[{name}] top-1 exclude_self={excl}: {got} in {ms:.1f} ms; oracle min over the join result {best:.7f}", flush=True)
            assert abs(dg - best) <= 1e-6 * best and abs(got["dist"] - best) <= 1e-6 * best
            assert not excl or got["h"] != got["t"]
        # top-k: the k smallest of the oracle-verified join result (which holds far more than k triples)
        k = 1000
        dall = np.sort(oracle.dist_triples(wl.E, wl.Rv, spec.p, full["h"], full["r"], full["t"]))
        t0 = time.perf_counter()
        tk = j.topk(E, Rv, spec.p, k)
        ms = (time.perf_counter() - t0) * 1e3
        print(f"[{name}] top-{k} in {ms:.1f} ms; largest of them {tk['dist'][-1]:.6f}", flush=True)
        assert tk["count"] == k
        dk = np.sort(oracle.dist_triples(wl.E, wl.Rv, spec.p, tk["h"], tk["r"], tk["t"]))
        assert np.allclose(dk, dall[:k], rtol=1e-6)
        key = (tk["r"].astype(np.int64) * spec.N + tk["h"]) * spec.N + tk["t"]
        assert np.unique(key).size == k
    finally:
        j.close()


def test_general_form_fullsize_c3():
    """kgc_join_ab on the TransE connectors of the L1 workload at full size (pruned): the same set as kgc_join, except for
    triples the float32 rounding of A = E + Rv moves across the threshold, which must lie in the boundary band."""
    import torch

    import paper_2307_12059_amd as kgc
    wl = workloads.generate("c3_l1")
    spec = wl.spec
    E = torch.from_numpy(wl.E).cuda(); Rv = torch.from_numpy(wl.Rv).cuda()
    A = (E.unsqueeze(0) + Rv.unsqueeze(1)).contiguous()
    cap = int(6 * spec.selectivity * spec.n_triples) + 4096
    j = kgc.Join(prune=kgc.KGC_PRUNE_ON)
    try:
        base = j.join(E, Rv, spec.p, wl.delta, cap)
        got = j.join_ab(A, E, spec.p, wl.delta, cap)
    finally:
        j.close()
    assert got["code"] == 0 and got["stats"]["tiles_pruned"] > 0.99 * got["stats"]["tiles_total"]
    N = spec.N
    kb = (base["r"].astype(np.int64) * N + base["h"]) * N + base["t"]
    kg = (got["r"].astype(np.int64) * N + got["h"]) * N + got["t"]
    assert np.unique(kg).size == kg.size
    diff = np.concatenate([np.setdiff1d(kb, kg), np.setdiff1d(kg, kb)])
    print(f"[c3_l1] general form: {got['count']} triples, {diff.size} differ from kgc_join", flush=True)
    if diff.size:
        r, rem = np.divmod(diff, N * N)
        h, t = np.divmod(rem, N)
        dref = oracle.dist_triples(wl.E, wl.Rv, spec.p, h.astype(np.int32), r.astype(np.int32), t.astype(np.int32))
        assert np.all(np.abs(dref - wl.delta) <= parity.BAND * wl.delta)
    # distances of the common triples against the oracle on the connectors the join saw
    Ah = (wl.E[got["h"][:2000]] + wl.Rv[got["r"][:2000]]).astype(np.float32).astype(np.float64)
    dab = np.abs(Ah - wl.E[got["t"][:2000]].astype(np.float64)).sum(-1)
    np.testing.assert_allclose(got["dist"][:2000], dab, rtol=parity.DIST_RTOL)
