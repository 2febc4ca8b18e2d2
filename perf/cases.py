"""The timed cases of the TransE similarity join: what a program that completes a knowledge graph asks of the library.

Inputs are entity embeddings in clusters and relations that translate one cluster onto another, as trained translation
models have them, drawn on the GPU from the seed.  The sizes are those of the repository's own workloads
(workloads/__init__.py: 2,000 to 1,000,000 entities, 8 to 1,345 relations, 32 to 200 dimensions) and of the model sizes
it names (128 to 512 dimensions).  The threshold is the quantile of the distance of two aligned entities (head in the
relation's source cluster, tail in its target cluster) that gives about the wanted number of hits.

A pass is one call of the public binding plus what its caller does with an unordered result: the records are put into
the order (relation, head, tail) on the GPU.  (The k-best search returns ordered records on the host by itself.)
"""
import math
from statistics import NormalDist

import torch

import paper_2307_12059_amd as kgc

# The largest estimated time of a drawn case, seconds at the matrix / vector rate of a join that prunes nothing: below
# what the largest listed cases take.
_DRAW_LIMIT_S = 0.25


def listed():
    def case(name, op, mode, N, R, d, p, dtype, rows, sigma, share, zipf=0.0, k=0):
        return {"name": name, "op": op, "mode": mode, "N": N, "R": R, "d": d, "p": p, "dtype": dtype, "rows": rows,
                "sigma": sigma, "share": share, "zipf": zipf, "k": k}

    return [
        # the smallest graphs: a call is a chain of short launches, with the default settings and with pruning off
        case("tiny_l2_pruned", "join", "pruned", 2_000, 8, 32, 2, "f32", 100, 0.1, 0.0455),
        case("tiny_l2_dense", "join", "dense", 2_000, 8, 32, 2, "f32", 100, 0.1, 0.0455),
        # a mid-size graph with many relation types: the benchmark's workload, default settings ...
        case("mid_l2_pruned", "join", "pruned", 15_000, 1_345, 100, 2, "f32", 30, 0.15, 0.25),
        # ... every pair scored, as a caller does who does not know the data to be clustered ...
        case("mid_l2_dense", "join", "dense", 15_000, 1_345, 100, 2, "f32", 30, 0.15, 0.25),
        # ... the thousand best triples instead of a threshold ...
        case("mid_l2_top1000", "topk", "pruned", 15_000, 1_345, 100, 2, "f32", 30, 0.15, 0.25, k=1_000),
        # ... and the structured-embedding model (L1, two maps per relation) on such entities
        case("mid_l1_se", "se", "pruned", 15_000, 64, 100, 1, "f32", 30, 0.15, 2e-5),
        # the L1 norm, few relation types
        case("l1_pruned", "join", "pruned", 40_000, 18, 100, 1, "f32", 200, 0.1, 0.04),
        case("l1_dense", "join", "dense", 40_000, 18, 100, 1, "f32", 200, 0.1, 0.04),
        # a large graph in bfloat16
        case("large_l2_pruned", "join", "pruned", 100_000, 200, 200, 2, "bf16", 50, 0.1, 0.4),
        case("large_l2_dense", "join", "dense", 100_000, 200, 200, 2, "bf16", 50, 0.1, 0.4),
        # a million entities whose cluster sizes follow Zipf's law
        case("scale_l2_pruned", "join", "pruned", 1_000_000, 1_000, 128, 2, "bf16", 100, 0.05, 0.1, zipf=1.1),
        # broad clusters, a long dimension and ragged sizes: pruning is on and finds nothing to prune
        case("broad_l2_pruned", "join", "pruned", 20_011, 37, 512, 2, "f32", 40, 0.7, 0.25),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _unpruned_seconds(c):
    """A rough time of the case if no pair can be skipped (which is so with pruning off, with broad clusters, and for
    the part of the entities that sits in clusters of fewer than two dozen)."""
    n = float(c["N"])
    if c["mode"] == "pruned" and c["sigma"] < 0.3 and c["rows"] >= 24:
        n *= 0.15 if c["zipf"] else 0.05
    pairs = n * n * c["R"]
    return pairs * 2.0 * c["d"] / (5e14 if c["p"] == 2 else 3.5e13)


def draw(rng):
    while True:
        op, mode, p = rng.choice([("join", "pruned", 2)] * 8 + [("join", "dense", 2)] * 3 + [("join", "pruned", 1)] * 3 +
                                 [("join", "dense", 1)] * 2 + [("topk", "pruned", 2)] * 2 + [("se", "pruned", 1)] * 2)
        c = {"op": op, "mode": mode, "p": p, "dtype": rng.choice(["f32", "bf16"])}
        if op == "se":
            c["N"], c["R"], c["d"] = _log_uniform(rng, 1_000, 20_000), _log_uniform(rng, 4, 64), _log_uniform(rng, 16, 200)
        else:
            c["N"] = _log_uniform(rng, 500, 400_000 if mode == "pruned" else 100_000)
            c["R"] = _log_uniform(rng, 4, 1_500)
            # half of the models have a round size, the others any
            c["d"] = rng.choice([32, 64, 100, 128, 200, 256, 512]) if rng.random() < 0.5 else _log_uniform(rng, 16, 512)
        c["rows"] = _log_uniform(rng, 8, 250)
        c["sigma"] = 0.7 if op == "join" and rng.random() < 0.2 else round(rng.uniform(0.05, 0.15), 3)
        c["zipf"] = 1.1 if op == "join" and mode == "pruned" and rng.random() < 0.25 else 0.0
        c["share"] = 2e-5 if op == "se" else round(rng.uniform(0.02, 0.4), 3)
        c["k"] = _log_uniform(rng, 10, 5_000) if op == "topk" else 0
        aligned = c["R"] * float(c["rows"]) ** 2
        if op == "topk" and (c["rows"] < 24 or c["k"] > 0.2 * aligned):
            continue
        if c["N"] < 4 * c["rows"] or c["share"] * aligned > 1e6 or c["N"] * float(c["N"]) * c["R"] > 2e14:
            continue
        if _unpruned_seconds(c) <= _DRAW_LIMIT_S:
            return c


def _cluster_labels(c, g):
    n, k = c["N"], max(2, round(c["N"] / c["rows"]))
    if not c["zipf"]:
        return torch.randint(0, k, (n,), generator=g, device="cuda"), k
    w = torch.arange(1, k + 1, dtype=torch.float64, device="cuda") ** -c["zipf"]
    sizes = (w / w.sum() * n).floor().clamp_(min=1).long()
    short = n - int(sizes.sum())
    sizes[0] += short                                    # the rounding remainder (of either sign) goes to the largest
    labels = torch.repeat_interleave(torch.arange(k, device="cuda"), sizes)
    return labels[torch.randperm(n, generator=g, device="cuda")], k


def _threshold(c, s, q):
    """The q-quantile of the L_p norm of d independent normal deviates of standard deviation s."""
    z, d = NormalDist().inv_cdf(q), c["d"]
    if c["p"] == 2:                                      # Wilson and Hilferty's approximation of the chi-square quantile
        return s * math.sqrt(d * max(1e-3, 1.0 - 2.0 / (9.0 * d) + z * math.sqrt(2.0 / (9.0 * d))) ** 3)
    return s * (math.sqrt(2.0 / math.pi) * d + z * math.sqrt((1.0 - 2.0 / math.pi) * d))


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda").manual_seed(seed)
    dtype = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    N, R, d, sigma = c["N"], c["R"], c["d"], c["sigma"]
    labels, k = _cluster_labels(c, g)
    centres = torch.randn((k, d), generator=g, device="cuda")
    E = (centres[labels] + sigma * torch.randn((N, d), generator=g, device="cuda")).to(dtype)
    state = {"case": c, "E": E}
    sizes = torch.bincount(labels, minlength=k).double()
    wanted = c["share"] * R * float(c["rows"]) ** 2
    if c["op"] == "se":
        # maps near the identity: both sides of an aligned pair lie in one cluster
        noise = 0.03 / math.sqrt(d)
        eye = torch.eye(d, device="cuda")
        state["W_lhs"] = (eye + noise * torch.randn((R, d, d), generator=g, device="cuda")).to(dtype).contiguous()
        state["W_rhs"] = (eye + noise * torch.randn((R, d, d), generator=g, device="cuda")).to(dtype).contiguous()
        aligned = R * float(N) * c["rows"]
        s = math.sqrt(2.0 * sigma * sigma + 2.0 * 0.03 * 0.03 * (1.0 + sigma * sigma))
        wanted = N * R + c["share"] * aligned            # (maps this close keep every entity near itself)
    else:
        src = torch.randint(0, k, (R,), generator=g, device="cuda")
        dst = (src + torch.randint(1, k, (R,), generator=g, device="cuda")) % k
        state["Rv"] = (centres[dst] - centres[src] + 0.02 * torch.randn((R, d), generator=g, device="cuda")).to(dtype)
        aligned = float((sizes[src] * sizes[dst]).sum())
        s = math.sqrt(2.0 * sigma * sigma + 0.02 * 0.02)
    q = c["share"] if c["op"] == "se" else wanted / max(1.0, aligned)
    state["delta"] = _threshold(c, s, min(0.5, max(1e-9, q)))
    # the table the caller collects a result in, in order; rows past the result hold -1
    state["cap"] = int(2 * wanted) + 16_384
    state["table"] = torch.empty((state["cap"], 4), dtype=torch.int32, device="cuda")
    state["out"] = torch.empty_like(state["table"])
    state["join"] = kgc.Join(dtype=c["dtype"], prune=kgc.KGC_PRUNE_OFF if c["mode"] == "dense" else kgc.KGC_PRUNE_AUTO)
    return state


def run(state):
    c, join = state["case"], state["join"]
    if c["op"] == "topk":
        return join.topk(state["E"], state["Rv"], c["p"], c["k"])
    if c["op"] == "se":
        got = join.join_se(state["E"], state["W_lhs"], state["W_rhs"], c["p"], state["delta"], state["cap"], fetch=False)
    else:
        got = join.join(state["E"], state["Rv"], c["p"], state["delta"], state["cap"], out=state["out"], fetch=False)
    count = min(got["count"], state["cap"])
    records, table = got["out"][:count], state["table"]
    # a record is h, r, t, dist: as two 64-bit words, (r, h) is the first of them and t the low half of the second
    words = records.view(torch.int64)
    key = torch.add(words[:, 1] & 0xFFFFF, words[:, 0], alpha=1 << 20)
    torch.index_select(records, 0, torch.argsort(key), out=table[:count])
    table[count:].fill_(-1)
    return {"count": got["count"], "triples": table[:, :3], "dist": table[:, 3].view(torch.float32)}


def work(case):
    c = case
    N, R, d, size = float(c["N"]), float(c["R"]), c["d"], 4 if c["dtype"] == "f32" else 2
    hits = c["share"] * R * float(c["rows"]) ** 2 if c["op"] != "se" else R * N
    if c["op"] == "topk":
        hits = c["k"]
    maps = 2.0 * R * d * d if c["op"] == "se" else R * d
    # every input once, every record once; the exact score of every hit
    need = {"bytes": (N * d + maps) * size + 16.0 * hits, "flops": 3.0 * d * hits + N * d}
    if c["op"] == "se":
        need["flops"] += 2.0 * 2.0 * R * N * d * d          # the connectors
    if c["mode"] == "dense":
        # L2: one contraction over the dimensions per pair, and two additions and a comparison for every relation of it;
        # L1: a subtraction and an addition per dimension of every triple
        need["flops"] += 2.0 * N * N * d + 3.0 * N * N * R if c["p"] == 2 else 2.0 * N * N * R * d
    return need


def tolerance(case):
    # The set of triples is decided in double precision and is the same for every correct implementation.  Distances
    # are float32 roundings of doubles (or roots of such roundings): one unit in the last place either way.
    return {"rel": 2.5e-7, "max": 5e-7}
