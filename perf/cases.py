"""The scoring calls whose speed this repository looks after, as a serving program makes them.

A case is one scoring step: the sub-item score tables of a batch of queries (Eq. 4), then the K best items by them
(Eq. 5 and TopK) - over the whole catalogue ("scan"), over a list of candidate items ("subset"), or over a catalogue
whose sub-ids take two bytes ("scan16").  Sizes are those of workloads.CONFIGS and of bench.py's sweeps; draw() gives
more steps of the same ranges.

Keys of a case:
  kind    scan | subset | scan16
  api     "prepared": the program marshalled its buffers once (binding.Prepared*) and only enqueues, as a serving loop
          does; "call": it calls the package's functions, which allocate their results, as in README.md
  N d m b items, embedding width, splits, sub-ids per split;  B K  queries, results per query
  codes   uniform | zipf | dup: sub-ids drawn uniformly; by Zipf(1.1) popularity per split; uniformly with 5 % of the
          rows copied from a lower id (exact ties)
  n order candidates of a subset step, and whether their list is "random" or "ascending"
"""
import math

import torch

import paper_2408_09992_amd as pq
from paper_2408_09992_amd import binding, workloads as W


def _case(name, kind, api, N, d, m, b, B, K, codes="uniform", n=0, order=""):
    return {"name": name, "kind": kind, "api": api, "N": N, "d": d, "m": m, "b": b, "B": B, "K": K, "codes": codes, "n": n, "order": order}


def listed():
    return [
        # the smallest catalogue anyone serves from a GPU: three launches and what the host does around them
        _case("tiny, functions", "scan", "call", 10_000, 64, 4, 256, 1, 10),
        # one user of a Gowalla-sized catalogue in a serving loop: the headline of bench.py
        _case("gowalla, one user", "scan", "prepared", 1_280_000, 512, 8, 256, 1, 10),
        # ... the data set's own (odd) number of items, a first-stage retrieval of 100 for a re-ranker, plain functions
        _case("gowalla, one user, K 100", "scan", "call", 1_271_638, 512, 8, 256, 1, 100),
        # a batch of users collected over a few milliseconds
        _case("gowalla, 64 users", "scan", "prepared", 1_280_000, 512, 8, 256, 64, 10),
        # offline or high-traffic serving: large batches, retrieval depth 100, popular sub-ids
        _case("serving, 1024 users", "scan", "prepared", 1_280_000, 512, 8, 256, 1024, 100, "zipf"),
        # finer codes, a handful of users, items with equal codes
        _case("finer codes, 16 users", "scan", "prepared", 5_000_000, 512, 16, 256, 16, 10, "dup"),
        # tens of millions of items: the stream of codes from memory
        _case("huge, one user", "scan", "prepared", 50_000_000, 512, 8, 256, 1, 10),
        _case("huge, 32 users", "scan", "prepared", 50_000_000, 512, 8, 256, 32, 10),
        # the finest codes of the paper's catalogue sweep, a ragged number of items
        _case("64 splits, one user", "scan", "prepared", 3_000_001, 512, 64, 256, 1, 10),
        # re-scoring the candidates of an earlier stage for four users
        _case("candidates, functions", "subset", "call", 1_280_000, 512, 8, 256, 4, 10, n=50_000, order="random"),
        # codebooks beyond one byte per sub-id: four users of the mid-size catalogue, one of the largest
        _case("wide ids, functions", "scan16", "call", 1_280_000, 512, 8, 1024, 4, 10),
        _case("wide ids, huge", "scan16", "prepared", 50_000_000, 512, 8, 1024, 1, 10),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread evenly over the logarithm."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choices(("scan", "subset", "scan16"), (6, 2, 2))[0]
    api = rng.choice(("prepared", "call"))
    B = 1 if rng.random() < 0.4 else _log_int(rng, 2, 1024)
    K = _log_int(rng, 1, 512)
    codes, n, order = "uniform", 0, ""
    if kind == "scan":
        m = rng.choices((4, 8, 16, 32, 64), (2, 6, 3, 1, 2))[0]
        b = 256
        most = 400_000_000 // m
        codes = rng.choices(("uniform", "zipf", "dup"), (4, 2, 1))[0]
    elif kind == "subset":
        m, b, most = rng.choice((4, 8, 16)), 256, 5_000_000
    else:
        m = rng.choice((4, 8, 16))
        b = _log_int(rng, 257, 32_768 // m)
        most = 400_000_000 // m
    # (no more lookups than the largest listed steps make in their time, whatever path the shape takes)
    lookups = 8.0e9 if m in (8, 16) and kind == "scan" and K <= 128 else 2.5e9
    if kind == "subset":
        N = _log_int(rng, 10_000, most)
        n = _log_int(rng, 1_000, max(1_000, min(N, int(lookups / (4 * B * m)))))
        order = rng.choice(("random", "ascending"))
        K = min(K, n)
    else:
        N = _log_int(rng, 1_000, max(1_000, min(most, int(lookups / (B * m)))))
        K = min(K, N)
    d = rng.choice([x for x in (64, 128, 256, 512) if x // m >= 4])
    return {"kind": kind, "api": api, "N": N, "d": d, "m": m, "b": b, "B": B, "K": K, "codes": codes, "n": n, "order": order}


def _codes(case, seed):
    """The code matrix, drawn on the GPU."""
    N, m, b = case["N"], case["m"], case["b"]
    if case["kind"] == "scan16":
        return W.codes_uniform_u16_device(N, m, b, seed)
    if case["codes"] != "zipf":
        G = W.codes_uniform_device(N, m, b, seed)
        if case["codes"] == "dup":
            g = torch.Generator(device="cuda").manual_seed(seed + 1)
            ids = torch.arange(N, device="cuda")
            src = (torch.rand(N, device="cuda", generator=g) * ids).long()
            take = torch.rand(N, device="cuda", generator=g) < 0.05
            G = G[torch.where(take, src, ids)]
        return G
    # popularity ranks by inverse CDF, then a bijection rank -> sub-id per split
    g = torch.Generator(device="cuda").manual_seed(seed)
    cdf = torch.from_numpy(W.zipf_cdf(b, 1.1)).float().cuda()
    perm = torch.from_numpy(W.zipf_permutations(m, b, seed)).cuda()
    G = torch.empty((N, m), dtype=torch.uint8, device="cuda")
    step = max(1, (1 << 26) // m)
    for lo in range(0, N, step):
        c = min(step, N - lo)
        rank = torch.searchsorted(cdf, torch.rand((c, m), device="cuda", generator=g)).clamp_(max=b - 1)
        G[lo:lo + c] = perm.gather(1, rank.t().contiguous()).t()
    return G


def prepare(case, seed):
    d, m, b, B, K = case["d"], case["m"], case["b"], case["B"], case["K"]
    g = torch.Generator(device="cuda").manual_seed(seed + 2)
    s = {"case": case, "K": K, "codes": _codes(case, seed),
         "centroids": torch.randn((m, b, d // m), device="cuda", generator=g) * d ** -0.5,
         "queries": torch.randn((B, d), device="cuda", generator=g)}
    if case["kind"] == "subset":
        V = torch.randperm(case["N"], device="cuda", generator=g)[:case["n"]].to(torch.int32)
        s["subset"] = V.sort().values.contiguous() if case["order"] == "ascending" else V.contiguous()
    if case["api"] == "prepared":
        s["tables"] = binding.PreparedSubitemScores(s["queries"], s["centroids"])
        S = s["tables"].S
        if case["kind"] == "subset":
            s["topk"] = binding.PreparedScoreTopKSubset(s["codes"], S, s["subset"], K)
        elif case["kind"] == "scan16":
            s["topk"] = binding.PreparedScoreTopKU16(s["codes"], S, K)
        else:
            s["topk"] = binding.PreparedScoreTopK(s["codes"], S, K)
    return s


def run(state):
    if "topk" in state:
        S = state["tables"]()
        ids, scores = state["topk"]()
    else:
        S = pq.pq_subitem_scores(state["queries"], state["centroids"])
        kind = state["case"]["kind"]
        if kind == "subset":
            ids, scores = pq.pq_score_topk_subset(state["codes"], S, state["subset"], state["K"])
        elif kind == "scan16":
            ids, scores = pq.pq_score_topk_u16(state["codes"], S, state["K"])
        else:
            ids, scores = pq.pq_score_topk(state["codes"], S, state["K"])
    return {"S": S, "ids": ids, "scores": scores}


def work(case):
    N, d, m, b, B, K = (case[k] for k in ("N", "d", "m", "b", "B", "K"))
    items = case["n"] if case["kind"] == "subset" else N
    row = m * (2 if case["kind"] == "scan16" else 1) + (4 if case["kind"] == "subset" else 0)
    return {"bytes": items * row + 4 * (B * d + b * d + B * m * b) + 8 * B * K,
            "flops": 2.0 * B * b * d + float(B) * items * (m - 1)}


def tolerance(case):
    # Eq. 4 and Eq. 5 are summed in a stated order and ties go to the lower id: the results are unique, bit for bit
    return "exact"
