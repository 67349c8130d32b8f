"""What the performance of this library is measured on: whole calls through the Python binding.

A case is a dict of plain values.  `kind` says which calls it makes:

    bucket  legend_train_bucket on one edge bucket (waits for the loss), then the node and relation embeddings are read
    epoch   legend_train_epoch over every bucket, then the same reads
    score   legend_score_edges of a list of test edges
    rank    legend_rank_edges of test triples against all nodes or one sampled candidate list

The training configurations are those of `workloads/graphs.py` (d, B, C, N, degree-weighted negatives, score, sides,
relation count, degree skew) and of the tests (losses, dimensions, ragged sizes).  Graphs are smaller than the
configurations' where the whole embedding table would take longer to read back than to train: what one batch costs
depends on its own sizes and on whether a row is touched once or often, and the large cases keep about as many table
rows as a batch has negatives.  Embeddings start at a standard deviation of 0.3, the size they have once training is
under way, through the library's own seeded fill; every pass of a training case trains the next epoch on the tables
the pass before left, as a training program does.  The learning rate is that of a run's later part: no time depends on
it, but Adagrad's first step on a row is the sign of its gradient times this rate, so that a gradient of zero within
rounding moves an element by twice the rate between two correct programs.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2505_09258_amd import binding as L

INIT_STD = 0.3
NODE_TAG, RELATION_TAG = 0x6E6F6465, 0x72656C73    # of the seeded fill
LEARNING_RATE = 0.02
SCORES = {"dot": L.SCORE_DOT, "distmult": L.SCORE_DISTMULT, "complex": L.SCORE_COMPLEX, "transe": L.SCORE_TRANSE_L1}
LOSSES = {"softmax": L.LOSS_SOFTMAX, "logistic": L.LOSS_LOGISTIC, "softmax_pos": L.LOSS_SOFTMAX_POS, "margin": L.LOSS_MARGIN}
SIDES = {"dst": L.CORRUPT_DST, "src": L.CORRUPT_SRC, "both": L.CORRUPT_BOTH}


def _train(name, kind, nodes, relations, edges, dim, batch, chunk, negs, *, degree_negs=0, score="dot", loss="softmax",
           sides="dst", partitions=1, capacity=0, skew=1.0, skew_q=34.0, edges_on="device"):
    """capacity 0: every partition is resident.  skew, skew_q: a node of rank x is an endpoint with density (x + q)^-s."""
    return dict(name=name, kind=kind, nodes=nodes, relations=relations, edges=edges, dim=dim, batch=batch, chunk=chunk,
                negs=negs, degree_negs=degree_negs, score=score, loss=loss, sides=sides, partitions=partitions,
                capacity=capacity, skew=skew, skew_q=skew_q, edges_on=edges_on)


def _test(name, kind, nodes, relations, dim, triples, *, candidates=0, score="dot", side="dst", partitions=1):
    """candidates 0: every node (kind rank)."""
    return dict(name=name, kind=kind, nodes=nodes, relations=relations, dim=dim, triples=triples, candidates=candidates,
                score=score, sides=side, partitions=partitions)


def listed():
    return [
        # the tiny configuration (c1), one batch per call: a program that follows the loss batch by batch; all latency
        _train("tiny_one_batch", "bucket", 10_000, 0, 1_000, 32, 1_000, 100, 64, skew=1.1, skew_q=1.0),
        # the tiny configuration, one whole epoch from edges in host memory: a hundred small batches
        _train("tiny_epoch", "epoch", 10_000, 0, 100_000, 32, 1_000, 100, 64, skew=1.1, skew_q=1.0, edges_on="host"),
        # the large social configuration (c4), the headline workload: many negatives, nearly all rows touched once per batch
        _train("social_dot", "bucket", 1_000_000, 0, 5_000_000, 100, 50_000, 50, 1_000),
        # the middle social configuration (c2): degree-weighted negatives, staged through the three-slot buffer; ragged buckets
        _train("social_staged_epoch", "epoch", 400_000, 0, 2_000_000, 100, 50_000, 50, 1_000, degree_negs=500,
               partitions=4, capacity=3, skew=0.91, skew_q=100.0),
        # the large knowledge-graph configuration (c5): ComplEx, both sides corrupted, many relations
        _train("knowledge_complex", "bucket", 1_000_000, 14_824, 2_000_000, 100, 50_000, 50, 1_000, score="complex",
               sides="both", skew=0.8, skew_q=1.0),
        # the small knowledge-graph configuration (c3): wide rows, a table smaller than a batch, one whole epoch
        _train("fb15k_distmult_d400", "bucket", 15_000, 1_345, 483_000, 400, 10_000, 100, 1_000, score="distmult",
               sides="both", skew=0.7, skew_q=1.0),
        # a point of the dimension sweep on the same graph: rows of 200 bytes, batches of 50 000
        _train("fb15k_complex_d50", "bucket", 15_000, 1_345, 483_000, 50, 50_000, 100, 1_000, score="complex",
               sides="both", skew=0.7, skew_q=1.0),
        # logistic loss, the widest rows of the fused kernel, odd batch and chunk sizes, an off-diagonal bucket
        _train("logistic_distmult_d128", "bucket", 120_001, 37, 301_000, 128, 20_011, 61, 333, degree_negs=33,
               score="distmult", loss="logistic", partitions=2, skew=0.7, skew_q=1.0),
        # the translational score on the social shape with one relation (the benchmark's --score transe)
        _train("social_transe", "bucket", 120_000, 1, 300_000, 100, 50_000, 50, 1_000, degree_negs=500, score="transe",
               skew=0.91, skew_q=100.0),
        # scoring a million test edges
        _test("score_million", "score", 1_000_000, 0, 100, 1_000_000, partitions=4),
        # link-prediction ranks against every node of the small knowledge graph (the benchmark's --rank)
        _test("rank_fb15k_all", "rank", 15_000, 1_345, 400, 10_000, score="distmult"),
        # ranks against one shared sample of a larger graph's nodes
        _test("rank_social_sampled", "rank", 480_000, 0, 100, 10_000, candidates=50_000, partitions=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _unnamed(case):
    return {k: v for k, v in case.items() if k != "name"}


def draw(rng):
    kind = rng.choice(["bucket", "bucket", "bucket", "epoch", "score", "rank"])
    score = rng.choice(["dot", "distmult", "complex", "transe"])
    dim = rng.choice([rng.randint(8, 128), 32, 50, 64, 100, 100, 100, rng.randint(129, 512), 200, 400])
    if score == "transe":
        dim = min(dim, 128)
    if score == "complex":
        dim += dim % 2
    relations = 0 if score == "dot" else _log(rng, 1, 15_000)
    if kind in ("score", "rank"):
        triples = _log(rng, 100, 10_000) if kind == "rank" else _log(rng, 1_000, 1_000_000)
        nodes = _log(rng, 5_000, 50_000) if kind == "rank" else _log(rng, 5_000, 500_000)
        return _unnamed(_test("", kind, nodes, relations, dim, triples, candidates=rng.choice([0, _log(rng, 500, 50_000)]),
                              score=score, side=rng.choice(["dst", "src"]), partitions=rng.choice([1, 2, 4])))
    batch = _log(rng, 500, 50_000)
    chunk = rng.choice([50, 50, 100, rng.randint(20, 130)])
    negs = rng.choice([1_000, _log(rng, 30, 1_500)])
    sides = rng.choice(["dst", "src", "both"])
    partitions = rng.choice([1, 2, 4]) if kind == "bucket" else rng.choice([1, 4, 5])
    # so many edges that a pass costs no more than a part of the largest listed case's
    per_edge = negs * dim * (2 if sides == "both" else 1) * (4 if score == "transe" else 1)
    most = max(2 * batch, min(1_000_000, int(1.0e11 / per_edge)))
    edges = _log(rng, min(batch, most // 2), most)
    rows = min(3_000_000 // dim, 400_000)
    return _unnamed(_train("", kind, _log(rng, 10_000, 10 * rows), relations, edges, dim, batch, chunk, negs,
                           degree_negs=rng.choice([0, negs // 2]), score=score,
                           loss=rng.choice(["softmax", "softmax", "softmax", "logistic", "softmax_pos", "margin"]),
                           sides=sides, partitions=partitions, capacity=3 if kind == "epoch" and partitions > 3 else 0,
                           skew=rng.choice([0.7, 0.91, 1.0]), skew_q=rng.choice([1.0, 34.0, 100.0]),
                           edges_on=rng.choice(["device", "host"])))


class _Model:
    """A context with its partitions resident; the library's memory goes with it."""

    def __init__(self, case, seed):
        train = case["kind"] in ("bucket", "epoch")
        self.nodes, self.dim, self.n = case["nodes"], case["dim"], case["partitions"]
        self.relations = case["relations"]
        self.capacity = case.get("capacity", 0) or self.n
        cfg = L.make_config(
            num_nodes=self.nodes, dim=self.dim, num_partitions=self.n, buffer_capacity=self.capacity,
            num_relations=self.relations, score=SCORES[case["score"]], loss=LOSSES[case.get("loss", "softmax")],
            corrupt=SIDES[case["sides"]], batch_size=case.get("batch", 1_000), chunk_size=case.get("chunk", 50),
            num_negs=case.get("negs", 50), num_degree_negs=case.get("degree_negs", 0), lr=LEARNING_RATE,
            init_std=INIT_STD, seed=seed)
        self.ctx = L.legend_init_partitions(cfg, None, None)
        self.epoch = 0
        if not (train and self.capacity < self.n):
            for p in range(self.n):
                L.legend_swap_partition(self.ctx, -1, p)
            L.legend_sync(self.ctx)

    def tables(self):
        out = {"node": L.legend_read_embeddings(self.ctx, L.TABLE_NODE_EMB, None, self.nodes, self.dim)}
        if self.relations:
            out["relation"] = L.legend_read_embeddings(self.ctx, L.TABLE_REL_EMB, None, self.relations, self.dim)
        return out

    def __del__(self):
        L.legend_destroy(self.ctx)


def _skewed(gen, count, size, s, q):
    """count draws of a rank in [0, size) with density (x + q)^-s, sent through a seeded permutation."""
    u = torch.rand(count, generator=gen, device="cuda", dtype=torch.float64)
    if abs(s - 1.0) < 1e-12:
        x = q * ((size + q) / q) ** u - q
    else:
        a, b = q ** (1.0 - s), (size + q) ** (1.0 - s)
        x = (a + u * (b - a)) ** (1.0 / (1.0 - s)) - q
    perm = torch.randperm(size, generator=gen, device="cuda")
    return perm[x.long().clamp_(0, size - 1)]


def _edge_list(case, gen, rows_src, rows_dst):
    m = case["edges"]
    src = _skewed(gen, m, rows_src, case["skew"], case["skew_q"])
    dst = _skewed(gen, m, rows_dst, case["skew"], case["skew_q"])
    rel = torch.zeros_like(src)
    if case["relations"] > 1:
        rel = _skewed(gen, m, case["relations"], 1.0, 1.0)
    return src, rel, dst


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    model = _Model(case, seed)
    state = {"kind": case["kind"], "model": model}
    n, nodes = case["partitions"], case["nodes"]
    rows = -(-nodes // n)
    if case["kind"] == "bucket":
        # with several partitions the bucket between the first and the last of them
        src, rel, dst = _edge_list(case, gen, rows, nodes - (n - 1) * rows)
        edges = torch.stack([src, rel, dst], 1).to(torch.int32)
        state["edges"] = edges if case["edges_on"] == "device" else edges.cpu().numpy()
    elif case["kind"] == "epoch":
        src, rel, dst = _edge_list(case, gen, nodes, nodes)
        bucket = (src // rows) * n + dst // rows
        order = torch.argsort(bucket, stable=True)
        edges = torch.stack([src % rows, rel, dst % rows], 1).to(torch.int32)[order]
        ends = torch.cumsum(torch.bincount(bucket, minlength=n * n), 0).tolist()
        parts = {divmod(b, n): edges[(ends[b - 1] if b else 0):ends[b]].contiguous() for b in range(n * n)}
        state["keep"] = parts
        if case["edges_on"] == "device":
            state["buckets"] = {k: (t.data_ptr(), t.shape[0]) for k, t in parts.items()}
            state["mem"] = L.MEM_DEVICE
        else:
            state["buckets"] = {k: t.cpu().numpy() for k, t in parts.items()}
            state["mem"] = L.MEM_HOST
    else:
        rng = np.random.default_rng(seed)
        m = case["triples"]
        state["src"], state["dst"] = rng.integers(0, nodes, m), rng.integers(0, nodes, m)
        state["rel"] = rng.integers(0, case["relations"], m).astype(np.int32) if case["relations"] else None
        state["side"] = SIDES[case["sides"]]
        state["candidates"] = rng.integers(0, nodes, case["candidates"]) if case["candidates"] else None
    torch.cuda.synchronize()        # the library works on streams of its own
    return state


def run(state):
    model = state["model"]
    if state["kind"] == "bucket":
        edges, epoch = state["edges"], model.epoch
        model.epoch += 1
        if isinstance(edges, np.ndarray):
            stats = L.legend_train_bucket(model.ctx, 0, model.n - 1, edges, epoch=epoch)
        else:
            stats = L.legend_train_bucket(model.ctx, 0, model.n - 1, edges.data_ptr(), m=edges.shape[0],
                                          edges_mem=L.MEM_DEVICE, epoch=epoch)
        return {"loss": stats["loss_sum"], **model.tables()}
    if state["kind"] == "epoch":
        stats = L.legend_train_epoch(model.ctx, model.n, state["buckets"], edges_mem=state["mem"], epoch=model.epoch)
        model.epoch += 1
        return {"loss": stats["loss_sum"], **model.tables()}
    if state["kind"] == "score":
        return L.legend_score_edges(model.ctx, state["src"], state["rel"], state["dst"])
    greater, equal, metrics = L.legend_rank_edges(model.ctx, state["src"], state["rel"], state["dst"], state["side"],
                                                  state["candidates"])
    return {"greater": greater, "equal": equal, "mrr": metrics["mrr"], "hits1": metrics["hits1"],
            "hits3": metrics["hits3"], "hits10": metrics["hits10"]}


def _touched(draws, rows):
    """Expected distinct rows of so many uniform draws."""
    return rows * -math.expm1(-draws / rows)


def work(case):
    d, nodes, rel = case["dim"], case["nodes"], max(case["relations"], 1)
    if case["kind"] == "score":
        m = case["triples"]
        return {"bytes": m * (8 * d + 24), "flops": 2 * m * d}
    if case["kind"] == "rank":
        m, c = case["triples"], case["candidates"] or nodes
        return {"bytes": 4 * d * (_touched(c, nodes) if case["candidates"] else nodes) + m * (4 * d + 32), "flops": 2 * m * c * d}
    sides = 2 if case["sides"] == "both" else 1
    flops = sides * 3 * 2 * case["edges"] * case["negs"] * d
    # every batch reads and writes embedding and state of the rows it touches (endpoints taken as uniform), and
    # reads its edges; the tables are read back once
    n, batch = case["partitions"], min(case["batch"], case["edges"])
    if case["kind"] == "epoch":
        batch = min(batch, -(-case["edges"] // (n * n)))
    batches = case["edges"] / batch
    draws = 2 * batch + sides * math.ceil(batch / case["chunk"]) * case["negs"]
    touched = _touched(draws, nodes if n == 1 else 2 * nodes / n) + (0 if case["score"] == "dot" else _touched(batch, rel))
    bytes_ = batches * (16 * d * touched + 12 * batch) + 8 * d * (nodes + (rel if case["relations"] else 0))
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """About four times what the tables differ by after two passes when every initial value is rounded once more (the
    seeded fill's scale raised by 2^-22): 2e-7 to 1.4e-4 and 0.18 of the root mean square for the product scores, up to
    3e-3 and 0.7 for the translational one, whose gradients are sums of signs; 3e-7 for scores; one count in 500 to
    1000 moves by one."""
    if case["kind"] == "score":
        return {"rel": 1e-6, "max": 4e-6}
    if case["kind"] == "rank":
        return {"rel": 1e-3, "differ": 0.008}
    if case["score"] == "transe":
        return {"rel": 0.013, "max": 0.99}
    return {"rel": 6e-4, "max": 0.7}


def _mix(z):
    """The output function of splitmix64 on int64 tensors (wrap-around arithmetic, logical shifts)."""
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * (0xBF58476D1CE4E5B9 - (1 << 64))
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * (0x94D049BB133111EB - (1 << 64))
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _fill(seed, tag, rows, dim):
    """The seeded initial table of include/legend.h's NULL tables, as float64."""
    golden = 0x9E3779B97F4A7C15 - (1 << 64)
    h = torch.tensor([seed], dtype=torch.int64, device="cuda")
    h = _mix(h + golden + tag)
    h = _mix(h + golden + torch.arange(rows, device="cuda")[:, None])
    h = _mix(h + golden + torch.arange(dim, device="cuda")[None, :])
    u = sum((h >> k) & 0xFFFF for k in (0, 16, 32, 48)) - 131070
    scale = float(np.float32(float(np.float32(INIT_STD)) * 1.7320508075688772 / 65536.0))
    return (u.to(torch.float32) * scale).double()


def _composed(case, a, r, side):
    """The row that meets the replaced endpoint: a times the relation, in the score's sense."""
    if case["score"] == "dot":
        return a
    if case["score"] == "transe":
        return a + r if side == "dst" else a - r
    if case["score"] == "distmult":
        return a * r
    h = case["dim"] // 2
    ar, ai, rr, ri = a[:, :h], a[:, h:], r[:, :h], r[:, h:]
    if side == "dst":
        return torch.cat([ar * rr - ai * ri, ar * ri + ai * rr], 1)
    return torch.cat([rr * ar + ri * ai, rr * ai - ri * ar], 1)


def exact(case, seed):
    """Scores and ranks of the seeded tables in 64 bits.  Training has none here: two passes of Adagrad from zero states
    enlarge a rounding to the size that `tolerance` states, so that a distance from 64 bits would say nothing."""
    if case["kind"] not in ("score", "rank"):
        return None
    nodes, m = case["nodes"], case["triples"]
    rng = np.random.default_rng(seed)
    src, dst = (torch.from_numpy(rng.integers(0, nodes, m)).cuda() for _ in range(2))
    E = _fill(seed, NODE_TAG, nodes, case["dim"])
    r = None
    if case["relations"]:
        rel = torch.from_numpy(rng.integers(0, case["relations"], m)).cuda()
        r = _fill(seed, RELATION_TAG, case["relations"], case["dim"])[rel]
    cand = torch.from_numpy(rng.integers(0, nodes, case["candidates"])).cuda() if case["candidates"] else None

    def against(q, rows):
        return -(q - rows).abs().sum(1) if case["score"] == "transe" else (q * rows).sum(1)

    if case["kind"] == "score":
        return against(_composed(case, E[src], r, "dst"), E[dst]).cpu().numpy()
    kept, true = (src, dst) if case["sides"] == "dst" else (dst, src)
    q = _composed(case, E[kept], r, case["sides"])
    f = against(q, E[true])
    ids = cand if cand is not None else torch.arange(nodes, device="cuda")
    greater, equal = (torch.zeros(m, dtype=torch.int64, device="cuda") for _ in range(2))
    step = 4096 if case["score"] != "transe" else max(1, int(3e7 / (m * case["dim"])))
    for lo in range(0, ids.numel(), step):
        part = ids[lo:lo + step]
        S = -(q[:, None] - E[part]).abs().sum(2) if case["score"] == "transe" else q @ E[part].T
        other = part[None, :] != true[:, None]
        greater += ((S > f[:, None]) & other).sum(1)
        equal += ((S == f[:, None]) & other).sum(1)
    rank = 1.0 + greater.double() + 0.5 * equal.double()
    return {"greater": greater.int().cpu().numpy(), "equal": equal.int().cpu().numpy(), "mrr": (1 / rank).mean().item(),
            **{f"hits{k}": (rank <= k).double().mean().item() for k in (1, 3, 10)}}
