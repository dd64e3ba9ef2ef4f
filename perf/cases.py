"""The work that a training or serving program has this library do, as cases that can be timed and compared.

A case names a graph shape (the configurations of synth.CONFIGS, possibly shrunk), the call and its sizes.  `prepare` builds
what the program keeps: the registered graph, the feature table, seed batches, the arena, the cache.  `run` is one pass of
its loop over the next batch: a minibatch sampled and its feature rows loaded (`step`), the rows of a minibatch loaded
through the LRU cache (`cached`), random walks and the rows (`walk`), or what a processor does with a sampled block besides
(`block`: neighbour mean fused with the feature load, and the frontier grouped by owner).
"""
import math

import numpy as np
import torch

import paper_2310_12403_amd as P
import synth

DEVICE = "cuda"
SAMPLERS = {"labor0": P.COOP_LABOR0, "ns": P.COOP_NS}
BATCHES = 8  # consecutive seed batches that a state walks through, again from the first one at the end

# What a case says where it does not say otherwise.
DEFAULTS = dict(op="step", graph="products", down=1, directed=False, sampler="labor0", kappa=1, batch=1024, fanouts="10,10,10",
                dim=128, half=False, arena=True, cache_rows=0, walk_length=3, walks=100, restart=0.5, owners=8)


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # A handful of vertices scored on request: two layers, every buffer from torch's allocator (the binding's default).
        # Launches, waits and host work are all there is.
        _case("few_seeds", graph="products", down=16, batch=24, fanouts="10,10", dim=100, arena=False),
        # The repository's tiny configuration: a training step on a small graph, uniform fanout-k sampling.
        _case("tiny_ns", graph="tiny", sampler="ns", batch=1024, dim=64),
        # A directed graph whose ids, batch, fanouts and row length are all odd (150-byte rows, 2-byte aligned), inside a
        # group of dependent batches: nothing divides anything.
        _case("ragged_directed_ns", graph="products", down=3, directed=True, sampler="ns", kappa=16, batch=4097, fanouts="15,7,3",
              dim=75, half=True),
        # The repository's products-shaped configuration at its stated batch.
        _case("products_labor", graph="products", batch=16384, dim=100),
        # The repository's reddit-shaped configuration: uniform sampling with 25/10/10 and 2,408-byte rows; the last frontier
        # is the whole graph.
        _case("reddit_ns", graph="reddit", sampler="ns", batch=8192, fanouts="25,10,10", dim=602),
        # The paper's cache study: reddit-shaped, batch 1,024, dependent batches, rows through a 60,000-row LRU cache.
        _case("reddit_cached_step", graph="reddit", kappa=16, batch=1024, dim=602, cache_rows=60000),
        # The headline: papers100M-shaped at full size, LABOR-0 with independent batches, batch 16,384.
        _case("papers_labor", graph="papers100M", batch=16384, half=True),
        # The same step inside a group of 16 dependent batches, on a quarter of the graph.
        _case("papers_labor_dependent", graph="papers100M", down=4, kappa=16, batch=16384, half=True),
        # The same graph with uniform fanout-k sampling.
        _case("papers_ns", graph="papers100M", down=4, sampler="ns", batch=16384, half=True),
        # The paper's random-walk sampler with its parameters: walks of 3 steps, 100 of them, restart probability 0.5.
        _case("papers_walk", op="walk", graph="papers100M", down=8, batch=4096, half=True),
        # The rows of consecutive dependent batches through an LRU cache that holds little more than one batch's inputs.
        _case("papers_cached", op="cached", graph="papers100M", down=4, kappa=16, batch=16384, half=True, cache_rows=2000000),
        # What a processor of the cooperative scheme does with its last block: mean over the sampled in-edges straight from
        # the table, and the frontier grouped by the vertices' owners.
        _case("papers_block", op="block", graph="papers100M", down=4, batch=16384, half=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: graphs from a few thousand vertices to a quarter of the papers100M shape, batches of
    one seed to twice the configurations' largest, one to four layers, rows of 1 to 768 elements of either type."""
    while True:
        op = rng.choice(["step"] * 7 + ["walk", "cached", "block"])
        graph = rng.choice(["tiny", "products", "products", "reddit", "papers100M", "papers100M"])
        down = {"tiny": 1, "products": _log_uniform(rng, 1, 40), "reddit": _log_uniform(rng, 1, 20),
                "papers100M": _log_uniform(rng, 4, 60)}[graph]
        layers = rng.choice([1, 2, 2, 3, 3, 3, 4])
        fanouts = ",".join(str(rng.choice([1, 3, 5, 7, 10, 10, 10, 15, 20, 25])) for _ in range(layers))
        c = dict(DEFAULTS, op=op, graph=graph, down=down, fanouts=fanouts, directed=graph != "papers100M" and rng.random() < 0.2,
                 sampler=rng.choice(["labor0", "ns"]), kappa=rng.choice([1, 1, 1, 4, 16, 64, 256]),
                 batch=min(_log_uniform(rng, 1, 65536), n_vertices(dict(graph=graph, down=down)) // (2 * BATCHES)),
                 dim=rng.choice([1, 64, 100, 128, 256, 602, 768, rng.randint(2, 768)]), half=rng.random() < 0.5, arena=rng.random() < 0.7)
        if op == "cached" or (op == "step" and rng.random() < 0.15):
            c["cache_rows"] = max(1, int(expected_sizes(c)[-1][0] * rng.uniform(0.3, 3.0)))
        if op == "walk":
            c.update(walk_length=rng.choice([1, 2, 3, 3, 4, 5]), walks=rng.choice([10, 33, 64, 100, 100, 150]), restart=rng.choice([0.0, 0.3, 0.5]))
        if op == "block":
            c["owners"] = rng.choice([2, 4, 8, 8, 16, 64])
        # no dearer than the headline, and a feature table of at most 20 GB
        if work(c)["bytes"] <= 0.5 * work(listed()[6])["bytes"] and n_vertices(c) * row_bytes(c) <= 2e10:
            return c


# ---- sizes -------------------------------------------------------------------------------------------------------------
def n_vertices(case):
    cfg = synth.CONFIGS[case["graph"]]
    return 1 << cfg["scale"] if cfg["kind"] == "rmat" else cfg["n"] // case["down"]


def row_bytes(case):
    return case["dim"] * (2 if case["half"] else 4)


def fanouts_of(case):
    return tuple(int(k) for k in case["fanouts"].split(","))


def expected_sizes(case):
    """[(|S^l|, |E^l|, entries in the lists of the vertices new at layer l)] for l = 0 .. L-1, then (|S^L|, 0, 0): the expected
    numbers for a graph of the case's degree law whose edges join vertices in proportion to their degrees."""
    cfg = synth.CONFIGS[case["graph"]]
    n = n_vertices(case)
    two_m = 2.0 * cfg["edges"] if cfg["kind"] == "rmat" else 2.0 * (cfg["m"] // case["down"])
    alpha = 1.0 / (cfg.get("exponent", 2.1) - 1.0)
    i0 = synth._chung_lu_offset(n, two_m, alpha)
    edge = np.unique(np.concatenate([[0], np.geomspace(1, n, 160).astype(np.int64)]))
    count = np.diff(edge).astype(np.float64)             # vertices per class of neighbouring ranks
    d = ((edge[:-1] + edge[1:]) / 2 + i0) ** -alpha
    d *= two_m / (d * count).sum()
    if case["directed"]:
        d, two_m = d / 2, two_m / 2
    p = np.full(len(d), min(1.0, case["batch"] / n))     # P(a vertex of the class is in S^l)
    before = np.zeros(len(d))
    sizes = []
    r = (np.arange(400) + 0.5) / 400
    for k in fanouts_of(case):
        kept = np.minimum(d, k)
        m = (count * p * kept).sum()
        sizes.append((float((count * p).sum()), float(m), float((count * (p - before) * d).sum())))
        if case["sampler"] == "ns" or case["op"] == "walk":
            hit = 1.0 - np.exp(-d * m / two_m)
        else:  # LABOR-0: t is sampled when some neighbour s in S^l has k / d_s >= r_t
            x = r ** 3                                   # small variates matter most
            mass = (count * p * d)[None, :] * (d[None, :] * x[:, None] <= k)
            hit = ((1.0 - np.exp(-d[None, :] * mass.sum(1)[:, None] / two_m)) * (3 * r ** 2 / 400)[:, None]).sum(0)
        before = p
        p = 1.0 - (1.0 - p) * (1.0 - np.minimum(hit, 1.0))
    sizes.append((float((count * p).sum()), 0.0, 0.0))
    return sizes


def work(case):
    """Bytes of one pass, each input read once and each output written once.  Sampling: the lists of the destinations (each
    vertex's once, however many layers it is a destination of), their bounds, and per layer the offsets, the edges' local and
    global sources and positions and the new vertices; loading: the rows in and out and the ids."""
    sizes = expected_sizes(case)
    n_last, row = sizes[-1][0], row_bytes(case)
    rows = n_last * (2 * row + 4)
    if case["op"] == "cached":
        return {"bytes": rows + 8 * n_last, "flops": 0}
    if case["op"] == "block":
        n_dst, m, _ = sizes[-2]
        return {"bytes": m * (row + 4) + n_dst * (row + 8) + n_last * 12, "flops": m * case["dim"]}
    total = rows
    for l, (n_dst, m, entries) in enumerate(sizes[:-1]):
        total += 24 * n_dst + 16 * m + 4 * sizes[l + 1][0]
        if case["op"] == "walk":  # every step reads an entry, and the bounds of the list that it leaves
            steps = case["walk_length"] * case["walks"]
            total += n_dst * steps * (4 + 16 * (1 - case["restart"]) * (1 - 1 / case["walk_length"]))
        else:
            total += 4 * entries
    return {"bytes": total, "flops": 0}


def tolerance(case):
    # Vertices, edges and copied rows are the same bytes.  The neighbour mean sums about ten numbers in 32 bits: summed from the
    # other end, or in 64 bits, fp32 results differ by 1e-7 (2-norm; 5e-7 at worst) and fp16 results by 1e-7, a unit in the
    # last place (at most 9.8e-4) of a few values.
    if case["op"] == "block":
        return {"rel": 4e-7, "max": 1e-3} if case["half"] else {"rel": 4e-7, "max": 2e-6}
    return "exact"


# ---- state -------------------------------------------------------------------------------------------------------------
def _room(case):
    """(vertices, edges of all layers, destinations of all layers) that the program's own buffers have room for."""
    n = n_vertices(case)
    most, vertices, edges, dsts = case["batch"], 0.0, 0.0, 0.0
    for (n_l, m, _), k in zip(expected_sizes(case), fanouts_of(case)):
        bound = k * most + 8 * math.sqrt(k * most) + 4096      # hardly ever exceeded, and for large batches far above ...
        edges += min(bound, 1.5 * m + 65536)                    # ... what is expected
        dsts += min(most, 1.5 * n_l + 65536) + 1
        most = min(n, most + bound)
    vertices = min(most, 1.5 * expected_sizes(case)[-1][0] + 65536)
    return int(vertices), int(edges), int(dsts)


def _sample(state, i):
    c = state["case"]
    seeds = state["seeds"][i % BATCHES]
    if state["arena"] is not None:
        state["arena"].reset()
    if c["op"] == "walk":
        return P.coop_sample_rw(state["graph"], seeds, state["fanouts"], c["walk_length"], c["walks"], c["restart"],
                                it=state["first"] + i, seed=state["seed"], arena=state["arena"])
    return P.coop_sample(state["graph"], seeds, state["fanouts"], SAMPLERS[c["sampler"]], it=state["first"] + i, kappa=c["kappa"],
                         seed=state["seed"], arena=state["arena"])


def prepare(case, seed):
    c = dict(DEFAULTS, **case)
    n = n_vertices(c)
    dtype = torch.float16 if c["half"] else torch.float32
    indptr, indices = synth.make_graph(c["graph"], device=DEVICE, scale_down=c["down"], seed=seed)
    flags = P.COOP_VALIDATE | P.COOP_SYMMETRIC
    if c["directed"]:
        indptr, indices = synth.directed_from_symmetric(indptr, indices, stream=seed)
        flags = P.COOP_VALIDATE
    indices = indices.contiguous()
    order = synth.permutation(n, 555 + seed, DEVICE)[:BATCHES * c["batch"]].to(torch.int32)
    vertices, edges, dsts = _room(c)
    state = {
        "case": c, "fanouts": fanouts_of(c), "seed": seed,
        "graph": P.coop_graph_load(indptr, indices, flags, torch_memory=True),
        "seeds": [order[b * c["batch"]:(b + 1) * c["batch"]].contiguous() for b in range(BATCHES)],
        "feat": synth.features(n, c["dim"], dtype, seed=seed, device=DEVICE),
        "arena": P.Arena((6 if c["graph"] == "papers100M" else 3) << 30) if c["arena"] else None,
        "first": 1000 + c["kappa"] // 3 - 1000 % c["kappa"],  # inside a group of dependent batches when there are groups
        "at": 0,
        # the training step's own buffers, sized once: a block leaves the sampler's memory before that is used again
        "rows": torch.zeros((vertices, c["dim"]), dtype=dtype, device=DEVICE),
        "ids": torch.zeros(vertices + edges, dtype=torch.int32, device=DEVICE),
        "places": torch.zeros(dsts + edges, dtype=torch.int64, device=DEVICE),
    }
    if c["cache_rows"]:
        state["cache"] = P.Cache(c["cache_rows"], n, c["dim"], dtype, n, device=DEVICE)
    if c["op"] == "cached":  # the inputs of consecutive batches, and a cache that has seen a round of them
        state["inputs"] = [_sample(state, i)[-1].src_ids.clone() for i in range(BATCHES)]
        for ids in state["inputs"]:
            state["cache"].gather(state["feat"], ids)
    if c["op"] == "block":
        last = _sample(state, 0)[-1]
        state["block"] = (last.indptr.clone(), last.col_global.clone(), last.src_ids.clone())
        state["groups"] = (torch.zeros(vertices, dtype=torch.int32, device=DEVICE), torch.zeros(vertices, dtype=torch.int32, device=DEVICE),
                           torch.zeros(c["owners"] + 1, dtype=torch.int64, device=DEVICE))
    return state


def run(state):
    c, i, rows = state["case"], state["at"], state["rows"]
    state["at"] = i + 1
    if c["op"] == "cached":
        ids = state["inputs"][i % BATCHES]
        return rows, state["cache"].gather(state["feat"], ids, out=rows)[1]
    if c["op"] == "block":
        indptr, col_global, src_ids = state["block"]
        P.coop_gather_mean(state["feat"], indptr, col_global, out=rows[:indptr.numel() - 1])
        ids, origin, offsets = state["groups"]
        P.coop_bucket_by_owner_static(src_ids, state["feat"].shape[0], c["owners"], P.COOP_OWNER_HASH, seed=state["seed"], out=ids,
                                      origin=origin, offsets=offsets)
        return rows, ids, origin, offsets
    blocks = _sample(state, i)
    n_miss = 0
    if c["cache_rows"]:
        n_miss = state["cache"].gather(state["feat"], blocks[-1].src_ids, out=rows)[1]
    else:
        P.coop_gather(state["feat"], blocks[-1].src_ids, out=rows)
    # the blocks: S^l is the front of S^{l+1}, so the last list of vertices holds them all (and gives the global sources)
    sizes = [n for b in blocks for n in (b.n_dst, b.n_src, b.n_edges)]
    n_edges = sum(b.n_edges for b in blocks)
    torch.cat([blocks[-1].src_ids] + [b.col_local for b in blocks], out=state["ids"][:blocks[-1].n_src + n_edges])
    torch.cat([b.indptr for b in blocks] + [b.eid for b in blocks],
              out=state["places"][:sum(b.n_dst + 1 for b in blocks) + n_edges])
    return rows, state["ids"], state["places"], sizes, n_miss
