"""The partitioner's work as its users have it done, for timing: each case is
one call (or one burst of requests) through the package's public entry points.

A case is a plain dict; its "entry" names the call and its "shape" the kind of
hypergraph, one of those the package's own workloads use:

  uniform   degrees uniform in [dmin, dmax], pins uniform, no locality
            (random hypergraphs)
  netlist   degrees power-law 2.5 on [2, 1000], four pins of five within
            2000 ids of the hyperedge's anchor (VLSI netlists), E = 1.2 N
  colnet    degrees power-law 2.1 on [dmin, 5000], pins uniform, E = N, a
            node weighs its number of hyperedges (column-net models of sparse
            matrices)

Hypergraphs are drawn on the GPU from the seed alone.  A pin drawn twice for a
hyperedge is kept once, so degrees can fall slightly short of the drawn ones.
"""
import math
import weakref

import numpy as np
import torch

import paper_2012_13618_amd as bp
from paper_2012_13618_amd import inputs

POLICIES = {"ldh": bp.LDH, "hdh": bp.HDH, "lwd": bp.LWD, "hwd": bp.HWD, "rand": bp.RAND}
# expected degrees of the power laws below (netlist: alpha 2.5 on [2, 1000])
NETLIST_DEGREE = 4.54


def _case(name, entry, shape, n, e, k, eps, dmin=2, dmax=1000, policy="ldh", weighted=False, graphs=1):
    return {"name": name, "entry": entry, "shape": shape, "nodes": n, "hedges": e, "k": k, "eps": eps,
            "dmin": dmin, "dmax": dmax, "policy": policy, "weighted": weighted, "graphs": graphs}


def listed():
    return [
        # the smallest everyday call: a thousand-node random hypergraph
        # bisected on the device; launches and round trips are all of it
        _case("uniform-1k-k2", "device", "uniform", 1000, 2000, 2, 0.05, dmax=8),
        # a small weighted hypergraph of ragged size with 1-pin hyperedges,
        # an odd number of parts and a weight policy (Table 1 of the paper)
        _case("weighted-12k-k5", "device", "uniform", 12347, 14503, 5, 0.05, dmin=1, dmax=12, policy="lwd",
              weighted=True),
        # a placement-sized netlist in a loop that may not allocate
        _case("netlist-41k-k2-noalloc", "noalloc", "netlist", 41003, 49204, 2, 0.05),
        # a netlist that comes from host memory: validated, copied,
        # partitioned and copied back by the one call
        _case("netlist-200k-k4-host", "host", "netlist", 200000, 240000, 4, 0.05),
        # a netlist of the size of the larger published benchmarks, bisected
        _case("netlist-1m-k2", "device", "netlist", 1000000, 1200000, 2, 0.05),
        # a mid-size sparse matrix without singleton columns, cut into many
        # parts (a distribution over 32 processes)
        _case("colnet-617k-k32", "device", "colnet", 617283, 617283, 32, 0.03, dmax=5000),
        # the package's benchmark workload: a four-million-row sparse matrix
        # over eight processes
        _case("colnet-4m-k8", "device", "colnet", 4000000, 4000000, 8, 0.03, dmin=1, dmax=5000),
        # the shape of the paper's Random-10M input, the largest single
        # hypergraph that it prints times for with that of 15 M nodes
        _case("uniform-10m-k2", "device", "uniform", 10000000, 10000000, 2, 0.1, dmax=21),
        # the batched form: many netlists of uneven size in one run, half
        # bisected, half cut in four; n is the largest member's node count
        _case("batch-256", "batch", "netlist", 200000, 240000, 4, 0.05, graphs=256),
        # a burst of requests at the server, pins log-uniform in [10k, 2M],
        # k of 2, 4 and 16, each waited for; n is the largest request's
        _case("serve-24", "serve", "netlist", 367000, 440400, 16, 0.05, graphs=24),
        # the quality of a given 16-part partition of a netlist
        _case("cut-1m-k16", "cut", "netlist", 1000000, 1200000, 16, 0.05),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    entry = rng.choice(["device", "device", "device", "device", "noalloc", "host", "batch", "serve", "cut"])
    if entry in ("batch", "serve"):
        n = _log_uniform(rng, 60000, 200000 if entry == "batch" else 367000)
        g = _log_uniform(rng, 12, 200) if entry == "batch" else rng.randint(8, 24)
        return _case("", entry, "netlist", n, int(round(1.2 * n)), 4 if entry == "batch" else 16, 0.05, graphs=g)
    shape = rng.choice(["uniform", "netlist", "colnet"])
    top = {"device": 3000000, "noalloc": 60000, "host": 400000, "cut": 2000000}[entry]
    n = _log_uniform(rng, 800, top)
    k = rng.choice([2, 2, 3, 4, 5, 8, 16, 32] if n <= 1200000 else [2, 3, 4, 8])
    if entry == "noalloc":
        k = min(k, 2)
    policy = rng.choice(["ldh", "ldh", "ldh", "hdh", "lwd", "hwd", "rand"])
    weighted = shape != "colnet" and rng.random() < 0.4
    dmin, dmax = 2, 1000
    e = int(round(1.2 * n))
    if shape == "uniform":
        dmin, dmax = rng.choice([1, 2]), rng.randint(5, 21)
        e = int(n * rng.uniform(0.9, 2.0))
    elif shape == "colnet":
        dmin, dmax, e = rng.choice([1, 2]), 5000, n
        n = min(n, 30000) if entry == "noalloc" else n
        e = n
    return _case("", entry, shape, n, e, k, rng.choice([0.03, 0.05, 0.1]), dmin, dmax, policy, weighted)


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _power_law(g, count, alpha, dmin, dmax):
    d = torch.arange(dmin, dmax + 1, dtype=torch.float64, device="cuda")
    cdf = torch.cumsum(d ** -alpha, 0)
    cdf /= cdf[-1].clone()
    u = torch.rand(count, dtype=torch.float64, device="cuda", generator=g)
    return dmin + torch.searchsorted(cdf, u, right=True).clamp_(max=dmax - dmin)


def _graph(shape, n, e, dmin, dmax, weighted, seed):
    """(num_nodes, offsets, pins, node_w, hedge_w) as int32 tensors on the GPU."""
    g = _gen(seed)
    if shape == "uniform":
        deg = torch.randint(dmin, dmax + 1, (e,), device="cuda", generator=g)
    else:
        deg = _power_law(g, e, 2.5 if shape == "netlist" else 2.1, dmin, dmax)
    deg.clamp_(max=n)
    he = torch.repeat_interleave(torch.arange(e, device="cuda"), deg)
    p = he.numel()
    node = torch.randint(0, n, (p,), device="cuda", generator=g)
    if shape == "netlist":
        w = min(4001, n)
        anchor = torch.randint(0, n, (e,), device="cuda", generator=g)
        near = (anchor[he] + torch.randint(0, w, (p,), device="cuda", generator=g) - w // 2) % n
        node = torch.where(torch.rand(p, device="cuda", generator=g) < 0.8, near, node)
    key = torch.unique_consecutive(torch.sort(he * n + node).values)
    off = torch.zeros(e + 1, dtype=torch.int32, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(key // n, minlength=e), 0).to(torch.int32)
    pins = (key % n).to(torch.int32)
    if shape == "colnet":
        nw = torch.bincount(pins, minlength=n).to(torch.int32)
    elif weighted:
        nw = torch.randint(1, 6, (n,), device="cuda", generator=g).to(torch.int32)
    else:
        nw = torch.ones(n, dtype=torch.int32, device="cuda")
    if weighted:
        hw = torch.randint(1, 6, (e,), device="cuda", generator=g).to(torch.int32)
    else:
        hw = torch.ones(e, dtype=torch.int32, device="cuda")
    return n, off, pins, nw, hw


def _members(case, seed):
    """Sizes, parts and seeds of the members of a batch or burst: node counts
    log-uniform up to the case's, the largest among them.  The sizes are the
    case's own, the hypergraphs the seed's."""
    rng = np.random.default_rng([case["nodes"], case["graphs"]])
    lo = 1000 if case["entry"] == "batch" else 1850
    u = rng.random(case["graphs"])
    u[0] = 1.0
    n = np.exp(math.log(lo) + u * (math.log(case["nodes"]) - math.log(lo))).round().astype(int)
    ks = [2, 4] if case["entry"] == "batch" else [2, 4, 16]
    seeds = np.random.default_rng(int(seed)).integers(1, 2**62, case["graphs"])
    return [(int(x), ks[i % len(ks)], int(s)) for i, (x, s) in enumerate(zip(n, seeds))]


def _host(graph, k, eps):
    n, off, pins, nw, hw = graph
    return inputs.Hypergraph(n, off.cpu().numpy(), pins.cpu().numpy(), nw.cpu().numpy(), hw.cpu().numpy(),
                             meta={"k": k, "eps": eps})


class _Served:
    """A server and the burst's hypergraphs; the server goes with it."""

    def __init__(self, graphs):
        self.graphs = graphs
        self.server = bp.Server()
        weakref.finalize(self, self.server.close)


def _given_parts(case, seed):
    """Parts of the kind that a partitioner gives: runs of ids, a tenth astray."""
    g = _gen(seed + 1)
    n, k = case["nodes"], case["k"]
    part = torch.arange(n, device="cuda") * k // n
    astray = torch.randint(0, k, (n,), device="cuda", generator=g)
    part = torch.where(torch.rand(n, device="cuda", generator=g) < 0.1, astray, part)
    return part.to(torch.int32)


def prepare(case, seed):
    entry, eps = case["entry"], case["eps"]
    if entry in ("batch", "serve"):
        gs = []
        for n, k, s in _members(case, seed):
            gs.append((_graph("netlist", n, int(round(1.2 * n)), 2, 1000, False, s), k))
        if entry == "serve":
            return case, _Served([_host(g, k, eps) for g, k in gs])
        # one buffer for all members' parts, each member's a view of it
        sizes = [g[0] for g, _ in gs]
        parts = torch.empty(sum(sizes), dtype=torch.int32, device="cuda")
        return (case, [bp.DeviceHypergraph(*g) for g, _ in gs], [k for _, k in gs], [eps] * len(gs), parts,
                list(parts.split(sizes)))
    g = _graph(case["shape"], case["nodes"], case["hedges"], case["dmin"], case["dmax"], case["weighted"], seed)
    prm = bp.params(policy=POLICIES[case["policy"]])
    if entry == "host":
        return case, _host(g, case["k"], eps), prm
    dh = bp.DeviceHypergraph(*g)
    if entry == "cut":
        return case, dh, _given_parts(case, seed)
    if entry == "noalloc":
        return case, dh, prm, torch.empty(case["nodes"], dtype=torch.int32, device="cuda")
    return case, dh, prm


def run(state):
    case = state[0]
    entry, k, eps = case["entry"], case["k"], case["eps"]
    if entry == "device":
        part, cut, status, rep = bp.partition_device(state[1], k, eps, state[2])
    elif entry == "noalloc":
        part, cut, status, rep = bp.partition_device_noalloc(state[1], k, eps, state[2], part_out=state[3])
    elif entry == "host":
        part, cut, status, rep = bp.partition_hg(state[1], k, eps, state[2])
    elif entry == "batch":
        _, cuts, status, reps = bp.partition_batch_device(state[1], state[2], state[3], parts_out=state[5])
        return {"parts": state[4], "cuts": np.array(cuts), "status": status,
                "heaviest": np.array([r.max_part_weight for r in reps])}
    elif entry == "serve":
        served = state[1]
        tickets = [served.server.submit(h) for h in served.graphs]
        got = [served.server.wait(t) for t in tickets]
        return {"parts": [x[0] for x in got], "cuts": np.array([x[1] for x in got]),
                "status": np.array([x[2] for x in got]),
                "heaviest": np.array([x[3].max_part_weight for x in got])}
    else:
        cut, heaviest = bp.compute_cut_device(state[1], state[2], k)
        return {"cut": cut, "heaviest": heaviest}
    return {"part": part, "cut": cut, "status": status, "heaviest": rep.max_part_weight}


def _pins(case, n, e):
    if case["shape"] == "uniform":
        return e * (case["dmin"] + case["dmax"]) / 2
    if case["shape"] == "netlist":
        return e * NETLIST_DEGREE
    d = np.arange(case["dmin"], case["dmax"] + 1, dtype=np.float64)
    p = d ** -2.1
    return e * float((d * p).sum() / p.sum())


def work(case):
    """The hypergraph read once and the parts written once (read once where
    they are given); one integer operation a pin."""
    sizes = [(case["nodes"], case["hedges"])]
    if case["entry"] in ("batch", "serve"):
        # the mean of a log-uniform node count, times the members
        lo = 1000 if case["entry"] == "batch" else 1850
        mean = (case["nodes"] - lo) / math.log(case["nodes"] / lo)
        sizes = [(mean, 1.2 * mean)] * case["graphs"]
    pins = sum(_pins(case, n, e) for n, e in sizes)
    total = sum(4 * (e + 1) + 4 * n + 4 * e + 4 * n for n, e in sizes) + 4 * pins
    return {"bytes": int(total), "flops": int(pins)}


def exact(case, seed):
    """The cut and the heaviest part, from plain torch in 64 bits; a partition
    is the method's whole-number result and has no such value."""
    if case["entry"] != "cut":
        return None
    n, off, pins, nw, hw = _graph(case["shape"], case["nodes"], case["hedges"], case["dmin"], case["dmax"],
                                  case["weighted"], seed)
    part = _given_parts(case, seed).long()
    k, e = case["k"], case["hedges"]
    he = torch.repeat_interleave(torch.arange(e, device="cuda"), (off[1:] - off[:-1]).long())
    touched = torch.zeros(e * k, dtype=torch.bool, device="cuda")
    touched[he * k + part[pins.long()]] = True
    spans = touched.view(e, k).sum(1)
    cut = int((hw.long() * (spans - 1).clamp(min=0)).sum())
    weights = torch.zeros(k, dtype=torch.int64, device="cuda").index_add_(0, part, nw.long())
    return {"cut": cut, "heaviest": int(weights.max())}
