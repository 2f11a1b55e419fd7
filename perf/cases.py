"""What the frame-parallel aggregation is used for, as cases that can be measured.

A case is a dynamic graph (a generator, its size, how much of it changes from snapshot to snapshot),
a frame of k of its snapshots, a feature width and layout, and what a program does with the frame:

  step       a new frame: overlap extraction, then one aggregation of all k snapshots
  slide      a new frame whose first k - 1 snapshots were in the frame before it: overlap extraction,
             then the aggregation of the entering snapshot alone (the other results are kept)
  aggregate  one more epoch on a frame that is there already: the aggregation alone
  layer      the same, with the layer's fully connected update behind it
  backward   directed graphs: the frame of the transposed operator, and the gradients through it

Sizes are those of the benchmark workloads and of the tests (1 thousand to 1 million nodes, 1 to 16
snapshots, 1 to 128 feature columns).  Graphs are made on the GPU from the seed alone: Chung-Lu or
R-MAT, undirected unless said otherwise, both directions stored, canonical CSR; adjacent snapshots
differ in a given fraction of their edges.  Features are uniform on [-1, 1), new for every snapshot.
"""
import math

import torch

import paper_2301_00391_amd as pipad

DEVICE = "cuda:0"

# The large case sets what a drawn case may cost: edge.feature updates, and entries of all snapshots.
MOST_UPDATES = 8 * 21_000_000 * 64
MOST_ENTRIES = 8 * 20_000_000


def _case(name, op, model, n, edges, k, churn, feat, layout="list", padded=True, out=0, static=False):
    c = {"name": name, "op": op, "model": model, "n": n, "edges": edges, "k": k, "churn": churn, "feat": feat,
         "layout": layout, "padded": padded, "out": out, "static": static}
    return c if name else {q: v for q, v in c.items() if q != "name"}


def listed():
    return [
        # a toy graph in the concatenated layout: what the calls themselves cost (launches, host path)
        _case("tiny step", "step", "chung-lu-2.5", 2_000, 8_000, 4, 0.05, 16, layout="wide"),
        # a small graph, epoch after epoch on the same frame through the call that allocates nothing (a
        # serving loop, a graph-captured training loop)
        _case("small epoch", "aggregate", "chung-lu-2.2", 20_000, 120_000, 4, 0.10, 32, static=True),
        # the small benchmark workload: a new frame each step
        _case("small step", "step", "chung-lu-2.2", 20_000, 120_000, 4, 0.10, 32),
        # the medium benchmark workload: a new frame each step
        _case("medium step", "step", "chung-lu-2.1", 200_000, 1_600_000, 8, 0.03, 64),
        # ... and its frames sliding by one snapshot, first-layer results kept
        _case("medium slide", "slide", "chung-lu-2.1", 200_000, 1_600_000, 8, 0.03, 64),
        # a hidden layer in training: aggregation and update in one call
        _case("medium layer", "layer", "chung-lu-2.1", 200_000, 1_600_000, 8, 0.03, 64, out=64),
        # a wide input layer (aggregation, then the multiplication), sizes that divide nothing
        _case("ragged layer", "layer", "chung-lu-2.3", 150_001, 900_001, 3, 0.20, 128, padded=False, out=40),
        # the backward pass on a directed graph
        _case("backward", "backward", "chung-lu-2.1", 200_000, 1_600_000, 4, 0.05, 64),
        # rows no vector load fits (30 columns, stored densely), an odd number of nodes and snapshots
        _case("ragged step", "step", "rmat", 99_991, 600_007, 5, 0.10, 30, padded=False),
        # the paper's own feature width, all snapshots concatenated, on a graph of real size
        _case("narrow epoch", "aggregate", "rmat", 1_000_000, 10_000_000, 8, 0.01, 2, layout="wide"),
        # hardly any overlap and wide features
        _case("low-overlap epoch", "aggregate", "chung-lu-2.3", 500_000, 5_000_000, 8, 0.40, 128),
        # the headline workload: one million nodes, ten million edges, a new frame each step
        _case("large step", "step", "rmat", 1_000_000, 10_000_000, 8, 0.01, 64),
    ]


def _spread(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """Another case of the same ranges: nodes, degree, churn and widths spread over their logarithms."""
    while True:
        op = rng.choice(["step", "step", "slide", "aggregate", "layer", "backward"])
        model = rng.choice(["rmat", "chung-lu-2.1", "chung-lu-2.2", "chung-lu-2.3", "chung-lu-2.5"])
        n = round(_spread(rng, 1_000, 1_000_000))
        edges = round(n * _spread(rng, 4, 20) / 2)
        k = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 12, 16])
        churn = round(_spread(rng, 0.01, 0.4), 3)
        feat = round(_spread(rng, 1, 128))
        if rng.random() < 0.6:  # most widths are round numbers
            feat = min(128, max(16, (feat + 8) // 16 * 16))
        layout = "wide" if op in ("step", "aggregate") and rng.random() < 0.3 else "list"
        padded = rng.random() < 0.6
        out = round(_spread(rng, 8, 128)) if op == "layer" else 0
        if op == "layer" and rng.random() < 0.6:
            out = max(16, (out + 8) // 16 * 16)
        static = op == "aggregate" and n <= 100_000 and rng.random() < 0.5
        if k * (2 * edges + n) * max(feat, out) <= MOST_UPDATES and 2 * k * edges <= MOST_ENTRIES:
            return _case(None, op, model, n, edges, k, churn, feat, layout, padded, out, static)


# ---- graphs ---------------------------------------------------------------------------------------


def _offset(n, edges, alpha):
    """The smallest i0 >= 1 for which no expected degree passes the square root of their sum."""
    lo, hi = 1.0, float(n)
    for _ in range(50):
        mid = math.sqrt(lo * hi)
        total = ((n + mid) ** (1.0 - alpha) - mid ** (1.0 - alpha)) / (1.0 - alpha)  # of the weights
        if mid ** -alpha / total * math.sqrt(2.0 * edges) > 1.0:
            lo = mid
        else:
            hi = mid
    return hi


def _pairs(model, n, edges, count, gen):
    """`count` random node pairs (both int64 on the GPU) of the model."""
    if model == "rmat":
        # quadrants 0.57 / 0.19 / 0.19 / 0.05 on the next power of two; ids past n are dropped
        u = torch.zeros(count, dtype=torch.int64, device=DEVICE)
        v = torch.zeros(count, dtype=torch.int64, device=DEVICE)
        for _ in range(max(1, (n - 1).bit_length())):
            r = torch.rand(count, device=DEVICE, generator=gen)
            u = u * 2 + (r >= 0.76).long()
            v = v * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).long()
        keep = (u < n) & (v < n)
        return u[keep], v[keep]
    # Chung-Lu: both ends drawn with probability proportional to (i + i0)^(-1 / (gamma - 1))
    alpha = 1.0 / (float(model.rsplit("-", 1)[1]) - 1.0)
    w = (torch.arange(n, dtype=torch.float64, device=DEVICE) + _offset(n, edges, alpha)).pow(-alpha)
    cdf = torch.cumsum(w, 0)
    cdf /= cdf[-1].clone()
    ends = torch.searchsorted(cdf, torch.rand(2 * count, dtype=torch.float64, device=DEVICE, generator=gen))
    ends.clamp_(max=n - 1)
    return ends[:count], ends[count:]


def _fresh_edges(case, count, present, gen):
    """`count` different undirected edges, as keys low * n + high, none of them in `present` (sorted)."""
    model, n, edges = case["model"], case["n"], case["edges"]
    have = torch.empty(0, dtype=torch.int64, device=DEVICE)
    while have.numel() < count:
        u, v = _pairs(model, n, edges, max(1024, int(1.5 * (count - have.numel()))), gen)
        lo, hi = torch.minimum(u, v), torch.maximum(u, v)
        key = (lo * n + hi)[lo != hi]
        if present.numel():
            at = torch.searchsorted(present, key).clamp_(max=present.numel() - 1)
            key = key[present[at] != key]
        have = torch.unique(torch.cat([have, key]))
    return have[torch.randperm(have.numel(), device=DEVICE, generator=gen)[:count]]


def _csr(n, edges, directed):
    """Canonical CSR of the undirected edges; a directed graph lacks one direction of half of them."""
    lo, hi = edges // n, edges % n
    forth, back = edges, hi * n + lo
    if directed:
        which = (edges * 2654435761 >> 7) & 3
        forth, back = forth[which != 0], back[which != 1]
    key = torch.cat([forth, back]).sort().values
    rows = torch.arange(n + 1, dtype=torch.int64, device=DEVICE) * n
    return torch.searchsorted(key, rows).to(torch.int32), (key % n).to(torch.int32)


def _snapshots(case, count, gen):
    n, m = case["n"], case["edges"]
    directed = case["op"] == "backward"
    edges = _fresh_edges(case, m, torch.empty(0, dtype=torch.int64, device=DEVICE), gen)
    got = [_csr(n, edges, directed)]
    change = round(case["churn"] * m)
    for _ in range(count - 1):
        kept = edges[torch.randperm(m, device=DEVICE, generator=gen)[change:]]
        if change:
            kept = torch.cat([kept, _fresh_edges(case, change, kept.sort().values, gen)])
        edges = kept
        got.append(_csr(n, edges, directed))
    return got


# ---- what a program has in hand, and a pass --------------------------------------------------------


def _matrices(case, feat, padded, gen=None):
    """k [n, feat] matrices (or one [n, k, feat] tensor): random with `gen`, else for results."""
    n, k = case["n"], case["k"]
    if case["layout"] == "wide":
        x = torch.empty((n, k, feat), dtype=torch.float32, device=DEVICE)
        return x.uniform_(-1, 1, generator=gen) if gen is not None else x
    stride = pipad.padded_row_stride(feat) if padded else feat
    got = []
    for _ in range(k):
        x = torch.empty((n, stride), dtype=torch.float32, device=DEVICE)
        if gen is not None:
            x.uniform_(-1, 1, generator=gen)
        got.append(x[:, :feat])
    return got


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    s = {"case": case, "snapshots": _snapshots(case, case["k"], gen)}
    # rows that are gathered are padded the way the library recommends, where the case says so;
    # results are dense
    s["X"] = _matrices(case, case["feat"], case["padded"], gen)
    s["Y"] = _matrices(case, case["feat"], False)
    if case["op"] in ("aggregate", "layer", "backward"):
        s["frame"] = pipad.frame_build_overlap(s["snapshots"])
    if case["op"] == "layer":
        s["W"] = torch.randn((case["feat"], case["out"]), device=DEVICE, generator=gen) / math.sqrt(case["feat"])
        s["bias"] = torch.randn(case["out"], device=DEVICE, generator=gen)
        s["H"] = _matrices(case, case["out"], False)
    return s


def run(s):
    case, op = s["case"], s["case"]["op"]
    if op == "step":
        frame = pipad.frame_build_overlap(s["snapshots"])
        return pipad.frame_aggregate(frame, s["X"], s["Y"])
    if op == "slide":
        frame = pipad.frame_build_overlap(s["snapshots"])
        last = case["k"] - 1
        pipad.frame_aggregate_subset(frame, [last], s["X"], s["Y"])
        return s["Y"][last]
    if op == "aggregate":
        return pipad.frame_aggregate(s["frame"], s["X"], s["Y"], static_scratch=case["static"])
    if op == "layer":
        # the aggregation results are kept too: the weight gradient needs them
        pipad.frame_aggregate_update(s["frame"], s["X"], s["W"], s["bias"], H=s["H"], A=s["Y"])
        return s["H"], s["Y"]
    back = pipad.frame_transpose(s["frame"])
    return pipad.frame_aggregate(back, s["X"], s["Y"])


def work(case):
    n, k, feat, out, op = case["n"], case["k"], case["feat"], case["out"], case["op"]
    nnz = (1.5 if op == "backward" else 2.0) * case["edges"]  # stored entries of a snapshot
    topology = 4 * k * (nnz + n + 1)
    if op in ("aggregate", "layer", "backward"):
        # the frame's parts are the input: the entries all snapshots share are there once
        shared = nnz * (1.0 - case["churn"]) ** (k - 1)
        topology = 4 * (shared + k * (nnz - shared)) + 4 * (k + 1) * (n + 1) + 4 * k * n
    taken = 1 if op == "slide" else k  # snapshots whose features are read and written
    features = 8 * taken * n * feat
    flops = 2 * taken * feat * (nnz + n)
    if op == "layer":
        features += 4 * k * n * out + 4 * (feat + 1) * out
        flops += 2 * k * n * feat * out
    return {"bytes": topology + features, "flops": flops}


def tolerance(case):
    return {"rel": 1e-5}  # sums of 32-bit floats, in any order
