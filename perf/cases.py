"""The calls whose speed matters, as a user's program makes them: k-hop sampling, cache lookup + gather +
FIFO insert, the two-level lookup, the overlapped minibatch loop, and the proximity-aware ordering.

Each case is a dict of plain values with a `kind`; `prepare` makes what a training program has in hand
(graph, features, warm cache, workspaces, seed batches), `run` is one pass through the public entry
points.  Graphs are power-law out-degree graphs with short-range edges on a hidden ring plus a few hubs,
the shape `paper_2112_08541_amd.inputs` generates, made on the GPU here because they are made often.
Everything is integers and bytes (feature rows are copied), so results are compared exactly.
"""
import math

import torch

from paper_2112_08541_amd import binding as B
from paper_2112_08541_amd.pipeline import NativePipeline

SEED_BATCHES = 8     # seed batches a state goes through in turn
ID_BATCHES = 6       # id batches a cache state goes through in turn
LOCAL_EDGES = 0.97   # share of short-range edges
REACH = 2000         # their mean distance on the ring


def listed():
    return [
        # One sampling call of a small graph (a test or a small dataset): launches and latency count.
        dict(name="sample tiny", kind="sample", nodes=10_000, mean_degree=10.0, dmin=2, seeds=512,
             fanouts="10,5", bits=32, placement="device"),
        # The ordinary training batch: Ogbn-products' shape, batch 1,024, fanout 15,10,5, the graph in HBM.
        dict(name="sample mid", kind="sample", nodes=2_450_000, mean_degree=50.0, dmin=5, seeds=1024,
             fanouts="15,10,5", bits=32, placement="device"),
        # Large batches with two wide hops on a larger graph.
        dict(name="sample wide", kind="sample", nodes=8_000_000, mean_degree=20.0, dmin=4, seeds=4096,
             fanouts="25,10", bits=32, placement="device"),
        # A graph that stays in page-locked host memory (64-bit offsets), as graphs of 10^9 edges do.
        dict(name="sample host graph", kind="sample", nodes=6_000_000, mean_degree=14.4, dmin=3, seeds=1024,
             fanouts="15,10,5", bits=64, placement="host"),
        # Feature retrieval of a small batch: most rows come from host memory, read in place.
        dict(name="cache tiny", kind="cache", nodes=10_000, row_bytes=400, ids=5_485, capacity=2_000),
        # Feature retrieval of an ordinary batch, cache of 20 % of the nodes, misses over the host link.
        dict(name="cache mid", kind="cache", nodes=2_450_000, row_bytes=400, ids=428_377, capacity=490_000),
        # The cache is large enough to hold every row it is asked for (bf16 x 512): the gather from HBM.
        dict(name="cache resident", kind="cache", nodes=600_000, row_bytes=1024, ids=302_709, capacity=600_000),
        # GPU cache of 10 % of the nodes, host tier of 30 % behind it, rows over the copy engine.
        dict(name="two level", kind="tier", nodes=1_000_000, row_bytes=512, ids=150_001, capacity=100_000,
             tier_rows=300_000, transport=1),
        # The overlapped loop on a small graph: 20 batches a pass, misses read in place.
        dict(name="epoch tiny", kind="epoch", nodes=10_000, mean_degree=10.0, dmin=2, batch=512, fanouts="10,5",
             row_bytes=400, cache_rows=2_000, staged=False, steps=20),
        # The overlapped loop as it is benchmarked: miss rows packed by host threads, copied, one output pass.
        dict(name="epoch mid", kind="epoch", nodes=2_450_000, mean_degree=50.0, dmin=5, batch=1024,
             fanouts="15,10,5", row_bytes=400, cache_rows=490_000, staged=True, steps=8),
        # Proximity-aware order of the training nodes, small graph: several sequences, many short levels.
        dict(name="order small", kind="order", nodes=100_000, mean_degree=10.0, dmin=2, train=10_000, sequences=5),
        # The same for the ordinary graph (two of the sequences that are merged).
        dict(name="order mid", kind="order", nodes=2_450_000, mean_degree=50.0, dmin=5, train=204_800, sequences=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sample", "sample", "cache", "cache", "tier", "epoch", "order"])
    if kind in ("sample", "epoch", "order"):
        nodes = _log_int(rng, 5_000, 2_450_000)
        mean = round(rng.uniform(8.0, 50.0), 1)
        graph = dict(nodes=nodes, mean_degree=mean, dmin=rng.randint(2, 5))
    if kind == "sample":
        return dict(kind=kind, **graph, seeds=_log_int(rng, 50, min(4096, nodes // 2)),
                    fanouts=rng.choice(["10,5", "15,10,5", "25,10", "20", "8,8", "5,5,5", "12,7,3", "33,3"]),
                    bits=rng.choice([32, 64]), placement=rng.choice(["device", "device", "device", "host", "host_col"]))
    if kind == "order":
        return dict(kind=kind, **graph, train=max(50, int(nodes * rng.uniform(0.05, 0.3))), sequences=rng.randint(1, 2))
    row_bytes = rng.choice([64, 272, 400, 512, 528, 1024])
    if kind == "epoch":
        staged = nodes >= 100_000
        return dict(kind=kind, **graph, batch=_log_int(rng, 200, 1024) if staged else _log_int(rng, 50, 500),
                    fanouts="15,10,5" if staged else rng.choice(["10,5", "8,4"]), row_bytes=min(row_bytes, 400),
                    cache_rows=max(100, int(nodes * rng.uniform(0.05, 0.4))), staged=staged, steps=rng.randint(3, 8))
    nodes = _log_int(rng, 5_000, min(2_000_000, 900_000_000 // row_bytes))
    ids = _log_int(rng, 200, nodes // 4)
    if kind == "cache":
        return dict(kind=kind, nodes=nodes, row_bytes=row_bytes, ids=ids,
                    capacity=max(16, int(nodes * rng.choice([0.05, 0.1, 0.2, 0.5, 1.0]))))
    ids = min(ids, 200_000)
    return dict(kind=kind, nodes=nodes, row_bytes=row_bytes, ids=ids, capacity=max(16, int(nodes * rng.uniform(0.05, 0.3))),
                tier_rows=int(nodes * rng.choice([0.0, 0.2, 0.5])), transport=rng.choice([0, 1, 2]))


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
    return g


def _pareto_exponent(mean, dmin, dmax):
    """Exponent whose Pareto law, cut at dmax, has the wanted mean."""
    lo, hi = 1.0001, 60.0
    t = dmax / dmin
    for _ in range(60):
        a = 0.5 * (lo + hi)
        m = dmin * (a / (a - 1.0) * (1.0 - t ** (1.0 - a)) + t ** (1.0 - a))
        lo, hi = (a, hi) if m > mean else (lo, a)
    return lo


def _csr(case, gen):
    """(row_ptr, col, ids by ring position) on the GPU."""
    n = case["nodes"]
    dmin = case["dmin"]
    dmax = int(max(4 * case["mean_degree"], min(20_000, n // 4)))
    a = _pareto_exponent(case["mean_degree"] + 0.5, dmin, dmax)
    u = torch.rand(n, generator=gen, device="cuda").clamp_(min=1e-7)
    deg = (dmin * u.pow_(-1.0 / a)).clamp_(max=dmax).to(torch.int64)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(deg, 0, out=row_ptr[1:])
    e = int(row_ptr[-1])
    id_at = torch.randperm(n, generator=gen, device="cuda").to(torch.int32)     # ring position -> node id
    at = torch.empty(n, dtype=torch.int32, device="cuda")
    at[id_at.long()] = torch.arange(n, dtype=torch.int32, device="cuda")
    reach = float(min(REACH, max(2, n // 16)))
    step = torch.empty(e, device="cuda").exponential_(1.0 / reach, generator=gen).ceil_()
    step.mul_(torch.rand(e, generator=gen, device="cuda").sub_(0.5).sign_())
    dst = torch.repeat_interleave(at, deg, output_size=e)
    dst += step.clamp_(-n // 2, n // 2).to(torch.int32)
    del step
    dst.remainder_(n)
    hubs = max(16, n // 16384)
    hub_pos = torch.randint(0, n, (hubs,), generator=gen, device="cuda", dtype=torch.int32)
    far = torch.nonzero(torch.rand(e, generator=gen, device="cuda") >= LOCAL_EDGES).squeeze(1)
    rank = (torch.rand(far.numel(), generator=gen, device="cuda").pow_(4.0) * hubs).to(torch.int64).clamp_(max=hubs - 1)
    dst[far] = hub_pos[rank]                                                     # Zipf 0.75 over the hubs
    return row_ptr, id_at[dst.long()], id_at


def _pinned(t):
    h = torch.empty(t.shape, dtype=t.dtype, pin_memory=True)
    h.copy_(t)
    return h


def _graph(case, gen, bits=32, placement="device"):
    row_ptr, col, id_at = _csr(case, gen)
    where = {"device": B.BGL_DEVICE, "host": B.BGL_HOST_PINNED, "host_col": B.BGL_HOST_PINNED_COL}[placement]
    rp = _pinned(row_ptr if bits == 64 else row_ptr.to(torch.int32))
    return B.Graph(rp, _pinned(col), where), id_at


def _fanouts(case):
    return [int(f) for f in case["fanouts"].split(",")]


def _seed_batches(gen, nodes, count, size):
    return torch.stack([torch.randperm(nodes, generator=gen, device="cuda")[:size] for _ in range(count)]).to(torch.int32)


def _rng_seeds(seed, count):
    return [(int(seed) * 0x9E3779B97F4A7C15 + 0xD1B54A32D192ED03 * (k + 1)) % (1 << 64) for k in range(count)]


def _features(case, gen):
    """Feature bytes in page-locked host memory."""
    words = torch.randint(-2**31, 2**31 - 1, (case["nodes"], case["row_bytes"] // 4), generator=gen, device="cuda",
                          dtype=torch.int32)
    return _pinned(words.view(torch.uint8))


def _id_batches(case, gen):
    """Distinct ids per batch; nodes differ in how often they are met, as a sampler's inputs do."""
    n, k = case["nodes"], case["ids"]
    popularity = torch.rand(n, generator=gen, device="cuda").clamp_(min=1e-6).log_().mul_(-0.5)
    batches = []
    for _ in range(ID_BATCHES):
        noise = torch.rand(n, generator=gen, device="cuda").clamp_(1e-7, 1 - 1e-7).log_().neg_().log_().neg_()
        ids = torch.topk(popularity + noise, k, sorted=True).indices
        batches.append(ids[torch.randperm(k, generator=gen, device="cuda")].to(torch.int32))
    return batches


def prepare(case, seed):
    gen = _generator(seed)
    s = dict(case=case, at=0)
    kind = case["kind"]
    if kind == "sample":
        s["graph"], _ = _graph(case, gen, case["bits"], case["placement"])
        s["sampler"] = B.Sampler(s["graph"], case["seeds"], _fanouts(case))
        s["sampler"].workspace.zero_()
        s["seeds"] = _seed_batches(gen, case["nodes"], SEED_BATCHES, case["seeds"])
        s["rng"] = _rng_seeds(seed, SEED_BATCHES)
    elif kind in ("cache", "tier"):
        feats = s["features"] = _features(case, gen)
        if kind == "cache":
            s["cache"] = B.Cache(case["capacity"], feats)
        else:
            s["cache"] = B.Cache(case["capacity"], None, num_nodes=case["nodes"], row_bytes=case["row_bytes"])
            s["cache"].set_write_through(True)
            s["tier"] = B.HostTier(feats.numpy(), case["tier_rows"], case["ids"])
            s["tier"].set_copy_engine(case["transport"])
        s["batches"] = _id_batches(case, gen)
        s["rows"] = torch.empty((case["ids"], case["row_bytes"]), dtype=torch.uint8, device="cuda")
        s["slot"] = torch.empty(case["ids"], dtype=torch.int32, device="cuda")
        s["miss_pos"] = torch.empty(case["ids"], dtype=torch.int32, device="cuda")
        for _ in range(ID_BATCHES):      # a training run is in its steady state: the cache has filled
            run(s)
    elif kind == "epoch":
        s["graph"], _ = _graph(case, gen)
        feats = s["features"] = _features(case, gen)
        s["cache"] = B.Cache(case["cache_rows"], None if case["staged"] else feats, num_nodes=case["nodes"],
                             row_bytes=case["row_bytes"])
        s["pipe"] = NativePipeline(s["graph"], s["cache"], case["batch"], _fanouts(case), case["row_bytes"])
        if case["staged"]:
            s["tier"] = B.HostTier(feats.numpy(), 0, s["pipe"].cap)
            s["tier"].set_copy_engine(2)
            s["pipe"].tier = s["tier"]
        for t in (s["pipe"].out_rows, s["pipe"].out_slot, *[x.workspace for x in s["pipe"].samplers]):
            t.zero_()
        s["seeds"] = _seed_batches(gen, case["nodes"], SEED_BATCHES, case["batch"])
        s["rng"] = _rng_seeds(seed, SEED_BATCHES)
        run(s)
    else:
        s["graph"], _ = _graph(case, gen)
        n, t, k = case["nodes"], case["train"], case["sequences"]
        s["train"] = torch.randperm(n, generator=gen, device="cuda")[:t].to(torch.int32).cpu().numpy()
        s["roots"] = torch.randint(0, n, (k,), generator=gen, device="cuda").cpu().numpy()
        s["shifts"] = torch.randint(0, t, (k,), generator=gen, device="cuda").cpu().numpy()
    torch.cuda.synchronize()
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    at = s["at"]
    s["at"] = at + 1
    if kind == "sample":
        b = at % SEED_BATCHES
        sb = s["sampler"].sample(s["seeds"][b], s["rng"][b] ^ (at // SEED_BATCHES))
        torch.cuda.current_stream().synchronize()       # the sizes of the blocks
        n, nnz = sb.sizes()
        # the arrays as the library hands them out, at their upper bounds (what lies beyond the sizes is not written)
        out = [n, nnz, sb.input_nodes()]
        for h in range(len(nnz)):
            out += [sb.row_ptr(h, sb.struct.cap_nodes[h]), sb.col_local(h, sb.struct.cap_edges[h])]
        return out
    if kind == "cache":
        ids, cache = s["batches"][at % ID_BATCHES], s["cache"]
        cache.lookup_gather(ids, case["ids"], s["rows"], s["slot"], s["miss_pos"])
        cache.insert_fifo(ids, s["miss_pos"], -1, s["rows"])
        cache.wait_rows()
        return [s["rows"], s["slot"], cache.n_hit_host]
    if kind == "tier":
        ids, cache = s["batches"][at % ID_BATCHES], s["cache"]
        hits = cache.lookup_gather_tiered(s["tier"], ids, case["ids"], s["rows"], s["slot"], s["miss_pos"])
        cache.insert_fifo(ids, s["miss_pos"], -1, s["rows"])
        cache.wait_rows()
        return [s["rows"], s["slot"], hits[0], hits[1]]
    if kind == "epoch":
        pipe, steps = s["pipe"], case["steps"]
        n_input, n_hit = pipe.run(s["seeds"], s["rng"], steps, first_step=at * steps)
        return dict(n_input=n_input, n_hit=n_hit, ids=pipe.last_ids, rows=pipe.out_rows, slots=pipe.out_slot)
    return B.order_proximity(s["graph"], s["train"], s["roots"], s["shifts"], case["train"])


# ------------------------------------------------------------------ what a pass cannot do without
def _sampled(case, seeds):
    """(frontier sizes, edges per hop) to expect: draws that land in a neighborhood met before repeat."""
    n, deg = case["nodes"], case["mean_degree"]
    sizes, edges = [float(seeds)], []
    for f in _fanouts(case):
        e = sizes[-1] * min(f, 0.75 * deg)
        edges.append(e)
        sizes.append(min(n, sizes[-1] + n * (1.0 - math.exp(-e / n))))
    return sizes, edges


def work(case):
    kind = case["kind"]
    if kind in ("sample", "epoch"):
        sizes, edges = _sampled(case, case["seeds"] if kind == "sample" else case["batch"])
        offset = case.get("bits", 32) // 8
        # per node its id and two offsets, per edge a column id read and a local id written, the blocks' row
        # pointers and the input nodes written
        one = sum(sizes[:-1]) * (4 + 2 * offset + 4) + sum(edges) * 8 + sizes[-1] * 4
        if kind == "sample":
            return {"bytes": one, "flops": 0}
        return {"bytes": case["steps"] * (one + sizes[-1] * (8 + 2 * case["row_bytes"])), "flops": 0}
    if kind in ("cache", "tier"):       # ids and slots, every row read once and written once
        return {"bytes": case["ids"] * (8 + 2 * case["row_bytes"]), "flops": 0}
    # every edge once, every node's offsets and its place in the order
    return {"bytes": case["sequences"] * (case["nodes"] * (4 * case["mean_degree"] + 12) + 4 * case["train"]), "flops": 0}


def tolerance(case):
    return "exact"      # ids, slots, counts and copied bytes
