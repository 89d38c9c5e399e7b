"""What the library is timed on: the work a program of offline-sampling training has it do.

Every case calls the public entry points of the package the way such a program does: buffers
and workspaces are made once per state and used again by every pass, and a pass starts from
the buffers the previous one left.  Five forms cover the entry points:

  step      one group of mini-batches through the whole path: sample_pack_group, then
            assemble_batches of every mini-batch (the benchmark's step on one stream)
  sample    sample_group alone, for a program that only wants the subgraphs
  pack      pack_group of node lists that came from another sampler
  assemble  assemble_batches of an existing packing result (an epoch over packed data)
  gather    gather_rows: filling a cache table, or individual packing
  freq      cache_by_frequency over a sampled group (cache configuration)
  minhash   minhash_order of the accessed, uncached nodes (disk-cache reordering)

Graphs are synthetic with R-MAT's marginals: node IDs are drawn bit by bit (a bit is 0 with
probability `skew`; 0.76 is R-MAT's 0.57 + 0.19, 0.5 gives a uniform graph), out-degrees are
Poisson with mean `deg` times the same weights, and IDs are then scattered by a multiplicative
permutation.  Features are N(0,1); the path treats rows as opaque bytes.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2405_05231_amd as dg

DEV = "cuda"
OUT_BUFFERS = 8  # output buffers the assembly uses in turn
MAX_LIST = 1 << 26  # entries of all node lists of a group
SIZES = {"f32": 4, "f16": 2, "u8": 1}


def listed():
    return [
        # one small group of four 64-seed mini-batches on a 10,000-node graph (workload T):
        # nothing but launches and round trips
        step("step-tiny", n=10_000, deg=10, skew=0.5, batches=4, seeds=64, fanouts="5,5", dim=16,
             cache=10.0),
        # one mini-batch at a time (inference on arriving requests)
        step("step-single", n=1_000_000, deg=16, batches=1, seeds=1024, fanouts="15,10,5",
             dim=128, cache=10.0),
        # a 1M-node graph, 32 mini-batches (workload M1)
        step("step-1m", n=1_000_000, deg=16, batches=32, seeds=1024, fanouts="15,10,5", dim=128,
             cache=10.0),
        # the flagship shape (L100: 512-byte rows, 64 mini-batches, three hops, 5% cached) on a
        # graph of a size that several states of it fit on the card
        step("step-large", n=32_000_000, deg=16, batches=64, seeds=1024, fanouts="15,10,5",
             dim=128, cache=5.0),
        # wide fp16 rows and two hops (W120)
        step("step-wide", n=12_000_000, deg=14, batches=64, seeds=1024, fanouts="25,15", dim=768,
             dtype="f16", cache=2.0),
        # a heavy tail, large fan-outs and 1 KiB rows (H65)
        step("step-heavy", n=8_000_000, deg=28, skew=0.75, batches=8, seeds=1024,
             fanouts="20,15,10", dim=256, cache=10.0),
        # subgraphs only, with sample_group's defaults (hash relabelling)
        case("sample-default", "sample", n=8_000_000, deg=16, skew=0.76, batches=16, seeds=1024,
             fanouts="15,10,5", layered=False, direct=False),
        # lists of another sampler, in any order, with the group's unique set; 400-byte rows
        # (100 fp32 features)
        case("pack-lists", "pack", n=8_000_000, skew=0.76, batches=32, draws=200_000, dim=100,
             dtype="f32", cache=5.0, unique=True),
        # rows that are no multiple of 16 bytes (385 fp32 features, 1540 bytes)
        case("assemble-ragged", "assemble", n=2_000_000, skew=0.76, batches=8, draws=150_000,
             dim=385, dtype="f32", cache=5.0),
        # a cache table of 200-byte rows (100 fp16 features)
        case("gather-narrow", "gather", n=8_000_000, rows=1_000_000, dim=100, dtype="f16"),
        # which nodes to cache, from a group's accesses on a large graph
        case("freq-cache", "freq", n=50_000_000, skew=0.76, batches=64, draws=200_000, cache=5.0),
        # the order of the disk cache's entries
        case("minhash", "minhash", n=32_000_000, skew=0.76, batches=64, draws=200_000, cache=5.0,
             hashes=2),
    ]


def case(name, form, **kw):
    return dict(kw, form=form, **({"name": name} if name else {}))


def step(name, n, deg, batches, seeds, fanouts, dim, cache, skew=0.76, dtype="f32", direct=True):
    return case(name, "step", n=n, deg=deg, skew=skew, batches=batches, seeds=seeds,
                fanouts=fanouts, dim=dim, dtype=dtype, cache=cache, direct=direct)


def draw(rng):
    """One more case of the listed ranges."""
    limit = max(work(c)["bytes"] for c in listed())
    while True:
        c = draw_any(rng)
        if fits(c) and work(c)["bytes"] <= limit:
            return c


def log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw_any(rng):
    form = rng.choice(["step", "step", "step", "step", "sample", "sample", "pack", "assemble",
                       "gather", "freq", "minhash"])
    skew = rng.choice([0.5, 0.75, 0.76])
    dtype = rng.choice(["f32", "f32", "f32", "f16", "u8"])
    dim = rng.choice([16, 32, 64, 100, 128, 128, 256, 300, 385, 602, 768, 1024])
    batches = log_int(rng, 1, 64)
    cache = rng.choice([0.0, 1.0, 2.0, 5.0, 10.0, 30.0])
    if form in ("step", "sample"):
        fanouts = rng.choice(["5,5", "10,10", "15,10,5", "15,10,5", "25,15", "20,15,10", "10",
                              "10,10,10", "40,10"])
        c = dict(n=log_int(rng, 10_000, 32_000_000), deg=rng.choice([4, 8, 14, 16, 28]),
                 skew=skew, batches=batches, seeds=log_int(rng, 32, 4096), fanouts=fanouts)
        if form == "sample":
            return case(None, "sample", layered=rng.random() < 0.4, direct=rng.random() < 0.5, **c)
        return step(None, dim=dim, dtype=dtype, cache=cache, direct=rng.random() < 0.8, **c)
    if form == "gather":
        n = log_int(rng, 10_000, 16_000_000)
        return case(None, "gather", n=n, rows=log_int(rng, 1000, min(n, 4_000_000)), dim=dim,
                    dtype=dtype)
    n = log_int(rng, 10_000, 50_000_000 if form in ("freq", "minhash") else 16_000_000)
    c = dict(n=n, skew=skew, batches=batches, draws=log_int(rng, 500, 400_000), cache=cache)
    if form == "freq":
        return case(None, "freq", **c)
    if form == "minhash":
        return case(None, "minhash", hashes=rng.choice([1, 2, 5]), **c)
    if form == "pack":
        return case(None, "pack", dim=dim, dtype=dtype, unique=rng.random() < 0.5, **c)
    return case(None, "assemble", dim=dim, dtype=dtype, **c)


def fits(c):
    """Whether three states of the case fit the card, and its seeds the graph."""
    rows = c["n"] * row_bytes(c) if "dim" in c else 0
    if rows > 20e9:
        return False
    if c["form"] not in ("step", "sample"):
        return True
    if c["seeds"] > c["n"] // 8 or c["n"] * c["deg"] > 6e8:
        return False
    node_cap, edge_cap = dg.sample_bounds(c["n"], int(c["n"] * c["deg"] * 1.1), c["seeds"],
                                          fanouts(c), layered=c.get("layered", False))
    return c["batches"] * max(node_cap, edge_cap) <= MAX_LIST and (
        "dim" not in c or work(c)["bytes"] <= 16e9)


def fanouts(c):
    return [int(f) for f in c["fanouts"].split(",")]


def row_bytes(c):
    return c["dim"] * SIZES[c["dtype"]]


# ---------------------------------------------------------------------------- inputs
def bits_of(n):
    return max(2, math.ceil(math.log2(n)))


def generator(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + stream)
    return g


def half_tables(n, skew):
    """Bit widths and cumulative weights of the high and low halves of an ID."""
    bits = bits_of(n)
    out = []
    for w in (bits - bits // 2, bits // 2):
        ones = torch.tensor([bin(i).count("1") for i in range(1 << w)], dtype=torch.float64)
        p = skew ** (w - ones) * (1 - skew) ** ones
        out.append((w, p.to(DEV), torch.cumsum(p, 0).float().to(DEV)))
    return out


def scatter(ids, n):
    """Multiplicative permutation of [0, n)."""
    m = int(n * 0.6180339887) | 1
    while math.gcd(m, n) != 1:
        m += 2
    return (ids * m) % n


def draw_ids(count, n, skew, g):
    """`count` node IDs of the graph's marginal, int32."""
    (_, _, hi), (lw, _, lo) = half_tables(n, skew)
    out = torch.empty(count, dtype=torch.int32, device=DEV)
    for i in range(0, count, 1 << 26):
        k = min(1 << 26, count - i)
        a = torch.searchsorted(hi, torch.rand(k, device=DEV, generator=g)).clamp_(max=len(hi) - 1)
        b = torch.searchsorted(lo, torch.rand(k, device=DEV, generator=g)).clamp_(max=len(lo) - 1)
        out[i:i + k] = scatter(((a << lw) | b) % n, n).int()
    return out


def make_graph(c, seed):
    """CSR graph: (offsets int64, indices int32)."""
    n, g = c["n"], generator(seed, 1)
    (_, hi, _), (lw, lo, _) = half_tables(n, c["skew"])
    ids = torch.arange(n, device=DEV)
    weight = hi[ids >> lw] * lo[ids & ((1 << lw) - 1)]
    weight *= n * c["deg"] / float(weight.sum())
    deg = torch.zeros(n, dtype=torch.int64, device=DEV)
    deg[scatter(ids, n)] = torch.poisson(weight, generator=g).long()
    offsets = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(deg, 0, out=offsets[1:])
    return offsets, draw_ids(int(offsets[-1]), n, c["skew"], g)


def make_features(c, seed):
    n, g = c["n"], generator(seed, 2)
    if c["dtype"] == "u8":
        return torch.randint(0, 256, (n, c["dim"]), dtype=torch.uint8, device=DEV, generator=g)
    kind = torch.float32 if c["dtype"] == "f32" else torch.float16
    return torch.randn((n, c["dim"]), dtype=kind, device=DEV, generator=g)


def make_cache(c, popularity):
    """The top `cache` percent of the nodes by popularity: (cache_slot [N], nodes)."""
    n, rows = c["n"], int(c["n"] * c["cache"] / 100)
    order = torch.sort(popularity, descending=True, stable=True).indices[:rows].int()
    slot = torch.full((n,), -1, dtype=torch.int32, device=DEV)
    slot[order.long()] = torch.arange(rows, dtype=torch.int32, device=DEV)
    return slot, order


def make_lists(c, seed):
    """One node list per mini-batch from another sampler: distinct nodes in no order.
    (nodes int32 [B, stride], counts)."""
    g = generator(seed, 3)
    lists = []
    for _ in range(c["batches"]):
        u = torch.unique(draw_ids(c["draws"], c["n"], c["skew"], g))
        lists.append(u[torch.randperm(u.numel(), device=DEV, generator=g)])
    counts = np.array([u.numel() for u in lists], dtype=np.int64)
    nodes = torch.zeros((c["batches"], min(c["draws"], c["n"])), dtype=torch.int32, device=DEV)
    for b, u in enumerate(lists):
        nodes[b, :u.numel()] = u
    return nodes, counts


def make_membership(c, nodes, counts):
    mask = torch.zeros(c["n"], dtype=torch.int64, device=DEV)
    for b, k in enumerate(counts):
        ids = nodes[b, :int(k)].long()
        mask[ids] |= (1 << b) - (1 << 64 if b == 63 else 0)
    return mask


def list_popularity(c, nodes, counts):
    p = torch.zeros(c["n"], dtype=torch.int32, device=DEV)
    for b, k in enumerate(counts):
        p[nodes[b, :int(k)].long()] += 1
    return p


def buffer(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def capacities(c):
    """Rows that a program of this shape makes room for: (packed rows, longest list, distinct
    nodes, disk-cache entries), the expected counts with a margin."""
    pairs, unique, rows_read, rows_packed, _ = list_work(c, *population_share(c)[:2])

    def room(x):
        return int(1.3 * x) + 4096
    return (room(rows_packed), room(pairs / c["batches"]), room(unique),
            max(1, int(0.8 * max(rows_read, 0.1 * unique))))


def sample_state(c, seed, want_direct):
    """Graph, seeds, output buffers and workspace of a sampling program."""
    offsets, indices = make_graph(c, seed)
    n, B, S = c["n"], c["batches"], c["seeds"]
    candidates = torch.nonzero(offsets[1:] > offsets[:-1]).squeeze(1).int()
    g = generator(seed, 4)
    picks = []  # per mini-batch distinct seeds with at least one neighbour
    for _ in range(B):
        at = torch.randint(0, candidates.numel(), (4 * S + 64,), device=DEV, generator=g)
        u = torch.unique(candidates[at])
        if u.numel() < S:
            u = candidates
        picks.append(u[torch.randperm(u.numel(), device=DEV, generator=g)[:S]])
    S = min(p.numel() for p in picks)
    seeds = torch.stack([p[:S] for p in picks]).contiguous()
    fan = fanouts(c)
    layered = c.get("layered", False)
    node_cap, edge_cap = dg.sample_bounds(n, indices.numel(), S, fan, layered=layered)
    out = dg.SampleResult(
        nodes=torch.zeros((B, node_cap), dtype=torch.int32, device=DEV),
        hop_ptr=np.zeros((B, len(fan) + 2), dtype=np.int64),
        edge_src=torch.zeros((B, edge_cap), dtype=torch.int32, device=DEV),
        edge_dst=torch.zeros((B, edge_cap), dtype=torch.int32, device=DEV),
        edge_ptr=np.zeros((B, len(fan) + 1), dtype=np.int64), sizes={}, timing=None)
    flags = dg.sample_flags(layered=layered, direct=want_direct)
    ws = buffer(dg._L.dg_sample_workspace_bytes(n, B, node_cap, edge_cap, flags))
    return dict(offsets=offsets, indices=indices, seeds=seeds, fan=fan, rng_seed=seed * 977 + 5,
                out=out, ws=ws, layered=layered, direct=want_direct)


def pack_buffers(c, loc, ids_cap, rows=None, unique=None):
    B, R = c["batches"], row_bytes(c)
    return dg.PackResult(
        packed=None if rows is None else torch.zeros((max(rows, 1), R), dtype=torch.uint8,
                                                     device=DEV),
        packed_ids=torch.zeros(max(ids_cap, 1), dtype=torch.int32, device=DEV),
        packed_ptr=torch.zeros(B + 1, dtype=torch.int64, device=DEV),
        packed_ptr_host=np.zeros(B + 1, dtype=np.int64), loc=loc, unique=unique, sizes={},
        timing=None, row_bytes=R)


def output_buffers(c, rows):
    return [torch.zeros((max(rows, 1), row_bytes(c)), dtype=torch.uint8, device=DEV)
            for _ in range(min(OUT_BUFFERS, c["batches"]))]


def prepare(case, seed):
    c = dict(case)
    return {"form": c["form"], **PREPARE[c["form"]](c, seed)}


def prepare_step(c, seed):
    s = sample_state(c, seed, c["direct"])
    n, B = c["n"], c["batches"]
    s["feats"] = make_features(c, seed)
    in_degree = torch.bincount(s["indices"], minlength=n)
    s["slot"], order = make_cache(c, in_degree)
    s["cache"] = s["feats"][order.long()].contiguous()
    s["member"] = torch.zeros(n, dtype=torch.int64, device=DEV)
    node_cap = s["out"].nodes.shape[1]
    s["pack_ws"] = buffer(dg._L.dg_sample_pack_workspace_bytes(n, B, node_cap))
    loc = torch.zeros((B, node_cap), dtype=torch.int32, device=DEV)
    # a first pass without rows checks the capacities, and leaves the masks clear for the
    # passes that follow
    s["pack"] = pack_buffers(c, loc, B * node_cap)
    sr, pr = sample_and_pack(s, entry_clear=False, tables_only=True)
    rows, longest, _, _ = capacities(c)
    if pr.sizes["packed_rows"] > rows or int(sr.node_count.max()) > longest:
        raise RuntimeError("the case's capacities are too small")
    s["pack"] = pack_buffers(c, loc, rows, rows)
    s["outs"] = output_buffers(c, longest)
    return s


def sample_and_pack(s, entry_clear, tables_only=False):
    return dg.sample_pack_group(
        s["offsets"], s["indices"], s["seeds"], s["fan"], s["rng_seed"], s["feats"], s["slot"],
        out=s["out"], pack_out=s["pack"], tables_only=tables_only, workspace=s["ws"],
        pack_workspace=s["pack_ws"], membership=s["member"], direct=s["direct"],
        entry_clear=entry_clear, exit_clear=True)


def prepare_sample(c, seed):
    return sample_state(c, seed, c["direct"])


def prepare_pack(c, seed):
    nodes, counts = make_lists(c, seed)
    slot, _ = make_cache(c, list_popularity(c, nodes, counts))
    s = dict(nodes=nodes, counts=counts, feats=make_features(c, seed), slot=slot,
             unique=c["unique"])
    total = int(counts.sum())
    s["ws"] = buffer(dg._L.dg_pack_workspace_bytes(c["n"], c["batches"], total))
    rows, _, unique, _ = capacities(c)
    s["pack"] = pack_buffers(
        c, torch.zeros_like(nodes), rows, rows,
        torch.zeros(unique, dtype=torch.int32, device=DEV) if c["unique"] else None)
    return s


def prepare_assemble(c, seed):
    nodes, counts = make_lists(c, seed)
    slot, order = make_cache(c, list_popularity(c, nodes, counts))
    feats = make_features(c, seed)
    pack = dg.pack_group(feats, slot, nodes, counts)
    return dict(pack=pack, counts=counts, cache=feats[order.long()].contiguous(),
                outs=output_buffers(c, nodes.shape[1]))


def prepare_gather(c, seed):
    g = generator(seed, 5)
    ids = torch.randperm(c["n"], device=DEV, generator=g)[:c["rows"]].int()
    return dict(feats=make_features(c, seed), ids=ids,
                out=torch.zeros((c["rows"], row_bytes(c)), dtype=torch.uint8, device=DEV))


def prepare_freq(c, seed):
    nodes, counts = make_lists(c, seed)
    return dict(mask=make_membership(c, nodes, counts), batches=c["batches"],
                rows=int(c["n"] * c["cache"] / 100),
                ws=buffer(dg._L.dg_cache_workspace_bytes(c["n"])))


def prepare_minhash(c, seed):
    nodes, counts = make_lists(c, seed)
    mask = make_membership(c, nodes, counts)
    slot, _ = make_cache(c, list_popularity(c, nodes, counts))
    # the disk has room for so many of the accessed nodes, the uncached ones first
    entries = torch.cat([torch.nonzero((mask != 0) & (slot < 0)),
                         torch.nonzero((mask != 0) & (slot >= 0))]).squeeze(1).int()
    entries = entries[:capacities(c)[3]].clone()
    g = generator(seed, 6)
    perms = torch.stack([torch.randperm(c["batches"], device=DEV, generator=g)
                         for _ in range(c["hashes"])]).int().contiguous()
    return dict(mask=mask, entries=entries, perms=perms, batches=c["batches"],
                ws=buffer(dg._L.dg_minhash_workspace_bytes(entries.numel())))


PREPARE = {"step": prepare_step, "sample": prepare_sample, "pack": prepare_pack,
           "assemble": prepare_assemble, "gather": prepare_gather, "freq": prepare_freq,
           "minhash": prepare_minhash}


# ---------------------------------------------------------------------------- the call
def run(s):
    return RUN[s["form"]](s)


def sampled(sr):
    return dict(nodes=sr.nodes, hop_ptr=sr.hop_ptr, edge_src=sr.edge_src, edge_dst=sr.edge_dst,
                edge_ptr=sr.edge_ptr)


def run_step(s):
    sr, pr = sample_and_pack(s, entry_clear=True)
    dg.assemble_batches(s["cache"], pr, sr.node_count, s["outs"])
    return dict(sampled(sr), loc=pr.loc, packed=pr.packed, packed_ids=pr.packed_ids,
                packed_ptr=pr.packed_ptr, outs=s["outs"])


def run_sample(s):
    return sampled(dg.sample_group(s["offsets"], s["indices"], s["seeds"], s["fan"],
                                   s["rng_seed"], out=s["out"], workspace=s["ws"],
                                   layered=s["layered"], direct=s["direct"]))


def run_pack(s):
    pr = dg.pack_group(s["feats"], s["slot"], s["nodes"], s["counts"], with_unique=s["unique"],
                       out=s["pack"], workspace=s["ws"])
    return dict(loc=pr.loc, packed=pr.packed, packed_ids=pr.packed_ids,
                packed_ptr=pr.packed_ptr, unique=pr.unique)


def run_assemble(s):
    dg.assemble_batches(s["cache"], s["pack"], s["counts"], s["outs"])
    return s["outs"]


def run_gather(s):
    return dg.gather_rows(s["feats"], s["ids"], out=s["out"])


def run_freq(s):
    slot, nodes, cached = dg.cache_by_frequency(s["mask"], s["batches"], s["rows"],
                                                workspace=s["ws"])
    return dict(slot=slot, nodes=nodes, cached=cached)


def run_minhash(s):
    order, signature = dg.minhash_order(s["mask"], s["batches"], s["entries"], s["perms"],
                                        workspace=s["ws"])
    return dict(order=order, signature=signature)


RUN = {"step": run_step, "sample": run_sample, "pack": run_pack, "assemble": run_assemble,
       "gather": run_gather, "freq": run_freq, "minhash": run_minhash}


# ---------------------------------------------------------------------------- its cost
class Population:
    """The nodes by class (number of 1 bits in the unscattered ID): expected counts follow
    from the classes' sizes and weights without sampling anything."""

    def __init__(self, c):
        bits = bits_of(c["n"])
        ones = np.arange(bits + 1)
        self.count = np.array([math.comb(bits, int(k)) for k in ones]) * c["n"] / 2.0 ** bits
        p = c["skew"] ** (bits - ones) * (1 - c["skew"]) ** ones
        self.p = p / float((p * self.count).sum())

    def distinct(self, draws, seen=0.0):
        """Share of each class hit after `draws` draws, `seen` of it hit before."""
        return 1 - (1 - seen) * np.exp(-draws * self.p)

    def cached(self, share):
        """Share of each class in a cache of `share` of the nodes, most popular first."""
        room, out = share * self.count.sum(), np.zeros_like(self.count)
        for k in np.argsort(-self.p):
            out[k] = min(1.0, room / self.count[k])
            room -= out[k] * self.count[k]
            if room <= 0:
                break
        return out


def mean_draws(lam, f):
    """E[min(Poisson(lam), f)]."""
    if f < 0:
        return lam
    out, term, below = 0.0, math.exp(-min(lam, 700.0)), 0.0
    for k in range(f):
        out += k * term
        below += term
        term *= lam / (k + 1)
    return out + f * max(0.0, 1 - below)


def list_work(c, pop, share):
    """Lists that hold `share` of each class: entries, distinct nodes, distinct uncached nodes,
    uncached entries, distinct cached nodes (of the whole group)."""
    B, count = c["batches"], pop.count
    union = 1 - (1 - share) ** B
    cached = pop.cached(c.get("cache", 0.0) / 100)
    return (B * (share * count).sum(), (union * count).sum(), (union * (1 - cached) * count).sum(),
            B * (share * (1 - cached) * count).sum(), (union * cached * count).sum())


def population_share(c):
    """(the population, the share of each class in one mini-batch's list, the bytes of its
    sampling over all mini-batches)."""
    pop = Population(c)
    if "fanouts" not in c:
        return pop, pop.distinct(c["draws"]), 0.0
    total, lam = 0.0, pop.p * c["n"] * c["deg"]
    live = 1 - np.exp(-lam)
    share = live * min(1.0, c["seeds"] / float((live * pop.count).sum()))
    front = share * pop.count
    for hop, f in enumerate(fanouts(c)):
        draws = float(sum(x * mean_draws(v, f) for x, v in zip(front, lam)))
        if hop == 0:
            draws /= float((front * live).sum() / front.sum())  # seeds have neighbours
        now = pop.distinct(draws, share)
        total += c["batches"] * (draws * (4 + 8) + 16 * float(front.sum()))
        front = (now if c.get("layered") else now - share) * pop.count
        share = now
    return pop, share, total


def work(case):
    """What a pass cannot do without: each input element it needs read once and each output
    element written once."""
    c, form = dict(case), case["form"]
    if form == "gather":
        return {"bytes": float(c["rows"]) * (2 * row_bytes(c) + 4), "flops": 0}
    if form == "freq":
        return {"bytes": 12.0 * c["n"] + 4 * c["n"] * c["cache"] / 100, "flops": 0}
    pop, share, total = population_share(c)
    pairs, unique, rows_read, rows_packed, cached_read = list_work(c, pop, share)
    if form == "sample":
        return {"bytes": total + 4 * pairs, "flops": 0}
    if form == "minhash":  # entry and membership word read, order and signature written
        return {"bytes": 20.0 * capacities(c)[3], "flops": 0}
    R = row_bytes(c)
    if form == "assemble":  # tables, each cache and packed row once, each output row
        return {"bytes": 4 * pairs + (cached_read + rows_packed + pairs) * R, "flops": 0}
    # packing: lists (read or written), cache slots, tables, packed IDs, rows
    total += 4 * pairs + 4 * unique + 4 * pairs + 4 * rows_packed + (rows_read + rows_packed) * R
    if form == "pack":
        return {"bytes": total + (4 * unique if c["unique"] else 0), "flops": 0}
    return {"bytes": total + 4 * pairs + (cached_read + rows_packed + pairs) * R, "flops": 0}


def tolerance(case):
    """Every output is an integer or a copied byte."""
    return "exact"
