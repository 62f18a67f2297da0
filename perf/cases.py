"""The work a user of this framework has it do, as timed cases.

Six kinds of call, each through the package's public entry points:

* ``sample``     one multi-hop sampling call (``Sampler.run``) over a batch or
                 a super-batch of consecutive batches;
* ``build``      the T-CSR of a COO (``tcsr_build``), workspace included;
* ``gather``     feature / state rows of sampled slots (``gather``);
* ``time``       time encoding of sampled slots (``time_encode``);
* ``mfg``        the blocks of every hop of a sampling call
                 (``tgl_mfg_export`` of the C ABI into buffers a program
                 keeps, since a block's sizes stay on the device);
* ``minibatch``  all of it for one training mini-batch: sample, blocks, state
                 lookup, time encoding.

Graphs have the shapes of the paper's datasets, drawn on the GPU from the
seed: ``wiki`` (bipartite, Zipf sides, times in seconds), ``gdelt`` (few
nodes, very long runs, integer time buckets), ``mag`` (citations, publication
years) and ``powerlaw`` (Zipf over one ranking, float times, the COO
shuffled).  Every list is chronological except the shuffled one.
"""
import ctypes
import math

import torch

import paper_2203_14883_amd as tgl
from paper_2203_14883_amd import binding

# Times of each family span [0, SPAN) (mag: publication years 1900..2020).
SPAN = {"wiki": 2.7e6, "gdelt": 170_000.0, "powerlaw": 1.0e8, "mag": 121.0}
# Valid share of hop 1's and of the later hops' slots, as sampled at the
# listed sizes: it sets how many roots a later hop has.
VALID = {"wiki": (0.95, 0.96), "gdelt": (1.0, 1.0), "mag": (0.51, 0.54), "powerlaw": (0.63, 0.93)}


def listed():
    return [
        # TGN on Wikipedia: one training batch, the smallest call there is
        dict(name="recent_wiki_batch", kind="sample", graph="wiki", nodes=9227, edges=157_474, batch=600, batches=1,
             fanouts="10", mode="recent", snapshots=1, length=0.0),
        # TGAT on Wikipedia: one training batch, two hops
        dict(name="uniform2_wiki_batch", kind="sample", graph="wiki", nodes=9227, edges=157_474, batch=600, batches=1,
             fanouts="10,10", mode="uniform", snapshots=1, length=0.0),
        # DySAT-like sampling (two hops inside three snapshots), 60,000-edge batch
        dict(name="snapshots2_powerlaw", kind="sample", graph="powerlaw", nodes=10_000_000, edges=100_000_000,
             batch=60_000, batches=1, fanouts="10,10", mode="uniform", snapshots=3, length=1.0e6),
        # GDELT at full size, 64 batches a call: most-recent in three snapshots
        dict(name="snapshots1_gdelt", kind="sample", graph="gdelt", nodes=16_682, edges=191_000_000, batch=4000,
             batches=64, fanouts="10", mode="recent", snapshots=3, length=1.0e4),
        # MAG's ratio of nodes to edges, 64 batches a call: TGAT over citations
        dict(name="uniform2_mag", kind="sample", graph="mag", nodes=37_400_000, edges=400_000_000, batch=4000,
             batches=64, fanouts="10,10", mode="uniform", snapshots=1, length=0.0),
        # a small graph's T-CSR, as a user rebuilds it when edges arrive
        dict(name="build_wiki", kind="build", graph="wiki", nodes=9227, edges=157_474, eid=False),
        # a large graph's T-CSR from an edge list in no order, float times
        dict(name="build_powerlaw", kind="build", graph="powerlaw", nodes=10_000_000, edges=100_000_000, eid=True),
        # a citation graph's T-CSR from a chronological edge list, few times
        dict(name="build_mag", kind="build", graph="mag", nodes=18_700_000, edges=200_000_000, eid=False),
        # MAG's 768-dim bf16 node features of 4M sampled slots
        dict(name="gather_mag_bf16", kind="gather", rows=12_000_000, slots=1 << 22, dims="768", dtype="bf16"),
        # TGL's 100-dim encoder over 8M sampled slots
        dict(name="time_f32", kind="time", slots=1 << 23, dim=100, dtype="f32"),
        # both hops' blocks of a 64-batch citation step
        dict(name="mfg_mag", kind="mfg", graph="mag", nodes=9_350_000, edges=100_000_000, batch=4000, batches=64,
             fanouts="10,10", mode="uniform", snapshots=1, length=0.0),
        # a whole TGN/TGAT mini-batch on Wikipedia: sample, blocks, memory,
        # mailbox and edge features, time encoding
        dict(name="minibatch_wiki", kind="minibatch", graph="wiki", nodes=9227, edges=157_474, batch=600, batches=1,
             fanouts="10,10", mode="uniform", snapshots=1, length=0.0),
    ]


def _log(rng, lo, hi):
    """A whole number spread over [lo, hi] by its logarithm, odd ones included."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST_EDGES = {"wiki": 3_000_000, "gdelt": 100_000_000, "mag": 150_000_000, "powerlaw": 60_000_000}


def _draw_graph(rng):
    graph = rng.choice(["wiki", "gdelt", "mag", "powerlaw"])
    edges = _log(rng, 20_000, _MOST_EDGES[graph])
    per_node = {"wiki": (8, 30), "gdelt": (500, 12_000), "mag": (6, 15), "powerlaw": (6, 20)}[graph]
    nodes = max(64, int(edges / rng.uniform(*per_node)))
    return dict(graph=graph, nodes=nodes, edges=edges)


def _draw_sample(rng):
    c = _draw_graph(rng)
    hops = rng.choice([1, 2, 2, 3])
    most = {1: 20, 2: 15, 3: 8}[hops]
    fan = [rng.randint(4, most) for _ in range(hops)]
    snapshots = rng.choice([1, 1, 1, 2, 3, 5])
    length = 0.0
    if snapshots > 1 or rng.random() < 0.2:
        length = SPAN[c["graph"]] * rng.uniform(0.01, 0.1)
    # slots of the last hop at most those of the largest listed case
    room = 60_000_000 // (snapshots * math.prod(fan) * 3)
    edges = _log(rng, 50, max(51, min(256_000, room, c["edges"] // 2)))
    batches = rng.choice([1, 1, 8]) if edges >= 800 else 1
    c.update(batch=max(1, edges // batches), batches=batches, fanouts=",".join(map(str, fan)),
             mode=rng.choice(["recent", "uniform", "uniform"]), snapshots=snapshots, length=length)
    return c


def draw(rng):
    kind = rng.choice(["sample", "sample", "sample", "build", "build", "gather", "time", "mfg", "minibatch"])
    if kind == "build":
        return dict(kind=kind, eid=rng.random() < 0.5, **_draw_graph(rng))
    if kind == "gather":
        dims = rng.choice([[100], [172], [768], [100, 172], [100, 372, 172], [188], [416, 188]])
        slots = _log(rng, 2_000, 3_000_000)
        return dict(kind=kind, rows=_log(rng, 5_000, 3_000_000), slots=slots, dims=",".join(map(str, dims)),
                    dtype=rng.choice(["f32", "bf16"]) if all(d % 8 == 0 for d in dims) else "f32")
    if kind == "time":
        return dict(kind=kind, slots=_log(rng, 2_000, 6_000_000), dim=rng.choice([100, 100, 64, 128, 172, 33, 101]),
                    dtype=rng.choice(["f32", "f32", "bf16"]))
    if kind == "minibatch":
        edges = _log(rng, 50_000, 3_000_000)
        fan = rng.choice([[10], [10, 10], [5, 8], [20]])
        return dict(kind=kind, graph="wiki", nodes=int(edges / rng.uniform(8, 30)), edges=edges,
                    batch=rng.choice([200, 600, 601, 1000, 4000]), batches=1, fanouts=",".join(map(str, fan)),
                    mode=rng.choice(["recent", "uniform"]), snapshots=1, length=0.0)
    return dict(kind=kind, **_draw_sample(rng))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------

def _zipf(n, s, size, gen, dev):
    """Node ids of [0, n) with about P(rank r) ~ r^-s (the inverse of the
    continuous law on [1, n + 1)), ranks in a random order."""
    ids = torch.randperm(n, generator=gen, device=dev, dtype=torch.int32)
    out = torch.empty(size, dtype=torch.int32, device=dev)
    for b in range(0, size, 1 << 25):
        e = min(size, b + (1 << 25))
        u = torch.rand(e - b, dtype=torch.float64, generator=gen, device=dev)
        x = u.mul_((n + 1.0) ** (1.0 - s) - 1.0).add_(1.0).pow_(1.0 / (1.0 - s))
        out[b:e] = ids[x.long().sub_(1).clamp_(0, n - 1)]
    return out


def _sorted_times(n, hi, gen, dev, whole):
    t = torch.rand(n, dtype=torch.float32, generator=gen, device=dev) * hi
    if whole:
        t.floor_()
    return t.sort().values


def _edges(case, gen, dev):
    """(src, dst, ts) of the case's graph in chronological order, and the node
    range negatives are drawn from."""
    n, m, graph = case["nodes"], case["edges"], case["graph"]
    if graph == "wiki":                                   # users first, one item per eight users
        users = max(1, n * 8 // 9)
        src = _zipf(users, 1.1, m, gen, dev)
        dst = _zipf(n - users, 1.3, m, gen, dev) + users
        return src, dst, _sorted_times(m, SPAN[graph], gen, dev, False), (users, n)
    if graph in ("gdelt", "powerlaw"):
        both = _zipf(n, 1.05 if graph == "gdelt" else 1.2, 2 * m, gen, dev)
        return both[:m].clone(), both[m:].clone(), _sorted_times(m, SPAN[graph], gen, dev, graph == "gdelt"), (0, n)
    # mag: papers ordered by year (more each year), heavy-tailed reference
    # lists to papers of the same or an earlier year
    ycdf = torch.pow(torch.tensor(1.04, dtype=torch.float64), torch.arange(121, dtype=torch.float64)).cumsum(0).to(dev)
    ycdf /= ycdf[-1].clone()
    year = torch.searchsorted(ycdf, torch.rand(n, dtype=torch.float64, generator=gen, device=dev)).clamp_(max=120)
    year = year.sort().values
    upto = torch.searchsorted(year, torch.arange(121, device=dev), right=True)      # papers of year <= y
    paper = torch.randperm(n, generator=gen, device=dev, dtype=torch.int32)
    deg = torch.rand(n, dtype=torch.float64, generator=gen, device=dev).clamp_(min=1e-9).pow_(-1.0 / 2.1)
    deg = deg.mul_(1.0e3).clamp_(max=1.0e7).long()
    deg = deg * m // int(deg.sum())
    short = m - int(deg.sum())                            # below n: each floor drops less than one
    deg[torch.randperm(n, generator=gen, device=dev)[:short]] += 1
    src = torch.repeat_interleave(paper, deg, output_size=m)
    y = torch.repeat_interleave(year, deg, output_size=m)
    pick = (torch.rand(m, dtype=torch.float64, generator=gen, device=dev) * upto[y]).long()
    dst = paper[pick]
    del pick
    return src, dst, (y + 1900).float(), (0, n)


def _gen(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed))


def _roots(case, src, dst, ts, neg, gen, dev):
    """Consecutive batches of [sources; destinations; negatives] from a random
    edge on: (roots, root times, index of the first root)."""
    per, nb = case["batch"], case["batches"]
    need = per * nb
    m = src.shape[0]
    e0 = int(torch.randint(m // 2, m - need + 1, (1,), generator=gen, device=dev)) if m - need > m // 2 else m - need
    e0 -= e0 % per if e0 >= per else 0
    s, d, t = (x[e0:e0 + need].view(nb, 1, per) for x in (src, dst, ts))
    g = torch.randint(neg[0], neg[1], (nb, 1, per), generator=gen, device=dev, dtype=torch.int32)
    return torch.cat([s, d, g], 1).reshape(-1).contiguous(), t.expand(nb, 3, per).reshape(-1).contiguous(), 3 * e0


def _fan(case):
    return tuple(int(k) for k in case["fanouts"].split(","))


def _prepare_sampler(case, gen, dev):
    src, dst, ts, neg = _edges(case, gen, dev)
    roots, rts, base = _roots(case, src, dst, ts, neg, gen, dev)
    if case["graph"] == "powerlaw":
        order = torch.randperm(src.shape[0], generator=gen, device=dev)
        src, dst, ts = src[order], dst[order], ts[order]
        g = tgl.tcsr_build(src, dst, ts, order, case["nodes"], True)
        del order
    else:
        g = tgl.tcsr_build(src, dst, ts, None, case["nodes"], True)
    smp = tgl.Sampler(roots.shape[0], _fan(case), case["snapshots"], device=dev)
    # a call writes the valid prefix of each later hop's buffers: what lies
    # past it is left as it was, so it is given a value once
    for bufs in (smp.nbr, smp.eid, smp.ts, smp.dt, smp.parent):
        for b in bufs:
            if b is not None:
                b.zero_()
    return dict(g=g, smp=smp, roots=roots, root_ts=rts, base=base, mode=case["mode"],
                length=case["length"] or math.inf, seed=7)


def _block_buffers(smp, h, dev):
    """One hop's block at capacity, with the export's workspace.  Past its
    valid prefix a block is left as it was."""
    k = smp.fanouts[h]
    groups = smp.caps[h] * (smp.snapshots if h == 0 else 1)

    def z(n, dtype):
        return torch.zeros(n, dtype=dtype, device=dev)

    out = dict(indptr=z(groups + 1, torch.int64), edge_dst=z(groups * k, torch.int64),
               edge_eid=z(groups * k, torch.int64), edge_dt=z(groups * k, torch.float32),
               src_nid=z(groups * (k + 1), torch.int32), src_ts=z(groups * (k + 1), torch.float32),
               sizes=z(2, torch.int64))
    c = binding.c_mfg(*(out[f].data_ptr() for f in ("indptr", "edge_dst", "edge_eid", "edge_dt", "src_nid", "src_ts",
                                                    "sizes")))
    return dict(out=out, c=c, groups=groups, ws=z(max(1, tgl.lib().tgl_mfg_workspace(groups)), torch.uint8))


def _encoder(dim, gen, dev):
    """TGL's frequency ladder, and phases as they are after some training."""
    omega = torch.pow(torch.tensor(10.0, dtype=torch.float64), -9.0 * torch.arange(dim, dtype=torch.float64)
                      / max(1, dim - 1)).float().to(dev)
    phi = torch.randn(dim, generator=gen, device=dev) * 0.1
    return omega, phi


def _slots(n, gen, dev, valid):
    """Which of n slots are valid: whole groups of ten, as a uniform hop gives."""
    keep = torch.rand((n + 9) // 10, generator=gen, device=dev) < valid
    return keep.repeat_interleave(10)[:n]


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = _gen(seed, dev)
    kind = case["kind"]
    if kind == "build":
        src, dst, ts, _ = _edges(case, gen, dev)
        if case["graph"] == "powerlaw":
            order = torch.randperm(src.shape[0], generator=gen, device=dev)
            src, dst, ts = src[order], dst[order], ts[order]
        else:
            order = None
        eid = None
        if case["eid"]:
            eid = order if order is not None else torch.arange(src.shape[0], device=dev) * 2 + 1
        return dict(kind=kind, src=src, dst=dst, ts=ts, eid=eid, nodes=case["nodes"])
    if kind == "gather":
        n, rows = case["slots"], case["rows"]
        dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
        dims = [int(d) for d in case["dims"].split(",")]
        tables = [(torch.empty(rows, d, dtype=dtype, device=dev).normal_(generator=gen), "node" if i < 2 else "edge")
                  for i, d in enumerate(dims)]
        ok = _slots(n, gen, dev, 0.5)
        nbr = torch.randint(0, rows, (n,), generator=gen, device=dev, dtype=torch.int32)
        eid = torch.randint(0, rows, (n,), generator=gen, device=dev)
        return dict(kind=kind, nbr=torch.where(ok, nbr, -1), eid=torch.where(ok, eid, -1), tables=tables)
    if kind == "time":
        n = case["slots"]
        dt = torch.empty(n, device=dev).exponential_(1.0 / 2.0e5, generator=gen)
        omega, phi = _encoder(case["dim"], gen, dev)
        return dict(kind=kind, dt=torch.where(_slots(n, gen, dev, 0.8), dt, -1.0), omega=omega, phi=phi,
                    dtype=torch.bfloat16 if case["dtype"] == "bf16" else torch.float32)
    s = _prepare_sampler(case, gen, dev)
    s["kind"] = kind
    if kind in ("mfg", "minibatch"):
        s["blocks"] = [_block_buffers(s["smp"], h, dev) for h in range(len(s["smp"].fanouts))]
    if kind == "mfg":
        _sample(s)
    if kind == "minibatch":
        n, m, smp = case["nodes"], case["edges"], s["smp"]
        s["tables"] = [(torch.randn(n, 100, generator=gen, device=dev), "node"),        # node memory
                       (torch.randn(n, 372, generator=gen, device=dev), "node"),        # mailbox: two memories, features
                       (torch.randn(m, 172, generator=gen, device=dev), "edge")]        # edge features
        s["omega"], s["phi"] = _encoder(100, gen, dev)
        s["rows"] = [[torch.zeros(b.shape[0], t.shape[1], device=dev) for t, _ in s["tables"]] for b in smp.nbr]
        s["enc"] = [torch.zeros(b.shape[0], 100, device=dev) for b in smp.nbr]
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------

def _sample(s):
    s["smp"].run(s["g"], s["roots"], s["root_ts"], s["mode"], s["length"], s["seed"], s["base"])


def _blocks(s):
    """Enqueues the export of every hop's block into the state's buffers."""
    smp, lib = s["smp"], tgl.lib()
    stream = torch.cuda.current_stream().cuda_stream
    for h, b in enumerate(s["blocks"]):
        prev = ctypes.byref(smp._outs[h - 1]) if h else None
        rc = lib.tgl_mfg_export(ctypes.byref(smp._outs[h]), prev, s["roots"].data_ptr(), s["root_ts"].data_ptr(),
                                smp.counts.data_ptr() + 8 * h, smp.snapshots if h == 0 else 1, smp.fanouts[h],
                                b["groups"], ctypes.byref(b["c"]), b["ws"].data_ptr(), b["ws"].numel(), stream)
        if rc:
            raise tgl.TglError(rc, "tgl_mfg_export")


def run(state):
    kind = state["kind"]
    if kind == "build":
        g = tgl.tcsr_build(state["src"], state["dst"], state["ts"], state["eid"], state["nodes"], True)
        return dict(indptr=g.indptr, entries=g.entries, ts=g.ts, nodes=g.nodes, ts_index=g.ts_index, hist=g.hist,
                    dir=g.dir)
    if kind == "gather":
        return tgl.gather(state["nbr"], state["eid"], state["tables"])
    if kind == "time":
        return tgl.time_encode(state["dt"], state["omega"], state["phi"], state["dtype"])
    smp = state["smp"]
    hops = range(len(smp.fanouts))
    if kind == "sample":
        _sample(state)
        return dict(nbr=smp.nbr, eid=smp.eid, ts=smp.ts, dt=smp.dt, parent=smp.parent, counts=smp.counts)
    if kind == "mfg":
        _blocks(state)
        return [b["out"] for b in state["blocks"]]
    _sample(state)
    _blocks(state)
    for h in hops:
        per = smp.fanouts[h] * (smp.snapshots if h == 0 else 1)
        count = smp.counts[h:h + 1]
        tgl.gather(smp.nbr[h], smp.eid[h], state["tables"], count=count, per_count=per, outs=state["rows"][h])
        tgl.time_encode(smp.dt[h], state["omega"], state["phi"], count=count, per_count=per, out=state["enc"][h])
    return dict(blocks=[b["out"] for b in state["blocks"]], rows=state["rows"], enc=state["enc"])


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------

def _hops(case):
    """Per hop: (roots, groups, slots, valid slots), from the family's shares."""
    roots = 3 * case["batch"] * case["batches"]
    out = []
    windows = case["snapshots"]
    for h, k in enumerate(_fan(case)):
        groups = roots * windows
        slots = groups * k
        valid = slots * VALID[case["graph"]][0 if h == 0 else 1]
        out.append((roots, groups, slots, valid))
        roots, windows = valid, 1
    return out


def work(case):
    kind = case["kind"]
    size = {"f32": 4, "bf16": 2}
    if kind == "build":
        m, M, n = case["edges"], 2 * case["edges"], case["nodes"]
        # edges in; indptr, records, timestamps, node records, search index,
        # histories and directories out
        return dict(bytes=m * (12 + (8 if case["eid"] else 0)) + n * (8 + 128) + M * (16 + 4 + 8) + M // 32 * 12,
                    flops=0)
    if kind == "gather":
        row = sum(int(d) for d in case["dims"].split(",")) * size[case["dtype"]]
        keys = 4 if len(case["dims"].split(",")) < 3 else 12
        return dict(bytes=case["slots"] * (keys + row + row // 2), flops=0)
    if kind == "time":
        return dict(bytes=case["slots"] * (4 + case["dim"] * size[case["dtype"]]), flops=2 * case["slots"] * case["dim"])
    hops = _hops(case)
    # a root's node and time, the record of a valid slot, the slot's four fields
    sample = sum((8 if h == 0 else 8 + 8) * r + 16 * v + 20 * s for h, (r, _, s, v) in enumerate(hops))
    # a slot's fields in; per edge destination, id, time difference and source out; per group its offset and node
    blocks = sum(4 * s + 16 * v + 28 * v + (8 + 8 + 8) * g for _, g, s, v in hops)
    if kind == "sample":
        return dict(bytes=sample, flops=0)
    if kind == "mfg":
        return dict(bytes=blocks, flops=0)
    row = (100 + 372 + 172) * 4
    # the tables are small: what is looked up is read from them once
    lookup = (472 * case["nodes"] + 172 * case["edges"]) * 4
    slots = sum(s for _, _, s, _ in hops)
    lookup = min(lookup, sum(v for _, _, _, v in hops) * row) + slots * (12 + row)
    return dict(bytes=sample + blocks + lookup + slots * (4 + 400), flops=2 * slots * 100)


def tolerance(case):
    """Sampling, building and the lookups pick, count and copy: every output
    is the same bits whatever the implementation (dt is one rounded
    difference).  Only the time encoding evaluates a function: each value is
    within 1e-6 of the exact cosine, so two correct ones differ by at most
    2e-6 (the values' root mean square is 0.7); over all values the present
    one is 3.3e-8 off in the 2-norm, and four times the difference of two
    such is 2e-7.  In bfloat16 a value moves by one step (2^-8 at most) where
    that changes its rounding, about one in 1e5."""
    if case["kind"] == "time" and case["dtype"] == "bf16":
        return {"rel": 5e-5, "max": 8e-3}
    if case["kind"] in ("time", "minibatch"):
        return {"rel": 2e-7, "max": 3e-6}
    return "exact"


def exact(case, seed):
    """The time encoding in 64 bits; the other kinds compute no number that
    is not exactly rounded already."""
    if case["kind"] != "time":
        return None
    s = prepare(case, seed)
    dt = s["dt"].double()
    out = torch.outer(dt, s["omega"].double()).add_(s["phi"].double()).cos_()
    return out.masked_fill_((dt < 0)[:, None], 0.0)
