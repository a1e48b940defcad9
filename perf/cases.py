"""What is timed: windows of the feature-fetch path through its drivers, and
the GraphSAGE forward pass on a window's rows.

A case is a dict of plain sizes and options.  `prepare` builds a seeded
power-law graph, feature shards and the driver (or a sampled window and the
layers' weights) on the GPU; `run` is one pass as a user's program makes it.

Two kinds of case:
  "fetch"  one pass = `windows` windows through FetchPipeline or
           LookaheadPipeline, into the caller's own output buffers.  The
           sequential drivers take the next of `cycle` windows in each pass,
           so that the persistent caches see a window they have not just held.
  "sage"   one pass = gg_sage_forward over one window's sampled blocks.

The graphs stand in for R-MAT graphs with (a, b, c) = (0.57, 0.19, 0.19): a
node's out-degree and its share of all neighbour entries are both
proportional to 0.76^zeros * 0.24^ones over the bits of its rank, and ranks
are spread over the ids.
"""
import math

import torch

from paper_2606_02916_amd import FetchPipeline, LookaheadPipeline, SageConsumer, gg

P_ZERO = 0.76                     # a + b of the R-MAT graphs
ELEM = {"fp32": 4, "fp16": 2}
TORCH = {"fp32": torch.float32, "fp16": torch.float16}

# Graph sizes are those of the repository's workloads (10K, 233K, 2.45M and
# 111M nodes) and generic ones between them.
TINY = dict(nodes=10_000, edges=100_000)
DENSE = dict(nodes=233_000, edges=114_000_000)
SPARSE = dict(nodes=2_450_000, edges=62_000_000)
PAPERS = dict(nodes=111_000_000, edges=1_600_000_000)


def _fetch(name, graph, dim, dtype, fanout, batch, W, driver, **kw):
    c = dict(kind="fetch", **graph, dim=dim, dtype=dtype, padded=True, fanout=fanout, batch=batch,
             W=W, driver=driver, book="range", parts=4, hot="", windows=1, cycle=4,
             per_batch=False, sim=False, layers="")
    c.update(kw)
    return dict(c, name=name) if name else c


def _sage(name, graph, dim, dtype, fanout, batch, W, layers, **kw):
    c = dict(kind="sage", **graph, dim=dim, dtype=dtype, padded=True, fanout=fanout, batch=batch,
             W=W, layers=layers)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: one window of four batches on a 10K-node graph,
        # owners by node id mod 4; launches and their gaps.
        _fetch("tiny_window", TINY, 64, "fp32", "10,5", 256, 4, "sequential", book="mod"),
        # Six windows of a single large batch: a program that cannot group
        # its batches.
        _fetch("one_batch_lookahead", SPARSE, 100, "fp32", "15,10,5", 4096, 1, "lookahead",
               windows=6, cycle=1),
        # The benchmark's workload: OGBN-Products-shaped, an epoch of six
        # windows on the look-ahead driver.
        _fetch("sparse_lookahead", SPARSE, 100, "fp32", "15,10,5", 1024, 16, "lookahead",
               windows=6, cycle=1),
        # Reddit-shaped: wide rows, high fan-out, two hops.
        _fetch("dense_lookahead", DENSE, 602, "fp32", "25,10", 1024, 8, "lookahead", windows=6,
               cycle=1),
        # OGBN-Papers100M-shaped, fp16 rows, everything in HBM.
        _fetch("papers_lookahead", PAPERS, 128, "fp16", "15,10,5", 1024, 16, "lookahead",
               windows=3, cycle=1),
        # The simulator's sweep: the hot set cut to a tenth of the window, so
        # that most remote rows take the miss path, and the window's counts
        # added to the running totals.
        _fetch("sparse_budget", SPARSE, 100, "fp32", "15,10,5", 1024, 16, "sequential",
               hot="1/10", sim=True),
        # A feature matrix as it comes, rows of 75 floats without padding,
        # one launch per batch, a persistent cache rebuilt by its delta,
        # owners by node id mod 8.
        _fetch("ragged_inplace", SPARSE, 75, "fp32", "10,10", 1000, 8, "inplace", padded=False,
               book="mod", parts=8, per_batch=True),
        # Reddit's 602 floats as they come (2,408-byte rows, unpadded),
        # two caches, whole-window gather.
        _fetch("dense_delta", DENSE, 602, "fp32", "25,10", 512, 8, "delta", padded=False),
        # The whole step: a window, then the GraphSAGE forward pass on it.
        _fetch("sparse_step", SPARSE, 100, "fp32", "15,10,5", 1024, 8, "inplace",
               layers="16,16,47"),
        # The forward pass alone on the three graphs' windows: small hidden
        # layers, wide inputs with a wide hidden layer, and fp16 inputs with
        # three hops of 128.
        _sage("sage_sparse", SPARSE, 100, "fp32", "15,10,5", 1024, 16, "16,16,47"),
        _sage("sage_dense", DENSE, 602, "fp32", "25,10", 1024, 8, "128,41"),
        _sage("sage_half", PAPERS, 128, "fp16", "15,10,5", 1024, 8, "128,128,64"),
    ]


def draw(rng):
    while True:
        c = _drawn(rng)
        w = _work(c)
        if w["bytes"] <= 6e9 and w["flops"] <= 6e10:
            return c


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _drawn(rng):
    nodes = _log(rng, 8_000, 6_000_000)
    edges = int(nodes * min(_log(rng, 8, 500), 150_000_000 // nodes + 1))
    batch = _log(rng, 100, 4096)
    fanout = rng.choice(["10,5", "15,10", "25,10", "15,10,5", "10,10,10", "5,5,5", "7,3"])
    W = rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 24])
    dtype = rng.choice(["fp32", "fp32", "fp16"])
    dim = _log(rng, 16, 640)
    dim += dim % 2 if dtype == "fp16" else 0
    graph = dict(nodes=nodes, edges=edges)
    layers = ",".join(str(_log(rng, 12, 128)) for _ in range(fanout.count(",") + 1))
    kind = rng.random()
    if kind < 0.35:
        return _sage("", graph, dim, dtype, fanout, batch, W, layers, padded=rng.random() < 0.6)
    if kind < 0.8:
        layers = ""
    driver = rng.choice(["sequential", "delta", "inplace", "lookahead", "lookahead"])
    look = driver == "lookahead"
    return _fetch("", graph, dim, dtype, fanout, batch, W, driver,
                  padded=rng.random() < 0.5, book=rng.choice(["range", "mod"]),
                  parts=rng.choice([2, 3, 4, 8]), hot=rng.choice(["", "", "", "1/10", "1/4"]),
                  windows=4 if look else 1, cycle=1 if look else 4, per_batch=(
                      not look and not layers and rng.random() < 0.4),
                  sim=rng.random() < 0.3, layers=layers)


# ---------------------------------------------------------------------------
# Seeded inputs.
# ---------------------------------------------------------------------------
def _ints(text):
    return [int(x) for x in text.split(",")] if text else []


def _halves(n):
    """The rank's low and high bits: (low bits, pmf of each half)."""
    bits = max((n - 1).bit_length(), 2)
    lo = bits // 2

    def pmf(k):
        p = torch.ones(1, dtype=torch.float64)
        for _ in range(k):
            p = torch.cat([p * P_ZERO, p * (1 - P_ZERO)])
        return p
    return lo, bits, pmf(lo), pmf(bits - lo)


class _Law:
    """The power law over n ids: neighbours drawn, expected degrees."""

    def __init__(self, n, edges, dev):
        self.n, self.dev = n, dev
        self.lo, self.bits, plo, phi = _halves(n)
        self.plo, self.phi = plo.to(dev, torch.float32), phi.to(dev, torch.float32)
        self.clo = plo.cumsum(0).to(dev, torch.float32)
        self.chi = phi.cumsum(0).to(dev, torch.float32)
        k = int(n * 0.6180339887) | 1
        while math.gcd(k, n) != 1:
            k += 2
        self.mul, self.inv = k % n or 1, pow(k, -1, n) if n > 1 else 0
        self.scale = edges           # the ids past n hold little of the law's mass

    def _id(self, rank):
        return rank.mul_(self.mul).add_(self.n // 3).remainder_(self.n)

    def neighbours(self, count, gen, out):
        """`count` ids by the law into out (int32)."""
        for a in range(0, count, 1 << 26):
            m = min(1 << 26, count - a)
            u = torch.rand(m, generator=gen, device=self.dev)
            r = torch.searchsorted(self.chi, u).clamp_(max=self.chi.numel() - 1)
            u = torch.rand(m, generator=gen, device=self.dev)
            r = r.mul_(1 << self.lo).add_(torch.searchsorted(self.clo, u)
                                          .clamp_(max=self.clo.numel() - 1))
            r = torch.where(r >= self.n, r - (1 << (self.bits - 1)), r)
            out[a:a + m] = self._id(r)
        return out

    def mean_degree(self, ids):
        rank = (ids.long() - self.n // 3).mul_(self.inv).remainder_(self.n)
        return self.phi[rank >> self.lo] * self.plo[rank & ((1 << self.lo) - 1)] * self.scale

    def csr(self, gen):
        deg = torch.empty(self.n, dtype=torch.float32, device=self.dev)
        for a in range(0, self.n, 1 << 25):
            b = min(self.n, a + (1 << 25))
            mean = self.mean_degree(torch.arange(a, b, device=self.dev))
            deg[a:b] = torch.poisson(mean, generator=gen)
        row_ptr = torch.zeros(self.n + 1, dtype=torch.int64, device=self.dev)
        torch.cumsum(deg, 0, dtype=torch.int64, out=row_ptr[1:])
        if int(deg.min()) < 0 or int(row_ptr.diff().min()) < 0:
            raise RuntimeError("the generated row offsets do not ascend")
        col = torch.empty(int(row_ptr[-1]), dtype=torch.int32, device=self.dev)
        self.neighbours(col.numel(), gen, col)
        if int(col.min()) < 0 or int(col.max()) >= self.n:
            raise RuntimeError("a generated neighbour is outside the graph")
        return row_ptr, col


def _generator(seed, dev):
    return torch.Generator(device=dev).manual_seed(int(seed) * 7919 + 11)


def _rows(n, case, gen, dev):
    """n feature rows, standard normal, at the case's stride (uint8)."""
    eb, dim = ELEM[case["dtype"]], case["dim"]
    width = _stride(case) // eb
    x = torch.empty((max(n, 1), width), dtype=TORCH[case["dtype"]], device=dev)
    x.normal_(generator=gen)
    return x if width == dim else _zero_tail(x, dim)


def _zero_tail(x, dim):
    x[:, dim:] = 0
    return x


def _row_bytes(case):
    return case["dim"] * ELEM[case["dtype"]]


def _stride(case):
    rb = _row_bytes(case)
    return (rb + 15) // 16 * 16 if case["padded"] else rb


def _seeds(case, batches, gen, dev):
    """`batches` batches of distinct seeds: a permutation's, over and over."""
    N, B = case["nodes"], case["batch"]
    perm = torch.randperm(N, generator=gen, device=dev)[:min(batches, N // B) * B]
    return perm.repeat(-(-batches * B // perm.numel()))[:batches * B]


def _layers(case, gen, dev):
    """(w_self, w_neigh, bias, relu) per layer, scaled to keep variances."""
    out, d = [], case["dim"]
    widths = _ints(case["layers"])
    for j, w in enumerate(widths):
        ws, wn = (torch.empty((d, w), device=dev).normal_(generator=gen).mul_((2 * d) ** -0.5)
                  for _ in range(2))
        b = torch.empty(w, device=dev).normal_(generator=gen).mul_(0.1)
        out.append((ws, wn, b, j + 1 < len(widths)))
        d = w
    return out


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = _generator(seed, dev)
    law = _Law(case["nodes"], case["edges"], dev)
    return (_prepare_fetch if case["kind"] == "fetch" else _prepare_sage)(case, gen, law, dev)


def _prepare_fetch(case, gen, law, dev):
    N, W, B, P = case["nodes"], case["W"], case["batch"], case["parts"]
    fan, stride = _ints(case["fanout"]), _stride(case)
    row_ptr, col = law.csr(gen)
    if N <= 100_000:
        row_ptr = row_ptr.int()
    mod = case["book"] == "mod"
    start = [m * N // P for m in range(P)] + [N]
    rows = [(N - m + P - 1) // P if mod else start[m + 1] - start[m] for m in range(P)]
    shards = [_rows(r, case, gen, dev).view(torch.uint8) for r in rows]
    nwin = max(case["windows"], case["cycle"])
    seeds = _seeds(case, nwin * W, gen, dev).int()
    off = [b * B for b in range(W + 1)]
    args = (row_ptr, col, P, gg.PART_MOD if mod else gg.PART_RANGE, 0, None if mod else start,
            shards, rows, _row_bytes(case), stride, W, fan, B)
    frac = tuple(_ints(case["hot"].replace("/", ","))) or None
    look = case["driver"] == "lookahead"
    if look:
        pipe = LookaheadPipeline(*args, device=dev, hot_frac=frac)
    else:
        pipe = FetchPipeline(*args, device=dev, hot_frac=frac, delta=case["driver"] == "delta",
                             inplace=case["driver"] == "inplace")
    # The caller's buffers, one per window: room for half as many rows again
    # as the law gives on average.  Bytes past a window's rows stay zero.
    ent, drawn, _ = _levels(case)
    cap = min(pipe.geo.out_cap, int(1.8 * ent[-1]) + 256)
    outs = []
    for k in range(nwin if not case["layers"] else 0):
        whole = torch.zeros((W * cap, stride), dtype=torch.uint8, device=dev)
        outs.append(whole.view(W, cap, stride) if case["per_batch"] else whole)
    lists = (min(pipe.geo.fcap, int(1.8 * W * sum(ent)) + 256 * W),
             min(pipe.geo.ncap, int(1.8 * W * sum(e * k for e, k in zip(ent, fan))) + 256 * W))
    for b in pipe.sets if look else [pipe.buf]:
        b.frontier_ids[:lists[0]] = 0
        b.nbr_ids[:lists[1]] = 0
        if case["layers"]:           # the driver's own buffer, of the worst case's rows
            b.win_out[:W * cap] = 0
    # `graph`: the drivers keep addresses; the caller keeps the tensors.
    st = dict(case=case, pipe=pipe, graph=(row_ptr, col), look=look, at=0, off=off, consumer=None,
              sim=None, outs=outs or [None] * nwin, rows=W * cap, lists=lists,
              seeds=seeds.split(W * B))
    if case["layers"]:
        st["consumer"] = SageConsumer(pipe.geo, _layers(case, gen, dev),
                                      gg.GG_F32 if case["dtype"] == "fp32" else gg.GG_F16,
                                      device=dev)
    if case["sim"]:
        coeffs = gg.make_sim_coeffs(P, 0.025, 1.6e-5, 5e-4, 3.2e-7, 1.25e9, _row_bytes(case), 30.0)
        st["sim"] = (coeffs, torch.zeros(gg.SIM_ACC_BYTES, dtype=torch.uint8, device=dev))
    return st


def _prepare_sage(case, gen, law, dev):
    """A window's sampled blocks drawn by the law, the gathered rows and the
    weights: what gg_sample_window and gg_gather_batch leave behind."""
    N, W = case["nodes"], case["W"]
    fan = _ints(case["fanout"])
    blocks = _blocks(case, gen, law, dev)
    x = _rows(blocks["keys"][-1].numel(), case, gen, dev)
    layers = _layers(case, gen, dev)
    wpb = gg.gg_bits_words(N)
    key = blocks["keys"][-1]
    word = torch.zeros(W * wpb, dtype=torch.int64, device=dev)
    b, u = key // N, key % N
    word.scatter_add_(0, b * wpb + (u >> 5), torch.ones_like(u) << (u & 31))
    bits = torch.where(word >= 1 << 31, word - (1 << 32), word).int()
    ids = torch.cat([k % N for k in blocks["keys"]]).int()
    edges = torch.arange(W, device=dev) * N
    off, base = [], 0
    noff, nbase = [], 0
    for l, k in enumerate(blocks["keys"]):
        first = torch.searchsorted(k, edges)
        off.append(first + base)
        base += k.numel()
        if l < len(fan):
            noff.append(first * fan[l] + nbase)
            nbase += k.numel() * fan[l]
    end = lambda v: torch.tensor([v], device=dev)           # noqa: E731
    smp = dict(ids=ids, off=torch.cat(off + [end(base)]),
               nbr=torch.cat([n.reshape(-1) for n in blocks["nbrs"]]).int(),
               noff=torch.cat(noff + [end(nbase)]), bits=bits,
               need=torch.zeros(2, dtype=torch.int64, device=dev))
    arr = gg.make_sage_layers(layers)
    # rows per level as the pipelines bound them: every draw a new node
    lev = min(case["batch"], N)
    for k in fan:
        lev = min(N, lev * (k + 1))
    cap = W * lev
    nseeds = blocks["keys"][0].numel()
    return dict(case=case, smp=smp, fan=fan, x=x, layers=layers, arr=arr, cap=cap, nseeds=nseeds,
                wsample=gg.make_wsample(smp["ids"], smp["off"], smp["nbr"], smp["noff"],
                                        smp["bits"], smp["need"]),
                out=torch.zeros((nseeds, layers[-1][0].shape[1]), device=dev),
                ws=torch.empty(gg.gg_ws_sage(N, W, cap, arr), dtype=torch.uint8, device=dev),
                status=torch.zeros(1, dtype=torch.int32, device=dev))


def _blocks(case, gen, law, dev):
    """keys[l]: b * N + id of every node of F_l, ascending; nbrs[l]: the ids
    each node of F_l drew at hop l, distinct, ascending, -1 where its degree
    is below the fan-out."""
    N, W = case["nodes"], case["W"]
    fan = _ints(case["fanout"])
    seeds = _seeds(case, W, gen, dev).view(W, -1) + N * torch.arange(W, device=dev)[:, None]
    keys, nbrs = [torch.unique(seeds)], []
    for k in fan:
        key = keys[-1]
        n = key.numel()
        deg = torch.poisson(law.mean_degree(key % N), generator=gen)
        v = law.neighbours(n * k, gen, torch.empty(n * k, dtype=torch.int32, device=dev)).long()
        v = v.view(n, k)
        v = torch.where(torch.arange(k, device=dev) < deg[:, None], v, N).sort(1).values
        v[:, 1:][v[:, 1:] == v[:, :-1]] = N
        v = v.sort(1).values
        v[v == N] = -1
        nbrs.append(v)
        drawn = (v + (key // N * N)[:, None])[v >= 0]
        keys.append(torch.unique(torch.cat([key, drawn])))
    return dict(keys=keys, nbrs=nbrs)


# ---------------------------------------------------------------------------
# One pass.
# ---------------------------------------------------------------------------
def run(st):
    if st["case"]["kind"] == "sage":
        gg.gg_sage_forward(st["wsample"], st["case"]["nodes"], st["case"]["W"], st["fan"], st["x"],
                           gg.GG_F32 if st["case"]["dtype"] == "fp32" else gg.GG_F16,
                           st["x"].stride(0) * st["x"].element_size(), st["cap"], st["arr"],
                           st["out"], st["nseeds"], st["status"], st["ws"])
        return dict(logits=st["out"], status=st["status"])
    case, pipe = st["case"], st["pipe"]
    W, L, got = case["W"], pipe.L, {}
    if st["look"]:
        for k in range(case["windows"]):
            _, buf = pipe.window(st["seeds"][k], st["off"], k * W, out=st["outs"][k],
                                 sim=st["sim"], consumer=st["consumer"])
            if st["outs"][k] is not None:
                got["rows%d" % k] = st["outs"][k].view(torch.int32)
        # the caller's stream reads the rows next
        torch.cuda.current_stream().wait_event(pipe.gathered_event(pipe.k - 1))
        stage, gather = buf.stage_stats, buf.gather_stats
    else:
        k = st["at"] % case["cycle"]
        st["at"] += 1
        pipe.window(st["seeds"][k], st["off"], k * W, outs=st["outs"][k], sim=st["sim"],
                    per_batch=case["per_batch"], consumer=st["consumer"])
        buf = pipe.buf
        if st["outs"][k] is not None:
            got["rows"] = st["outs"][k].view(torch.int32)
        stage, gather = pipe.stage_stats, pipe.gather_stats
    ids, nbrs = st["lists"]
    got.update(frontier=buf.frontier_ids[:ids], nbrs=buf.nbr_ids[:nbrs],
               off=buf.frontier_off[:(L + 1) * W + 1], noff=buf.nbr_off[:L * W + 1],
               bits=buf.frontier_bits, owner_off=buf.owner_off, status=pipe.status,
               stage=stage.view(torch.int64), gather=gather.view(torch.int64))
    if st["sim"]:
        got["sim"] = st["sim"][1].view(torch.int64)
    if st["consumer"]:
        got["rows"] = buf.win_out[:st["rows"]].view(torch.int32)
        got["logits"] = st["consumer"].out[:W * case["batch"]]
    return got


# ---------------------------------------------------------------------------
# What a pass cannot do without.
# ---------------------------------------------------------------------------
def _classes(case):
    """(nodes, neighbour probability, mean degree) of every popcount class."""
    n, bits = case["nodes"], max((case["nodes"] - 1).bit_length(), 2)
    got = []
    for j in range(bits + 1):
        c = math.comb(bits, j) * n / (1 << bits)
        p = P_ZERO ** (bits - j) * (1 - P_ZERO) ** j * (1 << bits) / n
        got.append((c, p, case["edges"] * p * n / (1 << bits)))
    return got


def _levels(case):
    """Expected sizes of one batch: entries per level, draws per hop, and
    the inclusion probability of every class at the last level."""
    cl, fan = _classes(case), _ints(case["fanout"])
    q = [min(1.0, case["batch"] / case["nodes"])] * len(cl)
    ent, drawn = [min(case["batch"], case["nodes"])], []
    for k in fan:
        d = sum(c * qi * k * (1 - math.exp(-lam / k)) for (c, p, lam), qi in zip(cl, q))
        q = [1 - (1 - qi) * math.exp(-d * p) for (c, p, lam), qi in zip(cl, q)]
        drawn.append(d)
        ent.append(sum(c * qi for (c, p, lam), qi in zip(cl, q)))
    return ent, drawn, q


def _work(case):
    """Bytes read and written once, operations, for one pass."""
    ent, drawn, q = _levels(case)
    W, fan, rb = case["W"], _ints(case["fanout"]), _row_bytes(case)
    flops = by = 0.0
    widths = _ints(case["layers"])
    if widths:
        # layer j: F_{L-j}'s own rows and the means of their neighbours, each
        # a product by d_in x d_out; the input rows and the lists read once
        d = case["dim"]
        for j, w in enumerate(widths):
            out = ent[len(ent) - 2 - j]
            flops += W * out * 4.0 * d * w + W * drawn[len(drawn) - 1 - j] * d
            by += 8.0 * d * w
            d = w
        by += W * (ent[0] * 4 * d + sum(e * 4 for e in ent) +
                   sum(e * k * 4 for e, k in zip(ent, fan)) + ent[-1] * rb)
    if case["kind"] == "sage":
        return dict(bytes=by, flops=flops)
    cl = _classes(case)
    remote = 1 - 1.0 / case["parts"]
    union = remote * sum(c * (1 - (1 - qi) ** W) for (c, p, lam), qi in zip(cl, q))
    both = remote * sum(c * (1 - (1 - qi) ** (2 * W)) for (c, p, lam), qi in zip(cl, q))
    staged = union
    if case["hot"]:
        a, b = _ints(case["hot"].replace("/", ","))
        staged = union * a / b
    elif case["driver"] != "sequential":
        staged = both - union                      # the rebuild delta
    bits = W * case["nodes"] / 8.0
    by += W * (ent[0] * 4 + sum(e * (4 + 16) for e in ent[:-1]) + ent[-1] * 4 +
               sum(d * 4 for d in drawn) + sum(e * k * 4 for e, k in zip(ent, fan)))
    by += bits + union * 12 + staged * (2.0 * rb + 8)
    by += W * ent[-1] * (2.0 * rb + 8)
    return dict(bytes=by * case["windows"], flops=flops * case["windows"])


def work(case):
    return _work(case)


def tolerance(case):
    # Ids, rows and counts are whole numbers and copied bytes.  The forward
    # pass sums up to a few hundred fp32 products per layer.
    return {"rel": 2e-6, "max": 4e-5} if case["layers"] else "exact"


# ---------------------------------------------------------------------------
# The forward pass in 64 bits.
# ---------------------------------------------------------------------------
def exact(case, seed):
    """The logits from the same blocks; rows, ids and counts have none."""
    if case["kind"] != "sage":
        return None
    dev = torch.device("cuda")
    gen = _generator(seed, dev)
    law = _Law(case["nodes"], case["edges"], dev)
    blocks = _blocks(case, gen, law, dev)
    N, keys = case["nodes"], blocks["keys"]
    x = _rows(keys[-1].numel(), case, gen, dev)
    h = None
    for j, (ws, wn, b, relu) in enumerate(_layers(case, gen, dev)):
        l = len(keys) - 2 - j
        nbr, own, above = blocks["nbrs"][l], keys[l], keys[l + 1]
        parts = []
        for a in range(0, own.numel(), 1 << 15):
            key, v = own[a:a + (1 << 15)], nbr[a:a + (1 << 15)]
            pos = torch.searchsorted(above, (v.clamp(min=0) + (key // N * N)[:, None]))
            get = (lambda i: x[i, :case["dim"]].double()) if h is None else (lambda i: h[i])
            ok = (v >= 0)
            s = torch.zeros((key.numel(), ws.shape[0]), dtype=torch.float64, device=dev)
            for t in range(v.shape[1]):
                s += get(pos[:, t]) * ok[:, t, None]
            y = (get(torch.searchsorted(above, key)) @ ws.double() +
                 s / ok.sum(1).clamp(min=1)[:, None] @ wn.double() + b.double())
            parts.append(y.clamp(min=0) if relu else y)
        h = torch.cat(parts)
    return dict(logits=h, status=None)
