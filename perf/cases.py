"""Timed workloads of the layout library: what a user's program calls, over the sizes it calls it with.

Every case works on a seeded variation graph of the model that the synthetic workloads use: a backbone of `backbone`
nodes with lengths 1 + Geometric(p_len), walked by `paths` haplotypes that take a single-nucleotide alternative at 5%
of the positions, skip short runs (1%) and invert short runs (0.2%).  Five kinds of call:

  layout   the initial layout and Alg. 1 on it, in the default order (schedule 0) or the paper's (1), also with data
           reuse (reuse, reduction)
  batch    several uneven graphs laid out together through one Batch handle
  sps      the sampled path stress of a finished layout, or of two layouts on the same pairs (compare)
  exact    the path stress over all step pairs of a finished layout
  train    one optimiser step on the differentiable stress: loss, backward, Adam
"""
import math

import numpy as np
import torch

import paper_2409_00876_amd as P

DEV = "cuda:0"


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # a small locus: the 2,000-node graph of the tests, the shortest layout a user runs
        dict(name="layout_tiny", kind="layout", backbone=2000, paths=8, p_len=0.2, schedule=0, reuse=1, reduction=1),
        # a gene region of a pangenome (tens of thousands of nodes)
        dict(name="layout_region", kind="layout", backbone=30011, paths=24, p_len=0.2, schedule=0, reuse=1,
             reduction=1),
        # the 1M-node backbone of the tests and the benchmark
        dict(name="layout_mid", kind="layout", backbone=1000000, paths=32, p_len=0.2, schedule=0, reuse=1,
             reduction=1),
        # a small chromosome: the coordinates and records of the chromosome workload's regime
        dict(name="layout_chromosome", kind="layout", backbone=4000037, paths=32, p_len=0.05, schedule=0, reuse=1,
             reduction=1),
        # the data-reuse variant at its 2x setting on a mid-size graph
        dict(name="layout_reuse", kind="layout", backbone=300007, paths=32, p_len=0.05, schedule=0, reuse=2,
             reduction=2),
        # uneven graphs laid out together, as the 24-chromosome batch is (scaled down)
        dict(name="batch_uneven", kind="batch", graphs=6, low=20000, high=200000, paths=32, p_len=0.05),
        # the metric on a small layout at its default 100 pairs per step
        dict(name="sps_tiny", kind="sps", backbone=2000, paths=8, p_len=0.2, pairs="uniform", m=100, compare=False),
        # the metric on a chromosome-like layout, 10 pairs per step, window-major order
        dict(name="sps_chromosome", kind="sps", backbone=1500001, paths=48, p_len=0.05, pairs="uniform_windowed",
             m=10, compare=False),
        # two layouts of one graph on the same power-law pairs (local structure)
        dict(name="sps_compare", kind="sps", backbone=200003, paths=16, p_len=0.2, pairs="power_law", m=10,
             compare=True),
        # the exact metric where it is affordable: a small graph
        dict(name="exact_small", kind="exact", backbone=20011, paths=8, p_len=0.2),
        # an optimiser step on a small graph: launches and latency
        dict(name="train_small", kind="train", backbone=20000, paths=8, p_len=0.2, pairs=100000),
        # an optimiser step on the 1M-node backbone with the benchmark's 1e7 pairs
        dict(name="train_mid", kind="train", backbone=1000000, paths=32, p_len=0.2, pairs=10000000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["layout", "batch", "sps", "exact", "train"], [45, 10, 20, 8, 17])[0]
    p_len = rng.choice([0.05, 0.1, 0.2])
    if kind == "layout":
        b = _log(rng, 600, 1500000)
        paths = rng.randint(4, 24 if b < 200000 else 40)
        reuse, reduction = rng.choice([(1, 1), (1, 1), (1, 1), (2, 1), (2, 2), (4, 2)])
        # the paper's order is several times slower: only where it stays below the largest listed case
        schedule = rng.choice([0, 0, 0, 1]) if b * paths < 2.5e7 else 0
        return dict(kind=kind, backbone=b, paths=paths, p_len=p_len, schedule=schedule, reuse=reuse,
                    reduction=reduction)
    if kind == "batch":
        n = rng.randint(2, 8)
        low = _log(rng, 1500, 40000)
        return dict(kind=kind, graphs=n, low=low, high=low * rng.randint(2, 12) + rng.randint(0, 99),
                    paths=rng.randint(4, 24), p_len=p_len)
    if kind == "sps":
        b = _log(rng, 600, 1500000)
        paths = rng.randint(4, 32)
        m = max(1, min(rng.choice([1, 3, 10, 30, 100]), int(3e8 / (b * paths))))
        return dict(kind=kind, backbone=b, paths=paths, p_len=p_len,
                    pairs=rng.choice(["uniform", "power_law", "uniform_windowed"]), m=m,
                    compare=rng.random() < 0.35)
    if kind == "exact":
        b = _log(rng, 300, 20000)
        return dict(kind=kind, backbone=b, paths=rng.randint(2, 8), p_len=p_len)
    b = _log(rng, 1500, 1000000)
    return dict(kind="train", backbone=b, paths=rng.randint(4, 32), p_len=p_len, pairs=_log(rng, 20000, 10000000))


# ---------------------------------------------------------------------------
# Graphs and finished layouts
# ---------------------------------------------------------------------------
def _graph(backbone, paths, p_len, seed):
    """(node_len, path_off, step_node as numpy; start coordinate of every node along the backbone, on the GPU)."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1000003 * int(seed) + 7)
    B = int(backbone)
    pos = torch.arange(B, device=DEV)

    def rand(n):
        return torch.rand(n, generator=gen, device=DEV)

    # the positions that have an alternative, their number fixed by the sizes (the share that `paths` walks would
    # visit); one path chosen for each takes it, the others with the probability that leaves 5% of the visits
    n_alt = int(round(B * (1.0 - 0.95 ** paths)))
    has_alt = torch.zeros(B, dtype=torch.bool, device=DEV)
    has_alt[torch.topk(rand(B), n_alt).indices] = True
    taker = (rand(B) * paths).long()
    rest = max(0.0, (0.05 * paths * B / max(1, n_alt) - 1.0) / max(1, paths - 1))
    snp = torch.stack([has_alt & ((rand(B) < rest) | (taker == p)) for p in range(paths)])
    ids = pos + torch.cumsum(has_alt, 0) - has_alt.long()  # id of a backbone node; its alternative is the next id
    n_nodes = B + n_alt
    length = torch.empty(B, device=DEV, dtype=torch.float64).geometric_(p_len, generator=gen).long()
    node_len = torch.ones(n_nodes, device=DEV, dtype=torch.int64)
    node_len[ids] = length
    begin = torch.cumsum(length, 0) - length
    node_at = torch.zeros(n_nodes, device=DEV, dtype=torch.float64)
    node_at[ids] = begin.double()
    alt = has_alt.nonzero().reshape(-1)
    node_at[ids[alt] + 1] = begin[alt].double()

    cells = (B + 255) // 256
    steps = []
    for p in range(paths):
        # skipped runs: 1% of the positions start one of 1..20
        start = (rand(B) < 0.01).nonzero().reshape(-1)
        stop = (start + 1 + (rand(start.numel()) * 20).long()).clamp_(max=B)
        mark = torch.zeros(B + 1, device=DEV, dtype=torch.int32)
        mark.index_add_(0, start, torch.ones_like(start, dtype=torch.int32))
        mark.index_add_(0, stop, -torch.ones_like(stop, dtype=torch.int32))
        skipped = torch.cumsum(mark[:B], 0) > 0
        skipped[0] = False
        # inverted runs: at most one of 1..20 in a cell of 256 positions
        at = torch.arange(cells, device=DEV) * 256 + (rand(cells) * 230).long()
        run = 1 + (rand(cells) * 20).long()
        run = torch.where(rand(cells) < 0.4, run, torch.zeros_like(run))
        cell = pos >> 8
        a, e = at[cell], at[cell] + run[cell]
        inside = (pos >= a) & (pos < e) & (e <= B)
        src = torch.where(inside, a + e - 1 - pos, pos)
        node = ids[src] + (snp[p][src] & ~inside).long()
        word = (node | (inside.long() << 31))[~skipped[src]]
        steps.append(word)
    path_off = np.zeros(paths + 1, dtype=np.uint64)
    path_off[1:] = np.cumsum([s.numel() for s in steps])
    step_node = torch.cat(steps).cpu().numpy().astype(np.uint32)
    return node_len.to(torch.int64).cpu().numpy().astype(np.uint32), path_off, step_node, node_at, node_len


def _finished(node_at, node_len, seed):
    """Coordinates of a finished layout, [2][n][2]: nodes along the x axis, a few nucleotides off their place."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7919 * int(seed) + 3)
    n = node_at.numel()
    c = torch.empty(2, n, 2, device=DEV, dtype=torch.float64)
    c[0, :, 0] = node_at
    c[0, :, 1] = node_at + node_len
    noise = torch.randn(2, n, 2, generator=gen, device=DEV, dtype=torch.float32).double()
    c[0] += 2.0 * noise[0]
    c[1] = 3.0 * noise[1]
    return c.float().reshape(-1).contiguous()


def _sizes(case):
    """Backbones of a batch, log-uniform between its ends (no seed: the sizes are the case's)."""
    n = case["graphs"]
    lo, hi = math.log(case["low"]), math.log(case["high"])
    return [int(round(math.exp(lo + (hi - lo) * ((0.37 + 0.61803398875 * k) % 1.0)))) for k in range(n)]


def _adam_state(n, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(104729 * int(seed) + 11)
    g = torch.randn(n, generator=gen, device=DEV) * 1e-7
    return 0.3 * g, 0.02 * g * g + 1e-17


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        graphs = []
        for k, b in enumerate(_sizes(case)):
            node_len, path_off, step_node, _, _ = _graph(b, case["paths"], case["p_len"], 64 * seed + k)
            graphs.append(P.Graph(node_len, path_off, step_node))
        coords = [g.new_coords() for g in graphs]
        for g, c in zip(graphs, coords):
            P.init_coords(g, c)
        params = P.LayoutParams(seed=24301 + seed)
        return dict(kind=kind, graphs=graphs, coords=coords, batch=P.Batch(graphs, coords, params))
    node_len, path_off, step_node, node_at, length = _graph(case["backbone"], case["paths"], case["p_len"], seed)
    s = dict(kind=kind, case=case, graph=P.Graph(node_len, path_off, step_node), seed=seed)
    if kind == "layout":
        s["coords"] = s["graph"].new_coords()
        s["params"] = P.LayoutParams(seed=24301 + seed, schedule=case["schedule"], reuse_factor=case["reuse"],
                                     step_reduction=case["reduction"])
        return s
    s["coords"] = _finished(node_at, length, seed)
    if kind == "sps" and case["compare"]:
        s["coords_b"] = _finished(node_at, length, seed + 5000)
    if kind == "train":
        s["coords"].requires_grad_(True)
        s["m"], s["v"] = _adam_state(s["coords"].numel(), seed)
        s["step"] = 0
        s["params"] = P.LayoutParams(seed=11 + seed)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "batch":
        for g, c in zip(s["graphs"], s["coords"]):
            P.init_coords(g, c)
        s["batch"].run()
        return s["coords"]
    case, g, c = s["case"], s["graph"], s["coords"]
    if kind == "layout":
        P.init_coords(g, c)
        P.layout(g, c, s["params"])
        return c
    if kind == "sps":
        if case["compare"]:
            return P.path_stress_compare(g, c, s["coords_b"], case["m"], seed=7 + s["seed"], pairs=case["pairs"])
        return P.path_stress(g, c, case["m"], seed=7 + s["seed"], pairs=case["pairs"])
    if kind == "exact":
        return P.path_stress_exact(g, c)
    loss = P.SampledPathStress.apply(c, g, case["pairs"], s["step"], s["params"])
    loss.backward()
    grad, c.grad = c.grad, None
    s["step"] += 1
    P.adam_step(c, grad, s["m"], s["v"], s["step"] + 10, lr=0.1)
    return dict(loss=loss.detach(), grad=grad, x=c.detach(), m=s["m"], v=s["v"])


def work(case):
    """Bytes: the step records (16 a step) and the coordinates (16 a node in, 16 out) once; operations: floating
    point ones of the sampled terms or pairs."""
    def size(b, paths):
        return 0.905 * b * paths, b * (2.0 - 0.95 ** paths)

    kind = case["kind"]
    if kind == "batch":
        got = [size(b, case["paths"]) for b in _sizes(case)]
        return dict(bytes=sum(16 * S + 32 * n for S, n in got), flops=sum(300 * S * 20 for S, n in got))
    S, n = size(case["backbone"], case["paths"])
    if kind == "layout":
        updates = 300 * S / case["reduction"] * case["reuse"]
        return dict(bytes=16 * S + 32 * n, flops=20 * updates)
    if kind == "sps":
        sides = 2 if case["compare"] else 1
        return dict(bytes=16 * S + 16 * n * sides, flops=12 * S * case["m"] * sides)
    if kind == "exact":
        return dict(bytes=16 * S + 16 * n, flops=36 * 0.5 * S * S / case["paths"])
    return dict(bytes=16 * min(S, 2.0 * case["pairs"]) + 16 * n + 16 * n * 7, flops=40 * case["pairs"])


# ---------------------------------------------------------------------------
# The same values in 64 bits, from the definitions of the header
# ---------------------------------------------------------------------------
M32 = 0xFFFFFFFF


def _philox(counter, word2, word3, seed):
    """Philox4x32-10 at the 64-bit counters of an int64 tensor: four int64 tensors of 32-bit words."""
    c0, c1 = counter & M32, (counter >> 32) & M32
    c2, c3 = torch.full_like(c0, word2), torch.full_like(c0, word3)
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wrap modulo 2^64
        c0, c1, c2, c3 = ((b >> 32) & M32) ^ c1 ^ k0, b & M32, ((a >> 32) & M32) ^ c3 ^ k1, a & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _scale(lo, hi, n):
    """floor(u64 * n / 2^64) of the words lo, hi, for n < 2^31 (a number or a tensor)."""
    return (hi * n + ((lo * n) >> 32)) >> 32


class _Reference:
    def __init__(self, case, seed):
        node_len, path_off, step_node, node_at, length = _graph(case["backbone"], case["paths"], case["p_len"], seed)
        self.coords, self.node_at, self.length = _finished(node_at, length, seed), node_at, length
        word = torch.from_numpy(step_node.astype(np.int64)).to(DEV)
        self.node, self.rev = word & 0x7FFFFFFF, word >> 31
        self.len = length[self.node]
        self.off = torch.from_numpy(path_off.astype(np.int64)).to(DEV)
        total = torch.cumsum(self.len, 0)
        self.S = int(path_off[-1])
        self.path = torch.bucketize(torch.arange(self.S, device=DEV), self.off[1:], right=True)
        before = torch.cat([total.new_zeros(1), total])
        self.pos = before[:-1] - before[self.off[:-1]][self.path]
        f = np.concatenate([[0.0], np.cumsum(np.arange(1, 1001, dtype=np.float64) ** -0.99)])
        self.zipf = torch.from_numpy(np.floor(f / f[-1] * 4294967295.0).astype(np.int64)).to(DEV)

    def power_law(self, i, start, size, r2, r3):
        up, down = start + size - 1 - i, i - start
        back = ((r3 >> 2) & 1).bool()
        back = torch.where(~back & (up == 0), torch.ones_like(back), torch.where(back & (down == 0),
                                                                                  torch.zeros_like(back), back))
        room = torch.where(back, down, up)
        n = room.clamp(max=1000)
        z = torch.searchsorted(self.zipf[1:].contiguous(), ((r2 * self.zipf[n]) >> 32) & M32, right=True) + 1
        return torch.where(back, i - z, i + z), room > 0

    def ends(self, i, j, r3):
        ei, ej = r3 & 1, (r3 >> 1) & 1
        d = (self.pos[i] + self.len[i] * (ei ^ self.rev[i]) - self.pos[j] - self.len[j] * (ej ^ self.rev[j])).abs()
        return 2 * self.node[i] + ei, 2 * self.node[j] + ej, d

    def segments(self, shift):
        cuts = torch.cat([torch.arange(0, self.S, 1 << shift, device=DEV), self.off[:-1]])
        start = torch.unique(cuts)
        start = start[start < self.S]
        stop = torch.cat([start[1:], start.new_full((1,), self.S)])
        return start, stop

    def chunks(self, n, step=1 << 23):
        for a in range(0, n, step):
            yield torch.arange(a, min(n, a + step), device=DEV)

    def windowed(self, shift, n, first, slot_stream, word2, seed):
        """The window-major listing: yields (r2, r3, i, start of the path, its size) over all n pairs; first(q) is
        the step of plain pair q."""
        start, stop = self.segments(shift)
        count = torch.zeros(start.numel(), dtype=torch.int64, device=DEV)
        for q in self.chunks(n):
            count += torch.bincount(torch.bucketize(first(q), start, right=True) - 1, minlength=start.numel())
        last = torch.cumsum(count, 0)
        for u in self.chunks(n):
            k = torch.bucketize(u, last, right=True)
            r0, r1, r2, r3 = _philox(u, word2, slot_stream << 24, seed)
            i = start[k] + _scale(r0, r1, stop[k] - start[k])
            p = self.path[i]
            yield r2, r3, i, self.off[p], self.off[p + 1] - self.off[p]


def _shift(S, top):
    def n(sh):
        return (S + (1 << sh) - 1) >> sh
    while top > 6 and n(top) < 16:
        top -= 1
    while n(top) > 32768:
        top += 1
    return top


def _sps_pairs(R, case, seed):
    m, key = case["m"], 7 + seed
    n = m * R.S

    def plain(q):
        p = R.path[q // m]
        r = _philox(q, 0, 1 << 24, key)
        return r, R.off[p], R.off[p + 1] - R.off[p]

    if case["pairs"] == "uniform_windowed":
        def first(q):
            r, start, size = plain(q)
            return start + _scale(r[0], r[1], size)
        for r2, r3, i, start, size in R.windowed(_shift(R.S, 14), n, first, 6, 0, key):
            yield i, start + ((r2 * size) >> 32), r3, None
        return
    for q in R.chunks(n):
        r, start, size = plain(q)
        i = start + _scale(r[0], r[1], size)
        if case["pairs"] == "power_law":
            j, good = R.power_law(i, start, size, r[2], r[3])
            yield i, torch.where(good, j, i), r[3], good
        else:
            yield i, start + ((r[2] * size) >> 32), r[3], None


def _exact_sps(case, seed):
    R = _Reference(case, seed)
    layouts = [R.coords]
    if case["compare"]:
        layouts.append(_finished(R.node_at, R.length, seed + 5000))
    xy = [c.double().reshape(2, -1) for c in layouts]
    got, skipped = [[] for _ in xy], 0
    for i, j, r3, good in _sps_pairs(R, case, seed):
        a, b, d = R.ends(i, j, r3)
        keep = d > 0 if good is None else good & (d > 0)
        skipped += int((~keep).sum())
        a, b, d = a[keep], b[keep], d[keep].double()
        for k, c in enumerate(xy):
            mag = torch.sqrt((c[0][a] - c[0][b]) ** 2 + (c[1][a] - c[1][b]) ** 2)
            got[k].append(((mag - d) / d) ** 2)
    got = [torch.cat(x) for x in got]
    n = got[0].numel()
    total = [float(x.sum()) for x in got]
    mean = [t / n for t in total]
    sd = [math.sqrt(float(((x - u) ** 2).sum()) / (n - 1)) for x, u in zip(got, mean)]
    if not case["compare"]:
        half = 1.96 * sd[0] / math.sqrt(n)
        return dict(mean=mean[0], ci_lo=mean[0] - half, ci_hi=mean[0] + half, stddev=sd[0], sum=total[0],
                    sumsq_dev=float(((got[0] - mean[0]) ** 2).sum()), n_valid=n, n_skipped=skipped)
    ratio = total[0] / total[1]
    diff = math.sqrt(float(((got[0] - ratio * got[1]) ** 2).sum()) / (n - 1))
    half = 1.96 * diff / (math.sqrt(n) * mean[1])
    return dict(mean_a=mean[0], mean_b=mean[1], ratio=ratio, ratio_ci_lo=ratio - half, ratio_ci_hi=ratio + half,
                sd_a=sd[0], sd_b=sd[1], sd_diff=diff, sum_a=total[0], sum_b=total[1], n_valid=n, n_skipped=skipped)


def _exact_all_pairs(case, seed):
    R = _Reference(case, seed)
    c = R.coords.double().reshape(2, -1, 2)
    total, count = 0.0, 0
    off = R.off.tolist()
    for p in range(len(off) - 1):
        at = slice(off[p], off[p + 1])
        node, rev, size, pos = R.node[at], R.rev[at], R.len[at], R.pos[at]
        n = node.numel()
        end = [(pos + size * (e ^ rev)).double() for e in (0, 1)]
        x, y = c[0][node], c[1][node]
        rows = max(1, (1 << 24) // n)
        for r in range(0, n, rows):
            i = torch.arange(r, min(n, r + rows), device=DEV)
            above = torch.arange(n, device=DEV)[None, :] > i[:, None]
            part = torch.zeros(i.numel(), n, dtype=torch.float64, device=DEV)
            valid = torch.zeros_like(part)
            for ei in (0, 1):
                for ej in (0, 1):
                    d = (end[ei][i][:, None] - end[ej][None, :]).abs()
                    mag = torch.sqrt((x[i, ei][:, None] - x[:, ej][None, :]) ** 2 +
                                     (y[i, ei][:, None] - y[:, ej][None, :]) ** 2)
                    good = (d > 0) & above
                    part += torch.where(good, ((mag - d) / d) ** 2, torch.zeros_like(d))
                    valid += good
            has = valid > 0
            total += float((part[has] / valid[has]).sum())
            count += int(has.sum())
    return total / count, count


def _exact_train(case, seed):
    R = _Reference(case, seed)
    n, key = case["pairs"], 11 + seed
    c = R.coords.double().reshape(2, -1)

    def first(q):
        r = _philox(q, 0, 2 << 24, key)
        return _scale(r[0], r[1], R.S)

    total, count = 0.0, 0
    grad = torch.zeros_like(c)
    for r2, r3, i, start, size in R.windowed(_shift(R.S, 10), n, first, 7, 0, key):
        j, good = R.power_law(i, start, size, r2, r3)
        a, b, d = R.ends(i, torch.where(good, j, i), r3)
        good = good & (d > 0) & (a != b)
        a, b, d = a[good], b[good], d[good].double()
        dx, dy = c[0][a] - c[0][b], c[1][a] - c[1][b]
        mag = torch.sqrt(dx * dx + dy * dy)
        total += float((((mag - d) / d) ** 2).sum())
        count += d.numel()
        f = torch.where(mag > 0, 2.0 * (mag - d) / (d * d) / mag, torch.zeros_like(mag))
        for k, v in ((0, f * dx), (1, f * dy)):
            grad[k].index_add_(0, a, v)
            grad[k].index_add_(0, b, -v)
    grad = (grad / count).reshape(-1)
    m, v = (t.double() for t in _adam_state(grad.numel(), seed))
    m = 0.9 * m + 0.1 * grad
    v = 0.999 * v + 0.001 * grad * grad
    t = 11
    x = R.coords.double() - 0.1 * (m / (1 - 0.9 ** t)) / (torch.sqrt(v / (1 - 0.999 ** t)) + 1e-8)
    return dict(loss=torch.tensor(total / count, dtype=torch.float64), grad=grad, x=x, m=m, v=v)


def exact(case, seed):
    kind = case["kind"]
    if kind == "sps":
        return _exact_sps(case, seed)
    if kind == "exact":
        return _exact_all_pairs(case, seed)
    if kind == "train":
        return _exact_train(case, seed)
    return None  # a layout is one of many that the concurrent updates may give
