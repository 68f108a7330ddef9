"""Measured cases of the Barnes-Hut t-SNE library: the calls a user's program
makes, over the range of sizes, embeddings and options it makes them with.

A run is: neighbour lists -> input similarities (once) -> a locality layout of P
(once, or again as Y evolves) -> about 1000 optimiser steps -> the cost.  Inputs
are seeded and synthetic, drawn on the GPU: clustered points without index
locality, k neighbours per point inside its cluster, Gaussian weights, P = (P +
P^T) / 2N; an early embedding is N(0, 1e-4 I), a late one is clustered.

    listed(), draw(rng)     the cases, and one more of the same ranges
    prepare(case, seed)     what the program has in hand before the call
    run(state)              one pass
    work(case)              bytes and flops a pass cannot do without
    tolerance(case)         how far another correct implementation may be off
    exact(case, seed)       the same outputs in 64 bits, by plain torch
"""
import math

import numpy as np
import torch

import paper_2212_11506_amd as bh

DEV = "cuda"


# ------------------------------------------------------------------ the cases
# call: "step" (one optimiser iteration in place), "gradient" (for a program with
# its own optimiser), "relayout" (a new layout, then a gradient through it),
# "affinities" (P from neighbour lists), "cost" (exact Z and KL).
# form: "layout" (P through its locality layout, the fast path) or "csr".
def _opt(name, call, n, **kw):
    c = dict(name=name, call=call, n=n, k=90, clusters=10, sizes="equal", phase="early", dups=0.0, theta=0.5,
             exaggeration=1.0, form="layout", dtype="f32", dim=2)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest real run: a few thousand points, where launches and latency count
        _opt("step_2k", "step", 2_000),
        # a script that hands its CSR matrix over as it is, at an odd size
        _opt("step_10k_csr", "step", 9_973, k=45, clusters=7, sizes="dirichlet", form="csr"),
        # a whole image data set (70k points), main phase of the schedule
        _opt("step_70k", "step", 70_000),
        # the headline run: single-cell data, 1.3M points, early exaggeration
        _opt("step_1300k", "step", 1_300_000, clusters=30, sizes="dirichlet", exaggeration=12.0),
        # its late phase at the accurate end of theta, with duplicated cells, an odd size
        _opt("gradient_1000k_fine", "gradient", 1_000_003, clusters=30, sizes="dirichlet", phase="late", dups=0.05,
             theta=0.2),
        # the largest: 5M points late in a run, clusters of very unequal size
        _opt("step_5000k", "step", 5_000_000, clusters=100, sizes="zipf", phase="late"),
        # data without clusters from a random start: rows reach the whole index range
        _opt("step_700k_connected", "step", 700_000, k=30, clusters=1, exaggeration=12.0),
        # double precision (the paper's default)
        _opt("gradient_200k_f64", "gradient", 200_000, clusters=20, sizes="dirichlet", phase="late", dtype="f64"),
        # a three-dimensional embedding
        _opt("step_150k_3d", "step", 150_001, k=60, clusters=12, sizes="dirichlet", dim=3),
        # the input similarities of the headline run
        _opt("affinities_1300k", "affinities", 1_300_000, clusters=30, sizes="dirichlet"),
        # a new layout once the embedding has taken shape, and the first gradient through it
        _opt("relayout_200k", "relayout", 200_003, clusters=20, sizes="dirichlet", phase="late"),
        # the cost a run reports: exact normaliser and KL divergence
        _opt("cost_70k", "cost", 70_000, phase="late"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "csr", "f64", "3d", "affinities", "relayout", "cost"], [5, 2, 2, 2, 2, 2, 1])[0]
    k = rng.choice([15, 30, 45, 60, 90, 150])
    phase = rng.choice(["early", "late"])
    opt = dict(k=k, phase=phase, theta=rng.choice([0.3, 0.5, 0.5, 0.8]), exaggeration=rng.choice([1.0, 12.0]),
               sizes=rng.choice(["equal", "dirichlet", "zipf"]))
    if phase == "late":
        opt["dups"] = rng.choice([0.0, 0.05])
    if kind == "step":
        n = _log_uniform(rng, 1_500, 1_500_000)
        call = rng.choice(["step", "step", "gradient"])
    elif kind == "csr":
        n, call = _log_uniform(rng, 1_200, 200_000), "step"
        opt["form"] = "csr"
    elif kind == "f64":
        n, call = _log_uniform(rng, 3_000, 400_000), rng.choice(["step", "gradient"])
        opt.update(dtype="f64", form=rng.choice(["layout", "layout", "csr"]))
    elif kind == "3d":
        n, call = _log_uniform(rng, 3_000, 400_000), rng.choice(["step", "gradient"])
        opt.update(dim=3, form=rng.choice(["layout", "layout", "csr"]))
    elif kind == "affinities":
        n, call = _log_uniform(rng, 5_000, 600_000), "affinities"
    elif kind == "relayout":
        n, call = _log_uniform(rng, 5_000, 400_000), "relayout"
    else:
        n, call = _log_uniform(rng, 3_000, 100_000), "cost"
    # clusters of a few hundred points and more, so that k neighbours exist
    opt["clusters"] = rng.randint(1, max(1, min(30, n // (5 * k))))
    c = _opt("", call, n, **opt)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs (plain torch)
def _cluster_sizes(case, rng):
    n, c, floor = case["n"], case["clusters"], min(2 * case["k"] + 2, case["n"] // case["clusters"])
    if case["sizes"] == "dirichlet":
        share = rng.dirichlet(np.ones(c))
    elif case["sizes"] == "zipf":
        share = np.arange(1, c + 1, dtype=np.float64) ** -1.1
    else:
        share = np.ones(c)
    sizes = floor + np.floor(share / share.sum() * (n - c * floor)).astype(np.int64)
    sizes[int(np.argmax(sizes))] += n - int(sizes.sum())
    return sizes


def _clusters(case, seed):
    """(order: points cluster by cluster, first position and size of every position's cluster, rng, generator)"""
    rng = np.random.Generator(np.random.PCG64([seed, case["n"]]))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(rng.integers(1 << 62)))
    sizes = torch.from_numpy(_cluster_sizes(case, rng)).to(DEV)
    order = torch.randperm(case["n"], generator=gen, device=DEV)
    start = torch.cumsum(sizes, 0) - sizes
    which = torch.repeat_interleave(torch.arange(sizes.numel(), device=DEV), sizes)
    return order, which, start, sizes, rng, gen


def _distinct(n, k, room, gen):
    """k distinct whole numbers below room[i] for every row i, ascending: [n, k] int32"""
    room = room.to(torch.float64).unsqueeze(1)

    def some(rows):
        r = room[rows]
        u = torch.rand((r.shape[0], k), generator=gen, device=DEV, dtype=torch.float32)
        return torch.minimum((u.double() * r).to(torch.int32), (r - 1).to(torch.int32))

    x = torch.empty((n, k), dtype=torch.int32, device=DEV)
    step = max(1, (1 << 27) // k)
    for a in range(0, n, step):
        rows = slice(a, min(n, a + step))
        x[rows] = torch.sort(some(rows), dim=1).values
    bad = torch.nonzero((x[:, 1:] == x[:, :-1]).any(1)).squeeze(1)
    while bad.numel():  # draw the repeated ones of a row again
        y = x[bad]
        again = torch.zeros_like(y, dtype=torch.bool)
        again[:, 1:] = y[:, 1:] == y[:, :-1]
        y = torch.sort(torch.where(again, some(bad), y), dim=1).values
        x[bad] = y
        bad = bad[(y[:, 1:] == y[:, :-1]).any(1)]
    return x


def _neighbours(case, which, start, sizes, gen):
    """k distinct other members of its own cluster for the point at every position: [n, k] positions"""
    n = case["n"]
    nb = _distinct(n, case["k"], (sizes - 1)[which], gen)
    own = (torch.arange(n, device=DEV) - start[which]).to(torch.int32).unsqueeze(1)
    nb += (nb >= own)
    nb += start[which].to(torch.int32).unsqueeze(1)
    return nb


def _symmetrised(n, src, dst, p):
    """CSR of (p + p^T) / 2n from distinct directed pairs"""
    key = torch.cat([src * n + dst, dst * n + src])
    del src, dst
    key, at = torch.sort(key)
    val = torch.cat([p, p])[at]
    del at
    twin = key[1:] == key[:-1]  # a pair listed in both directions comes twice in a row
    val[:-1] += torch.where(twin, val[1:], torch.zeros((), dtype=val.dtype, device=DEV))
    keep = torch.ones_like(key, dtype=torch.bool)
    keep[1:] = ~twin
    del twin
    key, val = key[keep], val[keep] / (2.0 * n)
    row = torch.div(key, n, rounding_mode="floor")
    ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(row, minlength=n), 0)
    return ptr, (key - row * n).to(torch.int32), val


def _embedding(case, order, which, sizes, rng, gen):
    n, dim = case["n"], case["dim"]
    y = torch.randn((n, dim), generator=gen, device=DEV, dtype=torch.float64)
    if case["phase"] == "early":
        y *= 1e-2
    else:
        c = sizes.numel()
        centre = torch.from_numpy(rng.uniform(-50.0, 50.0, (c, dim))).to(DEV)
        spread = torch.from_numpy(rng.uniform(0.1, 2.0, (c, 1))).to(DEV)
        y = centre[which] + spread[which] * y
        if case["dups"] > 0:  # some points copy the one before them in their cluster
            copy = torch.rand(n, generator=gen, device=DEV) < case["dups"]
            copy[0] = False
            copy[1:] &= which[1:] == which[:-1]
            copy[1:] &= ~copy[:-1].clone()
            y[1:] = torch.where(copy[1:].unsqueeze(1), y[:-1].clone(), y[1:])
    out = torch.empty_like(y)
    out[order] = y
    return out if case["dtype"] == "f64" else out.to(torch.float32)


def _inputs(case, seed):
    """Y and P = (row_ptr, col, val), in the caller's (shuffled) order"""
    order, which, start, sizes, rng, gen = _clusters(case, seed)
    n, k = case["n"], case["k"]
    nb = _neighbours(case, which, start, sizes, gen)
    w = torch.rand((n, k), generator=gen, device=DEV, dtype=torch.float32).mul_(3.0)
    w = torch.exp(-w.double().square_())
    w /= w.sum(1, keepdim=True)
    src = order.unsqueeze(1).expand(n, k).reshape(-1)
    ptr, col, val = _symmetrised(n, src, order[nb.reshape(-1)], w.reshape(-1))
    del nb, w, src
    val = val if case["dtype"] == "f64" else val.to(torch.float32)
    return _embedding(case, order, which, sizes, rng, gen), ptr, col, val


def _momentum_state(case, y, seed):
    """update and gains as they stand some way into a run"""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed * 7919 + case["n"])
    u = torch.randn(y.shape, generator=gen, device=DEV, dtype=torch.float64) * (0.01 * float(y.std()))
    g = 0.5 + torch.rand(y.shape, generator=gen, device=DEV, dtype=torch.float64)
    return u.to(y.dtype), g.to(y.dtype)


def _knn(case, seed):
    """Neighbour lists as a search returns them, by increasing distance, and the perplexity k / 3.  Half of a
    list is mutual (the nearest on a ring through the cluster, on either side); the rest are other members up
    to half the ring ahead, which never list the point back, so that P's entry count does not vary."""
    order, which, start, sizes, rng, gen = _clusters(case, seed)
    n, k = case["n"], case["k"]
    near = k // 4
    m = sizes[which].to(torch.int32).unsqueeze(1)
    ahead = _distinct(n, k - 2 * near, ((sizes - 1) // 2 - near)[which], gen) + (near + 1)
    ring = torch.arange(1, near + 1, dtype=torch.int32, device=DEV).expand(n, near)
    first = start[which].to(torch.int32).unsqueeze(1)
    own = torch.arange(n, dtype=torch.int32, device=DEV).unsqueeze(1) - first
    nb = first + (own + torch.cat([ring, m - ring, ahead], 1)) % m
    shuffle = torch.rand((n, k), generator=gen, device=DEV, dtype=torch.float32).argsort(1)
    idx = torch.empty((n, k), dtype=torch.int32, device=DEV)
    idx[order] = order[torch.gather(nb, 1, shuffle)].to(torch.int32)
    dist = torch.rand((n, k), generator=gen, device=DEV, dtype=torch.float32).mul_(3.0).sort(1).values
    return idx, dist, k / 3.0


# ------------------------------------------------------------------ the passes
def _schedule(case):
    early = case["exaggeration"] > 1.0
    return dict(learning_rate=max(case["n"] / 12.0, 200.0), momentum=0.5 if early else 0.8, min_gain=0.01)


_API = {  # (dtype, dim): matrix, layout, workspace size, gradient, step
    ("f32", 2): (bh.Csr, bh.Layout, bh.workspace_size, bh.gradient, bh.step),
    ("f64", 2): (bh.CsrF64, bh.LayoutF64, bh.workspace_size_f64, bh.gradient_f64, bh.step_f64),
    ("f32", 3): (bh.Csr, bh.Layout3, bh.workspace_size_3d, bh.gradient_3d, bh.step_3d),
}


def prepare(case, seed):
    s = {"case": case}
    n = case["n"]
    if case["call"] == "affinities":
        s["idx"], s["dist"], s["perplexity"] = _knn(case, seed)
        s["ws"] = torch.empty(bh.affinities_workspace_size(n, case["k"]), dtype=torch.uint8, device=DEV)
        return s
    csr, layout, size, s["gradient"], s["step"] = _API[case["dtype"], case["dim"]]
    s["Y"], ptr, col, val = _inputs(case, seed)
    s["P"] = csr(ptr, col, val)
    s["ws"] = torch.empty(size(n, s["P"].nnz), dtype=torch.uint8, device=DEV)
    s["grad"] = torch.empty_like(s["Y"])
    if case["form"] == "layout" and case["call"] in ("step", "gradient"):
        lay = layout(s["P"], s["Y"], workspace=s["ws"])
        # a 3-D layout without tiles is refused by the 3-D calls: the matrix itself serves
        if case["dim"] == 2 or lay.tiles:
            s["P"] = lay  # the layout holds its own copy of P
    if case["call"] == "step":
        s["update"], s["gains"] = _momentum_state(case, s["Y"], seed)
    return s


def run(s):
    c = s["case"]
    if c["call"] == "affinities":
        P, sigma2 = bh.affinities(s["idx"], s["dist"], s["perplexity"], workspace=s["ws"], sigma2=True)
        return {"row_ptr": P.row_ptr, "col": P.col, "val": P.val, "sigma2": sigma2}
    if c["call"] == "cost":
        z = bh.z_exact(s["Y"], workspace=s["ws"])
        return {"Z": np.float64(z), "kl": np.float64(bh.kl(s["Y"], s["P"], z, workspace=s["ws"]))}
    if c["call"] == "relayout":
        lay = bh.Layout(s["P"], s["Y"], workspace=s["ws"])
        grad, z = s["gradient"](s["Y"], lay, c["theta"], c["exaggeration"], grad=s["grad"], workspace=s["ws"])
        return {"grad": grad, "Z": np.float64(z)}
    if c["call"] == "gradient":
        grad, z = s["gradient"](s["Y"], s["P"], c["theta"], c["exaggeration"], grad=s["grad"], workspace=s["ws"])
        return {"grad": grad, "Z": np.float64(z)}
    s["step"](s["Y"], s["P"], c["theta"], c["exaggeration"], update=s["update"], gains=s["gains"], workspace=s["ws"],
              **_schedule(c))
    # The gains are left out: where a gradient is near zero its rounding decides between + 0.2 and x 0.8, which
    # moves a gain by a third and the embedding by nothing.  A pass reads the gains that the one before it wrote.
    return {"Y": s["Y"], "update": s["update"]}


# ------------------------------------------------------------------ floors and tolerances
def work(case):
    n, k, dim = case["n"], case["k"], case["dim"]
    f = 8 if case["dtype"] == "f64" else 4
    nnz = 2 * n * k
    entries = nnz * (4 + f) + 8 * (n + 1)
    # interactions of a point: about 7 ln n / theta^1.6 in the plane (measured 117 at 2k points, 202 at 70k,
    # 309 at 1.3M, theta 0.5), some four times as many in space; 14 flops each, 17 in space
    inter = n * min(n - 1.0, 7.0 * math.log(n) / case["theta"] ** 1.6 * (4 if dim == 3 else 1))
    if case["call"] == "affinities":
        # lists in, P and sigma^2 out; about 30 evaluations of a Gaussian row at some 20 flops a neighbour
        return {"bytes": 8 * n * k + 8 * nnz + 16 * n, "flops": 600.0 * n * k}
    if case["call"] == "cost":
        return {"bytes": 8 * n + entries, "flops": 7.0 * n * n + 50.0 * nnz}
    bytes_ = entries + n * dim * f * (2 if case["call"] != "step" else 6)
    if case["call"] == "relayout":
        bytes_ += 2 * entries  # the copy written, and read by the gradient
    return {"bytes": bytes_, "flops": inter * (17 if dim == 3 else 14) + nnz * (9 if dim == 2 else 12)}


def tolerance(case):
    # About four times what the calls differ from exact() by over some fifty drawn cases.
    if case["call"] == "affinities":
        return {"rel": 1e-7, "max": 2.5e-7}  # one rounding to 32 bits: 2.6e-8, largest 6e-8
    if case["call"] == "cost":
        return {"rel": 1e-7}  # pair terms in 32 bits: 2e-8
    if case["dtype"] == "f64":
        return {"rel": 2e-11, "max": 1e-9}  # 4.9e-12, most of it exact()'s own centres; largest 2e-11
    # Sums of some hundred to a thousand terms in 32 bits, of which attraction and repulsion cancel the more
    # the longer a phase lasts: up to 2.4e-5.  A cell near the acceptance bound is taken differently now and
    # then, which moves a single value by up to 9e-3.
    return {"rel": 1e-4, "max": 3.5e-2}


# ------------------------------------------------------------------ 64-bit values by plain torch
def _bits(dim):
    return (32, 64) if dim == 2 else (21, 63)


def _tree(y, theta2):
    """The compressed tree over the sorted Morton codes of y (float64), nodes in depth-first order."""
    n, dim = y.shape
    bits, top = _bits(dim)
    lo, hi = y.min(0).values, y.max(0).values
    cent, span = (lo + hi) * 0.5, float(0.5 * (hi - lo).max())
    scale = (2.0 ** (bits - 1)) / span if span > 0 else 0.0
    grid = ((y - (cent - span)) * scale).clamp(0, 2.0 ** bits - 1).to(torch.int64)
    code = torch.zeros(n, dtype=torch.int64, device=y.device)
    for b in range(bits):
        for d in range(dim):
            code |= ((grid[:, d] >> b) & 1) << (dim * b + d)
    flip = torch.tensor(-(1 << 63) if dim == 2 else 0, dtype=torch.int64, device=y.device)
    code, perm = torch.sort(code ^ flip, stable=True)
    ys = y[perm]
    diff = code[1:] ^ code[:-1]
    lam = torch.zeros(n - 1, dtype=torch.int64, device=y.device)  # levels two neighbours share
    for level in range(1, bits + 1):
        lam += (diff >> (top - dim * level)) == 0
    ends = torch.tensor([n], device=y.device)
    begin, end, lev = [torch.arange(n, device=y.device)], [torch.arange(1, n + 1, device=y.device)], \
        [torch.full((n,), bits + 1, device=y.device)]
    for level in range(bits + 1):
        first = torch.cat([torch.zeros(1, dtype=torch.int64, device=y.device), torch.nonzero(lam < level).squeeze(1) + 1])
        last = torch.cat([first[1:], ends])
        here = torch.nonzero(lam == level).squeeze(1)
        cell = torch.unique(torch.searchsorted(first, here, right=True) - 1)
        if level == 0:
            cell = torch.zeros(1, dtype=torch.int64, device=y.device)
        begin.append(first[cell])
        end.append(last[cell])
        lev.append(torch.full((cell.numel(),), level, device=y.device))
    begin, end, lev = torch.cat(begin), torch.cat(end), torch.cat(lev)
    key, at = torch.sort(begin * 64 + lev)
    begin, end, lev = begin[at], end[at], lev[at]
    skip = torch.searchsorted(key, end * 64)
    sums = torch.zeros((n + 1, dim), dtype=torch.float64, device=y.device)
    sums[1:] = torch.cumsum(ys - cent, 0)
    count = (end - begin).double()
    com = torch.where((end - begin == 1).unsqueeze(1), ys[begin], cent + (sums[end] - sums[begin]) / count.unsqueeze(1))
    side2 = (2.0 * span * torch.pow(2.0, -lev.double())) ** 2
    # a point is always taken; with theta = 0 nothing else is
    limit = torch.where(lev == bits + 1, -1.0, side2 / theta2 if theta2 > 0 else torch.inf)
    return perm, ys, begin, lev == bits + 1, skip, com, count, limit


def _repulsion(y, theta2):
    n, dim = y.shape
    perm, ys, begin, leaf, skip, com, count, limit = _tree(y, theta2)
    force = torch.zeros((n, dim), dtype=torch.float64, device=y.device)
    z = 0.0
    chunk = 1 << 16
    for a in range(0, n, chunk):
        m = min(chunk, n - a)
        pt = torch.arange(m, device=y.device)
        node = torch.zeros(m, dtype=torch.int64, device=y.device)
        f = torch.zeros((m, dim), dtype=torch.float64, device=y.device)
        while pt.numel():
            d = ys[a + pt] - com[node]
            d2 = d.square().sum(1)
            take = d2 > limit[node]
            own = leaf[node] & (begin[node] == a + pt)
            t = take & ~own
            w = 1.0 / (1.0 + d2[t])
            cw = count[node[t]] * w
            z += float(cw.sum())
            f.index_add_(0, pt[t], (cw * w).unsqueeze(1) * d[t])
            r = ~take & ~leaf[node]
            parent_pt, stop, child = pt[r], skip[node[r]], node[r] + 1
            pts, nodes = [], []
            while parent_pt.numel():
                pts.append(parent_pt)
                nodes.append(child)
                child = skip[child]
                more = child < stop
                parent_pt, stop, child = parent_pt[more], stop[more], child[more]
            pt = torch.cat(pts) if pts else pt[:0]
            node = torch.cat(nodes) if nodes else node[:0]
        force[a:a + m] = f
    out = torch.empty_like(force)
    out[perm] = force
    return out, z


def _entries(ptr, limit=1 << 25):
    """ranges of entries, with the row of each"""
    n, nnz = ptr.numel() - 1, int(ptr[-1])
    for a in range(0, nnz, limit):
        e = torch.arange(a, min(nnz, a + limit), device=ptr.device)
        yield slice(a, min(nnz, a + limit)), torch.searchsorted(ptr[1:], e, right=True).clamp_(max=n - 1)


def _attraction(y, ptr, col, val):
    f = torch.zeros_like(y)
    for s, row in _entries(ptr):
        d = y[row] - y[col[s].long()]
        f.index_add_(0, row, (val[s].double() / (1.0 + d.square().sum(1))).unsqueeze(1) * d)
    return f


def exact(case, seed):
    n = case["n"]
    if case["call"] == "affinities":
        return _exact_affinities(*_knn(case, seed))
    if n > 1_500_000:
        return None  # minutes
    y0, ptr, col, val = _inputs(case, seed)
    y = y0.double()
    if case["call"] == "cost":
        z = 0.0
        for a in range(0, n, 4096):
            d2 = sum((y[a:a + 4096, d, None] - y[None, :, d]) ** 2 for d in range(2))
            z += float((1.0 / (1.0 + d2)).sum())
        z -= n
        kl = 0.0
        for s, row in _entries(ptr):
            p = val[s].double()
            d2 = (y[row] - y[col[s].long()]).square().sum(1)
            kl += float(torch.where(p > 0, p * (torch.log(p.clamp_min(1e-300)) + torch.log1p(d2) + math.log(z)), 0.0).sum())
        return {"Z": torch.tensor(z, dtype=torch.float64), "kl": torch.tensor(kl, dtype=torch.float64)}
    num = float if case["dtype"] == "f64" else lambda x: float(np.float32(x))  # the call's own arguments
    rep, z = _repulsion(y, num(case["theta"]) ** 2)
    g = 4.0 * (num(case["exaggeration"]) * _attraction(y, ptr, col, val) - rep / z)
    if case["call"] != "step":
        return {"grad": g, "Z": torch.tensor(z, dtype=torch.float64)}
    sch = _schedule(case)
    u, gains = (t.double() for t in _momentum_state(case, y0, seed))
    gains = torch.where(u * g < 0, gains + num(0.2), gains * num(0.8)).clamp_min(num(sch["min_gain"]))
    u = num(sch["momentum"]) * u - num(sch["learning_rate"]) * gains * g
    return {"Y": y + u, "update": u}


def _exact_affinities(idx, dist, perplexity):
    n, k = idx.shape
    p = torch.empty((n, k), dtype=torch.float64, device=DEV)
    sigma2 = torch.empty(n, dtype=torch.float64, device=DEV)
    want = math.log(perplexity)
    for a in range(0, n, 1 << 18):
        d2 = dist[a:a + (1 << 18)].double().square_()
        d2 -= d2.min(1, keepdim=True).values

        def entropy(s2):
            t = d2 / (2.0 * s2).unsqueeze(1)
            w = torch.exp(-t)
            total = w.sum(1)
            return torch.log(total) + (t * w).sum(1) / total

        lo, hi = torch.zeros_like(d2[:, 0]), d2.max(1).values.clone()
        for _ in range(200):
            low = entropy(hi) < want
            if not bool(low.any()):
                break
            hi = torch.where(low, 2.0 * hi, hi)
        for _ in range(70):
            mid = 0.5 * (lo + hi)
            low = entropy(mid) < want
            lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
        w = torch.exp(-d2 / (2.0 * hi).unsqueeze(1))
        p[a:a + (1 << 18)] = w / w.sum(1, keepdim=True)
        sigma2[a:a + (1 << 18)] = hi
    src = torch.arange(n, device=DEV).unsqueeze(1).expand(n, k).reshape(-1)
    ptr, col, val = _symmetrised(n, src, idx.reshape(-1).long(), p.reshape(-1))
    return {"row_ptr": ptr, "col": col, "val": val, "sigma2": sigma2}
