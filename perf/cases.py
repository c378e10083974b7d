"""The workloads this library is timed on, each as a user's program runs it.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call (the
matrix and right-hand sides on the device, the handle with its analysis,
rewrite and schedule), ``run(state)`` is one pass through the public entry
points, ``work(case)`` the bytes and operations such a pass cannot do without,
and ``exact(case, seed)`` the same results from plain torch in 64 bits.

The matrices have the structures of the library's own benchmark inputs (the
random window, the 2D and 3D stencil factors with a near-serial tail, the power
law, the stand-ins for lung2 and torso2, the batch of window matrices), drawn
on the device from the seed. Off-diagonals are uniform in (-1, 1) on a grid of
2^-30, so that the diagonals 1 + sum |off-diagonals| do not depend on the order
of the sum; right-hand sides are uniform in (-1, 1).

Schedules: "default" is what a handle starts with, "tuned" runs the autotuner
in ``prepare``, and eight numbers are a schedule that a program keeps from an
earlier tuning (mode, thin_rows, wg_threads, wide_threads, lanes_per_row,
wide_grid, overlap, thin_cols).
"""
import math

import torch

import paper_2206_05843_amd as sp

FORMS = {"L": sp.LOWER, "LT": sp.LOWER_TRANS}
SYNC_FREE = "3,0,512,256,1,256,0,0"       # what the autotuner keeps on power-law matrices and for one column in 3D
THIN = "0,1024,1024,256,1,0,0,0"          # on the rewritten 2D stencil
PERSISTENT = "0,256,1024,256,1,4096,0,1"  # on the 3D stencil with many columns


def listed():
    return [
        # the smallest call: one solve of a small system, where latency and launches are all there is
        dict(name="window_2k", what="solve", matrix="window", n=2000, nrhs=1, schedule="tuned"),
        # a lung2-sized system after the paper's own rewriting rule: 26 fat levels and a few rewritten ones
        dict(name="lung2_avgcost", what="solve", matrix="lung2", n=109460, nrhs=1, rewrite="cost", schedule="tuned"),
        # a transposed (back-substitution) solve of a mesh matrix with a handful of right-hand sides by columns
        dict(name="torso2_trans_7rhs", what="solve", matrix="torso2", n=115967, form="LT", nrhs=7, schedule="tuned"),
        # the 2D stencil + chain after the naive rewrite, on its tuned schedule (one right-hand side)
        dict(name="stencil2d_naive", what="solve", matrix="stencil2d", k=1000, tail=20000, nrhs=1, rewrite="naive",
             schedule=THIN),
        # an unrewritten, untuned 2D stencil + chain of an odd size: what a program gets from analyze and solve alone
        dict(name="stencil2d_plain", what="solve", matrix="stencil2d", k=301, tail=4001, nrhs=1, schedule="default"),
        # one matrix of the size the learned policy is trained on, synchronisation-free
        dict(name="powerlaw_200k", what="solve", matrix="powerlaw", n=200003, window=2048, segments=8, nrhs=1,
             schedule=SYNC_FREE),
        # the large power law, rewritten, synchronisation-free
        dict(name="powerlaw_4m_naive", what="solve", matrix="powerlaw", n=4000000, window=4096, segments=8, nrhs=1,
             rewrite="naive", schedule=SYNC_FREE),
        # the largest: the 3D stencil factor with a tail and 32 right-hand sides by rows, graph replays
        dict(name="stencil3d_32rhs", what="solve", matrix="stencil3d", k=200, tail=5000, nrhs=32, rewrite="naive",
             rows=True, graph=True, schedule=PERSISTENT),
        # one application z = L^-T L^-1 r of an incomplete-Cholesky preconditioner inside a Krylov solver
        dict(name="precond_3d_1rhs", what="precond", matrix="stencil3d", k=101, tail=500, nrhs=1, rewrite="naive",
             schedule="tuned"),
        # many independent systems in one call, sixteen right-hand sides each
        dict(name="batch_512x16", what="batch", nmat=512, nmin=1000, nmax=50000, nrhs=16, schedule="tuned"),
        # preprocessing: analysis and naive rewriting of a power-law matrix, and its results
        dict(name="analyze_rewrite", what="setup", matrix="powerlaw", n=300007, window=1024, segments=8),
        # one gradient of the policy network on a batch of levels, and the inference of their probabilities
        dict(name="policy_gradient", what="policy", batch=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["window", "lung2", "torso2", "stencil2d", "powerlaw", "powerlaw", "stencil3d", "precond",
                       "batch", "setup", "policy"])
    if kind == "window":
        return dict(what="solve", matrix="window", n=_log(rng, 300, 60000), nrhs=rng.choice([1, 1, 3]),
                    schedule="default")
    if kind == "lung2":
        return dict(what="solve", matrix="lung2", n=_log(rng, 20000, 400000), nrhs=1,
                    rewrite=rng.choice(["cost", "naive"]), schedule="default")
    if kind == "torso2":
        return dict(what="solve", matrix="torso2", n=_log(rng, 20000, 250000), form=rng.choice(["L", "LT"]),
                    nrhs=rng.randint(1, 12), schedule="default")
    if kind == "stencil2d":
        k = _log(rng, 100, 1000)
        c = dict(what="solve", matrix="stencil2d", k=k, tail=rng.randint(0, 20 * k), nrhs=1,
                 schedule=rng.choice(["default", THIN]))
        if rng.random() < 0.5:
            c["rewrite"] = "naive"
        return c
    if kind == "powerlaw":
        c = dict(what="solve", matrix="powerlaw", n=_log(rng, 50000, 3000000), window=rng.randint(256, 4096),
                 segments=rng.randint(0, 16), nrhs=rng.choice([1, 1, 2]), schedule=SYNC_FREE)
        if rng.random() < 0.5:
            c["rewrite"] = "naive"
        return c
    if kind == "stencil3d":
        return dict(what="solve", matrix="stencil3d", k=_log(rng, 40, 150), tail=rng.randint(0, 3000),
                    nrhs=rng.randint(2, 32), rewrite="naive", rows=rng.random() < 0.5, schedule=PERSISTENT)
    if kind == "precond":
        return dict(what="precond", matrix="stencil3d", k=_log(rng, 40, 160), tail=rng.randint(0, 2000),
                    nrhs=rng.choice([1, 1, 4]), rewrite="naive", schedule=SYNC_FREE)
    if kind == "batch":
        nmax = _log(rng, 2000, 50000)
        return dict(what="batch", nmat=rng.randint(20, 500), nmin=rng.randint(300, nmax // 2), nmax=nmax,
                    nrhs=rng.choice([1, 4, 8, 13, 16]), schedule="default")
    if kind == "setup":
        return dict(what="setup", matrix="powerlaw", n=_log(rng, 50000, 1000000), window=rng.randint(256, 4096),
                    segments=rng.randint(0, 16))
    return dict(what="policy", batch=_log(rng, 256, 65536))


# ------------------------------------------------------------------ matrices
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, dtype=torch.float64, device="cuda", generator=g)


def _below(g, high):
    """One integer in [0, high) per entry of ``high`` (high >= 1)."""
    return torch.minimum((_rand(g, high.numel()) * high).long(), high - 1)


def _arange(a, b):
    return torch.arange(a, b, dtype=torch.int64, device="cuda")


def _csr(n, rows, cols, g):
    """CSR with the distinct pairs as off-diagonals and the diagonal last."""
    key = torch.unique(rows * n + cols)
    rows, cols = key // n, key % n
    off = (torch.randint(-(1 << 30) + 1, 1 << 30, (key.numel(),), device="cuda", generator=g).double()
           / float(1 << 30))
    count = torch.bincount(rows, minlength=n) if key.numel() else torch.zeros(n, dtype=torch.int64, device="cuda")
    rp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rp[1:] = torch.cumsum(count + 1, 0)
    at = _arange(0, key.numel()) + rows  # one diagonal before each earlier row's end
    ci = torch.empty(key.numel() + n, dtype=torch.int32, device="cuda")
    va = torch.empty(key.numel() + n, dtype=torch.float64, device="cuda")
    ci[at] = cols.int()
    va[at] = off
    ci[rp[1:] - 1] = _arange(0, n).int()
    va[rp[1:] - 1] = 1.0 + torch.zeros(n, dtype=torch.float64, device="cuda").index_add_(0, rows, off.abs())
    return rp.int(), ci, va


def _tail(g, first, count):
    """Chain rows: each reads its predecessor and two earlier rows."""
    q = _arange(first, first + count)
    a, c = _below(g, q - 1), _below(g, q - 1)
    return torch.cat([q, q, q]), torch.cat([a, c, q - 1])


def _window(g, n, window=64, draws=5):
    i = _arange(1, n).repeat_interleave(draws)
    lo = torch.clamp(i - window, min=0)
    return n, i, lo + _below(g, i - lo)


def _stencil(g, k, dims, tail):
    n = k ** dims
    p = _arange(0, n)
    rows, cols = [], []
    for d in range(dims):
        step = k ** d
        has = p[(p // step) % k > 0]
        rows.append(has)
        cols.append(has - step)
    if tail:
        r, c = _tail(g, n, tail)
        rows.append(r)
        cols.append(c)
    return n + tail, torch.cat(rows), torch.cat(cols)


def _levels_of(widths):
    w = torch.tensor(widths, dtype=torch.int64, device="cuda")
    start = torch.zeros(w.numel() + 1, dtype=torch.int64, device="cuda")
    start[1:] = torch.cumsum(w, 0)
    return w, start, torch.repeat_interleave(_arange(0, w.numel()), w)


def _poisson(g, mean, count):
    return torch.poisson(torch.full((count,), float(mean), device="cuda"), generator=g).long()


def _lung2(g, n):
    two = 453
    fat = 26
    base, rem = divmod(n - 2 * two, fat)
    w, start, lev = _levels_of([base + (i < rem) for i in range(fat)] + [2] * two)
    r = _arange(int(w[0]), n)
    lr = lev[r]
    near = start[lr - 1] + _below(g, w[lr - 1])
    head = r[lr < fat]
    er = torch.repeat_interleave(head, _poisson(g, 2.646, head.numel()))
    lo = start[torch.clamp(lev[er] - 3, min=0)]
    ec = lo + _below(g, start[lev[er]] - lo)
    thin = r[lr >= fat]
    tc = _below(g, start[fat].expand(thin.numel()))
    return n, torch.cat([r, er, thin]), torch.cat([near, ec, tc])


def _torso2(g, n, nlev=513, back=8, spread=2):
    tri = [min(i + 1, nlev - i) for i in range(nlev)]
    total = sum(tri)
    widths = [max(1, t * n // total) for t in tri]
    widths[nlev // 2] += n - sum(widths)
    w, start, lev = _levels_of(widths)
    r = _arange(widths[0], n)

    def near(rows, src):
        f = (rows - start[lev[rows]]).double() / w[lev[rows]].double()
        at = (f * w[src]).long() + torch.randint(-spread, spread + 1, (rows.numel(),), device="cuda", generator=g)
        return start[src] + torch.minimum(torch.clamp(at, min=0), w[src] - 1)

    er = torch.repeat_interleave(r, _poisson(g, 7.8, r.numel()))
    src = lev[er] - 1 - _below(g, torch.clamp(lev[er], max=back))
    return n, torch.cat([r, er]), torch.cat([near(r, lev[r] - 1), near(er, src)])


def _powerlaw(g, n, window, segments, mean=8.0, seglen=250, alpha=1.2):
    """Every row reads one row of its local window (its predecessor inside the
    near-serial segments) and further columns with power-law weights."""
    deg = _poisson(g, mean, n)
    deg[:1] = 0
    wl = torch.full((n,), window, dtype=torch.int64, device="cuda")
    for s in range(segments):
        st = ((s + 1) * n) // (segments + 1)
        wl[st:st + seglen] = 1
    r = torch.nonzero(deg > 0).flatten()
    lo = torch.clamp(r - wl[r], min=0)
    near = lo + _below(g, r - lo)
    er = torch.repeat_interleave(r, deg[r] - 1)
    top = float(n) ** (1.0 - alpha) - 1.0
    rank = torch.clamp(((1.0 + _rand(g, er.numel()) * top) ** (1.0 / (1.0 - alpha))).long() - 1, 0, n - 1)
    ec = torch.randperm(n, device="cuda", generator=g)[rank] % er
    return n, torch.cat([r, er]), torch.cat([near, ec])


def _matrix(case, g):
    """(n, row_ptr, col, val) on the device. The results of "setup" hold whole
    matrices, so its pattern is that of its sizes and only the values come
    from the seed."""
    kind = case["matrix"]
    values, g = g, _generator(case["n"]) if case["what"] == "setup" else g
    if kind == "window":
        n, r, c = _window(g, case["n"])
    elif kind == "lung2":
        n, r, c = _lung2(g, case["n"])
    elif kind == "torso2":
        n, r, c = _torso2(g, case["n"])
    elif kind == "powerlaw":
        n, r, c = _powerlaw(g, case["n"], case["window"], case["segments"])
    else:
        n, r, c = _stencil(g, case["k"], 2 if kind == "stencil2d" else 3, case["tail"])
    return (n,) + _csr(n, r, c, values)


def _batch(case, g):
    """The concatenated window matrices (local row pointers and columns) and
    the same as one block-diagonal pattern."""
    lo, hi, m = case["nmin"], case["nmax"], case["nmat"]
    ns = torch.randint(lo, hi + 1, (m,), device="cuda", generator=_generator(m + hi))  # the same for every seed
    off = torch.zeros(m + 1, dtype=torch.int64, device="cuda")
    off[1:] = torch.cumsum(ns, 0)
    n = int(off[-1])
    mat = torch.repeat_interleave(_arange(0, m), ns)
    p = _arange(0, n)
    loc = p - off[mat]
    i = p[loc > 0].repeat_interleave(5)
    li = i - off[mat[i]]
    first = torch.clamp(li - 64, min=0)
    rp, ci, va = _csr(n, i, off[mat[i]] + first + _below(g, li - first), g)
    ends = _arange(0, n + m) - torch.repeat_interleave(_arange(0, m), ns + 1)  # row pointer of each local entry
    base = torch.repeat_interleave(rp[off[:-1]].long(), ns + 1)
    rp_cat = (rp[ends].long() - base).int()
    entry = torch.repeat_interleave(p, (rp[1:] - rp[:-1]).long())
    ci_cat = (ci.long() - off[mat[entry]]).int()
    return ns, off, mat, (n, rp, ci, va), (rp_cat, ci_cat)


def _rhs(g, nrhs, n):
    return 2.0 * _rand(g, nrhs, n) - 1.0


# ------------------------------------------------------------------- programs
def _handle(case, form, matrix):
    h = sp.Handle()
    _, rp, ci, va = matrix
    h.analyze(rp, ci, va, form=FORMS[form])
    which = sp.ORIGINAL
    if case.get("rewrite"):
        if case["rewrite"] == "cost":
            h.rewrite(sp.THIN_COST, 0.0, 0.0)
        else:
            h.rewrite(sp.THIN_ROWS, 32, 4.0)
        which = sp.REWRITTEN
    if case["schedule"] == "tuned":
        h.autotune(which, case["nrhs"], rows=bool(case.get("rows")))
    elif case["schedule"] != "default":
        h.set_schedule(which, *[int(v) for v in case["schedule"].split(",")])
    h.prepare(which, case["nrhs"])
    return h, which


def _network(g, batch):
    """Parameters, standardised features, labels and weights of one minibatch."""
    w = [(64, 20, 20), (64, 1, 0), (64, 64, 64), (64, 1, 0), (1, 64, 64), (1, 1, 0)]
    parts = []
    for a, b, fan in w:
        lim = math.sqrt(6.0 / fan) if fan else 0.05
        parts.append(((2.0 * _rand(g, a * b) - 1.0) * lim).float())
    feat = torch.randn(batch, 20, device="cuda", generator=g)
    label = (_rand(g, batch) < 0.4).float()
    weight = torch.where(label > 0.5, 0.5 / 0.4, 0.5 / 0.6).float()
    norm = torch.cat([torch.randn(20, device="cuda", generator=g) * 0.1,
                      0.5 + torch.rand(20, device="cuda", generator=g)]).reshape(2, 20)
    return torch.cat(parts), feat, label, weight, norm


def prepare(case, seed):
    g = _generator(seed)
    if case["what"] == "policy":
        return dict(what="policy", net=_network(g, case["batch"]))
    if case["what"] == "batch":
        ns, off, mat, (n, _, _, va), (rp_cat, ci_cat) = _batch(case, g)
        h = sp.Handle()
        h.batch_analyze(ns.tolist(), rp_cat, ci_cat, va)
        if case["schedule"] == "tuned":
            h.autotune(sp.BATCH, case["nrhs"])
        b = _rhs(g, 1, n * case["nrhs"]).reshape(-1)
        return dict(what="batch", h=h, b=b, x=torch.empty_like(b), nrhs=case["nrhs"])
    m = _matrix(case, g)
    if case["what"] == "setup":
        return dict(what="setup", m=m, h=sp.Handle())
    b = _rhs(g, case["nrhs"], m[0])
    if case["what"] == "precond":
        return dict(what="precond", L=_handle(case, "L", m), LT=_handle(case, "LT", m), r=b, y=torch.empty_like(b),
                    z=torch.empty_like(b))
    h, which = _handle(case, case.get("form", "L"), m)
    if case.get("rows"):
        b = b.t().contiguous()
    s = dict(what="solve", h=h, which=which, b=b, x=torch.empty_like(b), rows=bool(case.get("rows")))
    if case.get("graph"):
        with torch.cuda.stream(torch.cuda.Stream()):
            s["graph"] = h.graph_create_rows(b, s["x"], which) if s["rows"] else h.graph_create(b, s["x"], which)
    return s


def run(s):
    if s["what"] == "policy":
        params, feat, label, weight, norm = s["net"]
        prob = sp.mlp_forward(params, feat, norm)
        grad, loss = sp.mlp_backward(params, feat, label, weight, norm)
        return dict(prob=prob, grad=grad, loss=loss)
    h = s["h"] if "h" in s else None
    if s["what"] == "batch":
        return h.batch_solve(s["b"], s["x"], s["nrhs"])
    if s["what"] == "setup":
        _, rp, ci, va = s["m"]
        nlev = h.analyze(rp, ci, va)
        level_ptr, level_rows, row_level = h.levels()
        st = h.rewrite(sp.THIN_ROWS, 32, 4.0)
        return dict(nlev=nlev, level_ptr=level_ptr, level_rows=level_rows, row_level=row_level,
                    nlev_after=st["nlev_after"], moved=st["rows_rewritten"], **h.rewritten())
    if s["what"] == "precond":
        (hl, wl), (ht, wt) = s["L"], s["LT"]
        hl.solve(s["r"], wl, x=s["y"])
        return ht.solve(s["y"], wt, x=s["z"])
    if "graph" in s:
        h.graph_launch(s["graph"])
        return s["x"]
    return h.solve_rows(s["b"], s["which"], s["x"]) if s["rows"] else h.solve(s["b"], s["which"], s["x"])


# ----------------------------------------------------------- what it has to do
def _size(case):
    """Rows, nonzeros and levels (about)."""
    kind = case.get("matrix")
    if case["what"] == "batch":
        n = case["nmat"] * (case["nmin"] + case["nmax"]) // 2
        return n, 5.83 * n, 0.136 * n
    if kind in ("stencil2d", "stencil3d"):
        d = 2 if kind == "stencil2d" else 3
        k, n = case["k"], case["k"] ** d
        return n + case["tail"], (d + 1) * n - d * n / k + 4 * case["tail"], d * (k - 1) + 1 + case["tail"]
    n = case["n"]
    return {"window": (n, 5.83 * n, 0.136 * n), "lung2": (n, 4.5 * n, 479), "torso2": (n, 8.9 * n, 513),
            "powerlaw": (n, 8.7 * n, 0.001 * n + 250 * case.get("segments", 0))}[kind]


def work(case):
    """Every nonzero once (value and column), the row pointer and level map of
    every row, the level pointers, every right-hand side read and every
    solution written once; two operations a nonzero and column."""
    if case["what"] == "policy":
        b = case["batch"]
        return dict(bytes=4.0 * (b * (20 + 20 + 3) + 3 * 5569), flops=b * (2 + 6) * 5440.0)
    n, nnz, nlev = _size(case)
    if case["what"] == "setup":  # reads L; writes its level sets, L' and T
        return dict(bytes=12.0 * nnz + 4.0 * n + 12.0 * n + 12.0 * nnz + 4.0 * n + 12.0 * n + 4.0 * n, flops=2.0 * nnz)
    times = 2 if case["what"] == "precond" else 1
    c = case["nrhs"]
    return dict(bytes=times * (12.0 * nnz + 8.0 * n + 4.0 * nlev + 16.0 * n * c), flops=times * 2.0 * nnz * c)


# ------------------------------------------------------------------ 64-bit results
def _solve64(n, rp, ci, va, b):
    """x of L x = b (b of shape (n, nrhs)), level by level in plain torch."""
    rp = rp.long()
    deg = rp[1:] - rp[:-1] - 1
    rows = torch.repeat_interleave(_arange(0, n), deg)
    rank = _arange(0, rows.numel()) - (torch.cumsum(deg, 0) - deg)[rows]
    at = rp[rows] + rank
    cols, vals = ci[at].long(), va[at]
    # level sets: rows whose last dependency has been placed
    order = torch.argsort(cols, stable=True)
    readers = rows[order]
    cp = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    cp[1:] = torch.cumsum(torch.bincount(cols, minlength=n), 0)
    left = deg.clone()
    now = torch.nonzero(deg == 0).flatten()
    sets = []
    while now.numel():
        sets.append(now)
        cnt = cp[now + 1] - cp[now]
        total = int(cnt.sum())
        if total == 0:
            break
        idx = torch.repeat_interleave(cp[now] - (torch.cumsum(cnt, 0) - cnt), cnt) + _arange(0, total)
        hit = readers[idx]
        left.index_add_(0, hit, torch.full_like(hit, -1))
        now = torch.unique(hit[left[hit] == 0])
    perm = torch.cat(sets)
    place = torch.empty_like(perm)
    place[perm] = _arange(0, n)
    most = max(1, int(deg.max()))
    pc = torch.zeros(most, n, dtype=torch.int64, device="cuda")
    pv = torch.zeros(most, n, dtype=torch.float64, device="cuda")
    pc[rank, place[rows]] = place[cols]
    pv[rank, place[rows]] = vals
    dg = va[rp[1:] - 1][perm]
    dp = deg[perm]
    x = torch.zeros(n, b.shape[1], dtype=torch.float64, device="cuda")
    ends = [0]
    for v in sets:
        ends.append(ends[-1] + v.numel())
    lev = torch.repeat_interleave(_arange(0, len(sets)), torch.tensor([v.numel() for v in sets], device="cuda"))
    deepest = torch.zeros(len(sets), dtype=torch.int64, device="cuda").scatter_reduce_(0, lev, dp, "amax").tolist()
    bp = b[perm]
    for i in range(len(sets)):
        s, e = ends[i], ends[i + 1]
        acc = bp[s:e]
        for d in range(deepest[i]):
            acc = acc - pv[d, s:e, None] * x[pc[d, s:e]]
        x[s:e] = acc / dg[s:e, None]
    return x[place]


def _reversed_transpose(n, rp, ci, va):
    """J L^T J (lower triangular, diagonal last); J reverses the rows."""
    rows = torch.repeat_interleave(_arange(0, n), (rp[1:] - rp[:-1]).long())
    r, c = n - 1 - ci.long(), n - 1 - rows
    order = torch.argsort(r * n + c)
    out = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    out[1:] = torch.cumsum(torch.bincount(r, minlength=n), 0)
    return out.int(), c[order].int(), va[order]


def _solve_form64(form, m, b):
    n, rp, ci, va = m
    if form == "L":
        return _solve64(n, rp, ci, va, b)
    return _solve64(n, *_reversed_transpose(n, rp, ci, va), b.flip(0)).flip(0)


def _policy64(params, feat, label, weight, norm):
    p = params.double()
    sizes, parts, o = [(64, 20), (64,), (64, 64), (64,), (64,), (1,)], [], 0
    for s in sizes:
        k = math.prod(s)
        parts.append(p[o:o + k].reshape(s).clone().requires_grad_(True))
        o += k
    w1, b1, w2, b2, w3, b3 = parts
    f = (feat.double() - norm[0].double()) * norm[1].double()
    h1 = torch.relu(f @ w1.t() + b1)
    h2 = torch.relu(h1 @ w2.t() + b2)
    z = (h2 * w3).sum(1) + b3
    loss = (weight.double() * (torch.clamp(z, min=0) - z * label.double() + torch.log1p(torch.exp(-z.abs())))).mean()
    grad = torch.autograd.grad(loss, parts)
    return dict(prob=torch.sigmoid(z).detach(), grad=torch.cat([v.reshape(-1) for v in grad]),
                loss=loss.detach().reshape(1))


def exact(case, seed):
    if case["what"] == "setup":
        return None
    g = _generator(seed)
    if case["what"] == "policy":
        return _policy64(*_network(g, case["batch"]))
    if case["what"] == "batch":
        ns, off, mat, (n, rp, ci, va), _ = _batch(case, g)
        c = case["nrhs"]
        b = _rhs(g, 1, n * c).reshape(-1)
        # matrix i's columns are n_i long and start at nrhs * its first row
        p = _arange(0, n)
        at = off[mat] * c + (p - off[mat])
        at = at[:, None] + ns[mat][:, None] * _arange(0, c)[None, :]
        out = torch.empty_like(b)
        out[at] = _solve64(n, rp, ci, va, b[at])
        return out
    m = _matrix(case, g)
    b = _rhs(g, case["nrhs"], m[0]).t()
    if case["what"] == "precond":
        x = _solve_form64("LT", m, _solve_form64("L", m, b))
    else:
        x = _solve_form64(case.get("form", "L"), m, b)
    return x.contiguous() if case.get("rows") else x.t().contiguous()
