"""The work a user of this framework has it do, as measurable cases.

Each case goes through the public entry points of ``paper_1902_09527_amd``
(``run``, ``KMeansMTI``, ``kmeanspp``, ``run_pp_best``) on float32 rows that
are already on the GPU, and counts the whole call: set-up, every iteration
and the outputs.  The inputs are Gaussian mixtures drawn on the GPU from the
seed, of the same recipes as ``synth`` (uniform or normal means, fixed or
varying spreads, equal / Dirichlet / Zipf weights, optionally anisotropic
components and uniform noise).

Kinds of case:
  run    one k-means run from given centroids (``stats``: with the inertia;
         ``spherical``: on the unit sphere), ended by ``iters`` or by ``tol``;
  steps  the same through a context, one iteration a call, the changed count
         read after each (a program with a stop rule or a log of its own);
  seed   k-means++ seeding with a workspace that the program keeps;
  best   k-means++ with ``r`` restarts, the run of the least inertia kept.
"""
import math

import numpy as np
import torch

import paper_1902_09527_amd as km

DEV = "cuda:0"
CHUNK = 1 << 22   # rows drawn at a time


def _case(name, kind, n, d, k, iters, tol=0.0, mix="iso", **more):
    c = {"kind": kind, "n": n, "d": d, "k": k, "iters": iters, "tol": tol, "mix": mix}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # The smallest call: a few thousand rows, where launches and host work count.
        _case("small-10k-d16-k8", "run", 10_000, 16, 8, 20),
        # Embedding rows of a power-of-two width, driven step by step by the
        # caller's own loop (changed count read each time).
        _case("steps-300k-d64-k50", "steps", 300_000, 64, 50, 20),
        # A table of measurements: odd row count and width, stopped by tol.
        _case("ragged-1M-d10-k25", "run", 999_983, 10, 25, 50, tol=0.001),
        # Spectral embedding of a large graph (the shape of the method's
        # 66M x 8 eigenvector data set), k = 10.
        _case("eigen-66M-d8-k10", "run", 66_000_000, 8, 10, 20, mix="aniso"),
        # Medium size, many clusters of uneven weight and spread.
        _case("blobs-1M-d32-k100", "run", 1_000_000, 32, 100, 30, mix="dirichlet"),
        # The benchmark's default workload: most rows stable, stopped by tol.
        _case("aniso-8M-d16-k10", "run", 8_000_000, 16, 10, 50, tol=0.001, mix="aniso"),
        # Wide rows and many clusters: the distances are a large contraction.
        _case("blobs-2M-d256-k1000", "run", 2_000_000, 256, 1000, 20, mix="normal"),
        # The largest row count that one run is used for here.
        _case("zipf-100M-d32-k64", "run", 100_000_000, 32, 64, 25, mix="zipf"),
        # A run whose objective is logged: the inertia of every step.
        _case("inertia-2M-d32-k64", "run", 2_000_000, 32, 64, 15, mix="dirichlet", stats=True),
        # Text or image embeddings clustered by the cosine.
        _case("sphere-400k-d128-k200", "run", 400_000, 128, 200, 15, mix="normal", spherical=True),
        # Seeding by itself, in the caller's workspace.
        _case("seed-4M-d32-k64", "seed", 4_000_000, 32, 64, 0, mix="dirichlet"),
        # The complete method on a modest table: four restarts, the best kept.
        _case("best4-200k-d16-k20", "best", 200_000, 16, 20, 25, r=4),
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["run"] * 7 + ["steps", "inertia", "sphere", "seed", "best"])
    common = rng.random() < 0.5   # half of the widths are the common ones, the rest anything
    d = rng.choice([8, 16, 32, 64, 128]) if common else _logu(rng, 2, 256)
    k = _logu(rng, 2, 1000 if kind in ("run", "sphere") else 128)
    n = _logu(rng, 2_000, 20_000_000)
    if kind == "best":
        n = min(n, 1_000_000)
    # at most 400 MB of rows, and well below the largest listed contraction
    n = min(n, 100_000_000 // d, 5_000_000_000 // (k * d))
    n = max(n, 40 * k)
    n += rng.randrange(1, 50)
    mix = rng.choice(["iso", "dirichlet", "zipf", "normal"] + (["aniso"] if d <= 32 and k <= 64 else []))
    if kind == "seed":
        return _case(None, "seed", n, d, k, 0, mix=mix)
    if kind == "best":
        return _case(None, "best", n, d, min(k, 64), rng.randrange(8, 20), mix=mix, r=rng.randrange(2, 5))
    tol = rng.choice([0.0, 0.001])
    iters = rng.randrange(8, 26) if tol == 0.0 else 40
    if kind == "inertia":
        return _case(None, "run", n, d, k, iters, tol=tol, mix=mix, stats=True)
    if kind == "sphere":
        return _case(None, "run", n, d, k, iters, tol=tol, mix="normal", spherical=True)
    return _case(None, kind, n, d, k, iters, tol=tol, mix=mix)


# --------------------------------------------------------------------------
# Inputs


def _mixture(case, g, d, k):
    """Means, spreads and cumulative weights of the case's k components."""
    mix = case["mix"]
    if mix == "normal":
        means = 2.0 * torch.randn(k, d, generator=g, device=DEV)
    else:
        scale = {"iso": 10.0, "aniso": 10.0, "dirichlet": 20.0, "zipf": 50.0}[mix]
        means = (torch.rand(k, d, generator=g, device=DEV) * 2 - 1) * scale
    lo, hi = {"iso": (1.0, 1.0), "normal": (1.0, 1.0), "dirichlet": (0.5, 2.0), "zipf": (1.0, 5.0),
              "aniso": (1.0, 1.0)}[mix]
    sig = lo + (hi - lo) * torch.rand(k, 1, generator=g, device=DEV)
    if mix == "dirichlet":
        w = -torch.log(torch.rand(k, generator=g, device=DEV).clamp_min(1e-6))
    elif mix == "zipf":
        w = torch.arange(1, k + 1, device=DEV, dtype=torch.float32) ** -1.1
    else:
        w = torch.ones(k, device=DEV)
    cum = torch.cumsum((w / w.sum()).double(), 0)
    return means, sig, cum


def _rows(case, g):
    n, d, k = case["n"], case["d"], case["k"]
    means, sig, cum = _mixture(case, g, d, k)
    factors = None
    if case["mix"] == "aniso":   # orthogonal directions with log-normal scales, 5 % uniform noise
        q = torch.linalg.qr(torch.randn(k, d, d, generator=g, device=DEV))[0]
        factors = (q * torch.exp(0.5 * torch.randn(k, 1, d, generator=g, device=DEV))).transpose(1, 2).contiguous()
        box = (means.abs().amax(0) + 3.0)[None, :]
    X = torch.empty(n, d, device=DEV)
    for i0 in range(0, n, CHUNK):
        m = min(CHUNK, n - i0)
        z = torch.searchsorted(cum, torch.rand(m, generator=g, device=DEV, dtype=torch.float64)).clamp_max_(k - 1)
        x = X[i0:i0 + m]
        x.normal_(generator=g)
        if factors is None:
            x.mul_(sig[z]).add_(means[z])
        else:
            y = torch.zeros_like(x)
            for j in range(k):   # k is small where the components are anisotropic
                y = torch.where((z == j)[:, None], x @ factors[j] + means[j], y)
            noise = torch.rand(m, 1, generator=g, device=DEV) < 0.05
            u = (torch.rand(m, d, generator=g, device=DEV) * 2 - 1) * box
            x.copy_(torch.where(noise, u, y))
    return X


def _start_rows(X, k, g):
    """k distinct rows of X."""
    n = X.shape[0]
    idx = torch.randint(0, n, (8 * k + 64,), generator=g, device=DEV).cpu().numpy()
    idx = idx[np.sort(np.unique(idx, return_index=True)[1])]   # first occurrences, in draw order
    if idx.size < k:
        idx = np.arange(k)
    return X[torch.from_numpy(idx[:k]).to(DEV)].contiguous()


def prepare(case, seed):
    g = torch.Generator(device=DEV).manual_seed(int(seed) * 1_000_003 + 17)
    c = dict(case)
    s = {"case": c, "X": _rows(c, g)}
    if c["kind"] in ("run", "steps"):
        s["C0"] = _start_rows(s["X"], c["k"], g)
    else:
        r = c.get("r", 1)
        s["U"] = torch.rand(r, c["k"], generator=g, device=DEV, dtype=torch.float64).cpu().numpy()
    if c["kind"] == "seed":
        need = km.kmeanspp_workspace_bytes(c["n"], c["d"], c["k"])
        s["ws"] = torch.empty(need + 256, dtype=torch.uint8, device=DEV)
    return s


# --------------------------------------------------------------------------
# One pass


def run(state):
    c = state["case"]
    X, kind = state["X"], c["kind"]
    if kind == "run":
        a, C, st = km.run(X, state["C0"], c["iters"], c["tol"], stats=c.get("stats", False),
                          spherical=c.get("spherical", False))
        out = {"assign": a, "C": C, "iterations": st["iterations"], "changed": st["changed_last"]}
        if c.get("stats"):
            out["inertia"] = st["inertia_last"]
        return out
    if kind == "steps":
        changed = []
        with km.KMeansMTI(X, state["C0"]) as ctx:
            while len(changed) < c["iters"]:
                changed.append(ctx.iterate(sync=True))
                if changed[-1] < c["tol"] * c["n"]:
                    break
            a, C = ctx.get()
        return {"assign": a, "C": C, "changed": np.array(changed, np.int64)}
    if kind == "seed":
        r = km.kmeanspp(X, c["k"], state["U"][0], workspace=state["ws"])
        return {"C": r["C"], "idx": r["idx"], "D2": r["D2"]}
    r = km.run_pp_best(X, c["k"], state["U"], c["iters"], c["tol"])
    return {"best": r["best"], "assign": r["assign"], "C": r["C"], "inertia": np.array(r["inertia"], np.float64)}


def work(case):
    """Rows in, assignment and centroids out.  The first step of a run has no
    bounds, so all its n k distances are due; a later step can leave out all
    but a test per row.  Seeding: the first seed's n distances and a test per
    row for each later seed."""
    n, d, k, T = case["n"], case["d"], case["k"], case["iters"]
    io = 4 * n * d + 8 * k * d
    if case["kind"] == "seed":
        return {"bytes": io + 8 * n, "flops": 3 * n * d + 2 * n * (k - 1)}
    r = case.get("r", 1)
    return {"bytes": io + 4 * n, "flops": r * (2 * n * k * d + 2 * n * (T - 1))}


def tolerance(case):
    # Float32 centroids of exact means are off by one rounding: against
    # exact() 2.5e-8 to 2.7e-8 in the 2-norm and at most 6e-8 in a value
    # (half a unit in the last place), the inertia by 2e-9.  Four times that.
    # No assignment and no count differed; one could where the two nearest
    # distances agree to about 1e-9.
    return {"rel": 1.1e-7, "max": 2.4e-7, "differ": 1e-6}


# --------------------------------------------------------------------------
# The same in 64 bits


def _nearest(X, C, prev=None):
    """Index of the nearest row of C (float64) for every row of X, and the
    squared distances; a previous index keeps an exact tie."""
    k = C.shape[0]
    c2 = (C * C).sum(1)
    a = torch.empty(X.shape[0], dtype=torch.int64, device=DEV)
    best = torch.empty(X.shape[0], dtype=torch.float64, device=DEV)
    step = max(1, min(X.shape[0], (1 << 27) // max(k, X.shape[1])))
    for i0 in range(0, X.shape[0], step):
        x = X[i0:i0 + step].double()
        e = c2[None, :] - 2.0 * (x @ C.t())
        v, j = e.min(1)
        if prev is not None:
            p = prev[i0:i0 + step]
            j = torch.where(e.gather(1, p[:, None])[:, 0] <= v, p, j)
        a[i0:i0 + step] = j
        best[i0:i0 + step] = v + (x * x).sum(1)
    return a, best


def _sums(X, a, k):
    """Per-cluster sums and counts: one-hot products over blocks of rows."""
    n, d = X.shape
    s = torch.zeros(k, d, dtype=torch.float64, device=DEV)
    ids = torch.arange(k, device=DEV)
    blk = 1024
    step = max(blk, (1 << 26) // max(k, d) // blk * blk)
    for i0 in range(0, n, step):
        x, b = X[i0:i0 + step].double(), a[i0:i0 + step]
        m = x.shape[0] // blk * blk
        if m:
            hot = (b[:m].view(-1, 1, blk) == ids[None, :, None]).double()
            s += torch.bmm(hot, x[:m].view(-1, blk, d)).sum(0)
        if m < x.shape[0]:
            s += (b[m:][None, :] == ids[:, None]).double() @ x[m:]
    return s, torch.bincount(a, minlength=k).double()


def _lloyd(X, C0, iters, tol, spherical=False):
    n, k = X.shape[0], C0.shape[0]
    C = C0.double()
    if spherical:
        X = torch.nn.functional.normalize(X.double(), dim=1, eps=1e-300).float()
        C = torch.nn.functional.normalize(C, dim=1, eps=1e-300)
    a, changed, inertia = None, [], 0.0
    for _ in range(iters):
        new, best = _nearest(X, C, a)
        changed.append(n if a is None else int((new != a).sum()))
        inertia = float(best.sum())
        a = new
        s, m = _sums(X, a, k)
        mean = s / m.clamp_min(1.0)[:, None]
        if spherical:
            norm = mean.norm(dim=1, keepdim=True)
            C = torch.where((m > 0)[:, None] & (norm > 0), mean / norm.clamp_min(1e-300), C)
        else:
            C = torch.where((m > 0)[:, None], mean, C)
        if changed[-1] < tol * n:
            break
    return a, C, changed, inertia


def _seed(X, k, u):
    n = X.shape[0]
    L = 0
    while (1 << L) < n:
        L += 1
    idx = [min(int(u[0] * n), n - 1)]
    D2 = None
    for t in range(k):
        if t:
            top = float(D2.max())
            S = 62 - math.frexp(top)[1] - L if top > 0 else 0
            w = torch.floor(D2 * 2.0 ** S).long()
            cum = torch.cumsum(w, 0)
            W = int(cum[-1])
            if W > 0:
                T = min(int(u[t] * float(W)), W - 1)
                idx.append(int(torch.searchsorted(cum, torch.tensor([T], device=DEV), right=True)))
            else:
                idx.append(min(int(u[t] * n), n - 1))
        c = X[idx[-1]].double()
        v = torch.empty(n, dtype=torch.float64, device=DEV)
        for i0 in range(0, n, CHUNK):
            v[i0:i0 + CHUNK] = (X[i0:i0 + CHUNK].double() - c).square().sum(1)
        D2 = v if D2 is None else torch.minimum(D2, v)
    idx = torch.tensor(idx, device=DEV)
    return X[idx], idx, D2


def exact(case, seed):
    s = prepare(case, seed)
    c, X = s["case"], s["X"]
    if c["kind"] in ("run", "steps"):
        a, C, changed, inertia = _lloyd(X, s["C0"], c["iters"], c["tol"], c.get("spherical", False))
        if c["kind"] == "steps":
            return {"assign": a, "C": C, "changed": np.array(changed, np.int64)}
        out = {"assign": a, "C": C, "iterations": len(changed), "changed": changed[-1]}
        if c.get("stats"):
            out["inertia"] = inertia
        return out
    if c["kind"] == "seed":
        C, idx, D2 = _seed(X, c["k"], s["U"][0])
        return {"C": C.double(), "idx": idx, "D2": D2}
    runs = [_lloyd(X, _seed(X, c["k"], u)[0], c["iters"], c["tol"]) for u in s["U"]]
    best = min(range(len(runs)), key=lambda q: runs[q][3])
    return {"best": best, "assign": runs[best][0], "C": runs[best][1],
            "inertia": np.array([q[3] for q in runs], np.float64)}
