"""The general incremental steps (any d; one lane per survivor on "lds-inc-vec",
matrix cores on "lds-inc") on the GPU.

KM_FLAG_FULL_SUMS takes the same problem through the general assignment kernel
(every row read and summed each step), which is pinned to the oracle: both
must give the same bits.  The sizes sit at the edges of the kernels' tiles:
16-dimension k-steps and their remainders, rows of 4-byte and of 16-byte
alignment, the 32-centroid blocks, 64-point sub-steps, the rule between the
two forms (k times d rounded up to 4, at most 256) and the largest k.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import check_assign, check_centroids

import paper_1902_09527_amd as km
from paper_1902_09527_amd import _native as N

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(DEV)


def _same(Xg, Cg, iters, **kw):
    a1, c1, s1 = km.run(Xg, Cg, iters, **kw)
    a2, c2, s2 = km.run(Xg, Cg, iters, full_sums=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a1, a2) and torch.equal(c1.view(torch.int32), c2.view(torch.int32))
    assert s1["iterations"] == s2["iterations"] and s1["changed_last"] == s2["changed_last"]
    return a1, c1, s1


CASES = [
    # n, d, k, path
    (1000, 1, 5, "lds-inc-vec"), (63, 3, 7, "lds-inc-vec"), (64 * 5 + 1, 4, 64, "lds-inc-vec"),
    (3000, 4, 65, "lds-inc"), (5000, 8, 32, "lds-inc-vec"), (5000, 8, 33, "lds-inc"),
    (2000, 12, 21, "lds-inc-vec"), (2001, 12, 22, "lds-inc"), (700, 10, 1, "lds-inc-vec"),
    (4097, 15, 32, "lds-inc"), (4096, 17, 33, "lds-inc"), (300000 + 7, 20, 64, "lds-inc"),
    (3001, 31, 65, "lds-inc"), (3000, 33, 100, "lds-inc"), (6000, 48, 128, "lds-inc"),
    (2500, 63, 30, "lds-inc"), (2500, 64, 31, "lds-inc"), (2500, 65, 40, "lds-inc"),
    (4000, 5, 129, "lds-inc"), (4001, 9, 256, "lds-inc"), (3000, 5, 257, "global-mfma"), (3000, 1, 257, "lds-vector"),
    (2000, 1, 257, "global-mfma"), (100001, 2, 260, "lds-vector"), (100001, 4, 260, "global-mfma"),
    (1500, 129, 33, "lds-inc"), (1201, 255, 20, "lds-inc"), (900, 600, 9, "lds-inc"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d-d%d-k%d" % c[:3])
@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "offset4"])
def test_general_step_matches_the_full_read_path(case, offset):
    n, d, k, path = case
    print("case", case, offset, flush=True)
    X, C0 = synth.blobs(n, d, k, seed=700 + n % 97 + d, spread=4.0, sigma=1.5, comps=max(1, k // 2))
    Cg = _gpu(C0)
    big = torch.zeros(n * d + offset, dtype=torch.float32, device=DEV)
    big[offset:] = _gpu(X).reshape(-1)
    Xg = big[offset:].view(n, d)     # rows at a 4-byte offset from 16-byte alignment with offset = 1
    with km.KMeansMTI(Xg, Cg) as ctx:
        assert ctx.path() == path
    a, c, st = _same(Xg, Cg, 12)
    if n < 10000:
        ref = oracle.lloyd(X, C0, 12)
        assert st["iterations"] == ref["iters"]
        check_assign(a.cpu().numpy(), ref["assign"], ref["best"], ref["second"])
        check_centroids(c.cpu().numpy(), ref["C"], X)


@pytest.mark.parametrize("d,k", [(7, 9), (24, 40), (70, 20)])
def test_general_step_out_of_range_rows_ties_and_spherical(d, k):
    X, C0 = synth.blobs(3000, d, k, seed=811 + d, spread=4.0, sigma=1.5)
    C0[1] = C0[0]                              # exact ties: the lower index wins every point
    X[500:700] = X[0]                          # duplicate rows
    Cg = _gpu(C0)
    _same(_gpu(X), Cg, 10)
    a, _, _ = km.run(_gpu(X), Cg, 1)
    assert not (a == 1).any()
    Xb = X.copy()
    Xb[1234] *= 1e6                            # far outside the sample's bound (f16 overflows: direct form)
    Xb[17] *= 1e-12
    _same(_gpu(Xb), Cg, 10)
    Cb = C0.copy()
    Cb[2] += 1e7                               # a centroid far outside the data keeps its place, empty
    _, c, _ = _same(_gpu(X), _gpu(Cb), 10)
    assert torch.equal(c[2], _gpu(Cb)[2])
    _same(_gpu(X), _gpu(np.abs(C0) + 0.1), 10, spherical=True)
    for scale in (1e-15, 1e15):                # the scaling of the f16 operands follows the data
        _same(_gpu(X * np.float32(scale)), _gpu(C0 * np.float32(scale)), 6)


@pytest.mark.parametrize("n,d,k", [(20000, 4, 9000), (6000, 40, 4097), (5000, 64, 200), (3000, 17, 300)])
def test_global_path_candidate_lists_match_oracle(n, d, k):
    # few components, so that many centroids share one: several candidates per
    # survivor and full lists; k past 4096 and 8192 centroids (list rounds)
    X, C0 = synth.blobs(n, d, k, seed=831 + d, spread=4.0, sigma=1.5, comps=12)
    for stats in (False, True):
        a, c, st = km.run(_gpu(X), _gpu(C0), 5, large_path=True, stats=stats)
        ref = oracle.lloyd(X, C0, 5)
        assert st["iterations"] == ref["iters"]
        check_assign(a.cpu().numpy(), ref["assign"], ref["best"], ref["second"])
        check_centroids(c.cpu().numpy(), ref["C"], X)


def test_general_step_with_infinite_and_nan_rows_ends():
    X, C0 = synth.blobs(2000, 20, 12, seed=821, spread=4.0, sigma=1.5)
    X[5, 3] = np.inf
    X[9, 0] = np.nan
    a, _, st = km.run(_gpu(X), _gpu(C0), 5)
    assert st["iterations"] == 5 and int(a.min()) >= 0 and int(a.max()) < 12


@pytest.mark.parametrize("n,d,k,kw", [(3001, 7, 9, {}), (3000, 24, 40, {}), (3000, 32, 40, {}), (5000, 64, 200, {}),
                                      (2000, 33, 300, {}), (3000, 24, 20, {"spherical": True}), (300, 20, 300, {})],
                         ids=lambda v: str(v))
def test_inertia_from_exact_sums(n, d, k, kw):
    # sum |x|^2 + sum_j (n_j |c_j|^2 - 2 c_j . S_j): a value's image is within
    # 2^(log2 n - 57) max |x| (the scale leaves log2 n bits to the sums and four to
    # values outside the sample): 2^-45 of max |x| at 3000 rows, and values above
    # 2^-20 of max |x| are exact.  Everything else is carried in double pairs, so
    # the inertia is within about 2^-43 of sum |x|^2 (1e-12 of it here; sum |x|^2
    # is below 100 times the inertia for k << n).
    X, C0 = synth.blobs(n, d, k, seed=841 + d, spread=4.0, sigma=1.5, comps=min(k, 30))
    if k == n:
        C0 = X.copy()
    Y = X.astype(np.float64)
    if kw:
        Y = (Y / np.linalg.norm(Y, axis=1, keepdims=True)).astype(np.float32).astype(np.float64)
    with km.KMeansMTI(_gpu(X), _gpu(C0), stats=True, **kw) as ctx:
        for _ in range(5):
            c = ctx.centroids64()
            ctx.iterate()
            a, _ = ctx.get(centroids=False)
            want = ((Y - c[a.cpu().numpy()]).astype(np.longdouble) ** 2).sum()
            assert abs(float(ctx.stats()["inertia_last"] - want)) <= 1e-12 * max(float(want), 1e-2 * (Y ** 2).sum())
        assert ctx.history()["inertia"][-1] == ctx.stats()["inertia_last"]
        if k == n:
            assert ctx.stats()["inertia_last"] == 0.0


def test_shapes_of_different_lds_need_alternate_on_one_kernel():
    # one kernel (two centroid blocks, aligned rows, d > 32) at 108, 54 and 108 KB
    # of LDS: its limit must not follow the last shape that set it
    runs = {}
    for d, k in ((100, 60), (36, 33), (100, 60), (36, 33)):
        X, C0 = synth.blobs(2000, d, k, seed=851 + d, spread=4.0, sigma=1.5)
        a, c, _ = _same(_gpu(X), _gpu(C0), 6)
        if (d, k) in runs:
            assert torch.equal(runs[(d, k)][0], a) and torch.equal(runs[(d, k)][1], c)
        runs[(d, k)] = (a, c)


@pytest.mark.parametrize("n,d,k,large", [(16000, 6, 138, False), (12000, 5, 60, False), (12000, 24, 60, False),
                                         (6000, 40, 90, False), (21000, 17, 294, False), (9000, 6, 50, True),
                                         (12000, 16, 12, False), (12000, 16, 40, False), (9000, 32, 100, True)],
                         ids=lambda v: str(v))
def test_tied_rows_fall_alike_on_every_path(n, d, k, large):
    # whole numbers projected to the unit sphere: many rows at equal distances
    # from two centroids, their float64 sums equal only when formed in one order
    rng = np.random.default_rng(861 + d)
    X = np.round(rng.normal(0.0, 1.2, (n, d))).astype(np.float32)
    X[np.abs(X).sum(1) == 0, 0] = 1.0
    Xg, Cg = _gpu(X), _gpu(X[rng.permutation(n)[:k]])
    a1, c1, s1 = km.run(Xg, Cg, 10, spherical=True, large_path=large)
    a2, c2, s2 = km.run(Xg, Cg, 10, spherical=True, generic=True)
    assert torch.equal(a1, a2) and torch.equal(c1.view(torch.int32), c2.view(torch.int32))
    assert s1["changed_last"] == s2["changed_last"]


@pytest.mark.parametrize("n,d,k,kw", [(3001, 7, 9, {}), (5000, 24, 40, {}), (4000, 5, 129, {"stats": True}),
                                      (3000, 5, 257, {}), (3000, 24, 40, {"generic": True})], ids=lambda v: str(v))
def test_captured_step_replays_as_every_step(n, d, k, kw):
    # the first call to iterate recorded into a graph: its replays are the
    # first, second, ... step, with eager work and synchronizations between
    X, C0 = synth.blobs(n, d, k, seed=871 + d, spread=4.0, sigma=1.5, comps=max(1, k // 2))
    Xg, Cg = _gpu(X), _gpu(C0)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), km.KMeansMTI(Xg, Cg, **kw) as ctx, km.KMeansMTI(Xg, Cg, **kw) as ref:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            ctx.iterate()
        for t in range(6):
            graph.replay()
            s.synchronize()
            ref.iterate(sync=True)
            a, c = ctx.get()
            b, e = ref.get()
            s.synchronize()
            assert torch.equal(a, b) and torch.equal(c.view(torch.int32), e.view(torch.int32)), t
        assert ctx.stats()["iterations"] == 6 and ctx.stats()["dist_computed"] == ref.stats()["dist_computed"]
        # recorded, and the next call made before any replay
        with km.KMeansMTI(Xg, Cg, **kw) as late:
            other = torch.cuda.CUDAGraph()
            with torch.cuda.graph(other, stream=s):
                late.iterate()
            for t in range(3):
                late.iterate(sync=True)
                other.replay()
            s.synchronize()
            a, c = late.get()
            b, e = ref.get()
            s.synchronize()
            assert torch.equal(a, b) and torch.equal(c.view(torch.int32), e.view(torch.int32))


@pytest.mark.parametrize("m", [2, 3, 5, 6, 7])
def test_global_path_keeps_every_candidate_of_a_survivor(m):
    # every centroid m times over: each survivor has m candidates (up to six go
    # on with it, seven are decided over all centroids); the lowest of equal
    # ones wins the first step
    n, d, k = 4000, 12, 300
    X, C0 = synth.blobs(n, d, k, seed=881 + m, spread=4.0, sigma=1.5)
    C0 = np.repeat(C0[:(k + m - 1) // m], m, axis=0)[:k]
    Xg, Cg = _gpu(X), _gpu(C0)
    a1, c1, s1 = km.run(Xg, Cg, 4, large_path=True)
    a2, c2, s2 = km.run(Xg, Cg, 4, generic=True)
    assert torch.equal(a1, a2) and torch.equal(c1.view(torch.int32), c2.view(torch.int32))
    assert s1["rechecks"] >= n
    a, _, _ = km.run(Xg, Cg, 1, large_path=True)
    assert int((a % m).max()) == 0


def test_open_contexts_of_the_global_path_step_in_turn():
    # the histogram's LDS is 4 k bytes (80 KB and 1 KB), the full decision's 8 d:
    # an open context must not lose its limit to one opened later
    shapes = ((20000, 4, 20000), (2000, 30, 300), (1500, 1152, 257))
    data = [synth.blobs(n, d, k, seed=891 + d, spread=4.0, sigma=1.5, comps=40) for n, d, k in shapes]
    want = [km.run(_gpu(X), _gpu(C0), 3, large_path=True) for X, C0 in data]
    ctxs = [km.KMeansMTI(_gpu(X), _gpu(C0), large_path=True) for X, C0 in data]
    for t in range(3):
        for ctx in ctxs:
            ctx.iterate(sync=True)
    for ctx, (a, c, _) in zip(ctxs, want):
        b, e = ctx.get()
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(c, e)
        ctx.close()


def test_global_path_refuses_wide_rows():
    X = torch.randn(300, 1153, device=DEV)
    with pytest.raises(N.KMError, match="d <= 1152"):
        km.KMeansMTI(X, X[:260].contiguous())


@pytest.mark.parametrize("d,k", [(24, 40), (70, 20), (5, 129)])
@pytest.mark.parametrize("scale", [1e-18, 1e-21, 1e-24, 1e-30])
def test_matrix_core_step_on_data_below_the_range_of_squares(d, k, scale):
    # |c|^2 is subnormal in float32 from about 1e-19 on and zero from 1e-23 on
    X, C0 = synth.blobs(3000, d, k, seed=901 + d, spread=4.0, sigma=1.5)
    X, C0 = X * np.float32(scale), C0 * np.float32(scale)
    with km.KMeansMTI(_gpu(X), _gpu(C0)) as ctx:
        assert ctx.path() == "lds-inc"
    a, c, st = km.run(_gpu(X), _gpu(C0), 8)
    ref = oracle.lloyd(X, C0, 8)
    assert st["iterations"] == ref["iters"]
    check_assign(a.cpu().numpy(), ref["assign"], ref["best"], ref["second"])
    check_centroids(c.cpu().numpy(), ref["C"], X)


@pytest.fixture
def leave_free():
    # fills the device up to the given number of free bytes
    held = []

    def fill(target):
        torch.cuda.empty_cache()
        km.kmeans.release_cache()
        while True:
            free = torch.cuda.mem_get_info()[0]
            if free - target < (32 << 20):
                return
            held.append(torch.empty(min(free - target, 16 << 30), dtype=torch.uint8, device=DEV))
    yield fill
    held.clear()
    torch.cuda.empty_cache()
    km.kmeans.release_cache()


def _path(X, C0, **kw):
    with km.KMeansMTI(X, C0, **kw) as ctx:
        ctx.iterate(sync=True)
        return ctx.path()


def test_route_of_many_centroids_follows_the_free_memory(leave_free):
    # 252 bytes a row on the global path, 8 on the general kernel
    g = torch.Generator(device=DEV)
    g.manual_seed(911)
    X = torch.randn(5_200_000, 2, generator=g, device=DEV)
    C0 = X[:400].contiguous()
    small = X[:3_500_000]
    want = km.run(small, C0, 2)
    torch.cuda.synchronize()
    leave_free(1536 << 20)
    assert _path(small, C0) == "lds-vector"        # needs 0.82 GiB, 1.5 free: not twice that
    got = km.run(small, C0, 2)
    torch.cuda.synchronize()
    assert torch.equal(want[0], got[0]) and torch.equal(want[1], got[1])


def test_kept_buffers_count_as_free_memory(leave_free):
    g = torch.Generator(device=DEV)
    g.manual_seed(912)
    X = torch.randn(9_000_000, 2, generator=g, device=DEV)
    C0 = X[:400].contiguous()
    leave_free(3072 << 20)
    first = _path(X[:5_200_000], C0)               # 1.22 GiB; its buffers are kept
    assert first == "global-mfma" and _path(X[:5_200_000], C0) == first
    assert _path(X, C0, large_path=True) == "global-mfma"   # 2.1 GiB: only where those are given back


@pytest.mark.parametrize("d", [1, 3, 16])
@pytest.mark.parametrize("k,distinct", [(65, 5), (128, 60), (200, 20), (256, 8), (300, 30), (700, 60)])
def test_many_candidates_of_duplicate_rows(d, k, distinct):
    # few distinct rows, so that centroids repeat: more candidates than a
    # survivor keeps, for many survivors of a batch or few (k <= 256); on the
    # global path 5001 survivors are more than 8 k at k = 300 and fewer at 700
    rng = np.random.default_rng(921 + d + k)
    rows = rng.normal(0.0, 3.0, (distinct, d)).astype(np.float32)
    X = rows[rng.integers(0, distinct, 5001)]
    X[::97] += np.float32(0.25)
    C0 = X[rng.permutation(5001)[:k]]
    _same(_gpu(X), _gpu(C0), 6)
    if k > 256:
        for scale in (1e-24, 1.0, 1e24):     # float32 squares vanish, hold, overflow
            a, c, _ = km.run(_gpu(X * np.float32(scale)), _gpu(C0 * np.float32(scale)), 6, large_path=True)
            ref = oracle.lloyd(X * np.float32(scale), C0 * np.float32(scale), 6)
            check_assign(a.cpu().numpy(), ref["assign"], ref["best"], ref["second"])
            check_centroids(c.cpu().numpy(), ref["C"], X * np.float32(scale))


@pytest.mark.parametrize("n,d,k", [(3000, 3, 100), (4001, 17, 33), (3000, 40, 70), (2500, 65, 200), (3000, 6, 300),
                                   (2000, 150, 260)])
def test_data_far_from_the_origin(n, d, k):
    # the split products are formed relative to the centroids' mean there
    X, C0 = synth.blobs(n, d, k, seed=931 + d, spread=4.0, sigma=1.5, comps=max(1, k // 3))
    rng = np.random.default_rng(931 + d)
    far = rng.normal(0.0, 400.0, d).astype(np.float32)
    X, C0 = X + far, C0 + far
    X[7] = 0.0                                # far from every centroid
    a, c, st = km.run(_gpu(X), _gpu(C0), 8)
    b, e, s2 = km.run(_gpu(X), _gpu(C0), 8, generic=True) if d * k < 5000 else (a, c, st)
    assert torch.equal(a, b) and torch.equal(c.view(torch.int32), e.view(torch.int32))
    ref = oracle.lloyd(X, C0, 8)
    assert st["iterations"] == ref["iters"]
    check_assign(a.cpu().numpy(), ref["assign"], ref["best"], ref["second"])
    check_centroids(c.cpu().numpy(), ref["C"], X)
    # float64 decisions are near ties alone, not every survivor
    assert st["rechecks"] < 0.05 * n * st["iterations"]


@pytest.mark.parametrize("n,d,k", [(1_300_001, 3, 7), (4_700_003, 5, 7), (700_001, 12, 21), (2_300_017, 8, 10),
                                   (600_007, 40, 20), (1_200_001, 40, 60), (1_200_001, 40, 100), (700_001, 40, 200),
                                   (1_200_003, 24, 20), (900_001, 9, 200)], ids=lambda v: str(v))
def test_waves_of_many_tiles_match_the_full_read_path(n, d, k):
    # sizes at which a wave takes two or four sub-steps a tile and several tiles
    # from the block's counter, its queue carried from one to the next; the last
    # tile is short
    g = torch.Generator(device=DEV)
    g.manual_seed(941 + d + k)
    m = torch.randn(k, d, generator=g, device=DEV) * 3
    X = (m[torch.randint(k, (n,), generator=g, device=DEV)] + torch.randn(n, d, generator=g, device=DEV)).contiguous()
    C0 = X[torch.randperm(n, generator=g, device=DEV)[:k]].contiguous()
    with km.KMeansMTI(X, C0) as ctx:
        assert ctx.path() in ("lds-inc-vec", "lds-inc")
    _, _, st = _same(X, C0, 5)
    assert st["clause1_skips"] > 0


def test_two_columns_on_the_sphere_are_a_line():
    X, C0 = synth.blobs(4000, 2, 300, seed=951, spread=4.0, sigma=1.5)
    Xg, Cg = _gpu(X), _gpu(C0 + np.float32(0.01))
    for kw, path in (({"spherical": True}, "lds-vector"), ({}, "global-mfma")):
        with km.KMeansMTI(Xg, Cg, **kw) as ctx:
            assert ctx.path() == path
        _same(Xg, Cg, 6, **kw)
