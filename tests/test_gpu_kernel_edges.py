"""Kernels at the edges of their ranges: first and last tile, remainders, and
both sides of every size rule, against numpy / scipy in FP64."""
import math

import numpy as np
import pytest
import scipy.linalg

from tests.gpu_util import requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.fixture(scope="module")
def handle():
    import paper_2105_00578_amd as sx
    return sx.Handle(0)


@pytest.mark.parametrize("w,m", [(1, 1), (2, 1), (2, 2), (7, 7), (8, 3), (22, 7), (23, 7),
                                 (31, 9), (32, 9), (33, 11), (47, 16)])
def test_rayleigh_ritz_orders(handle, w, m):
    """Odd and even orders, one / two / five blocks per thread.  The pencil's
    condition is that of Z^T Z for a 300 x w normal Z (below 10), so a
    backward-stable solve has errors of some w * 2^-53 ||GA||, w^2 with the
    norms' bounds: 1e-12 ||GA|| leaves a factor above 4."""
    from paper_2105_00578_amd import _lib
    rng = np.random.default_rng(100 + w)
    Z = rng.standard_normal((300, w))
    GB = Z.T @ Z
    A = rng.standard_normal((w, w))
    GA = A + A.T
    Y, th, kept, bd = _lib.rayleigh_ritz(handle, m, GA, GB)
    assert bd == 0 and kept == w
    ref = scipy.linalg.eigh(GA, GB, eigvals_only=True)[:m]
    scale = np.linalg.norm(GA) / 300
    assert np.allclose(th, ref, rtol=0, atol=1e-12 * scale)
    assert np.allclose(Y.T @ GB @ Y, np.eye(m), atol=1e-12)
    assert np.allclose(GA @ Y, GB @ Y @ np.diag(th), atol=1e-12 * np.linalg.norm(GA))


@pytest.mark.parametrize("n,nev,gen", [(63, 1, 0), (64, 2, 1), (65, 3, 0), (128, 5, 1),
                                       (129, 8, 0), (140, 9, 1), (90, 16, 1)])
def test_adjoint_cg_edges(handle, n, nev, gen):
    """Row counts around the CG's 64-row tiles, odd and even widths, one and
    two pairs of columns per thread, against the dense gradient.  Both solves
    stop at 1e-13 of the right-hand side and the gap terms of these spectra
    are above 1e-4: 1e-8 of the largest entry."""
    import torch
    import paper_2105_00578_amd as sx
    from oracle import adjoint
    from tests.gpu_util import dev, random_graph, upload
    g = random_graph(n, 6.0 / n, n + nev, np.float64)
    rp, col, w = upload(g)
    G = sx.Graph(handle, rp, col, w)
    rng = np.random.default_rng(nev)
    a = rng.standard_normal(nev)
    C = rng.standard_normal((g.n, nev))
    problem = sx.GENERALIZED if gen else sx.COMBINATORIAL
    gd, lam, V = adjoint.grad_dense(g.rowptr, g.col, g.w, problem, nev, a, C)
    args = (handle, G, problem, lam, torch.from_numpy(V).to(dev()), a,
            torch.from_numpy(C).to(dev()))
    grad = sx.eig_backward(*args, cg_tol=1e-13, cg_max_iter=5000).cpu().numpy()
    assert np.abs(grad - gd).max() <= 1e-8 * np.abs(gd).max()
    its, res = sx.backward_info(handle)
    assert 0 < its <= 5000 and res <= 1e-13
    # a limit inside a batch of steps is kept, and reported
    if its > 3:
        sx.eig_backward(*args, cg_tol=1e-13, cg_max_iter=3, allow_not_converged=True)
        its3, res3 = sx.backward_info(handle)
        assert its3 == 3 and res3 > 1e-13


def _graph_of(kind):
    import graphgen
    from tests.gpu_util import star_graph
    if kind == "grid":            # one lane per row, int16 offsets
        n, (u, v) = graphgen.grid3d_7pt(9, 8, 7)
        return graphgen.csr_from_edges(n, u, v, None)
    if kind == "brick":           # staged rows, weights
        n, (u, v) = graphgen.brick27(8, 7, 6)
        return graphgen.csr_from_edges(n, u, v, graphgen.uniform_weights(u.size, 4,
                                                                         dtype=np.float64))
    if kind == "rmat":            # every degree class
        return graphgen.rmat_graph(11, seed=2, weight_seed=3, weight_dtype=np.float64)
    if kind.startswith("ring"):   # n vertices, d neighbours each: staged chunks of 64 rows
        n, d = map(int, kind[4:].split("x"))
        u = np.repeat(np.arange(n), d // 2)
        v = (u + np.tile(np.arange(1, d // 2 + 1), n)) % n
        return graphgen.csr_from_edges(n, u, v, graphgen.uniform_weights(u.size, 4))
    return star_graph(17000)      # a hub row in chunks


@pytest.mark.parametrize("m", range(1, 17))
@pytest.mark.parametrize("kind", ["grid", "brick", "rmat", "hub", "ring127x26", "ring64x32",
                                  "ring129x34", "ring97x48"])
def test_products_every_width(handle, kind, m):
    """Every block width on every row class, from a base that is only aligned
    to its elements: L X, five Chebyshev steps (also in place) and the GMRES
    polynomial against FP64 numpy.  Errors of a product are at most some
    deg u ||x|| (deg 17000 for the hub); a polynomial of 5 steps multiplies
    them by less than 100 on these spectra."""
    import torch
    import paper_2105_00578_amd as sx
    from oracle import laplacian as lap, precond
    from tests.gpu_util import dev, upload
    g = _graph_of(kind)
    rp, col, w = upload(g)
    G = sx.Graph(handle, rp, col, w)
    rng = np.random.default_rng(m)
    X64 = rng.standard_normal((g.n, m))
    roots = [1.9, 0.1, 1.0, 0.4]
    for npd, td, tol in ((np.float32, torch.float32, 3e-6), (np.float64, torch.float64, 1e-14)):
        Xh = X64.astype(npd)
        buf = torch.zeros(g.n * m + 1, dtype=td, device=dev())
        X = buf[1:].view(g.n, m)
        X.copy_(torch.from_numpy(Xh))
        ref = Xh.astype(np.float64)
        LX = lap.apply(g.rowptr, g.col, g.w, ref)
        Y = sx.laplacian_apply(handle, G, X).cpu().numpy()
        assert np.abs(Y - LX).max() <= tol * np.abs(LX).max()
        d = lap.degrees(g.rowptr, g.col, g.w)
        for problem in (sx.COMBINATORIAL, sx.GENERALIZED):
            gen = problem == sx.GENERALIZED
            hi = 2.0 if gen else 2.0 * d.max()
            H0 = precond.chebyshev(g.rowptr, g.col, g.w, ref, 5, hi / 20, hi,
                                   dinv=1.0 / d if gen else None, problem=problem)
            o = sx.Options(problem=problem, precond=sx.PRECOND_CHEBYSHEV, cheb_degree=5,
                           cheb_ratio=20.0)
            H = sx.precond_apply(handle, G, o, X).cpu().numpy()
            assert np.abs(H - H0).max() <= 100 * tol * np.abs(H0).max()
            Xc = X.clone()
            sx.precond_apply(handle, G, o, Xc, out=Xc)     # in place
            assert np.array_equal(Xc.cpu().numpy(), H)
        P0 = precond.gmres_poly_apply(g.rowptr, g.col, g.w, sx.GENERALIZED, ref, roots)
        P = sx.poly_apply(handle, G, sx.GENERALIZED, roots, X).cpu().numpy()
        assert np.abs(P - P0).max() <= 100 * tol * np.abs(P0).max()


def _split_case(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal((n, 3))
    if kind == "ties":                # a few values: the order is by id
        return rng.integers(0, 3, (n, 3)).astype(np.float64)
    if kind == "constant":
        return np.zeros((n, 3))
    if kind == "sorted":              # sections are ranges of one coordinate
        return np.sort(rng.standard_normal((n, 1)), axis=0)
    x = rng.standard_normal((n, 3)) * 10.0 ** rng.integers(-30, 30, (n, 3))   # localised
    x[rng.random((n, 3)) < 0.3] = 0.0
    x[rng.random((n, 3)) < 0.1] = -0.0
    x[0, 0], x[1, 0] = np.inf, -np.inf
    return x


@pytest.mark.parametrize("kind", ["normal", "ties", "constant", "sorted", "wide"])
@pytest.mark.parametrize("n,K", [(2, 2), (5, 4), (2047, 64), (2049, 24), (70000, 48), (70000, 61),
                                 (70000, 64 * 63), (40000, 256)])
def test_split_bins_vs_oracle(handle, kind, n, K):
    """Sizes around the sample's, section and cut counts on both sides of the
    sample bins' limits (61 and 4032 = 7 3 3 2^6 cuts at once or by levels),
    ties, one value, localised values and infinities, with and without vertex
    weights, both types: the oracle's parts, exactly."""
    import graphgen
    import torch
    import paper_2105_00578_amd as sx
    from oracle import split as osplit
    from tests.gpu_util import dev
    rng = np.random.default_rng(n + K)
    x = _split_case(kind, n, rng)
    g = graphgen.csr_from_edges(n, np.arange(n - 1), np.arange(1, n))
    for weighted in (False, True):
        vw = rng.integers(1, 50, n).astype(np.int32) if weighted else None
        G = sx.Graph(handle, torch.from_numpy(g.rowptr.astype(np.int32)),
                     torch.from_numpy(g.col.astype(np.int32)), None,
                     None if vw is None else torch.from_numpy(vw))
        for dt in (np.float32, np.float64):
            xc = x.astype(dt)
            ref = osplit.split_mj(xc, K, vwgt=vw)
            got = sx.split(handle, G, torch.from_numpy(xc).to(dev()), K).cpu().numpy()
            assert np.array_equal(got, ref), (weighted, dt)


@pytest.mark.parametrize("kind", ["rows", "empty_runs", "one_row", "hub_edges"])
@pytest.mark.parametrize("wd", [None, np.float32, np.float64])
def test_cut_chunks_vs_numpy(handle, kind, wd):
    """Chunks of 4096 entries whose rows number few, none (a row over several
    chunks) or more than the 4096 staged ones (runs of empty rows, also at a
    chunk's first and last entry): the exact cut and part weights."""
    import graphgen
    import torch
    import paper_2105_00578_amd as sx
    rng = np.random.default_rng(5)
    if kind == "rows":
        n, (u, v) = graphgen.brick27(17, 13, 11)
    elif kind == "empty_runs":        # 3 x 9000 isolated vertices between three rings
        u, v, n = [], [], 0
        for size in (4096, 2048, 700):
            a = n + np.arange(size)
            u.append(a)
            v.append(np.roll(a, -1))
            n += size + 9000
        u, v = np.concatenate(u), np.concatenate(v)
    elif kind == "one_row":
        n = 13000
        u, v = np.zeros(n - 1, dtype=np.int64), np.arange(1, n)
    else:                             # hubs of 4096 entries: rows end with chunks
        n = 4 * 4097
        u = np.repeat(np.arange(4) * 4097, 4096)
        v = u + 1 + np.tile(np.arange(4096), 4)
    w = None if wd is None else graphgen.uniform_weights(u.size, 3, dtype=wd)
    g = graphgen.csr_from_edges(n, u, v, w)
    for rpt in (np.int32, np.int64):
        G = sx.Graph(handle, torch.from_numpy(g.rowptr.astype(rpt)),
                     torch.from_numpy(g.col.astype(np.int32)),
                     None if w is None else torch.from_numpy(g.w), validate=True)
        for K in (2, 9000):
            part = rng.integers(0, K, n).astype(np.int32)
            cross = part[u] != part[v]
            want = math.fsum(w[cross].astype(np.float64)) if w is not None else float(cross.sum())
            cut, cut2, imb, pw = sx.quality(handle, G, torch.from_numpy(part).cuda(), K)
            cnt = np.bincount(part, minlength=K)
            assert cut == want and cut2 == 2 * want and pw == cnt.tolist()
            assert imb == cnt.max() * K / n


@pytest.mark.parametrize("log_range", [0, 24, 25, 26, 39])
@pytest.mark.parametrize("deg", [4, 32, 34])
def test_refine_sum_widths(handle, log_range, deg):
    """Rows at the four-lane kernels' degree limit and past it, and FP32
    weight ranges on both sides of what 64-bit sums hold: the oracle's parts,
    exactly."""
    import graphgen
    import torch
    import paper_2105_00578_amd as sx
    from oracle import refine
    from tests.gpu_util import dev, upload
    n, half = 700, deg // 2
    u = np.repeat(np.arange(n), half)          # a circulant graph of degree `deg`
    v = (u + 1 + np.tile(np.arange(half), n)) % n
    rng = np.random.default_rng(deg + log_range)
    w = ((1.0 + rng.random(u.size)) * 2.0 ** rng.integers(0, log_range + 1, u.size) * 0.7)
    w = w.astype(np.float32)
    w[0], w[1] = 0.7, np.float32(0.7) * np.float32(2.0) ** log_range
    g = graphgen.csr_from_edges(n, u, v, w)
    rp, col, wd = upload(g)
    G = sx.Graph(handle, rp, col, wd)
    K = 6
    part0 = ((np.arange(n) * K // n + (rng.random(n) < 0.3)) % K).astype(np.int32)
    pd = torch.from_numpy(part0.copy()).to(dev())
    cut, imb, kept, moves = sx.refine(handle, G, pd, K, eps=0.2)
    ref, kept_ref, moves_ref = refine.refine(g.rowptr, g.col, g.w, part0, K, eps=0.2)
    assert np.array_equal(pd.cpu().numpy(), ref) and (kept, moves) == (kept_ref, moves_ref)
    assert moves > 0


@pytest.mark.parametrize("leaves", [1024, 1025, 1536, 64 * 512, 64 * 512 + 1, 130 * 512 + 7])
@pytest.mark.parametrize("f32", [False, True])
def test_single_column_hub_rows_vs_numpy(handle, leaves, f32):
    """The last row of a wavefront, the first hub, and hubs of 64 chunks of 512
    entries (one per lane that combines them), 65 and 131.  A lane adds at most
    4 entries twice over, 64 lanes 6 times, at most 3 chunks and 6 times again,
    and each difference is rounded: below 24 roundings of the sum of |terms|."""
    import torch
    import paper_2105_00578_amd as sx
    from tests.gpu_util import star_graph, upload
    g = star_graph(leaves)
    G = sx.Graph(handle, *upload(g))
    dt, eps = (np.float32, 2.0 ** -24) if f32 else (np.float64, 2.0 ** -53)
    x = np.random.default_rng(leaves).standard_normal(g.n).astype(dt)
    y = sx.laplacian_apply(handle, G, torch.from_numpy(x).cuda()).cpu().numpy()
    row = np.repeat(np.arange(g.n), np.diff(g.rowptr))
    t = x.astype(np.float64)[row] - x.astype(np.float64)[g.col]
    bound = 24 * eps * np.bincount(row, np.abs(t), g.n)
    want = np.array([math.fsum(t[a:b]) for a, b in zip(g.rowptr[:-1], g.rowptr[1:])])
    assert np.all(np.abs(y.astype(np.float64) - want) <= bound)


@pytest.mark.parametrize("wd", [None, np.float64])
def test_cut_from_chunk_to_chunk_vs_numpy(handle, wd):
    """More than 2 x 2048 chunks of 1024 entries, so that every block goes over
    several: a row of five whole chunks that ends with one, 3000 empty rows
    behind it, rows of one entry (1024 to a chunk, 1280 staged) with none, one
    in 5 and one in 3 empty between them, runs of 40,000 empty rows between
    chunks and inside them, and rows of 2 and 3 entries.  Weights are multiples
    of 1/8, so numpy's sums are exact."""
    import graphgen
    import torch
    import paper_2105_00578_amd as sx
    rng = np.random.default_rng(11)
    u, v, n = [], [], 0

    def pairs(ids):
        u.append(ids[0::2])
        v.append(ids[1::2])

    hub = 5 * 1024                    # vertex 0 and its leaves, 3000 rows further on
    u.append(np.zeros(hub, dtype=np.int64))
    v.append(3001 + np.arange(hub))
    n = 3001 + hub
    for every in (0, 5, 3):           # rows of one entry, each `every`-th row empty
        ids = n + np.arange(1_200_000)
        n += ids.size
        if every:
            ids = ids[np.arange(ids.size) % every != 0]
        pairs(ids[:ids.size // 2 * 2])
    for size in (1024, 1500, 1024, 2048, 3000):
        n += 40_000                   # a run of empty rows
        pairs(n + np.arange(size))
        n += size
    path = n + np.arange(900_000)     # rows of 2 entries, and of 3 where chords end
    u += [path[:-1], path[:-7:11]]
    v += [path[1:], path[:-7:11] + 5]
    n += path.size + 2000             # empty rows at the end
    u, v = np.concatenate(u), np.concatenate(v)
    w = None if wd is None else (rng.integers(1, 64, u.size) / 8).astype(wd)
    g = graphgen.csr_from_edges(n, u, v, w)
    assert g.col.size > 2 * 2048 * 1024
    for rpt in (np.int32, np.int64):
        G = sx.Graph(handle, torch.from_numpy(g.rowptr.astype(rpt)),
                     torch.from_numpy(g.col.astype(np.int32)),
                     None if w is None else torch.from_numpy(g.w), validate=True)
        part = rng.integers(0, 7, n).astype(np.int32)
        cross = part[u] != part[v]
        want = float(cross.sum()) if w is None else float(w[cross].sum())
        cut, _, _, pw = sx.quality(handle, G, torch.from_numpy(part).cuda(), 7)
        assert cut == want and pw == np.bincount(part, minlength=7).tolist()


@pytest.mark.parametrize("nev", range(1, 17))
@pytest.mark.parametrize("kind", ["short", "long"])
def test_solver_widths_vs_dense(handle, kind, nev):
    """Blocks of every width, with exactly their columns (rows of at most 4
    neighbours) and padded (20 to 30 neighbours), 257 rows, so that the update
    has a block of one row.  Each value lies within its residual of an
    eigenvalue (Weinstein), and the solver stops at
    ||r|| <= tol max(theta, theta_1): that bound against the dense values, plus
    the rounding of an FP32 product (2^-20 of ||L||) in mixed precision.  (One
    vector: the value is 0, and no residual is small beside that.)"""
    import graphgen
    import paper_2105_00578_amd as sx
    from tests.gpu_util import upload
    n, rng = 257, np.random.default_rng(nev)
    i = np.arange(n)
    if kind == "short":
        u, v = np.concatenate([i[:-1], i[:-16]]), np.concatenate([i[1:], i[16:]])
    else:
        u = np.repeat(i, 12)
        v = (u + 1 + np.tile(np.arange(12) ** 2, n)) % n
    w = 0.5 + rng.random(u.size)
    g = graphgen.csr_from_edges(n, u, v, w)
    L = np.zeros((n, n))
    np.add.at(L, (np.repeat(i, np.diff(g.rowptr)), g.col), -g.w)
    L[i, i] = -L.sum(axis=1)
    ref = np.linalg.eigvalsh(L)
    G = sx.Graph(handle, *upload(g))
    for prec, tol in ((sx.FP64, 1e-7), (sx.MIXED, 1e-4)):
        opts = sx.options_default(True, sx.PRECOND_JACOBI, precision=prec, tol=tol, max_iter=3000)
        lam, V, st = sx.eigensolve(handle, G, nev, opts, allow_not_converged=nev == 1)
        scale = np.maximum(ref[:nev], ref[min(1, nev - 1)])
        slack = 1e-12 if prec == sx.FP64 else 2.0 ** -20 * ref[-1]
        assert np.all(np.abs(np.array(lam) - ref[:nev]) <= 1.01 * tol * np.abs(scale) + slack)
        x = V.double().cpu().numpy()
        assert np.allclose(x.T @ x, np.eye(nev), atol=1e-9 if prec == sx.FP64 else 1e-4)
