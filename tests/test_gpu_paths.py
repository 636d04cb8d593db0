"""Kernel variants at the edges of their tiles and dispatch rules, against the oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import spai_oracle as O
from paper_2511_09753_amd import workloads as W
from tests.helpers import (TOL_F64, history_array, history_from_oracle, oracle_rule, parse_state,
                           pattern_diff, rel_err, require_gpu, value_err)

pytestmark = pytest.mark.gpu


def _spai():
    require_gpu()
    from paper_2511_09753_amd import spai as S
    S.load()
    return S


def _random_symmetric(n, per_row, seed):
    rng = np.random.default_rng(seed)
    m = n * per_row // 2
    r, c, v = rng.integers(0, n, m), rng.integers(0, n, m), rng.standard_normal(m)
    U = sp.triu(sp.coo_matrix((v, (r, c)), shape=(n, n)).tocsr(), 1)
    A = (U + U.T + sp.diags(rng.standard_normal(n))).tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("n,steps,per_row", [
    (1, 1, 0), (2, 2, 2), (255, 63, 6), (256, 64, 6), (257, 65, 40), (300, 130, 6),
    (1025, 68, 9)])
def test_lanczos_passes_at_tile_edges(n, steps, per_row):
    """Rows around a 256-row tile, basis vectors around the 64 a workgroup takes at once,
    rows of up to about 40 entries (four lanes share one).  Both sides run the same
    process in float64 and differ by the order of their sums: 1e-9 of the spectral scale."""
    S = _spai()
    A = _random_symmetric(n, per_row, n)
    v0 = np.random.default_rng(steps).standard_normal(n)
    g = S.spectrum(A, v0, steps=steps)
    o = O.lanczos(A, steps, v0)
    scale = max(abs(o[0]), abs(o[1]))
    assert g[4] == o[4]
    assert abs(g[0] - o[0]) <= 1e-9 * scale and abs(g[1] - o[1]) <= 1e-9 * scale
    assert abs(g[2] - o[2]) <= 1e-7 * scale and abs(g[3] - o[3]) <= 1e-7 * scale


def test_lanczos_stops_in_an_invariant_subspace():
    """Three distinct eigenvalues: the process ends after three steps, although the host
    looks only every 64."""
    S = _spai()
    A = sp.diags(np.repeat([1.0, 2.0, 5.0], 200)).tocsr()
    lo, hi, _, _, k = S.spectrum(A, np.random.default_rng(0).standard_normal(600), steps=200)
    assert k == 3
    assert lo == pytest.approx(1.0, rel=1e-12) and hi == pytest.approx(5.0, rel=1e-12)


def _pattern_with(n, long_row, per_row, seed):
    """Symmetric pattern with about per_row entries a row and one row (and column) of
    long_row entries, diagonal included."""
    rng = np.random.default_rng(seed)
    m = max(n * (per_row - 1) // 2, 1)
    r, c = rng.integers(0, n, m), np.empty(m, dtype=np.int64)
    c = (r + rng.integers(1, min(40, max(n - 1, 2)), m)) % n
    k = rng.choice(n - 1, long_row - 1, replace=False) + 1 if long_row > 1 else np.empty(0, int)
    U = sp.coo_matrix((np.ones(m + len(k)), (np.r_[r, np.zeros(len(k), int)], np.r_[c, k])),
                      shape=(n, n)).tocsr()
    P = (U + U.T + sp.identity(n)).tocsr()
    P.sort_indices()
    return P


@pytest.mark.parametrize("n,rows_a,long_a,rows_m,long_m", [
    (1, 1, 1, 1, 1),
    (70, 3, 1, 5, 16),        # 16 lanes a row of M
    (70, 3, 1, 5, 17),        # 32
    (90, 3, 1, 5, 33),        # 64: eight rows of A's row at most
    (90, 3, 30, 2, 1),        # a long row of A: many rounds
    (200, 3, 1, 3, 64),       # the longest row that the lean kernel takes
    (200, 3, 1, 3, 65),       # and the first that it leaves
    (300, 5, 1, 12, 1),
    (400, 2, 60, 2, 1),       # more than eight rounds: left
    (600, 2, 1, 2, 240),      # a column of M near the tile's 256
])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_loss_rows_at_the_edges_of_their_tiles(n, rows_a, long_a, rows_m, long_m, precision):
    """Value and both gradients (unsymmetric values) on patterns around the lane-group
    widths, rounds and row lengths of the lean kernel and the rows that it leaves to the
    larger tile.  float64: sums of at most a few hundred products in another order, 1e-12
    of the largest entry; float32 values: 1e-5."""
    S = _spai()
    rng = np.random.default_rng(n + long_m)
    A = _pattern_with(n, long_a, rows_a, 1)
    M = _pattern_with(n, long_m, rows_m, 2)
    A.data = rng.standard_normal(A.nnz)
    M.data = 0.3 * rng.standard_normal(M.nnz)
    tol = 1e-12 if precision == "f64" else 1e-5
    o = S.Options(precision=precision)
    assert S.loss_fwd(A, M, o) == pytest.approx(O.loss(A, M), rel=tol)
    gA, gM = S.loss_bwd(A, M, dL=0.5, options=o)
    oA, oM = O.loss_grad(A, M)
    oA, oM = (0.5 * sp.csr_matrix(x)[tuple(p.nonzero())] for x, p in ((oA, A), (oM, M)))
    oA, oM = np.asarray(oA).ravel(), np.asarray(oM).ravel()
    assert np.max(np.abs(gA - oA)) <= tol * np.max(np.abs(oA))
    assert np.max(np.abs(gM - oM)) <= tol * np.max(np.abs(oM))


def test_loss_row_beyond_the_tile_is_refused():
    """Rows that select 510 entries or more are refused, as before the lean kernel."""
    S = _spai()
    n = 600
    A = _pattern_with(n, 64, 2, 3)
    M = _pattern_with(n, 1, 12, 4)
    longest = max(M[A.indices[A.indptr[i]:A.indptr[i + 1]]].nnz for i in range(n))
    assert longest >= 510
    with pytest.raises(S.SpaiError) as e:
        S.loss_fwd(A, M)
    assert e.value.code == -7


@pytest.mark.parametrize("kind,n,nrhs", [
    ("geo", 1, 1), ("geo", 2, 3), ("geo", 9, 32), ("geo", 257, 1), ("geo", 1024, 1),
    ("geo", 1023, 4), ("geo", 585, 7), ("geo", 512, 8), ("geo", 273, 15), ("geo", 272, 15),
    ("geo", 240, 17), ("geo", 129, 31), ("geo", 128, 32), ("grid", 32, 2), ("grid", 9, 5),
    ("grid", 32, 4)])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_pcg_in_one_workgroup_equals_the_launched_solve(kind, n, nrhs, precision):
    """Small solves run in one workgroup; with phase timing the same solve is launched
    product by product.  The sums are the same: bitwise equal, also where the terms' layout
    is at its limits (rows per XCD range, blocks of rows, padded right-hand sides), at
    iteration caps, and where a right-hand side is zero."""
    S = _spai()
    A = W.laplace2d(n) if kind == "grid" else \
        W.geometric_graph(n, 3) if n > 2 else sp.csr_matrix(np.diag(np.arange(1.0, n + 1)))
    n = A.shape[0]
    B = W.rhs(n, nrhs, 11)
    if nrhs > 4:
        B[:, 3] = 0.0
    out = []
    for prof in (False, True):
        h = S.SPAI(A, "lomr", "global", 2.0, True, max_iter=12,
                   options=S.Options(precision=precision, profile=prof))
        h.iterate(12)
        out.append([h.pcg(B, rtol=1e-9, max_iter=m) for m in (0, 1, 2, 7, 10000)])
        h.close()
    for a, b in zip(*out):
        assert a[3] == b[3]
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert np.array_equal(a[2], b[2])


@pytest.mark.parametrize("n", [1025, 2049, 8193, 16500])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 5, 16, 31])
def test_pcg_narrow_products_against_the_oracle(n, nrhs):
    """Sizes around the chunks of the narrow products (up to 1024 rows a workgroup, eight
    ranges) on irregular rows of up to about 25 entries.  Eight iterations, before a CG
    recurrence lets rounding grow (with a nearly indefinite M the two drift apart by 1e-6 in
    40): X is then a few sums of products away from B, 1e-12."""
    S = _spai()
    A = W.geometric_graph(n, n)
    M = sp.csr_matrix(O.lomr(A, oracle_rule(A, "column", 1.0, True), 6).M)
    B = W.rhs(n, nrhs, n + nrhs)
    X, it, _, rc = S.pcg_solve(A, M, B, rtol=1e-8, max_iter=8)
    Xo, ito, _ = O.pcg_block(A, M, B, rtol=1e-8, max_iter=8)
    assert rc in (S.SPAI_OK, S.SPAI_MAXITER) and list(it) == list(ito)
    assert np.max(np.abs(X - Xo)) <= 1e-12 * np.max(np.abs(Xo))


# the selection of a global cap takes one workgroup up to 2048 columns; the walks over the
# candidates take groups of columns, the bounds tiles of 128 columns or more
@pytest.mark.parametrize("n", [1, 7, 65, 127, 129, 513, 2047, 2048, 2049, 4101])
@pytest.mark.parametrize("method", ["mr", "cg", "lomr"])
@pytest.mark.parametrize("mode,value", [("global", 2.0), ("column", 3.0)])
def test_builds_at_the_edges_of_the_size_rules(n, method, mode, value):
    S = _spai()
    A = W.geometric_graph(n, 11 + n)
    h = S.SPAI(A, method, mode, value, True, max_iter=6)
    _, hist, _ = h.iterate(6)
    M = h.get()
    h.close()
    ref = O.run(method, A, oracle_rule(A, mode, value, True), 6)
    want = np.asarray(ref.resid[1:len(hist) + 1])
    assert len(hist) == ref.iters
    # a converged residual (n = 1, 7) is rounding: absolute against the first
    assert np.all(np.abs(np.asarray(hist) - want) <= 1e-10 * want + 1e-13 * ref.resid[0])
    assert pattern_diff(M, ref.M) == (set(), set())
    assert value_err(M, ref.M) <= 1e-9


@pytest.mark.parametrize("method", ["mr", "cg", "lomr"])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_floors_from_their_first_size_on(method, precision):
    """50,653 columns (the floors start at 49,152): none, the default and floors that every
    iteration fails give the same bits."""
    S = _spai()
    A = W.lognormal3d(37, 41)
    runs = []
    for frac in (0.0, 0.75, 4.0):
        h = S.SPAI(A, method, "global", 2.0, True, max_iter=5,
                   options=S.Options(precision=precision, floor_frac=frac))
        _, hist, _ = h.iterate(5)
        runs.append((hist, h.get(), history_array(h)))
        h.close()
    for hist, M, rec in runs[1:]:
        assert np.array_equal(hist, runs[0][0])
        assert (M != runs[0][1]).nnz == 0
        assert np.array_equal(rec, runs[0][2])


# constant coefficients: thousands of candidates share the cut's magnitude, so the collected
# keys neither fit one workgroup's LDS (2025 columns) nor thin out from pass to pass (2116)
@pytest.mark.parametrize("side", [45, 46])
@pytest.mark.parametrize("method", ["mr", "lomr"])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_selection_among_ties(side, method, precision):
    S = _spai()
    A = W.laplace2d(side)
    h = S.SPAI(A, method, "global", 1.5, True, max_iter=4, options=S.Options(precision=precision))
    _, hist, _ = h.iterate(4)
    M = h.get()
    h.close()
    ref = O.run(method, A, oracle_rule(A, "global", 1.5, True), 4)
    want = np.asarray(ref.resid[1:len(hist) + 1])
    if precision == "f64":
        assert np.all(np.abs(np.asarray(hist) - want) <= 1e-10 * want)
        assert pattern_diff(M, ref.M) == (set(), set())
        assert value_err(M, ref.M) <= 1e-9
    else:
        # float32 values: the cut's tie band is decided on rounded values, so only the
        # first step (its candidates have a handful of distinct magnitudes) is compared
        assert abs(hist[0] - want[0]) <= 1e-5 * want[0]


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_export_of_an_unsymmetric_state(precision):
    """A restored state may hold any M; the export transposes one that is not symmetric."""
    S = _spai()
    A = W.lognormal3d(8, 7)
    n = A.shape[0]
    h = S.SPAI(A, "mr", "global", 2.0, True, max_iter=8, options=S.Options(precision=precision))
    h.iterate(4)
    M = h.get()
    state = bytearray(h.get_state())
    hd, lists = parse_state(bytes(state))
    cp, ix, vl = lists[0]
    q = int(cp[n // 2])
    j = n // 2
    assert ix[q] != j                                  # an off-diagonal entry of column j
    o = hd["list_offsets"][0] + 8 * (n + 1) + 4 * int(cp[n]) + vl.itemsize * q
    state[o:o + vl.itemsize] = np.asarray([2 * vl[q]], dtype=vl.dtype).tobytes()
    h.set_state(bytes(state))
    got = h.get()
    h.close()
    want = M.tolil()
    want[int(ix[q]), j] = 2 * float(vl[q])
    want = want.tocsr()
    want.sort_indices()
    assert np.array_equal(got.indptr, want.indptr) and np.array_equal(got.indices, want.indices)
    assert np.array_equal(got.data, want.data)


# the scores' resident tier ends at 128 candidates a column and a few hundred rows of its
# residual: a generous cap on denser graphs takes some columns past either end
@pytest.mark.parametrize("name,make,cap", [
    ("lognormal7", lambda: W.lognormal3d(7, 3), 6.0),
    ("geo400", lambda: W.geometric_graph(400, 9), 6.0),
    ("geo900", lambda: W.geometric_graph(900, 4), 3.0),
    ("one", lambda: W.geometric_graph(1, 4), 3.0)])
@pytest.mark.parametrize("method", ["mr", "lomr"])
def test_scores_at_the_ends_of_their_tier(name, make, cap, method):
    S = _spai()
    A = make()
    m = O.cap_counts(A, "global", cap, True)
    h = S.SPAI(A, method, "global", cap, True, max_iter=5, options=S.Options(drop_score=True))
    _, hist, _ = h.iterate(5)
    M = h.get()
    h.close()
    ref = O.run(method, A, O.DropRule(mode="global", m=m, score=True), 5)
    want = np.asarray(ref.resid[1:len(hist) + 1])
    assert np.all(np.abs(np.asarray(hist) - want) <= 1e-10 * want + 1e-13 * ref.resid[0])
    assert pattern_diff(M, ref.M) == (set(), set())
    assert value_err(M, ref.M) <= 1e-9


def _arrow(n, spokes, seed):
    """2 I with one row and column coupled to `spokes` others: its columns of M, R and P are
    as wide as that, all the others narrow."""
    rng = np.random.default_rng(seed)
    hub = n // 3
    to = np.sort(rng.choice(np.delete(np.arange(n), hub), spokes, replace=False))
    v = rng.uniform(0.5, 1.0, spokes) / np.sqrt(spokes)
    U = sp.coo_matrix((v, (np.full(spokes, hub), to)), shape=(n, n)).tocsr()
    A = (U + U.T + 2.0 * sp.identity(n)).tocsr()
    A.sort_indices()
    return A


# wide columns, whose rows are collected in a bitmap up to 131,072 rows and in a hash set
# beyond: every column wide (2600 rows, lists past the large tile), and one of 3000 or 900
# entries among narrow ones on either side of the limit
@pytest.mark.parametrize("name,make,cap,iters,fmt", [
    ("all", lambda: _random_symmetric(2600, 9, 3) + 16.0 * sp.identity(2600), 40.0, 4, "ell"),
    ("all", lambda: _random_symmetric(2600, 9, 3) + 16.0 * sp.identity(2600), 40.0, 4, "csr"),
    ("below", lambda: _arrow(131072, 3000, 5), 1.5, 2, "csr"),
    ("above", lambda: _arrow(131073, 3000, 5), 1.5, 2, "csr"),
    ("large", lambda: _arrow(50000, 900, 6), 1.5, 2, "csr")])
@pytest.mark.parametrize("method", ["mr", "cg", "lomr"])
def test_wide_columns(name, make, cap, iters, fmt, method):
    S = _spai()
    A = make().tocsr()
    A.sort_indices()
    h = S.SPAI(A, method, "global", cap, True, max_iter=iters, options=S.Options(a_format=fmt))
    _, hist, _ = h.iterate(iters)
    M = h.get()
    h.close()
    ref = O.run(method, A, oracle_rule(A, "global", cap, True), iters)
    want = np.asarray(ref.resid[1:len(hist) + 1])
    assert np.all(np.abs(np.asarray(hist) - want) <= 1e-10 * want)
    assert pattern_diff(M, ref.M) == (set(), set())
    assert value_err(M, ref.M) <= 1e-9


def _state_with_direction(buf, k, j, value):
    """The LOMR state `buf` with every value of P and P^T zero and P's column j given an
    entry `value` in row k (a row after the column's last)."""
    hd, lists = parse_state(buf)
    n, (cp, ix, vl) = hd["n"], lists[1]
    q = int(cp[j + 1])
    assert q == cp[j] or ix[q - 1] < k
    cp2 = cp + (np.arange(n + 1) > j)
    vt = vl.dtype
    P = (cp2, np.insert(ix, q, k), np.insert(np.zeros(len(vl), vt), q, value))
    PT = (lists[2][0], lists[2][1], np.zeros(len(lists[2][2]), vt))
    head = bytearray(buf[:hd["list_offsets"][0]])
    np.frombuffer(head, dtype=np.int64, count=13)[9] += 1          # header: entries of P
    out = bytes(head)
    for c, i, v in (lists[0], P, PT, lists[3]):
        out += c.astype(np.int64).tobytes() + i.astype(np.int32).tobytes() + v.astype(vt).tobytes()
    return out


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_a_nan_direction_is_no_candidate_under_a_column_cap(precision):
    """A NaN in P (the step then falls back to MR, as it does with P = 0) adds no candidate
    of P: the iterate and the drop record are those of the same state with a zero there."""
    S = _spai()
    A = W.aniso2d(24, 1.0, 1.0)
    n = A.shape[0]
    h = S.SPAI(A, "lomr", "column", 3.0, True, max_iter=8, options=S.Options(precision=precision))
    h.iterate(3)
    st = h.get_state()
    runs = []
    for value in (0.0, np.nan):
        h.set_state(_state_with_direction(st, n - 1, 0, value))
        h.iterate(1)
        runs.append((history_array(h)[3], h.get()))
    assert h.stats()["mr_fallbacks"] >= 1
    h.close()
    assert np.array_equal(runs[0][0], runs[1][0])
    assert (runs[0][1] != runs[1][1]).nnz == 0


def _kernels_of(call, name):
    """Milliseconds of every kernel named `name` that call() launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.device_time / 1e3 for e in prof.events()
            if name in e.name and str(e.device_type).endswith("CUDA")]


@pytest.mark.parametrize("n,nrhs", [(1024, 1), (300, 3), (512, 8)])
def test_a_stagnating_small_solve_is_cut_into_launches(n, nrhs):
    """rtol = 0 on a matrix of condition 1e12: thousands of iterations.  No launch runs more
    than 1024 of them, and the solve is that of the product-by-product launches bit for bit
    (also where max_iter is a multiple of 1024, and one more)."""
    S = _spai()
    d = np.sqrt(np.random.default_rng(n).permutation(np.logspace(0, 12, n)))
    T = sp.diags([np.full(n, 2.0), np.full(n - 1, -1.0), np.full(n - 1, -1.0)], [0, 1, -1])
    A = sp.csr_matrix(sp.diags(d) @ T @ sp.diags(d))
    A = sp.csr_matrix((A + A.T) / 2)
    A.sort_indices()
    B = W.rhs(n, nrhs, 7)
    caps = (1024, 1025, 2048, 2500)
    out, launches = [], 0
    for prof in (False, True):
        h = S.SPAI(A, "mr", "global", 2.0, True, max_iter=2, options=S.Options(profile=prof))
        if not prof:
            launches = len(_kernels_of(lambda: h.pcg(B, rtol=0.0, max_iter=2500), "k_pcg_tiny"))
        out.append([h.pcg(B, rtol=0.0, max_iter=m) for m in caps])
        h.close()
    assert max(out[0][-1][1]) > 2048 and 2 <= launches <= 3
    for a, b in zip(*out):
        assert a[3] == b[3]
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert np.array_equal(a[2], b[2])


def test_dots_of_20000_rows_keep_their_place_beside_the_residual():
    """Random rows of 30 entries: in the second step a residual column has 900 entries and the
    dots reach all 20,000 rows.  The dots took 13 times the residual's time with a hash set
    and a sort (both kernels hashing), 54 times with the products entered in an LDS table
    too small for them first, and 20 times where they enter a bitmap (both kernels)."""
    S = _spai()
    A = _random_symmetric(20000, 60, 1)      # (half of the drawn entries are dropped)
    A = (A + sp.diags(np.asarray(abs(A).sum(axis=1)).ravel() + 1.0)).tocsr()
    A.sort_indices()
    h = S.SPAI(A, "mr", "global", 1.0, True, max_iter=2,
               options=S.Options(profile=True, a_format="csr"))
    h.iterate(1)
    before = h.profile()[0]
    h.iterate(1)
    after = h.profile()[0]
    h.close()
    ratio = (after["dots"] - before["dots"]) / (after["resid"] - before["resid"])
    print("dots / residual: %.1f" % ratio)
    assert ratio <= 35.0


def _power_pattern(A, k):
    B = sp.csr_matrix((np.ones(A.nnz), A.indices, A.indptr), shape=A.shape)
    P = B
    for _ in range(k - 1):
        P = sp.csr_matrix(P @ B)
        P.data[:] = 1.0
    P.sort_indices()
    return P


@pytest.mark.parametrize("make,k", [
    (lambda: W.lognormal3d(10, 4), 3),       # columns of up to 63 entries
    (lambda: W.grid9(20, 4), 3),             # 49
    (lambda: W.laplace2d(24), 5),            # 61
    (lambda: W.laplace2d(24), 4)])           # 41
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_loss_gradients_on_wide_patterns(make, k, precision):
    """M on pattern(A^k), its columns beyond the lean kernel's 32 entries: tolerances as above."""
    S = _spai()
    A = make()
    M = _power_pattern(A, k)
    M.data = 0.1 * np.random.default_rng(k).standard_normal(M.nnz)
    tol = 1e-12 if precision == "f64" else 1e-5
    gA, gM = S.loss_bwd(A, M, options=S.Options(precision=precision))
    for g, o, p in zip((gA, gM), O.loss_grad(A, M), (A, M)):
        o = np.asarray(sp.csr_matrix(o)[tuple(p.nonzero())]).ravel()
        assert np.max(np.abs(g - o)) <= tol * np.max(np.abs(o))


def _best_time(call, reps=10):
    import time

    import torch
    best = np.inf
    for _ in range(reps):
        torch.cuda.synchronize()
        t = time.perf_counter()
        call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_gradient_in_m_keeps_its_place_beside_the_gradient_in_a():
    """Nine-point graph, M on pattern(A^3): both gradients leave the lean kernel.  The one in M
    took 1.3 times the one in A with a kernel of its own, 6.2 times with the rows' kernel."""
    import torch
    S = _spai()
    A = W.grid9(256, 3)
    M = _power_pattern(A, 3)
    M.data = np.random.default_rng(0).standard_normal(M.nnz)
    dev = [torch.sparse_csr_tensor(torch.from_numpy(X.indptr.astype(np.int64)),
                                   torch.from_numpy(X.indices.astype(np.int64)),
                                   torch.from_numpy(X.data), size=X.shape).cuda() for X in (A, M)]
    ta = _best_time(lambda: S.loss_bwd(*dev, want_m=False))
    tm = _best_time(lambda: S.loss_bwd(*dev, want_a=False))
    print("gradient in M / in A: %.2f" % (tm / ta))
    assert tm <= 3.0 * ta


@pytest.mark.parametrize("eigs,steps,enqueued", [(1, 1, 1), (3, 3, 4), (5, 5, 16), (12, 12, 16)])
def test_lanczos_enqueues_few_steps_past_its_end(eigs, steps, enqueued):
    """A process of `steps` steps (as many distinct eigenvalues) enqueues no more than the host
    needs to see its end: the passes of 1, 4 or 16 steps, three each, and one for ||v0||."""
    S = _spai()
    A = sp.diags(np.repeat(np.linspace(1.0, 3.0, eigs), 600 // eigs)).tocsr()
    v0 = np.random.default_rng(eigs).standard_normal(A.shape[0])
    got = []
    n = len(_kernels_of(lambda: got.append(S.spectrum(A, v0, steps=200)[4]), "k_lz_pass"))
    assert got[0] == steps
    assert 0 < n <= 1 + 3 * enqueued


@pytest.mark.parametrize("nrhs", [1, 3, 4, 7])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_small_solves_with_long_rows_are_launched(nrhs, precision):
    """One workgroup takes a small solve only where A and M have few entries (with 150 a row,
    512 rows and three right-hand sides it took 145 us an iteration, launched 84): the rows of
    a cap of 24 nnz(A) are left to the launched products, those of 2 are not, and either way
    the solve is the launched one bit for bit."""
    S = _spai()
    A = W.lognormal3d(8, 1)
    B = W.rhs(A.shape[0], nrhs, 5)
    for cap, launched in ((2.0, False), (24.0, True)):
        out = []
        for prof in (False, True):
            h = S.SPAI(A, "lomr", "global", cap, True, max_iter=12,
                       options=S.Options(precision=precision, profile=prof))
            h.iterate(12)
            if not prof:
                assert (len(_kernels_of(lambda: h.pcg(B, rtol=1e-9), "k_spmm")) > 0) == launched
            out.append(h.pcg(B, rtol=1e-9))
            h.close()
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
        assert np.array_equal(out[0][2], out[1][2])


def _kernel_names(call, name):
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return {e.name for e in prof.events() if name in e.name}


# 512 workgroups of 64 (32 right-hand sides) or 256 rows (4), and 1024 of 128 (8), are the last
# with 1024 threads
@pytest.mark.parametrize("n,nrhs,threads", [
    (32768, 31, 1024), (32769, 31, 256), (131072, 3, 1024), (131073, 3, 256),
    (131072, 5, 1024), (131073, 5, 256)])
@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_pcg_narrow_products_on_either_side_of_their_widths(n, nrhs, threads, precision):
    """A few iterations against the oracle (M rounded to float32 on the mixed path), as above."""
    S = _spai()
    A = sp.csr_matrix(W.geometric_graph(n, 3))
    d = sp.diags(1.0 / np.sqrt(A.diagonal()))
    M = sp.csr_matrix(d @ (sp.identity(n) - 0.05 * (d @ A @ d - sp.identity(n))) @ d)
    M = sp.csr_matrix((M + M.T) / 2)
    M.sort_indices()
    if precision == "mixed":
        M.data = M.data.astype(np.float32).astype(np.float64)
    B = W.rhs(n, nrhs, 3)
    got = []
    names = _kernel_names(lambda: got.append(S.pcg_solve(
        A, M, B, rtol=1e-8, max_iter=4, options=S.Options(precision=precision))), "k_spmm_narrow")
    assert names and all((", %d>" % (threads // 256)) in x for x in names)
    Xo, ito, _ = O.pcg_block(A, M, B, rtol=1e-8, max_iter=4)
    assert list(got[0][1]) == list(ito)
    assert np.max(np.abs(got[0][0] - Xo)) <= 1e-12 * np.max(np.abs(Xo))


@pytest.mark.parametrize("method", ["mr", "cg", "lomr"])
def test_floors_in_use_against_the_oracle(method):
    """50,653 columns, where floors are in use: residual history and drop record against the
    oracle with the default floor, which leaves candidates unwritten (its second pass hardly
    ever runs), and with one (a million cuts) that every iteration fails (the second pass then writes them)."""
    S = _spai()
    A = W.lognormal3d(37, 41)
    iters = 6
    ref = getattr(O, method)(A, oracle_rule(A, "global", 2.0, True), iters)
    written = {}
    for frac in (0.0, 0.75, 1e6):
        h = S.SPAI(A, method, "global", 2.0, True, max_iter=iters,
                   options=S.Options(floor_frac=frac))
        _, hist, _ = h.iterate(iters)
        written[frac] = h.profile()[2]["cand_m"]
        rec = history_array(h)
        M = h.get()
        h.close()
        assert rel_err(hist, ref.resid[1:]) <= TOL_F64
        assert np.array_equal(rec, history_from_oracle(ref))
        assert pattern_diff(M, ref.M) == (set(), set())
        assert value_err(M, ref.M) <= 1e-9
    assert written[0.75] < written[0.0] == written[1e6]


@pytest.mark.parametrize("n", [1, 2, 64])
def test_get_waits_and_copies_little(n):
    """A small export is waits and copies: one copy for the size, and one before the three
    lists (four more, with a wait each, took 20 us of 128 more than the host's transposition)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    S = _spai()
    A = sp.csr_matrix(sp.diags([np.full(n, 3.0), np.full(max(n - 1, 0), -1.0),
                                np.full(max(n - 1, 0), -1.0)], [0, 1, -1], shape=(n, n)))
    h = S.SPAI(A, "lomr", "global", 2.0, True, max_iter=4)
    h.iterate(3)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        M = h.get()
        torch.cuda.synchronize()
    h.close()
    ref = O.run("lomr", A, oracle_rule(A, "global", 2.0, True), 3)
    assert pattern_diff(M, ref.M) == (set(), set()) and value_err(M, ref.M) <= 1e-12
    assert 0 < sum("DtoH" in e.name for e in prof.events()) <= 5


@pytest.mark.parametrize("precision", ["f64", "mixed"])
def test_loss_calls_allocate_once(precision):
    """Value and gradients on device matrices take one block a call, the float32 copies of the
    mixed path among it (two more blocks made it slower than float64)."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    S = _spai()
    A = W.grid9(20, 4)
    M = sp.csr_matrix(W.square_pattern(A))
    M.data = 0.1 * np.random.default_rng(1).standard_normal(M.nnz)
    dev = [torch.sparse_csr_tensor(torch.from_numpy(X.indptr.astype(np.int64)),
                                   torch.from_numpy(X.indices.astype(np.int64)),
                                   torch.from_numpy(X.data), size=X.shape).cuda() for X in (A, M)]
    o = S.Options(precision=precision)
    L, g = S.loss_fwd(*dev, o), S.loss_bwd(*dev, options=o)     # (torch's blocks are then cached)
    tol = 1e-12 if precision == "f64" else 1e-5
    assert L == pytest.approx(O.loss(A, M), rel=tol)
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        S.loss_fwd(*dev, o)
        S.loss_bwd(*dev, options=o)
        torch.cuda.synchronize()
    assert 0 < sum(e.name == "hipMalloc" for e in prof.events()) <= 2
    del g
