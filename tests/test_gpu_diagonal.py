"""GPU: matrices whose rows share column offsets are read as diagonals, 128
rows at a time (plans of every kind of slice: one value per diagonal, a value
per row, both, the matrix's first and last rows, and slices that fall back to
the sliced layout because a row is unsorted or repeats a column).  One launch
per power and the persistent kernels give the oracle's bits for every count of
right-hand sides, for row counts around the slice height, in both row
orders, with infinities and NaN next to rows that do not read them."""
import contextlib
import ctypes
import types

import numpy as np
import pytest

import oracle
import workloads as w

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
mpk = pytest.importorskip("paper_2405_12525_amd")


def banded(n, offsets, seed, vary=(), drop=0.0, odd_rows=False):
    """Row i holds i + d for the offsets d that stay inside, each left out with
    probability `drop`; diagonals in `vary` have a value per row, the others
    one value (-0.0 for the first).  odd_rows: a few rows are unsorted, repeat
    a column or are empty."""
    g = np.random.default_rng(seed)
    const = {d: float(v) for d, v in zip(offsets, g.standard_normal(len(offsets)))}
    const[offsets[0]] = -0.0
    rp, cols, vals = [0], [], []
    for i in range(n):
        c = [i + d for d in offsets if 0 <= i + d < n and g.random() >= drop]
        v = [float(g.standard_normal()) if k - i in vary else const[k - i] for k in c]
        if odd_rows and i % 300 == 7:
            c, v = c[::-1], v[::-1]
        elif odd_rows and i % 300 == 9 and c:
            c, v = c + [c[-1]], v + [0.5]
        elif odd_rows and i % 300 == 11:
            c, v = [], []
        cols += c
        vals += v
        rp.append(len(cols))
    return w.CSR(n, np.array(rp, np.int32), np.array(cols, np.int32), np.array(vals, np.float64))


def check(A, R, p=3, value_bits=64, x=None, reorder="none", order="original"):
    x = w.uniform_vectors(A.n, R, 17 * A.n + R) if x is None else x
    ref = oracle.powers(A, x, p, value_bits=value_bits)
    P = mpk.Plan(A, value_bits=value_bits, reorder=reorder, order=order)
    xd = torch.from_numpy(x).cuda()
    for tune in (None, dict(schedule="powers", chunk_nnz=900), dict(schedule="wave", lag=3, chunk_nnz=900)):
        if tune:
            P.tune(**tune)
        Y, B = P.run(xd, p), P.run_baseline(xd, p)
        P.sync()
        assert np.array_equal(Y.cpu().numpy().reshape(ref.shape), ref, equal_nan=True), (A.n, R, tune)
        assert np.array_equal(B.cpu().numpy().reshape(ref.shape), ref, equal_nan=True), (A.n, R, tune)
    P.close()


OFFS = [-40, -3, -1, 0, 1, 2, 40]


@pytest.mark.parametrize("n", [1, 3, 127, 128, 129, 255, 256, 257, 640, 1001])
@pytest.mark.parametrize("R", [1, 2, 3, 16])
def test_row_counts_around_the_slice_height(n, R):
    check(banded(n, OFFS, n), R)
    check(banded(n, OFFS, n + 1, vary=OFFS), R)


@pytest.mark.parametrize("R", list(range(1, 17)))
@pytest.mark.parametrize("vary", [(), (0,), (-3, 1, 40), tuple(OFFS)])
def test_every_rhs_count_and_kind_of_diagonal(R, vary):
    check(banded(900, OFFS, R, vary=vary, drop=0.1), R)
    check(banded(900, OFFS, R, vary=vary), R, value_bits=32)


@pytest.mark.parametrize("m", range(1, 10))
def test_list_lengths(m):
    offs = [-5, -4, -2, -1, 0, 1, 3, 4, 7][:m]
    check(banded(700, offs, m, vary=offs[::2]), 1)
    check(banded(700, offs, m, vary=offs[1::2]), 4)


@pytest.mark.parametrize("reorder,R", [("none", 1), ("none", 5), ("bfs", 1), ("bfs", 4)])
def test_slices_that_fall_back(reorder, R):
    check(banded(4000, OFFS, 3, vary=(1,), drop=0.05, odd_rows=True), R, reorder=reorder)


@pytest.mark.parametrize("R", [1, 2, 3])
def test_infinities_and_nan_stay_in_their_columns(R):
    A = banded(700, OFFS, 5, vary=(2,), drop=0.2)
    x = w.uniform_vectors(A.n, R, 6)
    x[0, 0], x[130, R - 1], x[131, 0], x[699, R - 1] = np.inf, np.nan, -np.inf, np.inf
    x[200] = -0.0
    A.val[A.rowptr[300]] = np.inf
    A.val[A.rowptr[301]] = np.nan
    with np.errstate(invalid="ignore"):
        check(A, R, p=2, x=x)


@pytest.mark.parametrize("R", [1, 2, 5])
def test_recurrence_and_sums(R):
    A = w.anderson_3d(9)          # periodic: wrapped rows at both ends of every line
    x = w.random_sign_unit_vectors(A.n, R, 12)
    xd = torch.from_numpy(x).cuda()
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(11, 0.7)
    be = be + 0.25
    for bits in (64, 32):
        P = mpk.Plan(A, value_bits=bits)
        assert np.array_equal(P.run_recur(xd, al, be, ga).cpu().numpy(),
                              oracle.recur(A, x, al, be, ga, value_bits=bits))
        ra, rb = oracle.poly_sums(A, x, al, be, ga, wa, wb, value_bits=bits)
        for run in (P.run_poly, P.run_baseline_poly):
            acc = run(xd, wa, wb, al, be, ga)[0].cpu().numpy()
            assert np.array_equal(acc[0], ra) and np.array_equal(acc[1], rb)
        P.close()


@pytest.mark.parametrize("side,R", [(5, 1), (12, 3), (16, 2)])
def test_more_powers_than_a_segment_holds(side, R):
    """p = 70 on one workgroup per column (5^3, 12^3) and on launches (16^3)."""
    A = w.anderson_3d(side)
    x = w.random_sign_unit_vectors(A.n, R, side)
    xd = torch.from_numpy(x).cuda()
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(70, 3.0)
    P = mpk.Plan(A)
    ref = oracle.recur(A, x, al, be, ga)
    assert np.array_equal(P.run_recur(xd, al, be, ga).cpu().numpy(), ref)
    assert np.array_equal(P.run(xd, 70).cpu().numpy(), oracle.powers(A, x, 70))
    ra, rb = oracle.poly_sums(A, x, al, be, ga, wa, wb)
    acc, ring = P.run_poly(xd, wa, wb, al, be, ga)
    acc = acc.cpu().numpy()
    assert np.array_equal(acc[0], ra) and np.array_equal(acc[1], rb)
    assert np.array_equal(ring.cpu().numpy()[1], ref[69])
    P.close()


def test_unaligned_vectors_and_captured_run():
    A = w.stencil_3d27(12)
    x = w.uniform_vectors(A.n, 1, 4)
    buf = torch.zeros(A.n + 1, dtype=torch.float64, device="cuda")
    out = torch.zeros(4 * A.n + 1, dtype=torch.float64, device="cuda")
    xd, Y = buf[1:], out[1:].view(4, A.n)          # 8-byte aligned only
    xd.copy_(torch.from_numpy(x[:, 0]))
    ref = oracle.powers(A, x, 4)[:, :, 0]
    P = mpk.Plan(A)
    P.run(xd, 4, Y)
    assert np.array_equal(Y.cpu().numpy(), ref)
    G = P.capture(xd, 4, Y)
    for _ in range(3):
        Y.fill_(np.nan)
        torch.cuda.synchronize()
        G.launch()
        assert np.array_equal(Y.cpu().numpy(), ref)
    G.close()
    status = torch.full((1,), 7, dtype=torch.int32).pin_memory()
    Y.fill_(np.nan)
    P.run_noalloc(xd, 4, Y, status=status)         # run before: prepared
    torch.cuda.synchronize()
    assert int(status[0]) == 0 and np.array_equal(Y.cpu().numpy(), ref)
    P.close()


@pytest.mark.parametrize("R", [1, 4, 16])
def test_vectors_past_the_caches(R):
    """A periodic lattice whose planes are wider than an XCD's L2 holds and
    whose vectors exceed the memory-side cache: streamed results and values,
    blocks dealt in runs of an eighth of a plane; the persistent kernel, which
    reads the sliced layout, gives the same bits."""
    side, planes = (330, 40) if R == 1 else (160, 64 // R * 8)
    offs = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    n = side * side * planes
    g = np.random.default_rng(R)
    A = w._lattice_stencil((side, side, planes), offs, [0.25] * 7, True, "torus")
    if R == 1:                       # a value per entry: 244 MB of them
        A.val = g.standard_normal(A.nnz)
    x = torch.from_numpy(g.uniform(-1, 1, (n, R))).cuda()
    co = mpk.chebyshev_coefficients(3)
    P = mpk.Plan(A, reorder="none")
    Y, Z = P.run(x, 3), P.run_recur(x, *co)
    P.tune(schedule="powers", workgroups=512)
    Yp, Zp = P.run(x, 3), P.run_recur(x, *co)
    P.sync()
    assert torch.equal(Y, Yp) and torch.equal(Z, Zp)
    P.close()


@pytest.mark.parametrize("side,R,bits", [(23, 1, 64), (24, 3, 32), (82, 1, 64), (84, 1, 32),
                                         (83, 16, 64)])
def test_plan_order_runs_on_diagonals_of_the_callers_order(side, R, bits):
    """BFS plans in their own order: small ones as they are, large ones (2^19 rows,
    2^23 elements) converted, on two streams at once, after which a captured and
    a no-allocation run of the same shape are taken as before."""
    A = w.stencil_3d27(side)
    p = 5
    x = w.uniform_vectors(A.n, R, side)
    ref = oracle.powers(A, x, p, value_bits=bits)
    co = mpk.chebyshev_coefficients(p)
    cref = oracle.recur(A, x, *co, value_bits=bits)
    P = mpk.Plan(A, value_bits=bits, order="plan")
    xp = P.permute(torch.from_numpy(x).cuda(), to_plan=True)
    assert np.array_equal(xp.cpu().numpy(), x[P.levels()[1]])
    torch.cuda.synchronize()

    def back(Y):
        return P.permute(Y.reshape(p, A.n, R), to_plan=False).cpu().numpy()
    streams = [torch.cuda.Stream() for _ in range(2)]
    jobs = []
    for i in range(6):
        with torch.cuda.stream(streams[i % 2]):
            Y = torch.empty((p, A.n, R), dtype=torch.float64, device="cuda")
            (P.run if i < 4 else lambda x, p, Y, stream: P.run_recur(x, *co, Y=Y, stream=stream))(
                xp, p, Y, stream=streams[i % 2])
            jobs.append(Y)
    P.sync()
    torch.cuda.synchronize()
    for i, Y in enumerate(jobs):
        assert np.array_equal(back(Y), ref if i < 4 else cref), i
    Y = torch.empty((p, A.n, R), dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=streams[0]):
        P.run(xp, p, Y=Y, stream=streams[0])
    for _ in range(2):
        Y.fill_(np.nan)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(back(Y), ref)
    Y.fill_(np.nan)
    P.run_noalloc(xp, p, Y)
    assert np.array_equal(back(Y), ref)
    assert np.array_equal(back(P.run_baseline(xp, p)), ref)
    del g
    P.close()


@pytest.mark.parametrize("R", [1, 2, 3, 7, 16])
@pytest.mark.parametrize("nvec", [1, 3, 4, 9])
def test_permute_moves_every_row(R, nvec):
    for A in (w.stencil_3d27(11), w.banded_random(3000, half_width=90)):   # with and without the inverse map
        P = mpk.Plan(A, order="plan")
        perm = P.levels()[1]
        v = np.random.default_rng(R).standard_normal((nvec, A.n, R))
        vd = torch.from_numpy(v).cuda()
        q = P.permute(vd, to_plan=True)
        assert np.array_equal(q.cpu().numpy(), v[:, perm])
        assert np.array_equal(P.permute(q, to_plan=False).cpu().numpy(), v)
        P.close()


def near_band(n, seed, wide):
    """Rows with one to 23 symmetric neighbours within 600 rows, shuffled within
    windows of 3000 rows; wide: 40 rows also have one anywhere."""
    g = np.random.default_rng(seed)
    cnt = g.integers(0, 12, size=n)
    src = np.repeat(np.arange(n, dtype=np.int64), cnt)
    dst = src + g.integers(1, 601, size=src.size)
    src, dst = src[dst < n], dst[dst < n]
    if wide:
        src = np.concatenate([src, g.integers(0, n, size=40)])
        dst = np.concatenate([dst, g.integers(0, n, size=40)])
    i = np.arange(n, dtype=np.int64)
    new = np.argsort(np.argsort(i // 3000 + g.random(n)))
    src, dst = new[src], new[dst]
    key = np.unique(np.concatenate([src * n + dst, dst * n + src, i * n + i]))
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    return w.CSR(n, rp.astype(np.int32), (key % n).astype(np.int32), g.standard_normal(key.size))


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("order,bits", [("original", 64), ("original", 32), ("plan", 64)])
def test_windowed_rows(wide, order, bits):
    """A shuffled band in BFS order, read through a ring of input rows in LDS by
    one right-hand side: powers, recurrence and weighted sums give the oracle's
    bits, also where some entries lie outside the windows."""
    A = near_band((1 << 20) + 333, 5 + wide, wide)
    x = w.uniform_vectors(A.n, 1, 9)
    P = mpk.Plan(A, value_bits=bits, order=order)
    xd = torch.from_numpy(x).cuda()
    if order == "plan":
        xd = P.permute(xd, to_plan=True)

    def back(Y):
        Y = Y.reshape(-1, A.n, 1)
        return (P.permute(Y, to_plan=False) if order == "plan" else Y).cpu().numpy()
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(3, 0.4)
    be = be + 0.5
    assert np.array_equal(back(P.run(xd, 3)), oracle.powers(A, x, 3, value_bits=bits))
    assert np.array_equal(back(P.run_baseline_recur(xd, al, be, ga)),
                          oracle.recur(A, x, al, be, ga, value_bits=bits))
    acc, _ = P.run_poly(xd, wa, wb, al, be, ga)
    ra, rb = oracle.poly_sums(A, x, al, be, ga, wa, wb, value_bits=bits)
    got = back(acc)
    assert np.array_equal(got[0], ra) and np.array_equal(got[1], rb)
    P.close()


@pytest.mark.parametrize("rem", [1, 127, 128, 129])
@pytest.mark.parametrize("R", [1, 3, 16])
def test_slice_height_where_every_power_fills_the_device(rem, R):
    n = (1 << 15) + rem
    check(banded(n, OFFS, rem, vary=(-3, 1, 40), drop=0.1), R, p=2)
    check(banded(n, OFFS, rem, vary=(1,), drop=0.05, odd_rows=True), R, p=2, value_bits=32)
    check(banded(n, OFFS, rem, vary=OFFS, drop=0.19), R, p=2)   # near the limit on missing entries


@pytest.mark.parametrize("slots", [8, 9, 16, 17])
@pytest.mark.parametrize("n,R", [(63, 1), (65, 5), (4096, 16), (4097, 16), (24576, 1)])
def test_few_elements(slots, n, R):
    """Rows without common offsets, about `slots` long, empty ones among them,
    with sizes on both sides of the limits: the oracle's bits."""
    g = np.random.default_rng(slots)
    cnt = np.minimum(n, slots - (g.random(n) < 0.1))
    cnt[::64] = 0
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(cnt)
    A = w.CSR(n, rp, g.integers(0, n, size=rp[-1]).astype(np.int32), g.standard_normal(rp[-1]))
    x = w.uniform_vectors(n, R, 4)
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(4, 0.6)
    for bits, reorder in ((64, "none"), (32, "none"), (64, "bfs")):
        P = mpk.Plan(A, value_bits=bits, reorder=reorder)
        xd = torch.from_numpy(x).cuda()
        for Y, ref in ((P.run_baseline(xd, 3), oracle.powers(A, x, 3, value_bits=bits)),
                       (P.run_recur(xd, al, be, ga), oracle.recur(A, x, al, be, ga, value_bits=bits)),
                       (P.run_baseline_poly(xd, wa, wb, al, be, ga)[0],
                        np.stack(oracle.poly_sums(A, x, al, be, ga, wa, wb, value_bits=bits)))):
            assert np.array_equal(Y.cpu().numpy().reshape(ref.shape), ref), (bits, reorder)
        P.close()


@pytest.mark.parametrize("length", [500, (1 << 22) + 100])
def test_band_with_a_long_row(length):
    """One row of a wide irregular band is long (repeated columns, taken
    literally), beyond 2^22 entries in the second case: every entry counts."""
    A = near_band((1 << 20) + 333, 11, False)
    g = np.random.default_rng(length)
    row, e0, e1 = 4000, int(A.rowptr[4000]), int(A.rowptr[4001])
    col = g.integers(row - 500, row + 501, size=length).astype(np.int32)
    val = g.integers(-8, 9, size=length).astype(np.float64)
    rp = A.rowptr.copy()
    rp[row + 1:] += length - (e1 - e0)
    A = w.CSR(A.n, rp, np.concatenate([A.col[:e0], col, A.col[e1:]]),
              np.concatenate([A.val[:e0], val, A.val[e1:]]))
    x = w.uniform_vectors(A.n, 1, 3)
    P = mpk.Plan(A, reorder="none")
    xd = torch.from_numpy(x).cuda()
    ref = oracle.powers(A, x, 2)
    assert np.array_equal(P.run_baseline(xd, 2).cpu().numpy().reshape(ref.shape), ref)
    assert np.array_equal(P.run(xd, 2).cpu().numpy().reshape(ref.shape), ref)
    P.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 3000])
@pytest.mark.parametrize("R", range(4, 17))
def test_csr_rows_of_many_right_hand_sides(n, R):
    """Rows of uneven length, empty and long ones among them, around the rows
    that a workgroup takes: powers, recurrence and sums give the oracle's bits."""
    g = np.random.default_rng(n)
    cnt = g.integers(0, 12, size=n)
    cnt[::max(1, n // 3)] = 40
    cnt[n // 2] = 0
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(cnt)
    A = w.CSR(n, rp, g.integers(0, n, size=rp[-1]).astype(np.int32), g.standard_normal(rp[-1]))
    x = w.uniform_vectors(n, R, 4)
    xd = torch.from_numpy(x).cuda()
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(3, 0.6)
    for bits, reorder in ((64, "bfs"), (32, "none")):
        P = mpk.Plan(A, value_bits=bits, reorder=reorder)
        for Y, ref in ((P.run(xd, 2), oracle.powers(A, x, 2, value_bits=bits)),
                       (P.run_baseline_recur(xd, al, be, ga),
                        oracle.recur(A, x, al, be, ga, value_bits=bits)),
                       (P.run_baseline_poly(xd, wa, wb, al, be, ga)[0],
                        np.stack(oracle.poly_sums(A, x, al, be, ga, wa, wb, value_bits=bits)))):
            assert np.array_equal(Y.cpu().numpy().reshape(ref.shape), ref), (bits, reorder)
        P.close()


@pytest.mark.parametrize("R", [1, 2, 3])
@pytest.mark.parametrize("slices", [4095, 4097])
def test_csr_slices_one_by_one_and_in_pairs(R, slices):
    """Slice counts on both sides of where workgroups take two."""
    n, g = 256 * slices - 5, np.random.default_rng(R)     # a slice holds at most 256 rows
    cnt = np.where(np.arange(n) % 64 == 0, 9, 1)
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(cnt)
    col = np.repeat(np.arange(n), cnt) + g.integers(-50, 51, size=rp[-1])
    A = w.CSR(n, rp, np.clip(col, 0, n - 1).astype(np.int32), g.standard_normal(rp[-1]))
    x = w.uniform_vectors(n, R, 5)
    P = mpk.Plan(A, reorder="none")
    ref = oracle.powers(A, x, 2)
    assert np.array_equal(P.run_baseline(torch.from_numpy(x).cuda(), 2).cpu().numpy().reshape(ref.shape), ref)
    P.close()


@pytest.mark.parametrize("n,R", [(8192, 16), (20000, 4), (60000, 16)])
def test_default_run_of_a_small_band_is_no_slower_than_a_persistent_one(n, R):
    """A default run of a small irregular matrix fills the device: measured at
    0.14 to 0.5 of the persistent kernel's time, 1.3 to 1.8 where it did not."""
    A = w.banded_random(n)
    P = mpk.Plan(A)
    xd = torch.from_numpy(w.uniform_vectors(n, R, 6)).cuda()
    Y = torch.empty((8, n, R), dtype=torch.float64, device="cuda")

    def fastest():
        times = []
        for _ in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(4):
                P.run(xd, 8, Y)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times)
    default = fastest()
    P.tune(schedule="wave", lag=4096)
    assert default < fastest()
    P.close()


def times_of_default_and_persistent_runs(P, x, p):
    Y = torch.empty((p,) + tuple(x.shape), dtype=torch.float64, device="cuda")

    def fastest():
        times = []
        for _ in range(12):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(4):
                P.run(x, p, Y)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times)
    default = fastest()
    P.tune(schedule="wave", lag=4096)
    return default, fastest()


@pytest.mark.parametrize("n,k", [(400000, 16), (60000, 100)])
def test_default_run_of_near_columns_is_no_slower_than_a_persistent_one(n, k):
    """Rows of equal length without common offsets (sliced layout, 16-bit
    offsets), one right-hand side: measured at 1.0 of the persistent kernel's
    time, which the default runs; 1.6 to 1.7 with a launch per power."""
    g = np.random.default_rng(k)
    col = np.arange(n)[:, None] + g.integers(-2000, 2001, size=(n, k))
    A = w.CSR(n, np.arange(0, n * k + 1, k, dtype=np.int32),
              np.sort(np.clip(col, 0, n - 1), axis=1).reshape(-1).astype(np.int32),
              g.standard_normal(n * k))
    P = mpk.Plan(A, reorder="none")
    x = torch.from_numpy(w.uniform_vectors(n, 1, 6)).cuda()
    default, persistent = times_of_default_and_persistent_runs(P, x, 8)
    assert default < 1.25 * persistent
    P.close()


def test_default_run_of_a_five_point_plane_in_plan_order_is_no_slower_than_a_persistent_one():
    """A plane whose matrix stays in the memory-side cache, one right-hand side:
    the persistent kernel, 1.10 to 1.17 of whose time conversion takes."""
    A = w.stencil_2d5(1500)
    P = mpk.Plan(A, order="plan")
    x = torch.from_numpy(w.uniform_vectors(A.n, 1, 6)).cuda()
    default, persistent = times_of_default_and_persistent_runs(P, x, 8)
    assert default < 1.08 * persistent
    P.close()


def shifted(shape, by):
    """A vector array `by` doubles past a 128-byte boundary."""
    n = int(np.prod(shape))
    return torch.full((n + 16,), np.nan, dtype=torch.float64, device="cuda")[by:by + n].view(shape)


@pytest.mark.parametrize("first", ["aligned", "unaligned", "sums"])
@pytest.mark.parametrize("R", [1, 2, 4])
def test_one_run_prepares_every_form_of_its_shape(first, R):
    """A plan whose default runs take the persistent kernel or one launch per
    power by the alignment of their output and by whether they sum: one run of
    any kind, then no-allocation and captured runs of the others, from a fresh
    plan each."""
    A, p = w.anderson_3d(96), 4                    # 884,736 rows, a multiple of 16
    x = w.uniform_vectors(A.n, R, 3)
    xd = torch.from_numpy(x).cuda()
    al, be, ga, wa, wb = mpk.cheb_time_coefficients(p, 0.5)
    ref = mpk.Plan(A).run_baseline(xd, p)
    ya, yu = shifted((p, A.n, R), 0), shifted((p, A.n, R), 1)
    assert ya.data_ptr() % 128 == 0 and yu.data_ptr() % 128 == 8
    sums = [torch.empty((2, A.n, R), dtype=torch.float64, device="cuda") for _ in range(4)]
    P = mpk.Plan(A, reorder="bfs", order="plan")
    xp = P.permute(xd, to_plan=True)
    refp = P.permute(ref, to_plan=True)
    P.run_baseline_poly(xp, wa, wb, al, be, ga, acc=sums[0], work=sums[1])
    P.close()
    calls = {"aligned": lambda P, **k: P.run(xp, p, ya, **k),
             "unaligned": lambda P, **k: P.run(xp, p, yu, **k),
             "sums": lambda P, **k: P.run_poly(xp, wa, wb, al, be, ga, acc=sums[2], work=sums[3], **k)}
    outs = {"aligned": (ya, refp), "unaligned": (yu, refp), "sums": (sums[2], sums[0])}
    for kind, (out, want) in outs.items():
        if kind == first:
            continue
        P = mpk.Plan(A, reorder="bfs", order="plan")
        if kind == "sums":                         # checks the pattern; another p
            P.run_poly(xp, wa[:3], wb[:3], al[:2], be[:2], ga[:2], acc=sums[2], work=sums[3])
        calls[first](P)
        P.sync()
        if kind != "sums":
            out.fill_(np.nan)
            P.run_noalloc(xp, p, out)
            torch.cuda.synchronize()
            assert torch.equal(out.view(want.shape), want), (first, kind)
        s = torch.cuda.Stream()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            calls[kind](P, stream=s)
        for _ in range(2):
            out.fill_(np.nan)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(want.shape), want), (first, kind)
        del g
        P.close()


@pytest.mark.parametrize("counts", [(1,), (1, 9), (16, 1)])
def test_prepared_runs_that_convert_allocate_nothing(counts):
    """A plan-order lattice whose runs use vectors in the caller's numbering:
    they are there once prepare was called with the counts that run."""
    A, p = w.stencil_3d27(101), 3
    mpk.use_torch_allocator(True)
    try:
        P = mpk.Plan(A, order="plan")
        for R in counts:
            P.prepare(p, R)
        allocs = mpk.allocator_stats["allocs"]
        for R in counts:
            x = torch.from_numpy(w.uniform_vectors(A.n, R, R)).cuda()
            Y = P.run(x, p)
            P.sync()
            assert mpk.allocator_stats["allocs"] == allocs, R
            P2 = P.run_baseline(x, p)
            P.sync()
            assert torch.equal(Y, P2)
        P.close()
    finally:
        mpk.use_torch_allocator(False)


@contextlib.contextmanager
def allocations(refuse):
    """Every allocation of the library through torch, numbered from 0; refuse(i,
    bytes): it gets none.  Yields the list of sizes asked for."""
    lib, pool, sizes = mpk.lib(), {}, []

    def alloc(nbytes, _):
        sizes.append(nbytes)
        if refuse(len(sizes) - 1, nbytes):
            return 0
        t = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
        pool[t.data_ptr()] = t
        return t.data_ptr()

    def free(p, _):
        torch.cuda.synchronize()
        pool.pop(p, None)
    fa = ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)(alloc)
    ff = ctypes.CFUNCTYPE(None, ctypes.c_void_p, ctypes.c_void_p)(free)
    assert lib.mpk_set_allocator(ctypes.cast(fa, ctypes.c_void_p),
                                 ctypes.cast(ff, ctypes.c_void_p), None) == 0
    try:
        yield sizes
    finally:
        lib.mpk_set_allocator(None, None, None)


def test_conversion_without_memory_for_its_vectors():
    """Where the vectors cannot be had, a run takes its own order, and asks for
    them once."""
    A, p = w.stencil_3d27(84), 3
    x = torch.from_numpy(w.uniform_vectors(A.n, 1, 1)).cuda()
    limit = [None]
    with allocations(lambda i, b: limit[0] is not None and b > limit[0]) as sizes:
        P = mpk.Plan(A, order="plan")
        limit[0] = A.n * 8
        P.prepare(p, 1)
        before = sum(b > limit[0] for b in sizes)
        outs = [P.run(x, p) for _ in range(3)]
        P.sync()
        assert sum(b > limit[0] for b in sizes) == before
        limit[0] = None
        Q = mpk.Plan(A, order="plan")
        ref = Q.run(x, p)
        Q.sync()
        assert all(torch.equal(Y, ref) for Y in outs)
        Q.close()
        P.close()


@pytest.mark.parametrize("matrix,reorder,optional", [("diagonals", "none", 2), ("diagonals", "bfs", 2),
                                                     ("windows", "none", 2), ("windows", "bfs", 3)])
@pytest.mark.parametrize("device", [False, True])
def test_plans_do_without_layouts_that_memory_is_short_for(matrix, reorder, optional, device):
    """Each allocation of a plan refused in turn: those of the diagonal slices or
    the windowed rows leave a plan that runs, every other one fails it."""
    A = (banded(6000, OFFS, 4, vary=OFFS) if matrix == "diagonals"
         else near_band((1 << 20) + 333, 5, False))
    x = torch.from_numpy(w.uniform_vectors(A.n, 1, 1)).cuda()
    M = types.SimpleNamespace(n=A.n, rowptr=torch.from_numpy(A.rowptr).cuda(),
                              col=torch.from_numpy(A.col).cuda(),
                              val=torch.from_numpy(A.val).cuda()) if device else A
    with allocations(lambda i, b: i == nth[0]) as sizes:
        nth = [-1]
        P = mpk.Plan(M, reorder=reorder)
        count, ref = len(sizes), P.run_baseline(x, 2)
        P.sync()
        P.close()
        done = 0
        for k in range(count):
            nth[0] = len(sizes) + k
            try:
                P = mpk.Plan(M, reorder=reorder)
            except mpk.MPKError as e:
                assert "ENOMEM" in str(e)
                continue
            nth[0] = -1
            done += 1
            assert torch.equal(P.run_baseline(x, 2), ref) and torch.equal(P.run(x, 2), ref)
            P.sync()
            P.close()
    assert done == optional


def two_lists(a, b, n=12800):
    """Offsets 0 and 5, their values a[0], a[1] and b[0], b[1] in alternating
    slices of 128 rows."""
    rp, cols, vals = [0], [], []
    for i in range(n):
        v = (a, b)[i // 128 % 2]
        cols += [c for c in (i, i + 5) if c < n]
        vals += v[:len(cols) - rp[-1]]
        rp.append(len(cols))
    return w.CSR(n, np.array(rp, np.int32), np.array(cols, np.int32), np.array(vals, np.float64))


def plan_sizes(A):
    with allocations(lambda i, b: False) as sizes:
        P = mpk.Plan(A, reorder="none")
        P.close()
    return list(sizes)


@pytest.mark.parametrize("a,b", [((1.0, 2.0), (-1.0, 2.0)), ((0.0, 2.0), (-0.0, 2.0)),
                                 ((1.0, -2.0), (-1.0, 2.0))])
def test_lists_that_differ_in_a_sign_are_shared(a, b):
    """Two lists that differ in a value's sign: each is stored once, as two
    that differ in a value are."""
    assert plan_sizes(two_lists(a, b)) == plan_sizes(two_lists((1.0, 2.0), (3.0, 2.0)))
    check(two_lists(a, b), 1)
    check(two_lists(a, b), 2)


def list_hash(values):
    """State of the hash of a list of offsets 0 and 5 that every row has, before
    its last value is mixed in."""
    h, mask = 1469598103934665603, (1 << 64) - 1
    for off, v in zip((0, 5), list(values) + [None]):
        for word in (off, 0xffffffff, 0xffffffff, 0xffffffff, 0xffffffff, 1):
            h = (h ^ word) * 1099511628211 & mask
        if v is None:
            return h
        h = (h ^ int(np.float64(v).view(np.uint64))) * 1099511628211 & mask
        h ^= h >> 29


@pytest.mark.parametrize("R", [1, 2, 3])
def test_different_lists_of_equal_hash(R):
    """Two lists of the same hash: found out, and every slice gets its own."""
    a, g = (1.0, 2.0), np.random.default_rng(1)
    while True:
        b0 = float(g.uniform(-2, 2))
        bits = int(np.float64(a[1]).view(np.uint64)) ^ list_hash(a[:1]) ^ list_hash([b0])
        b1 = float(np.uint64(bits).view(np.float64))
        if 0.01 < abs(b1) < 100:
            break
    A = two_lists(a, (b0, b1))
    assert len(plan_sizes(A)) == len(plan_sizes(two_lists(a, (b0, 3.0)))) + 1   # built twice
    check(A, R)
    check(A, R, reorder="bfs")


def test_autotuned_choices_of_constant_and_general_values_are_kept_apart():
    """One pattern, one value per diagonal and then a value per entry: the second
    is timed on its own (candidates build schedules; a choice taken over builds
    nothing), and a general matrix of other values takes that choice over."""
    A, B, C = (w.stencil_3d27(23) for _ in range(3))
    B.val = np.random.default_rng(1).standard_normal(A.nnz)
    C.val = np.random.default_rng(2).standard_normal(A.nnz)
    x = torch.from_numpy(w.uniform_vectors(A.n, 1, 1)).cuda()
    built = []
    with allocations(lambda i, b: False) as sizes:
        for M in (A, B, C):
            P = mpk.Plan(M)
            before = len(sizes)
            P.autotune(x, 5, reps=1)
            built.append(len(sizes) - before)
            P.close()
    assert built[0] > 0 and built[1] > 0 and built[2] == 0


@pytest.mark.parametrize("n", [1024, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("R", [1, 2, 3, 16])
def test_small_matrices_around_the_limits_of_one_launch(n, R):
    """One value per diagonal, a value per row on one of them, and on all; lists
    of two groups and of three."""
    for offs in (OFFS, OFFS + [41, 60]):
        for vary in ((), (0,), tuple(offs)):
            A = banded(n, offs, n, vary=vary)
            x = w.uniform_vectors(n, R, 8)
            P = mpk.Plan(A, reorder="none")
            ref = oracle.powers(A, x, 4)
            xd = torch.from_numpy(x).cuda()
            assert np.array_equal(P.run(xd, 4).cpu().numpy().reshape(ref.shape), ref), (offs, vary)
            P.close()


def half_irregular(n, share, seed, const=False):
    """16 entries a row: shared offsets, but in a share of each 256 rows anywhere
    within +-2000; every row within 1..16 entries in a fifth of those."""
    g = np.random.default_rng(seed)
    offs = np.array([-1001, -1000, -999, -101, -100, -99, -2, -1, 0, 1, 2, 99, 100, 101, 1000, 1001])
    i = np.arange(n)
    away = (g.random((n + 255) // 256) < share)[i // 256]
    col = np.where(away[:, None], i[:, None] + g.integers(-2000, 2001, size=(n, 16)), i[:, None] + offs) % n
    col = np.sort(col, axis=1)
    keep = np.ones((n, 16), bool)
    for r in np.flatnonzero(away)[::640]:
        keep[r:r + 3, g.integers(0, 17):] = False
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(keep.sum(axis=1))
    val = np.full((n, 16), 0.05) if const else g.standard_normal((n, 16)) * 0.2
    return w.CSR(n, rp, col[keep].astype(np.int32), val[keep])


@pytest.mark.parametrize("n", [50001, 100003])
@pytest.mark.parametrize("share", [0.1, 0.45])
def test_slices_without_a_list_beside_others(n, share):
    """Both in one matrix, in both row orders, for every number of right-hand
    sides: the oracle's bits."""
    A = half_irregular(n, share, n)
    for R in range(1, 17):
        x = w.uniform_vectors(n, R, R)
        xd = torch.from_numpy(x).cuda()
        ref = oracle.powers(A, x, 2)
        for reorder in ("none", "bfs") if R in (1, 2, 3, 8) else ("none",):
            P = mpk.Plan(A, reorder=reorder)
            assert np.array_equal(P.run(xd, 2).cpu().numpy().reshape(ref.shape), ref), (R, reorder)
            P.close()


@pytest.mark.parametrize("n,R,limit", [(250000, 2, 1.15), (2000000, 1, 1.1)])
def test_runs_of_half_irregular_matrices_are_no_slower_than_the_sliced_layout(n, R, limit):
    """Against an explicitly tuned persistent run, which reads the sliced layout:
    measured at 0.7 and 1.0 of its time, 1.1 and 1.3 with slices read element by
    element."""
    P = mpk.Plan(half_irregular(n, 0.45, 7), reorder="none")
    x = torch.from_numpy(w.uniform_vectors(n, R, 6)).cuda()
    default, persistent = times_of_default_and_persistent_runs(P, x, 8)
    assert default < limit * persistent
    P.close()


def test_default_run_of_very_uneven_rows_is_no_slower_than_a_persistent_one():
    """Rows of 22 entries on average and some 500 at most, three right-hand sides:
    the persistent kernel, 1.29 of whose time a launch per power takes."""
    n, g = 300000, np.random.default_rng(3)
    cnt = np.clip(2 / (g.random(n) + 0.004), 1, 500).astype(np.int64)
    src = np.repeat(np.arange(n), cnt)
    dst = np.clip(src + (g.standard_normal(src.size) * 2000).astype(np.int64), 0, n - 1)
    key = np.unique(np.concatenate([src * n + dst, dst * n + src]))
    rp = np.zeros(n + 1, np.int32)
    rp[1:] = np.cumsum(np.bincount(key // n, minlength=n))
    P = mpk.Plan(w.CSR(n, rp, (key % n).astype(np.int32), g.standard_normal(key.size)), reorder="none")
    x = torch.from_numpy(w.uniform_vectors(n, 3, 6)).cuda()
    default, persistent = times_of_default_and_persistent_runs(P, x, 6)
    assert default < 1.12 * persistent
    P.close()


def test_vectors_for_more_right_hand_sides_that_memory_is_short_for():
    """One set for each count is made larger for the next by prepare; where that
    fails, the smaller one stays and is used."""
    A = w.stencil_3d27(101)
    limit = [None]
    with allocations(lambda i, b: limit[0] is not None and b > limit[0]) as sizes:
        P = mpk.Plan(A, order="plan")
        P.prepare([3], [1, 9])
        limit[0] = 9 * 24 * A.n
        P.prepare([3], [16])
        before = len(sizes)
        for R in (1, 9, 16):
            x = torch.from_numpy(w.uniform_vectors(A.n, R, 2)).cuda()
            Y = P.run(x, 3)
            P.sync()
            assert torch.equal(Y, P.run_baseline(x, 3)), R
            P.sync()
        assert len(sizes) == before
        P.close()
