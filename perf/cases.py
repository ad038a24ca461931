"""The workloads whose speed this repository is judged by.

Each case is one call (or the few calls) that a program using the matrix
power kernel makes again and again on a plan it keeps: the powers
y_k = A^k x, the three-term recurrence, one Chebyshev time step, the
p x SpMV form, a captured graph, and the conversion between row numberings.
The matrices are those of the repository's benchmark and serving pool (2D
5-point, 3D 27-point, Anderson lattices, random bands), plus the 27-point
pattern with a coefficient of its own at every entry, as a discretised
operator with varying material has it.

A case holds:

    matrix   lap2d | stencil27 | varcoef27 | anderson | banded
    size     side of the lattice, or rows of the band
    p, R     powers and right-hand sides
    bits     64 or 32: stored value width (vectors are always doubles)
    form     powers | recur | step | baseline | graph | permuted
    reorder  bfs | none: the plan's row order
    tuned    whether the program ran the autotuner on its plan
"""
import math
import types

import torch

import paper_2405_12525_amd as mpk

# One time step of length dt needs somewhat more than dt powers.
STEP_DT = {16: 1.0, 32: 10.0, 64: 30.0}


def _case(name, matrix, size, p, R=1, bits=64, form="powers", reorder="none", tuned=False):
    return dict(name=name, matrix=matrix, size=size, p=p, R=R, bits=bits, form=form,
                reorder=reorder, tuned=tuned)


def listed():
    return [
        # the smallest call: a 64^2 Laplacian on a plan with every default
        _case("lap2d_64_p4", "lap2d", 64, 4, reorder="bfs"),
        # a small serving request; the server runs p x SpMV wherever blocking
        # is not clearly faster
        _case("lap2d_100_p16_r4_baseline", "lap2d", 100, 16, 4, form="baseline", reorder="bfs"),
        # a small lattice stepped in a loop, replayed from a captured graph
        _case("anderson_50_p12_graph", "anderson", 50, 12, form="graph"),
        # a mid-size plane, two vectors, float values, default plan
        _case("lap2d_1000_p10_r2_fp32", "lap2d", 1000, 10, 2, 32, reorder="bfs"),
        # general coefficients, odd row count and right-hand sides, default plan
        _case("varcoef27_101_p7_r3", "varcoef27", 101, 7, 3, reorder="bfs"),
        # a block of 16 vectors on a mid-size cube
        _case("stencil27_64_p16_r16", "stencil27", 64, 16, 16, tuned=True),
        # the benchmark's headline workload
        _case("stencil27_128_p8", "stencil27", 128, 8, tuned=True),
        # the same pattern with general coefficients
        _case("varcoef27_128_p8", "varcoef27", 128, 8, tuned=True),
        # the benchmark's irregular matrix
        _case("banded_4m_p6", "banded", 1 << 22, 6, reorder="bfs", tuned=True),
        # the benchmark's Chebyshev recurrence on 8 vectors, float values
        _case("anderson_160_cheb16_r8_fp32", "anderson", 160, 16, 8, 32, form="recur", tuned=True),
        # a long time step of two complex states
        _case("anderson_96_step64_r4", "anderson", 96, 64, 4, form="step", tuned=True),
        # a program that works in the plan's numbering and converts in and out
        _case("stencil27_96_p8_permuted", "stencil27", 96, 8, form="permuted", reorder="bfs"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# most entries per row, to bound a drawn case's cost
_WIDTH = {"lap2d": 5, "stencil27": 27, "varcoef27": 27, "anderson": 7, "banded": 16}


def _rows(case):
    s = case["size"]
    return {"lap2d": s * s, "banded": s}.get(case["matrix"], s ** 3)


def _cost(case):
    """Bytes that p separate products move."""
    n, R = _rows(case), case["R"]
    return case["p"] * (n * _WIDTH[case["matrix"]] * (4 + case["bits"] // 8) + 16 * n * R)


def draw(rng):
    top = max(_cost(c) for c in listed())
    while True:
        matrix = rng.choice(["lap2d", "stencil27", "varcoef27", "anderson", "banded"])
        size = {"lap2d": lambda: _log_int(rng, 32, 1400), "banded": lambda: _log_int(rng, 8192, 1 << 22),
                "anderson": lambda: _log_int(rng, 12, 160)}.get(matrix, lambda: _log_int(rng, 12, 128))()
        form = rng.choice(["powers"] * 5 + ["recur"] * 2 + ["baseline"] * 2 + ["step", "graph", "permuted"])
        p, R = rng.randint(2, 32), rng.choice([1, 1, 1, 2, 3, 4, 5, 6, 8, 12, 16])
        if form == "step":  # real and imaginary columns; a spectrum inside [-1, 1]
            matrix, size = "anderson", _log_int(rng, 12, 128)
            p, R = rng.choice(sorted(STEP_DT)), rng.choice([2, 4, 6, 8])
        c = _case("", matrix, size, p, R, rng.choice([64, 64, 32]), form, rng.choice(["bfs", "none"]),
                  rng.random() < 0.4)
        del c["name"]
        if form == "permuted":
            c["reorder"] = "bfs"
        if _cost(c) <= top and p * _rows(c) * R * 8 <= 4.5e9:
            return c


# ---------------------------------------------------------------- inputs

def _generator(seed, salt):
    return torch.Generator(device="cuda").manual_seed(seed * 7 + salt)


def _csr(cols, vals, mask):
    n = cols.shape[0]
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = mask.sum(dim=1).cumsum(0)
    return types.SimpleNamespace(n=n, rowptr=rowptr.int(), col=cols[mask].int(), val=vals[mask])


def _lattice(dims, offsets, periodic, vals):
    """Rows i = x + Lx*(y + Ly*z), columns ascending in each row; vals: (n, k)
    in the order of the offsets."""
    Lx, Ly, Lz = dims
    n = Lx * Ly * Lz
    i = torch.arange(n, device="cuda")
    x, y, z = i % Lx, (i // Lx) % Ly, i // (Lx * Ly)
    cols = torch.empty((n, len(offsets)), dtype=torch.int32, device="cuda")
    mask = torch.ones((n, len(offsets)), dtype=torch.bool, device="cuda")
    for j, (dx, dy, dz) in enumerate(offsets):
        a, b, c = x + dx, y + dy, z + dz
        if periodic:
            a, b, c = a % Lx, b % Ly, c % Lz
        else:
            mask[:, j] = (a >= 0) & (a < Lx) & (b >= 0) & (b < Ly) & (c >= 0) & (c < Lz)
        cols[:, j] = (a + Lx * (b + Ly * c)).int()
    if periodic:  # wrapped neighbours are out of order at the faces
        cols, at = cols.sort(dim=1)
        vals = vals.gather(1, at)
    return _csr(cols, vals, mask)


def _matrix(case, seed):
    kind, L = case["matrix"], case["size"]
    f64 = dict(dtype=torch.float64, device="cuda")
    if kind == "lap2d":
        offs = [(0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0)]
        return _lattice((L, L, 1), offs, False, torch.tensor([-1., -1., 4., -1., -1.], **f64).expand(L * L, 5))
    if kind in ("stencil27", "varcoef27"):
        offs = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
        if kind == "stencil27":
            w = torch.full((27,), -1.0, **f64)
            w[13] = 26.0
            vals = w.expand(L ** 3, 27)
        else:
            vals = torch.rand((L ** 3, 27), generator=_generator(seed, 1), **f64) * 2 - 1
        return _lattice((L, L, L), offs, False, vals)
    if kind == "anderson":  # hopping -1, on-site energies in [-8.25, 8.25], scaled into [-1, 1]
        offs = [(0, 0, -1), (0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
        vals = torch.full((L ** 3, 7), -1.0 / 14.25, **f64)
        vals[:, 3] = (torch.rand(L ** 3, generator=_generator(seed, 2), **f64) * 2 - 1) * (8.25 / 14.25)
        return _lattice((L, L, L), offs, True, vals)
    # random band: about 15 neighbours within 5000 rows, mirrored, rows
    # shuffled within windows of 65536
    n, g = L, _generator(seed, 3)
    cnt = torch.poisson(torch.full((n,), 7.5, device="cuda"), generator=g).long()
    src = torch.repeat_interleave(torch.arange(n, device="cuda"), cnt)
    dst = src + torch.randint(1, 5001, src.shape, generator=g, device="cuda")
    src, dst = src[dst < n], dst[dst < n]
    i = torch.arange(n, device="cuda")
    new = torch.argsort(torch.argsort((i // 65536) + torch.rand(n, generator=g, **f64)))
    src, dst = new[src], new[dst]
    key = torch.unique(torch.cat([src * n + dst, dst * n + src, i * n + i]))
    row = key // n
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.bincount(row, minlength=n).cumsum(0)
    val = torch.randn(key.numel(), generator=g, **f64)
    return types.SimpleNamespace(n=n, rowptr=rowptr.int(), col=(key - row * n).int(), val=val)


def _vectors(case, seed, n):
    """Uniform block vectors, or normalised random states for a time step."""
    x = torch.rand((n, case["R"]), generator=_generator(seed, 4), dtype=torch.float64, device="cuda") * 2 - 1
    return x / x.norm(dim=0) if case["form"] == "step" else x


def prepare(case, seed):
    A = _matrix(case, seed)
    x = _vectors(case, seed, A.n)
    form, p, R = case["form"], case["p"], case["R"]
    plan = mpk.Plan(A, value_bits=case["bits"], reorder=case["reorder"],
                    order="plan" if form == "permuted" else "original")
    Y = torch.empty((p, A.n, R), dtype=torch.float64, device="cuda")
    if case["tuned"] and form != "baseline" and p >= 4:
        plan.autotune(x, p, Y=Y, recur={"recur": True, "step": 2}.get(form, False))
    s = dict(plan=plan, x=x, Y=Y, p=p, form=form)
    if form == "recur":
        s["coefs"] = mpk.chebyshev_coefficients(p)
    elif form == "step":
        del s["Y"], Y
        s["dt"], s["out"] = STEP_DT[p], torch.empty_like(x)
    elif form == "graph":
        s["graph"] = plan.capture(x, p, Y)
    elif form == "permuted":
        s["xp"], s["Yp"] = torch.empty_like(x), torch.empty_like(Y)
    return s


def run(s):
    plan, x, p, form = s["plan"], s["x"], s["p"], s["form"]
    if form == "powers":
        return plan.run(x, p, s["Y"])
    if form == "recur":
        return plan.run_recur(x, *s["coefs"], Y=s["Y"])
    if form == "baseline":
        return plan.run_baseline(x, p, s["Y"])
    if form == "graph":
        return s["graph"].launch()
    if form == "step":
        return plan.cheb_time_step(x, s["dt"], p, out=s["out"])
    plan.permute(x, to_plan=True, out=s["xp"])
    plan.run(s["xp"], p, s["Yp"])
    return plan.permute(s["Yp"], to_plan=False, out=s["Y"])


def _nnz(case):
    """Stored entries (the band: on average)."""
    L, n = case["size"], _rows(case)
    return {"lap2d": 5 * n - 4 * L, "stencil27": (3 * L - 2) ** 3, "varcoef27": (3 * L - 2) ** 3,
            "anderson": 7 * n, "banded": 16 * n}[case["matrix"]]


def work(case):
    """The matrix read once, the input read once, every result written once."""
    n, nnz, p, R = _rows(case), _nnz(case), case["p"], case["R"]
    vectors = 2 if case["form"] == "step" else p + 1
    flops = 2 * nnz * R * p + (2 * n * R * (p - 1) if case["form"] in ("recur", "step") else 0)
    return {"bytes": 4 * (n + 1) + (4 + case["bits"] // 8) * nnz + 8 * n * R * vectors, "flops": flops}


def exact(case, seed):
    A = _matrix(case, seed)
    x = _vectors(case, seed, A.n)
    row = torch.repeat_interleave(torch.arange(A.n, device="cuda", dtype=torch.int32), A.rowptr.long().diff())
    step = (1 << 25) // case["R"]

    def times(v):
        y = torch.zeros_like(v)
        for a in range(0, A.val.numel(), step):
            b = slice(a, a + step)
            y.index_add_(0, row[b], A.val[b, None] * v[A.col[b]])
        return y

    p = case["p"]
    if case["form"] == "step":  # exp(-i dt H) by Taylor steps of length at most 1
        parts = math.ceil(STEP_DT[p])
        h = STEP_DT[p] / parts
        for _ in range(parts):
            term, total = x, x.clone()
            for k in range(1, 22):
                t = times(term) * (h / k)  # -i (a + i b) = b - i a
                term = torch.stack([t[:, 1::2], -t[:, 0::2]], dim=2).reshape(t.shape)
                total += term
            x = total
        return x
    Y = [x]
    for k in range(p):
        y = times(Y[-1])
        if case["form"] == "recur" and k > 0:
            y = 2 * y - Y[-2]
        Y.append(y)
    return torch.stack(Y[1:])
