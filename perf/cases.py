"""Workloads that the solver's speed is judged by.

``listed()`` names twelve solves as a user's program makes them through
``helm.Plan`` and ``helm.Batch``; ``draw(rng)`` gives further ones of the same
ranges.  A case is a dict of plain values:

  grid       node counts, "n1xn2" or "n1xn2xn3" (batches: several, comma separated)
  omega      wavenumber (batches: comma separated)
  spacing    "unit" (h_j = 1/(n_j - 1), the unit square / cube of the paper) or
             "uniform" (one mesh size 1/(max n - 1) on every axis: a channel)
  nrhs       right-hand sides per solve
  precision  "fp64" or "mixed" (complex64 storage + FP64 refinement)
  entry      "solve", "static" (the allocation-free call), "residual", "batch"
  check      FP64 residual check and refinement to 1e-10
  transform  "fft" or "dense"
"""

import math

import numpy as np
import torch

from paper_1809_03808_amd import helm, inputs

TWO_PI = 2.0 * math.pi


def _case(name, grid, omega, nrhs=1, precision="fp64", spacing="unit", entry="solve", check=True, transform="fft"):
    c = dict(grid=grid, omega=omega, nrhs=nrhs, precision=precision, spacing=spacing, entry=entry, check=check,
             transform=transform)
    if name is not None:
        c["name"] = name
    return c


def listed():
    batch = inputs.batched_2d_problems(count=8, seed=4000)
    return [
        # the smallest problem of the test suite: a call is launches and one wait
        _case("2d_128_fp64", "128x128", 80.0),
        # a serving loop that may not allocate: one plain solve, nothing read back
        _case("2d_257_static_plain", "257x257", inputs.omega_for_ppw(257, 12.0), entry="static", check=False),
        # a wave guide with ragged sides, several sources
        _case("2d_513x200_mixed_x4", "513x200", inputs.omega_for_ppw(513, 11.0), 4, "mixed", spacing="uniform"),
        # the largest 2D shape of the paper (2^k + 1 nodes, omega = 2 pi)
        _case("2d_2049_fp64", "2049x2049", TWO_PI),
        # the large 2D workload in both precisions
        _case("2d_4096_fp64", "4096x4096", inputs.omega_for_ppw(4096, 10.0)),
        _case("2d_4096_mixed", "4096x4096", inputs.omega_for_ppw(4096, 10.0), 1, "mixed"),
        # the matrix-core transform, which the tuner takes at this size
        _case("2d_257_dense_mixed_x4", "257x257", inputs.omega_for_ppw(257, 12.0), 4, "mixed", transform="dense"),
        # a small 3D box with odd sides
        _case("3d_61x75x90_fp64", "61x75x90", inputs.omega_for_ppw(90, 10.0), spacing="uniform"),
        # 2^k + 1 nodes in 3D, two sources
        _case("3d_129_mixed_x2", "129x129x129", inputs.omega_for_ppw(129, 10.0), 2, "mixed"),
        # the medium 3D workload
        _case("3d_256_fp64", "256x256x256", inputs.omega_for_ppw(256, 10.0)),
        # the largest 3D grid with several sources (four of the benchmark's sixteen: three states fit the card)
        _case("3d_512_mixed_x4", "512x512x512", inputs.omega_for_ppw(512, 10.0), 4, "mixed"),
        # uneven problems in one graph launch
        _case("2d_batch8_mixed_x4", ",".join("%dx%d" % p["grid"] for p in batch),
              ",".join(repr(p["omega"]) for p in batch), 4, "mixed", entry="batch"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    """A node count in [lo, hi]: a power of two, 2^k + 1 (the paper's), or any."""
    n = _log_uniform(rng, lo, hi)
    kind = rng.random()
    if kind < 0.3:
        n = 1 << int(round(math.log2(n)))
    elif kind < 0.6:
        n = (1 << int(round(math.log2(n)))) + 1
    return min(max(n, lo), hi)


def _uniform_omega(grid, ppw):
    return inputs.omega_for_ppw(max(grid), ppw)


def draw(rng):
    kind = rng.random()
    precision = "mixed" if rng.random() < 0.5 else "fp64"
    ppw = rng.uniform(8.0, 20.0)
    if kind < 0.42:  # 2D solves, square-ish to channels
        grid = (_side(rng, 65, 4096), _side(rng, 65, 4096))
        n = grid[0] * grid[1]
        nrhs = rng.choice([1, 1, 2, 4, 7]) if n < 1 << 22 else 1
        return _case(None, "%dx%d" % grid, _uniform_omega(grid, ppw), nrhs, precision, "uniform",
                     check=precision == "mixed" or rng.random() < 0.8)
    if kind < 0.78:  # 3D solves
        grid = tuple(_side(rng, 24, 384) for _ in range(3))
        n = grid[0] * grid[1] * grid[2]
        nrhs = rng.choice([1, 1, 2, 4, 7]) if n < 1 << 23 else 1
        return _case(None, "%dx%dx%d" % grid, _uniform_omega(grid, ppw), nrhs, precision, "uniform",
                     check=precision == "mixed" or rng.random() < 0.8)
    if kind < 0.85:  # dense transforms
        grid = (_side(rng, 65, 513), _side(rng, 65, 1025))
        return _case(None, "%dx%d" % grid, _uniform_omega(grid, ppw), rng.choice([1, 2, 4]), precision, "uniform",
                     transform="dense")
    if kind < 0.91:  # the allocation-free entry point
        grid = (_side(rng, 65, 513), _side(rng, 65, 513))
        return _case(None, "%dx%d" % grid, _uniform_omega(grid, ppw), rng.choice([1, 2]), precision, "uniform",
                     entry="static", check=precision == "mixed" or rng.random() < 0.5)
    if kind < 0.96:  # residuals of given fields
        grid = (_side(rng, 65, 2049), _side(rng, 65, 2049)) if rng.random() < 0.5 else \
            tuple(_side(rng, 24, 256) for _ in range(3))
        return _case(None, "x".join(str(n) for n in grid), _uniform_omega(grid, ppw), rng.choice([1, 2, 4]), "fp64",
                     "uniform", entry="residual")
    sides = [_side(rng, 129, 1025) for _ in range(rng.randint(3, 6))]
    return _case(None, ",".join("%dx%d" % (n, n) for n in sides),
                 ",".join(repr(inputs.omega_for_ppw(n, rng.uniform(8.0, 20.0))) for n in sides),
                 rng.choice([1, 2, 4]), "mixed", entry="batch")


def _problems(case):
    """[(grid, omega, h)] of a case (one entry unless it is a batch)."""
    grids = [tuple(int(n) for n in g.split("x")) for g in str(case["grid"]).split(",")]
    omegas = [float(w) for w in str(case["omega"]).split(",")]
    out = []
    for g, w in zip(grids, omegas):
        h = inputs.spacing(g) if case["spacing"] == "unit" else (1.0 / (max(g) - 1),) * len(g)
        out.append((g, w, h))
    return out


def _gaussian(shape, seed):
    """Complex Gaussian loads, so that every eigenmode is excited."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    out = torch.empty(shape, dtype=torch.complex128, device="cuda")
    torch.view_as_real(out).normal_(0.0, 1.0, generator=gen)
    return out


def _inputs(case, seed):
    fs = [_gaussian((case["nrhs"],) + g, 1000003 * seed + i) for i, (g, _, _) in enumerate(_problems(case))]
    us = None
    if case["entry"] == "residual":
        us = [_gaussian((case["nrhs"],) + g, 1000003 * seed + 500 + i) for i, (g, _, _) in enumerate(_problems(case))]
    return fs, us


def prepare(case, seed):
    prec = helm.PREC_MIXED if case["precision"] == "mixed" else helm.PREC_FP64
    tf = helm.TRANSFORM_DENSE if case["transform"] == "dense" else helm.TRANSFORM_FFT
    plans = [helm.Plan(g, h, w, precision=prec, check=case["check"], transform=tf) for g, w, h in _problems(case)]
    fs, us = _inputs(case, seed)
    state = {"entry": case["entry"], "plans": plans, "f": fs}
    state["u"] = us if us is not None else [torch.empty_like(f) for f in fs]
    if case["entry"] == "batch":
        state["batch"] = helm.Batch(plans, max_nrhs=case["nrhs"])
    if case["entry"] == "residual":
        state["r"] = torch.empty_like(fs[0])
    return state


def run(state):
    entry = state["entry"]
    if entry == "batch":
        state["batch"].solve(state["f"], state["u"])
        return list(state["u"])
    plan, f, u = state["plans"][0], state["f"][0], state["u"][0]
    if entry == "residual":
        rel = plan.residual(u, f, state["r"])
        return [state["r"], rel]
    if entry == "static":
        plan.solve_static(f, u)
    else:
        plan.solve(f, u)
    return [u]


def work(case):
    """f (and u for a residual) read once, the result written once; flops of
    the transforms along the periodised axes (5 n log2 n each way) and of one
    tridiagonal solve per line (about 30 per unknown), or of the stencil."""
    b = fl = 0.0
    for g, _, _ in _problems(case):
        n = float(np.prod([float(x) for x in g])) * case["nrhs"]
        if case["entry"] == "residual":
            b += 48.0 * n
            fl += (2.0 * 3 ** len(g)) * 4 * n
        else:
            b += 32.0 * n
            fl += n * (30.0 + sum(10.0 * math.log2(x) for x in g[:-1]))
    return {"bytes": b, "flops": fl}


# ---------------------------------------------------------------------------
# 64-bit reference values: separation of variables with dense eigenvectors of
# all axes but one (the longest), Thomas along that one, iterative refinement
# ---------------------------------------------------------------------------

def _pencil(n, h, omega):
    """(K, M) of one axis with absorbing faces, linear elements."""
    K = np.zeros((n, n), dtype=np.complex128)
    M = np.zeros((n, n))
    i = np.arange(n)
    K[i, i] = 2.0 / h
    M[i, i] = 4.0 * h / 6.0
    K[0, 0] = K[-1, -1] = 1.0 / h - 1j * omega
    M[0, 0] = M[-1, -1] = 2.0 * h / 6.0
    K[i[:-1], i[1:]] = K[i[1:], i[:-1]] = -1.0 / h
    M[i[:-1], i[1:]] = M[i[1:], i[:-1]] = h / 6.0
    return K, M


def _tri(A, x, axis):
    """Tridiagonal (dense-stored, numpy) matrix times x along an axis."""
    n = A.shape[0]
    shape = [1] * x.dim()
    d = torch.from_numpy(np.ascontiguousarray(np.diag(A).astype(np.complex128))).to(x.device)
    shape[axis] = n
    y = x * d.view(shape)
    off = complex(A[0, 1])
    y.narrow(axis, 0, n - 1).add_(x.narrow(axis, 1, n - 1), alpha=off)
    y.narrow(axis, 1, n - 1).add_(x.narrow(axis, 0, n - 1), alpha=off)
    return y


def _apply(pencils, omega, u):
    """A u: -omega^2 M(x)..(x)M + sum_j M(x)..K_j..(x)M over trailing axes."""
    d = len(pencils)
    out = None
    for j in range(-1, d):
        t = u
        for a in range(d):
            K, M = pencils[a]
            t = _tri(K if a == j else M, t, t.dim() - d + a)
        if j < 0:
            t = t * (-omega * omega)
        out = t if out is None else out + t
    return out


def _sov(grid, h, omega, f):
    d = len(grid)
    line = int(np.argmax(grid))  # Thomas along the longest axis
    pencils = [_pencil(grid[a], h[a], omega) for a in range(d)]
    vecs, lam = {}, {}
    for a in range(d):
        if a == line:
            continue
        K, M = pencils[a]
        w, V = np.linalg.eig(np.linalg.solve(M.astype(np.complex128), K))
        V = V / np.sqrt(np.sum(V * (M @ V), axis=0))  # V^T M V = I
        vecs[a] = torch.from_numpy(V).to(f.device)
        lam[a] = torch.from_numpy(w).to(f.device)
    K, M = pencils[line]
    n = grid[line]

    def along(V, x, axis):  # V x along an axis
        y = x.movedim(axis, 0)
        s = y.shape
        return (V @ y.reshape(s[0], -1)).reshape(s).movedim(0, axis)

    def solve(r):
        x = r
        for a in vecs:
            x = along(vecs[a].T.contiguous(), x, 1 + a)
        x = x.movedim(1 + line, 0).contiguous()  # [n][nrhs][other axes]
        sig = torch.full((1,) * (x.dim() - 1), -omega * omega, dtype=torch.complex128, device=f.device)
        for i, a in enumerate(sorted(vecs)):
            shape = [1] * (x.dim() - 1)
            shape[1 + i] = grid[a]
            sig = sig + lam[a].view(shape)
        e = sig * M[0, 1] + complex(K[0, 1])
        piv = [None] * n
        for i in range(n):
            p = sig * M[i, i] + complex(K[i, i])
            if i:
                m = e / piv[i - 1]
                p = p - m * e
                x[i] -= m * x[i - 1]
            piv[i] = p
        x[n - 1] /= piv[n - 1]
        for i in range(n - 2, -1, -1):
            x[i] = (x[i] - e * x[i + 1]) / piv[i]
        x = x.movedim(0, 1 + line)
        for a in vecs:
            x = along(vecs[a], x, 1 + a)
        return x

    u = solve(f)
    for _ in range(2):
        u = u + solve(f - _apply(pencils, omega, u))
    return u


def exact(case, seed):
    if case["entry"] == "batch":
        return None  # the same solves as single ones, and long eigenproblems
    (grid, omega, h), = _problems(case)
    total = float(np.prod([float(n) for n in grid])) * case["nrhs"]
    if sorted(grid)[-2] > 700 or total > 3e7:
        return None  # the dense eigenproblems or the sweeps would take too long
    fs, us = _inputs(case, seed)
    f = fs[0]
    if case["entry"] == "residual":
        pencils = [_pencil(grid[a], h[a], omega) for a in range(len(grid))]
        r = f - _apply(pencils, omega, us[0])
        nr = torch.linalg.vector_norm(r.reshape(case["nrhs"], -1), dim=1)
        nf = torch.linalg.vector_norm(f.reshape(case["nrhs"], -1), dim=1)
        return [r, (nr / nf).cpu().numpy()]
    return [_sov(grid, h, omega, f)]
