"""The work that users of this library have it do, as timed cases.

Every case is a call (or the short sequence of calls a time step makes) on the
public binding: solves of one right-hand side with the FP64 or the FP32
V-cycle, batches of right-hand sides, a coefficient update, a whole setup, the
paper's preconditioner, and a stream of requests to the server.  The operators
are those of this repository's benchmark and tests, generated here on the GPU:

* ``lap7``: the 7-point Laplacian on an n^3 grid (homogeneous Dirichlet);
* ``varcoef7``: -div(k grad p) on an n^3 grid with a log-normal coefficient
  per cell, drawn from the seed;
* ``q1``: the trilinear finite-element Laplacian on n^3 elements stretched
  vertically by 1.05 (27-point rows, Dirichlet top, one pinned node), with the
  discrete divergence of a smooth random velocity field (64 Fourier modes) as
  right-hand side.
"""
from __future__ import annotations

import math
import time
from types import SimpleNamespace

import numpy as np
import torch

import paper_2210_16660_amd as pamg

TOL = 1e-6
STRETCH = 1.05
EXACT_MAX_ROWS = 600_000      # larger systems take a plain CG too long

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # the smallest whole solve: ten levels, launch latency
        dict(name="lap7_32_f64", kind="solve", op="lap7", n=32, precision="f64", krylov="fcg"),
        # a serving-sized operator (n odd) with the FP32 cycle under plain PCG
        dict(name="varcoef7_75_f32", kind="solve", op="varcoef7", n=75, precision="f32", krylov="cg"),
        # aggregates of up to four, ragged size
        dict(name="q1_95_f64_agg2", kind="solve", op="q1", n=95, precision="f64", krylov="fcg", agg_steps=2),
        # the benchmark's operator at its two sizes, and the FP32 cycle between them
        dict(name="q1_128_f64", kind="solve", op="q1", n=128, precision="f64", krylov="fcg"),
        dict(name="q1_161_f32", kind="solve", op="q1", n=161, precision="f32", krylov="fcg"),
        dict(name="q1_256_f64", kind="solve", op="q1", n=256, precision="f64", krylov="fcg"),
        # sixteen consecutive time steps' right-hand sides at once
        dict(name="batch16_q1_128_f32", kind="batch", op="q1", n=128, precision="f32", nrhs=16),
        # a few right-hand sides on a mid-sized operator
        dict(name="batch5_varcoef7_61_f64", kind="batch", op="varcoef7", n=61, precision="f64", nrhs=5),
        # a time step with new coefficients: hierarchy update, then the solve
        dict(name="update_varcoef7_83_f64", kind="update", op="varcoef7", n=83, precision="f64"),
        # a new operator: setup and its first solve
        dict(name="setup_q1_64_f64", kind="setup", op="q1", n=64, precision="f64"),
        # the paper's preconditioner: smoothed prolongators over aggregates of
        # up to eight, four hybrid Gauss-Seidel sweeps on each side
        dict(name="paper_q1_56_f64", kind="paper", op="q1", n=56, precision="f64"),
        # requests on several cached operators, answered by the server
        dict(name="serve_varcoef7_24_70", kind="serve", op="varcoef7", n=24, n_max=70, operators=5, requests=40),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "batch", "update", "setup", "paper", "serve"])
    op = rng.choice(["q1", "varcoef7", "lap7"])
    precision = rng.choice(["f64", "f32"])
    if kind == "solve":
        n = _log_size(rng, 24, 170 if op == "q1" else 200)
        c = dict(kind=kind, op=op, n=n, precision=precision, krylov=rng.choice(["fcg", "fcg", "cg"]))
        if op == "q1" and rng.random() < 0.3:
            c["agg_steps"] = rng.choice([2, 3])
        return c
    if kind == "batch":
        return dict(kind=kind, op=op, n=_log_size(rng, 24, 110), precision=precision, nrhs=rng.randint(2, 16))
    if kind == "update":
        return dict(kind=kind, op="varcoef7", n=_log_size(rng, 24, 130), precision=precision)
    if kind == "setup":
        return dict(kind=kind, op=op, n=_log_size(rng, 24, 96), precision=precision)
    if kind == "paper":
        return dict(kind=kind, op="q1", n=_log_size(rng, 24, 64), precision=precision)
    n = rng.randint(24, 40)
    return dict(kind=kind, op="varcoef7", n=n, n_max=rng.randint(n + 8, 96), operators=rng.randint(2, 6),
                requests=rng.randint(8, 48))


# ------------------------------------------------------------------ operators


def _csr(vals, cols, mask):
    """Host CSR from (rows, candidates) tables on the GPU, columns ascending."""
    rp = torch.zeros(mask.shape[0] + 1, dtype=torch.int64, device=mask.device)
    torch.cumsum(mask.sum(1), 0, out=rp[1:])
    return SimpleNamespace(n=int(mask.shape[0]), row_ptr=rp.to(torch.int32).cpu().numpy(),
                           col=cols[mask].cpu().numpy(), val=vals[mask].cpu().numpy())


def _couplings(n, seed):
    """Edge couplings (x, y, z) of the 7-point operator; seed None: constant coefficient."""
    s = float((n + 1) ** 2)
    if seed is None:
        one = [torch.full(sh, s, dtype=torch.float64, device="cuda")
               for sh in ((n, n, n + 1), (n, n + 1, n), (n + 1, n, n))]
        return one
    g = torch.Generator(device="cuda").manual_seed(seed)
    k = torch.exp(torch.randn((n + 1,) * 3, generator=g, dtype=torch.float64, device="cuda"))   # [z, y, x] cells
    cx = ((k[:-1, :-1, :] + k[:-1, 1:, :]) + (k[1:, :-1, :] + k[1:, 1:, :])) * 0.25 * s
    cy = ((k[:-1, :, :-1] + k[:-1, :, 1:]) + (k[1:, :, :-1] + k[1:, :, 1:])) * 0.25 * s
    cz = ((k[:, :-1, :-1] + k[:, :-1, 1:]) + (k[:, 1:, :-1] + k[:, 1:, 1:])) * 0.25 * s
    return [cx, cy, cz]


def _seven_point(n, seed):
    cx, cy, cz = _couplings(n, seed)
    west, east = cx[:, :, :-1], cx[:, :, 1:]
    south, north = cy[:, :-1], cy[:, 1:]
    down, up = cz[:-1], cz[1:]
    diag = ((west + east) + (south + north)) + (down + up)
    vals = torch.stack([-down, -south, -west, diag, -east, -north, -up], -1).reshape(-1, 7)
    i = torch.arange(n, device="cuda")
    z, y, x = torch.meshgrid(i, i, i, indexing="ij")
    inside = torch.stack([z > 0, y > 0, x > 0, x >= 0, x < n - 1, y < n - 1, z < n - 1], -1).reshape(-1, 7)
    off = torch.tensor([-n * n, -n, -1, 0, 1, n, n * n], dtype=torch.int32, device="cuda")
    cols = torch.arange(n ** 3, dtype=torch.int32, device="cuda")[:, None] + off
    return _csr(vals, cols, inside)


def _heights(n, stretched):
    if not stretched:
        return torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    k = torch.arange(n + 1, dtype=torch.float64, device="cuda")
    z = (STRETCH ** k - 1.0) / (STRETCH ** n - 1.0)
    return z[1:] - z[:-1]


def _line_matrices(h):
    """Mass, stiffness and convection rows (offsets -1, 0, 1) of linear elements of lengths h."""
    m, k, c = (torch.zeros(h.numel() + 1, 3, dtype=torch.float64, device="cuda") for _ in range(3))
    m[:-1, 1] += h / 3
    m[1:, 1] += h / 3
    m[:-1, 2] = m[1:, 0] = h / 6
    k[:-1, 1] += 1 / h
    k[1:, 1] += 1 / h
    k[:-1, 2] = k[1:, 0] = -1 / h
    c[0, 1], c[-1, 1] = -0.5, 0.5
    c[:-1, 2], c[1:, 0] = 0.5, -0.5
    return m, k, c


def _q1(n):
    p = n + 1
    m, k, _ = _line_matrices(_heights(n, False))
    mz, kz, _ = _line_matrices(_heights(n, True))
    mz, kz = mz[:n], kz[:n]                                    # the top layer is eliminated

    def product(z, y, x):
        return (z[:, None, None, :, None, None] * y[None, :, None, None, :, None]) * x[None, None, :, None, None, :]

    vals = product(mz, m, k)
    vals += product(mz, k, m)
    vals += product(kz, m, m)
    vals = vals.reshape(-1, 27)
    d = torch.arange(-1, 2, device="cuda", dtype=torch.int32)
    off = (d[:, None, None] * (p * p) + d[None, :, None] * p + d[None, None, :]).reshape(27)
    cols = torch.arange(p * p * n, device="cuda", dtype=torch.int32)[:, None] + (off - 1)
    i = torch.arange(p, device="cuda")
    line = torch.stack([i > 0, i >= 0, i < n], 1)
    deep = torch.stack([i[:n] > 0, i[:n] >= 0, i[:n] < n - 1], 1)
    mask = (deep[:, None, None, :, None, None] & line[None, :, None, None, :, None] & line[None, None, :, None, None, :])
    mask = mask.reshape(-1, 27) & (cols >= 0)                  # node 0 is pinned
    return _csr(vals[1:], cols[1:], mask[1:])


def _operator(case, seed, n=None):
    n = n or case["n"]
    if case["op"] == "q1":
        return _q1(n)
    return _seven_point(n, None if case["op"] == "lap7" else seed)


# ------------------------------------------------------------------ right-hand sides


def _divergence(n, seed):
    """Discrete divergence of a random smooth velocity field on the stretched mesh."""
    rng = np.random.default_rng(seed)
    wave = []
    while len(wave) < 64:
        c = rng.integers(-8, 9, 3)
        if 0 < int((c * c).sum()) <= 64:
            wave.append(c)
    wave = torch.tensor(np.array(wave), dtype=torch.float64, device="cuda")
    amp = torch.tensor(rng.uniform(-1, 1, (3, 64)), device="cuda")
    phase = torch.tensor(rng.uniform(0, 2 * np.pi, 64), device="cuda")
    h, hz = _heights(n, False), _heights(n, True)
    x = torch.arange(n + 1, dtype=torch.float64, device="cuda") / n
    z = torch.cat([torch.zeros(1, dtype=torch.float64, device="cuda"), torch.cumsum(hz, 0)])
    m, _, c = _line_matrices(h)
    mz, _, cz = _line_matrices(hz)

    def line(rows, angle):
        """A tridiagonal matrix times (cos, sin) of every mode, as a complex array."""
        e = torch.polar(torch.ones_like(angle), angle)
        y = rows[:, 1:2] * e
        y[1:] += rows[1:, 0:1] * e[:-1]
        y[:-1] += rows[:-1, 2:3] * e[1:]
        return y

    ax, ay = 2 * np.pi * x[:, None] * wave[:, 0], 2 * np.pi * x[:, None] * wave[:, 1]
    az = 2 * np.pi * z[:, None] * wave[:, 2] + phase
    parts = []
    for comp in range(3):
        fx = line(c if comp == 0 else m, ax)
        fy = line(c if comp == 1 else m, ay)
        fz = line(cz if comp == 2 else mz, az)[:n] * amp[comp]
        parts.append((torch.einsum("zm,ym->zym", fz, fy).reshape(-1, 64), fx))
    zy = torch.cat([p[0] for p in parts], 1)
    xs = torch.cat([p[1] for p in parts], 1)
    b = zy.real @ xs.imag.t().contiguous() + zy.imag @ xs.real.t().contiguous()
    return b.reshape(-1)[1:].contiguous()


def _rhs(case, rows, seed, count, n=None):
    """(count, rows): successive time steps (5 % changes) on the finite-element
    operator, independent uniform fields on the others."""
    if case["op"] != "q1":
        g = torch.Generator(device="cuda").manual_seed(seed + 1)
        return torch.rand((count, rows), generator=g, dtype=torch.float64, device="cuda") * 2 - 1
    out = [_divergence(case["n"], seed)]
    for t in range(1, count):
        d = _divergence(case["n"], seed + 7919 * t)
        out.append(out[-1] + d * (0.05 * out[0].norm() / d.norm()))
    return torch.stack(out)


# ------------------------------------------------------------------ prepare and run


def _options(case):
    if case["kind"] == "paper":
        return dict(agg_steps=3, smooth_prolongator=1, smoother="hgs")
    return dict(agg_steps=case.get("agg_steps", 1))


def _serve_sizes(case):
    k = case["operators"]
    return [round(case["n"] * (case["n_max"] / case["n"]) ** (i / max(1, k - 1))) for i in range(k)]


def prepare(case, seed):
    f32 = int(case.get("precision") == "f32")
    if case["kind"] == "serve":
        server = pamg.Server(hbm_budget_bytes=16 << 30, setup_workers=4)
        ops = [_operator(case, seed * 64 + i, n) for i, n in enumerate(_serve_sizes(case))]
        reqs = []
        for j in range(case["requests"]):
            key = (j * 7 + j // len(ops)) % len(ops)
            b = _rhs(case, ops[key].n, seed * 4096 + j, 1)[0]
            reqs.append((key, ops[key], b, torch.empty_like(b)))
        state = dict(kind="serve", server=server, requests=reqs)
        run(state)                                   # the operators are cached from here on
        return state
    A = _operator(case, seed)
    if case["kind"] == "setup":
        b = _rhs(case, A.n, seed, 1)[0]
        return dict(kind="setup", A=A, f32=f32, b=b, precision=case["precision"])
    H = pamg.Hierarchy(A, build_f32=f32, **_options(case))
    count = case.get("nrhs", 1)
    B = _rhs(case, A.n, seed, count)
    state = dict(kind=case["kind"], H=H, precision=case["precision"], krylov=case.get("krylov", "fcg"))
    if case["kind"] == "batch":
        H.batch_config(pamg.PREC_F32 if f32 else pamg.PREC_F64)      # the engine and its tuning are kept
        state.update(B=B, X=torch.empty_like(B))
    else:
        state.update(b=B[0].contiguous(), x=torch.empty_like(B[0]))
    if case["kind"] == "update":
        # a program between time steps has updated before: the plans exist
        H.update_values(torch.from_numpy(_operator(case, seed + 1).val).cuda())
        state["values"] = torch.from_numpy(_operator(case, seed + 2).val).cuda()
    return state


def run(state):
    kind = state["kind"]
    if kind == "serve":
        server, reqs = state["server"], state["requests"]
        for tag, (key, A, b, x) in enumerate(reqs):
            server.submit(key, A, b, x, tol=TOL, tag=tag)
        left = len(reqs)
        while left:
            done = server.poll()
            for c in done:
                if c.status != pamg.OK:
                    raise RuntimeError(f"request {c.tag}: status {c.status}")
            left -= len(done)
            if left:
                time.sleep(5e-5)
        return [x for _, _, _, x in reqs]
    if kind == "setup":
        H = pamg.Hierarchy(state["A"], build_f32=state["f32"])
        x = torch.empty_like(state["b"])
        H.solve(state["b"], x, tol=TOL, precision=state["precision"])
        sizes = H.level_sizes()
        H.close()
        return {"x": x, "rows": np.array(sizes[0]), "entries": np.array(sizes[1])}
    H = state["H"]
    if kind == "batch":
        H.solve_batch(state["B"], state["X"], tol=TOL, precision=state["precision"])
        return {"X": state["X"]}
    if kind == "update":
        H.update_values(state["values"])
    H.solve(state["b"], state["x"], tol=TOL, precision=state["precision"], krylov=state["krylov"])
    return {"x": state["x"]}


# ------------------------------------------------------------------ work and exact values


def _counts(op, n):
    if op == "q1":
        p = n + 1
        line = 3 * p - 2
        return p * p * n - 1, line * line * (3 * n - 2) - 8 - 7
    return n ** 3, 7 * n ** 3 - 6 * n * n


def work(case):
    """The operator's entries (value and column) read once, the right-hand
    sides read once and the solutions written once; a multiply and an add per
    entry and right-hand side."""
    if case["kind"] == "serve":
        sizes = _serve_sizes(case)
        per = [_counts(case["op"], n) for n in sizes]
        share = case["requests"] / len(per)
        return {"bytes": float(sum(12 * nnz + 16 * rows * share for rows, nnz in per)),
                "flops": float(sum(2 * nnz * share for _, nnz in per))}
    rows, nnz = _counts(case["op"], case["n"])
    count = case.get("nrhs", 1)
    return {"bytes": float(12 * nnz + 16 * rows * count), "flops": float(2 * nnz * count)}


def _plain_cg(A, B):
    """A x = b in FP64 by Jacobi-preconditioned conjugate gradients, to the rounding level."""
    a = torch.sparse_csr_tensor(torch.from_numpy(A.row_ptr).cuda().long(), torch.from_numpy(A.col).cuda().long(),
                                torch.from_numpy(A.val).cuda(), size=(A.n, A.n))
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    dinv = torch.from_numpy(1.0 / A.val[rows == A.col]).cuda()
    out = []
    for b in B:
        x, r = torch.zeros_like(b), b.clone()
        z = dinv * r
        p, rz, stop = z.clone(), r @ z, 1e-13 * float(b.norm())
        for it in range(20000):
            q = (a @ p[:, None])[:, 0]
            alpha = rz / (p @ q)
            x += alpha * p
            r -= alpha * q
            if it % 50 == 49 and float(r.norm()) <= stop:
                break
            z = dinv * r
            new = r @ z
            p = z + (new / rz) * p
            rz = new
        out.append(x)
    return torch.stack(out)


def exact(case, seed):
    if case["kind"] == "serve":
        return None                                  # many systems of one kind: the batch cases say it
    rows, _ = _counts(case["op"], case["n"])
    count = case.get("nrhs", 1)
    if rows * count > EXACT_MAX_ROWS * 2 or rows > EXACT_MAX_ROWS:
        return None
    A = _operator(case, seed + 2 if case["kind"] == "update" else seed)
    X = _plain_cg(A, _rhs(case, A.n, seed, count))
    if case["kind"] == "batch":
        return {"X": X}
    if case["kind"] == "setup":
        return {"x": X[0], "rows": None, "entries": None}
    return {"x": X[0]}
