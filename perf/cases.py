"""Workloads of the solver as a simulator's program runs them.

A case is one repeated call sequence: new block values come in, the
preconditioner is refactored, one or more right-hand sides are solved (a
Newton step), or one of its parts alone.  Inputs are the synthetic grids of
the benchmark (3x3 FP64 blocks on a Cartesian grid, optional inactive cells
and non-neighbour connections), drawn on the device from the seed; a case's
pattern belongs to the case, as a grid does to a simulation, and the seed
draws the values.
"""

from __future__ import annotations

import numpy as np
import torch

import paper_2309_11488_amd as rs

ORDER = {"colour": rs.ORDER_GRAPH_COLOUR, "level": rs.ORDER_LEVEL_SET, "rcm": rs.ORDER_RCM_LEVEL_SET}
PREC = {"fp64": rs.PREC_FP64, "fp32": rs.PREC_FP32_FACTORS}
SERVE_GRIDS = ((25, 20, 20), (50, 50, 20), (100, 100, 20))


def _case(name, kind, nx, ny, nz, **over):
    c = dict(name=name, kind=kind, nx=nx, ny=ny, nz=nz, sigma=1.0, masked=False, order="colour", prec="fp64",
             batch=1, rhs=1, reduction=1e-2, wells=0, parts=0, queued=False)
    c.update(over)
    if not name:
        del c["name"]
    return c


def listed():
    return [
        # the smallest Newton step: a 4 000-cell sector model, bound by latency and launches
        _case("step_4k_colour", "step", 20, 20, 10),
        # the same call with the binding's default ordering (level sets) on a 10 000-cell grid
        _case("step_10k_level", "step", 25, 20, 20, order="level"),
        # NORNE-class grid (inactive cells, 2 % non-neighbour connections), the benchmark's c2:
        # one factorisation, ten right-hand sides
        _case("step_96k_colour", "step", 46, 112, 22, masked=True, rhs=10, queued=True),
        # the same grid under level scheduling (the paper's other ordering): thousands of thin levels
        _case("step_96k_level", "step", 46, 112, 22, masked=True, order="level"),
        # the same grid with the simulator's other Krylov solver, mixed precision
        _case("gmres_96k_colour", "gmres", 46, 112, 22, masked=True, prec="fp32"),
        # Block-Jacobi-ILU0 with 150 partitions under level scheduling, no non-neighbour connections
        _case("step_113k_jacobi", "step", 46, 112, 22, order="level", parts=150),
        # standard wells kept separate on a 50 000-cell grid
        _case("step_50k_wells", "step", 50, 50, 20, wells=3),
        # BigModel class, the benchmark's default workload, and the same with FP32-stored factors
        _case("step_1m_fp64", "step", 100, 100, 100, sigma=2.0, queued=True),
        _case("step_1m_fp32", "step", 100, 100, 100, sigma=2.0, prec="fp32", queued=True),
        # the benchmark's ensemble: 64 realisations of one grid in one call, mixed precision
        _case("ensemble_64x48k", "step", 40, 40, 30, prec="fp32", batch=64, queued=True),
        # a program with its own Krylov method: one preconditioner application and one product with A
        _case("apply_spmv_200k", "apply", 100, 100, 20),
        # a burst of requests of mixed sizes to the request server, mixed precision
        _case("serve_burst", "serve", 25, 20, 20, prec="fp32", rhs=24),
    ]


def draw(rng):
    """One more case of the same ranges: sizes over their logarithm (odd ones among them), each kind and option."""
    kind = rng.choice(["step", "step", "step", "step", "gmres", "apply", "serve"])
    order = rng.choice(["colour", "colour", "colour", "level", "rcm"])
    batch = 1
    if kind == "step" and order == "colour" and rng.random() < 0.3:
        batch = rng.randint(2, 48)
    most = 1_000_000 if order == "colour" else 90_000
    cells = int(round(4000 * (most / 4000) ** rng.random())) // batch + 1000
    cells = min(cells, 900_000)
    nx = max(3, int(cells ** (1 / 3) * rng.uniform(0.6, 1.6)))
    ny = max(3, int((cells / nx) ** 0.5 * rng.uniform(0.6, 1.6)))
    nz = max(3, int(cells / (nx * ny)))
    c = _case("", kind, nx, ny, nz, sigma=rng.choice([1.0, 2.0]), order=order, prec=rng.choice(["fp64", "fp32"]),
              batch=batch, masked=batch == 1 and rng.random() < 0.4, queued=rng.random() < 0.5)
    if kind == "serve":
        c.update(nx=25, ny=20, nz=20, rhs=rng.randint(8, 24), masked=False, order="colour", prec=rng.choice(["fp64", "fp32"]),
                 sigma=1.0 + 0.5 * rng.random())
    elif kind == "step" and batch == 1:
        c["rhs"] = rng.choice([1, 1, 2, 5])
        if rng.random() < 0.2:
            c["wells"] = rng.randint(1, 5)
        elif order == "level" and rng.random() < 0.4:
            c["parts"] = rng.randint(4, 150)
    return c


# ------------------------------------------------------------------ inputs

def _pattern(case, shape=None):
    """Rows of the active cells: (n, u, v, cell coordinates); u, v the directed connections, pattern fixed by the case."""
    nx, ny, nz = shape or (case["nx"], case["ny"], case["nz"])
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * nx + 1009 * ny + nz)
    cell = torch.arange(nx * ny * nz, device="cuda").reshape(nz, ny, nx)
    u = torch.cat([cell[:, :, :-1].reshape(-1), cell[:, :-1, :].reshape(-1), cell[:-1].reshape(-1)])
    v = torch.cat([cell[:, :, 1:].reshape(-1), cell[:, 1:, :].reshape(-1), cell[1:].reshape(-1)])
    row = cell.reshape(-1)
    if case["masked"]:
        active = torch.rand(nx * ny * nz, generator=g, device="cuda") < 0.85
        row = torch.where(active, torch.cumsum(active, 0) - 1, -1)
        keep = active[u] & active[v]
        u, v = row[u[keep]], row[v[keep]]
        n = int(active.sum())
        have = torch.sort(u * n + v)[0]
        m = int(round(0.02 * u.numel()))
        p = torch.randint(0, n, (2, 2 * m), generator=g, device="cuda")
        lo, hi = p.min(0)[0], p.max(0)[0]
        key = torch.unique((lo * n + hi)[lo < hi])
        at = torch.searchsorted(have, key).clamp(max=have.numel() - 1)
        key = key[have[at] != key]
        key = key[torch.randperm(key.numel(), generator=g, device="cuda")[:m]]
        u, v = torch.cat([u, key // n]), torch.cat([v, key % n])
    else:
        n = nx * ny * nz
    cells = torch.nonzero(row >= 0).reshape(-1)
    return n, torch.cat([u, v]), torch.cat([v, u]), cells


def _csr(n, u, v):
    """BCSR arrays of the pattern, and where each directed connection and each diagonal block is stored."""
    d = torch.arange(n, device="cuda")
    rows, cols = torch.cat([u, d]), torch.cat([v, d])
    order = torch.argsort(rows * n + cols)
    pos = torch.empty_like(order)
    pos[order] = torch.arange(order.numel(), device="cuda")
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=n), 0)
    return ptr, cols[order], pos[:u.numel()], pos[u.numel():]


def _values(n, u, v, pos, dpos, sigma, g):
    """Block values: harmonic-mean transmissibilities of a log-normal permeability, the diagonal the sum of its row's couplings plus an accumulation term."""
    half = u.numel() // 2
    k = torch.exp(sigma * torch.randn(n, generator=g, device="cuda", dtype=torch.float64))
    a = 0.5 + torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    t = 2 * k[u[:half]] * k[v[:half]] / (k[u[:half]] + k[v[:half]])
    t = torch.cat([t, t])
    eye = torch.eye(3, device="cuda", dtype=torch.float64)
    c = t[:, None, None] * (eye + 0.2 * (2 * torch.rand(u.numel(), 3, 3, generator=g, device="cuda", dtype=torch.float64) - 1))
    diag = a[:, None, None] * (eye + 0.1 * (2 * torch.rand(n, 3, 3, generator=g, device="cuda", dtype=torch.float64) - 1))
    vals = torch.empty(u.numel() + n, 3, 3, device="cuda", dtype=torch.float64)
    vals[pos] = -c
    vals[dpos] = 0.0
    # a fixed order of the additions: the row's stored blocks one after another
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = torch.cumsum(torch.bincount(u, minlength=n) + 1, 0)
    for e in range(int((ptr[1:] - ptr[:-1]).max())):
        rows = torch.nonzero(ptr[:-1] + e < ptr[1:]).reshape(-1)
        diag[rows] -= vals[ptr[rows] + e]
    vals[dpos] = diag
    return vals


def _wells(case, cells, n, seed):
    """Vertical standard wells: columns of the grid and layers fixed by the case, values by the seed."""
    nx, ny, nz, nw = case["nx"], case["ny"], case["nz"], case["wells"]
    fixed = np.random.default_rng(nx * ny + nw)
    row = np.full(nx * ny * nz, -1, np.int64)
    row[cells.cpu().numpy()] = np.arange(n)
    columns = row.reshape(nz, ny * nx)
    cols = [c for c in fixed.permutation(nx * ny) if (columns[:, c] >= 0).any()][:nw]
    ptr, perf = [0], []
    for c in cols:
        rows = columns[:, c][columns[:, c] >= 0]
        perf.extend(rows[int(fixed.integers(0, len(rows))):].tolist())
        ptr.append(len(perf))
    r = np.random.default_rng(seed)
    e = np.vstack([np.eye(3), np.full((1, 3), 1 / 3)])
    wi = np.exp(case["sigma"] * r.standard_normal(len(perf)))[:, None, None]
    b = wi * (e + 0.1 * r.uniform(-1, 1, (len(perf), 4, 3)))
    cc = wi * (e + 0.1 * r.uniform(-1, 1, (len(perf), 4, 3)))
    scale = np.array([wi[p:q].sum() for p, q in zip(ptr, ptr[1:])])[:, None, None]
    dinv = (np.eye(4) + 0.1 * r.uniform(-1, 1, (len(cols), 4, 4))) / (2 * scale)
    return np.array(ptr, np.int32), np.array(perf, np.int32), b, cc, dinv


def _parts(case, cells):
    """Partition of the cells into `parts` columns of the grid (a user's own domain decomposition)."""
    nx, ny, p = case["nx"], case["ny"], case["parts"]
    px = max(1, min(nx, int(round((p * nx / ny) ** 0.5))))
    py = max(1, min(ny, p // px))
    i, j = cells % nx, (cells // nx) % ny
    return ((j * py // ny) * px + i * px // nx).to(torch.int32)


def _system(case, seed, shape=None, batch=None):
    """The matrix and right-hand sides of a case, all on the device."""
    batch = case["batch"] if batch is None else batch
    n, u, v, cells = _pattern(case, shape)
    ptr, col, pos, dpos = _csr(n, u, v)
    g = torch.Generator(device="cuda")
    g.manual_seed(7919 * int(seed) + 17)
    vals = torch.stack([_values(n, u, v, pos, dpos, case["sigma"], g) for _ in range(batch)])
    b = torch.randn(case["rhs"], batch, n, 3, generator=g, device="cuda", dtype=torch.float64)
    return dict(n=n, ptr=ptr.to(torch.int32), col=col.to(torch.int32), vals=vals, b=b, cells=cells)


def _serve_order(case):
    """Which grid each request of the burst is for (fixed by the case; the seed draws the values)."""
    return np.random.default_rng(case["rhs"]).integers(0, len(SERVE_GRIDS), case["rhs"]).tolist()


def prepare(case, seed):
    if case["kind"] == "serve":
        server = rs.Server(hbm_budget_bytes=64 << 30, max_slots=4, precision=PREC[case["prec"]])
        systems, ids = [], []
        for k, shape in enumerate(SERVE_GRIDS):
            s = _system(dict(case, rhs=2), 31 * int(seed) + k, shape)
            ids.append(server.add_pattern(s["ptr"].cpu().numpy(), s["col"].cpu().numpy()))
            systems.append(dict(vals=s["vals"][0], b=s["b"][:, 0]))
        torch.cuda.synchronize()
        order = _serve_order(case)
        x = [torch.empty_like(systems[k]["b"][0]) for k in order]
        # resident instances, as a running server has them
        for ticket in [server.submit(ids[k], systems[k]["vals"], systems[k]["b"][i % 2], x[i], reduction=case["reduction"])
                       for i, k in enumerate(order)]:
            server.wait(ticket)
        return dict(case=case, server=server, ids=ids, systems=systems, order=order, x=x)
    s = _system(case, seed)
    vals = s["vals"] if case["batch"] > 1 else s["vals"][0]
    part = None if not case["parts"] else _parts(case, s["cells"]).cpu().numpy()
    solver = rs.Solver(s["ptr"], s["col"], vals, ordering=ORDER[case["order"]], precision=PREC[case["prec"]], part=part)
    if case["queued"]:
        rs.ilu0_set_option(solver.M, rs.OPT_FACTOR_ASYNC, 1)
    if case["wells"]:
        rs.bcsr_set_wells(solver.A, *_wells(case, s["cells"], s["n"], seed))
    state = dict(case=case, solver=solver, vals=vals, b=s["b"], x=[torch.empty_like(b) for b in s["b"]])
    if case["kind"] == "apply":
        solver.factor()
        state["y"] = torch.empty_like(s["b"][0])
    return state


# -------------------------------------------------------------------- run

def run(state):
    case = state["case"]
    if case["kind"] == "serve":
        server, systems = state["server"], state["systems"]
        tickets = [server.submit(state["ids"][k], systems[k]["vals"], systems[k]["b"][i % 2], state["x"][i],
                                 reduction=case["reduction"]) for i, k in enumerate(state["order"])]
        done = [server.wait(t) for t in tickets]
        return {"x": [d[0] for d in done], "steps": [d[2]["half_steps"] for d in done][:24]}
    solver = state["solver"]
    if case["kind"] == "apply":
        z = rs.ilu0_apply(solver.M, state["b"][0], state["x"][0], 0, case["batch"])
        return {"z": z, "y": rs.bcsr_spmv(solver.A, z, state["y"])}
    solver.factor(state["vals"])
    out, steps = [], []
    for b, x in zip(state["b"], state["x"]):
        if case["kind"] == "gmres":
            x, status, info = solver.solve_gmres(b, x, restart=30, reduction=case["reduction"], max_iter=200)
        else:
            x, status, info = solver.solve(b, x, reduction=case["reduction"], max_iter=200)
        out.append(x)
        steps.append(np.array([i["half_steps"] for i in info]))
    return {"x": out, "steps": steps}


# ------------------------------------------------------------------- work

def _sizes(case, shape=None):
    nx, ny, nz = shape or (case["nx"], case["ny"], case["nz"])
    cells = nx * ny * nz
    pairs = (nx - 1) * ny * nz + nx * (ny - 1) * nz + nx * ny * (nz - 1)
    if case["masked"]:
        cells, pairs = 0.85 * cells, 1.02 * 0.7225 * pairs
    return cells, cells + 2 * pairs


def work(case):
    """Bytes and operations of one pass with the matrix, the factors and each vector passing once per use: a
    factorisation reads A and writes the factors; an iteration has two applications (factors and indices)
    and two products (A and indices) and about 20 vectors; steps counted as the grids usually need."""
    tb = 4 if case["prec"] == "fp32" else 8
    if case["kind"] == "serve":
        total = {"bytes": 0.0, "flops": 0.0}
        for k in _serve_order(case):
            one = work(dict(case, kind="step", rhs=1, nx=SERVE_GRIDS[k][0], ny=SERVE_GRIDS[k][1], nz=SERVE_GRIDS[k][2]))
            total = {m: total[m] + one[m] for m in total}
        return total
    n, nnzb = _sizes(case)
    app = (9 * tb + 4) * nnzb + 48 * n
    mul = 76 * nnzb + 52 * n
    if case["kind"] == "apply":
        return {"bytes": float(app + mul), "flops": float(36 * nnzb)}
    factor = (72 + 9 * tb + 4) * nnzb
    its = 3 if case["sigma"] <= 1.0 else 5
    if case["kind"] == "gmres":
        solve = 2 * its * (app + mul + 24 * n * 10)
    else:
        solve = its * (2 * app + 2 * mul + 24 * n * 20)
    ops = 108 * nnzb + case["rhs"] * its * 4 * 18 * nnzb
    return {"bytes": float(case["batch"] * (factor + case["rhs"] * solve)), "flops": float(case["batch"] * ops)}


# ------------------------------------------------------------------ exact

class _Plain:
    """Block ILU0 and its application in plain FP64 torch, level by level, on a given matrix and row order."""

    def __init__(self, ptr, col, vals, perm, part=None):
        n = ptr.numel() - 1
        self.n, dev = n, vals.device
        rows = torch.repeat_interleave(torch.arange(n, device=dev), (ptr[1:] - ptr[:-1]).long())
        cols = col.long()
        self.rows, self.cols, self.vals = rows, cols, vals
        if part is not None:
            keep = part[rows] == part[cols]
            rows, cols, vals = rows[keep], cols[keep], vals[keep]
        inv = torch.empty_like(perm)
        inv[perm] = torch.arange(n, device=dev)
        r, c = inv[rows], inv[cols]
        order = torch.argsort(r * n + c)
        r, c, a = r[order], c[order], vals[order].clone()
        key = r * n + c
        first = torch.searchsorted(r, torch.arange(n + 1, device=dev))
        diag = torch.searchsorted(key, torch.arange(n, device=dev) * (n + 1))
        self.perm, self.first, self.diag, self.c = perm, first, diag, c
        self.lower = self._levels(r, c, c < r, False)
        self.upper = self._levels(r, c, c > r, True)
        self.dinv = torch.zeros(n, 3, 3, dtype=torch.float64, device=dev)
        for q in self.lower:
            lo = first[q]
            for t in range(int((diag[q] - lo).max())):
                i = q[lo + t < diag[q]]
                e = first[i] + t
                k = c[e]
                l = a[e] @ self.dinv[k]
                a[e] = l
                cnt = first[k + 1] - diag[k] - 1
                own = torch.repeat_interleave(torch.arange(i.numel(), device=dev), cnt)
                off = torch.arange(own.numel(), device=dev) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
                f = diag[k[own]] + 1 + off
                want = i[own] * n + c[f]
                at = torch.searchsorted(key, want).clamp(max=key.numel() - 1)
                hit = key[at] == want
                a[at[hit]] -= l[own[hit]] @ a[f[hit]]
            self.dinv[q] = torch.linalg.inv(a[diag[q]])
        self.a = a

    def _levels(self, r, c, dep, backward):
        """Rows grouped by the length of their dependency chain (host loop over the rows)."""
        n = self.n
        rr, cc = r[dep].cpu().numpy(), c[dep].cpu().numpy()
        ptr = np.searchsorted(rr, np.arange(n + 1)).tolist()
        cc = cc.tolist()
        depth = [0] * n
        for i in (range(n - 1, -1, -1) if backward else range(n)):
            best = 0
            for e in range(ptr[i], ptr[i + 1]):
                d = depth[cc[e]] + 1
                best = d if d > best else best
            depth[i] = best
        depth = torch.tensor(depth, device=r.device)
        order = torch.argsort(depth, stable=True)
        return list(torch.split(order, torch.bincount(depth).tolist()))

    def apply(self, v):
        y = v[self.perm].clone()
        for q in self.lower[1:]:
            y[q] -= self._row_sums(self.first[q], self.diag[q], y)
        z = torch.empty_like(y)
        for q in self.upper:
            z[q] = (self.dinv[q] @ (y[q] - self._row_sums(self.diag[q] + 1, self.first[q + 1], z))[..., None])[..., 0]
        out = torch.empty_like(z)
        out[self.perm] = z
        return out

    def _row_sums(self, lo, hi, x):
        s = torch.zeros(lo.numel(), 3, dtype=torch.float64, device=x.device)
        for t in range(int((hi - lo).max()) if lo.numel() else 0):
            m = lo + t < hi
            e = lo[m] + t
            s[m] += (self.a[e] @ x[self.c[e]][..., None])[..., 0]
        return s

    def mul(self, x, wells=None):
        y = torch.zeros_like(x)
        y.index_add_(0, self.rows, (self.vals @ x[self.cols][..., None])[..., 0])
        if wells is not None:
            ptr, perf, b, c, dinv = wells
            for w in range(len(ptr) - 1):
                p = slice(int(ptr[w]), int(ptr[w + 1]))
                t = dinv[w] @ (b[p] @ x[perf[p]][..., None]).sum(0)
                y.index_add_(0, perf[p], -(c[p].transpose(1, 2) @ t)[..., 0])
        return y


def _bicgstab(m, b, reduction, max_iter, wells):
    x, r, rhat = torch.zeros_like(b), b.clone(), b
    p = v = torch.zeros_like(b)
    rho_old = alpha = omega = torch.ones((), dtype=torch.float64, device=b.device)
    tol = reduction * b.norm()
    for it in range(1, max_iter + 1):
        rho = (rhat * r).sum()
        p = r + (rho / rho_old) * (alpha / omega) * (p - omega * v)
        ph = m.apply(p)
        v = m.mul(ph, wells)
        alpha = rho / (rhat * v).sum()
        s = r - alpha * v
        if s.norm() <= tol:
            return x + alpha * ph, 2 * it - 1
        sh = m.apply(s)
        t = m.mul(sh, wells)
        omega = (t * s).sum() / (t * t).sum()
        x = x + alpha * ph + omega * sh
        r = s - omega * t
        if r.norm() <= tol:
            return x, 2 * it
        rho_old = rho
    return x, 2 * max_iter


def _gmres(m, b, restart, reduction, max_iter, wells):
    x, steps, tol, r = torch.zeros_like(b), 0, float(reduction * b.norm()), b
    while True:
        beta = r.norm()
        basis, h, g = [r / beta], np.zeros((restart + 1, restart)), np.zeros(restart + 1)
        g[0], stop = float(beta), False
        rot = []
        for j in range(restart):
            w = m.mul(m.apply(basis[j]), wells)
            for _ in range(2):
                coef = [(w * q).sum() for q in basis]
                for i, (q, a) in enumerate(zip(basis, coef)):
                    w = w - a * q
                    h[i, j] += float(a)
            h[j + 1, j] = float(w.norm())
            basis.append(w / w.norm())
            for k, (cs, sn) in enumerate(rot):
                h[k, j], h[k + 1, j] = cs * h[k, j] + sn * h[k + 1, j], -sn * h[k, j] + cs * h[k + 1, j]
            d = np.hypot(h[j, j], h[j + 1, j])
            rot.append((h[j, j] / d, h[j + 1, j] / d))
            h[j, j], h[j + 1, j] = d, 0.0
            g[j + 1], g[j] = -rot[j][1] * g[j], rot[j][0] * g[j]
            steps += 1
            if abs(g[j + 1]) <= tol or steps >= max_iter:
                stop = True
                break
        y = np.linalg.solve(np.triu(h[:j + 1, :j + 1]), g[:j + 1])
        x = x + m.apply(sum(float(a) * q for a, q in zip(y, basis)))
        if stop:
            return x, steps
        r = b - m.mul(x, wells)
        if float(r.norm()) <= tol:
            return x, steps


def _order(case, s, shape=None):
    """The row order: natural, or the two colours of a full grid with the lowest interior cell's colour first."""
    n = s["n"]
    if case["order"] != "colour":
        return torch.arange(n, device="cuda")
    nx, ny, nz = shape or (case["nx"], case["ny"], case["nz"])
    at = torch.arange(n, device="cuda")
    colour = (at % nx + at // nx % ny + at // (nx * ny) + 1) % 2
    return torch.argsort(colour, stable=True)


def exact(case, seed):
    """Plain FP64 torch.  None for the orders that this file does not restate (colouring of an irregular
    grid, reverse Cuthill-McKee)."""
    if (case["masked"] and case["order"] == "colour") or case["order"] == "rcm":
        return None
    if case["kind"] == "serve":
        plain, b = [], []
        for k, shape in enumerate(SERVE_GRIDS):
            s = _system(dict(case, rhs=2), 31 * int(seed) + k, shape)
            plain.append(_Plain(s["ptr"], s["col"], s["vals"][0], _order(case, s, shape)))
            b.append(s["b"][:, 0])
        done = {}
        x = []
        for i, k in enumerate(_serve_order(case)):
            if (k, i % 2) not in done:
                done[k, i % 2] = _bicgstab(plain[k], b[k][i % 2], case["reduction"], 200, None)[0]
            x.append(done[k, i % 2])
        return {"x": x, "steps": [None for _ in x][:24]}
    s = _system(case, seed)
    part = _parts(case, s["cells"]) if case["parts"] else None
    wells = None
    if case["wells"]:
        ptr, perf, b, c, dinv = _wells(case, s["cells"], s["n"], seed)
        wells = (ptr, *(torch.tensor(t, device="cuda") for t in (perf.astype(np.int64), b, c, dinv)))
    x = [torch.empty_like(b) for b in s["b"]]
    z = y = None
    for k in range(case["batch"]):
        m = _Plain(s["ptr"], s["col"], s["vals"][k], _order(case, s), part)
        if case["kind"] == "apply":
            z = m.apply(s["b"][0, 0])[None]
            return {"z": z, "y": m.mul(z[0])[None]}
        for i in range(case["rhs"]):
            solve = (lambda b: _gmres(m, b, 30, case["reduction"], 200, wells)) if case["kind"] == "gmres" else (
                lambda b: _bicgstab(m, b, case["reduction"], 200, wells))
            x[i][k] = solve(s["b"][i, k])[0]
    return {"x": x, "steps": [None for _ in x]}
