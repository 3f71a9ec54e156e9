"""Launches whose rows wait on each other through the result itself (the
single-launch sweeps): bit for bit the per-level launches, whatever the
number of rows a level holds (one XCD below 1 000, all XCDs above), tiles
that a level fills exactly or not, rows longer than one walk batch, batches,
and inputs that hold NaN, the mark's own bit pattern among them."""

import numpy as np
import pytest

import oracle
import paper_2309_11488_amd as rs
from synth import make_ensemble, make_grid_system

pytestmark = pytest.mark.gpu



def rel_block_err(a, b):
    return np.abs(a - b).max(initial=0.0) / max(np.abs(b).max(initial=0.0), 1e-300)


MARK = np.array([0x7FF4BEEF7FF4BEEF], np.uint64).view(np.float64)[0]


def _pattern(name):
    """(rowptr, colidx, vals) with vals (batch, nnzb, 3, 3), diagonally dominant."""
    if name.startswith("grid"):
        nx, ny, nz = (int(t) for t in name[4:].split("x"))
        s = make_grid_system(nx, ny, nz, seed=nx + ny)
        return s.rowptr, s.colidx, s.vals
    if name == "nnc":
        s = make_grid_system(19, 13, 11, active_frac=0.85, nnc_frac=0.05, seed=3, sigma=2.0)
        return s.rowptr, s.colidx, s.vals
    if name == "ensemble":
        s = make_ensemble(12, 10, 9, seeds=[1, 2, 3])
        return s.rowptr, s.colidx, s.vals
    kind, n = name.split("_")
    n = int(n)
    rng = np.random.default_rng(n)
    if kind == "diag":       # one level of independent rows
        mask = np.eye(n, dtype=bool)
    elif kind == "chain":    # one row a level
        mask = np.eye(n, dtype=bool) | np.eye(n, k=-1, dtype=bool) | np.eye(n, k=1, dtype=bool)
    else:                    # every row holds every column
        mask = np.ones((n, n), bool)
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    colidx = np.nonzero(mask)[1].astype(np.int32)
    rows = np.nonzero(mask)[0]
    vals = rng.uniform(-1, 1, (1, len(colidx), 3, 3)) / (3.0 * n if kind == "dense" else 9.0)
    vals[0, rows == colidx] += 2.0 * np.eye(3)
    return rowptr, colidx, vals


PATTERNS = ["diag_1", "diag_63", "diag_64", "diag_65", "chain_1", "chain_2", "chain_70", "dense_9", "dense_40",
            "grid7x5x3", "grid16x8x8", "grid23x17x11", "nnc", "ensemble"]


@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
@pytest.mark.parametrize("ordering", [rs.ORDER_LEVEL_SET, rs.ORDER_GRAPH_COLOUR, rs.ORDER_NATURAL])
@pytest.mark.parametrize("name", PATTERNS)
def test_single_launch_sweeps_equal_per_level(name, ordering, precision):
    rowptr, colidx, vals = _pattern(name)
    n, batch = len(rowptr) - 1, vals.shape[0]
    rng = np.random.default_rng(5)
    clean = rng.standard_normal((batch, n, 3))
    holed = clean.copy()
    holed[:, 0, 0], holed[:, n // 2, 2], holed[:, n - 1, 1] = MARK, np.inf, np.nan
    with rs.Solver(rowptr, colidx, vals, ordering=ordering, precision=precision) as s:
        s.factor()
        for v in (clean, holed, clean):
            rs.ilu0_set_option(s.M, rs.OPT_SWEEP_TILES, 0)
            want = rs.ilu0_apply(s.M, v, n_sys=batch)
            rs.ilu0_set_option(s.M, rs.OPT_SWEEP_TILES, 1)
            for _ in range(2):
                got = rs.ilu0_apply(s.M, v, n_sys=batch)
                assert np.array_equal(got, want, equal_nan=True)


@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
@pytest.mark.parametrize("name", ["chain_3", "chain_70", "dense_9", "dense_40", "grid16x8x8", "grid40x17x11", "nnc",
                                  "ensemble", "wide_ensemble"])
def test_single_launch_factorisation_equals_the_oracle(name, precision):
    """Factors of patterns whose factorisation is one launch (more than two
    levels), short rows and rows past the register width, with and without
    updates of U blocks, on one XCD and on all (an ensemble wide enough):
    the oracle's under the same ordering, and again after a refactorisation
    with other values."""
    if name == "wide_ensemble":
        s = make_ensemble(40, 17, 11, seeds=list(range(24)))
        rowptr, colidx, vals = s.rowptr, s.colidx, s.vals
    else:
        rowptr, colidx, vals = _pattern(name)
    n, nnzb = len(rowptr) - 1, len(colidx)
    with rs.Solver(rowptr, colidx, vals[::-1].copy() * 2.0, ordering=rs.ORDER_LEVEL_SET, precision=precision) as s:
        s.factor()
        st, bad = s.factor(vals)
        assert st == rs.OK and (bad == -1).all()
        for k in (0, vals.shape[0] - 1):
            lu, dinv = rs.ilu0_get_factors(s.M, k, n, nnzb)
            perm, _, _ = rs.ilu0_get_schedule(s.M, n)
            prow, pcol, pv = oracle.permute(rowptr, colidx, vals[k], perm)
            st, _, olu, odinv = oracle.ilu0(prow, pcol, pv)
            assert st == oracle.OK
            offd = pcol != np.repeat(np.arange(n), np.diff(prow))
            for got, want in ((lu[offd], olu[offd]), (dinv, odinv)):
                if precision == rs.PREC_FP64:
                    assert rel_block_err(got, want) <= 1e-12
                else:
                    w32 = want.astype(np.float32)
                    assert np.all(np.abs(got - w32.astype(np.float64)) <= np.spacing(np.abs(w32)).astype(np.float64))


def test_single_launch_factorisation_reports_a_zero_pivot():
    rowptr, colidx, vals = _pattern("grid16x8x8")
    vals = vals.copy()
    row = 700
    for p in range(rowptr[row], rowptr[row + 1]):
        vals[0, p, 1] = 0.0
    with rs.Solver(rowptr, colidx, vals, ordering=rs.ORDER_LEVEL_SET) as s:
        st, bad = s.factor()
        assert st == rs.ZERO_PIVOT and bad[0] == row
        st, bad = s.factor(_pattern("grid16x8x8")[2])
        assert st == rs.OK and bad[0] == -1


APPLY_PATTERNS = ["diag_1", "diag_65", "chain_2", "chain_257", "dense_9", "dense_40", "grid7x5x3", "grid16x8x8",
                  "grid23x17x15", "grid19x18x18", "nnc", "big_nnc", "ensemble"]


@pytest.mark.parametrize("variant", [0, 4, 8])
@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
@pytest.mark.parametrize("ordering", [rs.ORDER_GRAPH_COLOUR, rs.ORDER_RCM_LEVEL_SET])
@pytest.mark.parametrize("name", APPLY_PATTERNS)
def test_application_and_product_in_one_launch(name, ordering, precision, variant):
    """BiCGStab whose applications and products are one launch each (small
    systems) against the separate launches (which a solve takes while its
    sweeps are timed): the same bits, for tiles of 84 rows (up to 6 000 rows)
    and of 252, filled exactly or not, every number of waves a partial, with
    and without fused rows and lower parts, and with graphs off (separate
    launches again), after a solve that stopped at its iteration limit."""
    if name == "big_nnc":
        s = make_grid_system(31, 23, 12, active_frac=0.9, nnc_frac=0.03, seed=6)
        rowptr, colidx, vals = s.rowptr, s.colidx, s.vals
    else:
        rowptr, colidx, vals = _pattern(name)
    n, batch = len(rowptr) - 1, vals.shape[0]
    b = np.random.default_rng(8).standard_normal((batch, n, 3))

    def outcomes(s, red, max_iter):
        x, st, info = s.solve(b, reduction=red, max_iter=max_iter)
        return x, st, [(i["status"], i["half_steps"], i["final_norm"], i["true_rel_residual"]) for i in info]

    with rs.Solver(rowptr, colidx, vals, ordering=ordering, precision=precision) as s:
        rs.ilu0_set_option(s.M, rs.OPT_SPMV_VARIANT, variant)
        s.factor()
        for red, max_iter in ((0.0, 3), (1e-8, 200)):
            rs.rsolve_profile_enable(1 << rs.PROF_LSWEEP)
            try:
                want = outcomes(s, red, max_iter)
                assert rs.rsolve_profile_get(rs.PROF_LSWEEP)[1] > 0
            finally:
                rs.rsolve_profile_enable(0)
            for graph in (0, 1, 1):
                rs.ilu0_set_option(s.M, rs.OPT_USE_GRAPH, graph)
                got = outcomes(s, red, max_iter)
                assert np.array_equal(got[0], want[0], equal_nan=True) and got[1:] == want[1:]


def test_one_launch_application_recovers_from_a_wait_that_gives_up():
    s = make_grid_system(17, 13, 9, active_frac=0.85, nnc_frac=0.03, seed=4)
    b = s.b[:, 0]
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_GRAPH_COLOUR) as sol:
        sol.factor()
        want, st, _ = sol.solve(b)
        assert st == rs.OK
        default = rs.ilu0_get_option(sol.M, rs.OPT_SPIN_LIMIT)
        rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, 0)
        with pytest.raises(rs.RsolveError) as e:
            for _ in range(5):
                sol.solve(b)
        assert e.value.status == rs.HIP_ERROR
        rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, default)
        for _ in range(2):
            x, st, _ = sol.solve(b)
            assert st == rs.OK and np.array_equal(x, want)


@pytest.mark.parametrize("n", [1, 341, 342, 12_000, 350_000, 720_001])
def test_polled_reduction_adds_every_partial(n):
    """||b|| over one workgroup, a second one that holds a single entry, many
    (up to 1 024: one pass of the polling workgroup), more (several passes)
    and more tiles than workgroups: a sum of 3n squares is within
    3n eps of the exact one in any order, so the norm is too; the same twice."""
    eye = np.tile(np.eye(3), (n, 1, 1))
    b = np.random.default_rng(n).standard_normal((1, n, 3))
    with rs.Solver(np.arange(n + 1), np.arange(n), eye, ordering=rs.ORDER_GRAPH_COLOUR) as s:
        s.factor()
        norms = [s.solve(b, reduction=0.0, max_iter=0)[2][0]["r0_norm"] for _ in range(2)]
    want = np.linalg.norm(b)
    assert norms[0] == norms[1] and abs(norms[0] - want) <= 3 * n * np.finfo(np.float64).eps * want


@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
@pytest.mark.parametrize("restart", [3, 30])
@pytest.mark.parametrize("name", ["chain_257", "dense_40", "grid16x8x8", "grid23x17x15", "nnc", "big_nnc", "ensemble"])
def test_gmres_with_applications_in_one_launch(name, restart, precision):
    """GMRES on a small system against the separate launches (graphs off): the
    same bits, over restarts and with systems of a batch that stop apart."""
    if name == "big_nnc":
        s = make_grid_system(31, 23, 12, active_frac=0.9, nnc_frac=0.03, seed=6)
        rowptr, colidx, vals = s.rowptr, s.colidx, s.vals
    else:
        rowptr, colidx, vals = _pattern(name)
    n, batch = len(rowptr) - 1, vals.shape[0]
    b = np.random.default_rng(9).standard_normal((batch, n, 3))
    b[0] *= np.linspace(1.0, 1e4, n)[:, None]
    with rs.Solver(rowptr, colidx, vals, ordering=rs.ORDER_GRAPH_COLOUR, precision=precision) as s:
        s.factor()
        got = []
        for graph in (0, 1, 1):
            rs.ilu0_set_option(s.M, rs.OPT_USE_GRAPH, graph)
            x, st, info = s.solve_gmres(b, restart=restart, reduction=1e-5, max_iter=60)
            got.append((x, st, [(i["status"], i["half_steps"], i["final_norm"], i["true_rel_residual"]) for i in info]))
    for g in got[1:]:
        assert np.array_equal(g[0], got[0][0]) and g[1:] == got[0][1:]


@pytest.mark.parametrize("tiles", [0, 1])
def test_queued_applications_keep_the_handle_in_order_across_streams(tiles):
    """A device caller's application returns before its work is done; the
    handle's next call works in the same buffers, on whatever stream."""
    torch = pytest.importorskip("torch")
    s = make_grid_system(37, 31, 23, seed=8)
    rng = np.random.default_rng(2)
    v = torch.from_numpy(rng.standard_normal((6, s.n, 3))).cuda()
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_GRAPH_COLOUR) as sol:
        rs.ilu0_set_option(sol.M, rs.OPT_SWEEP_TILES, tiles)
        sol.factor()
        want = [rs.ilu0_apply(sol.M, v[k].cpu().numpy()[None]) for k in range(6)]
        xw, st, _ = sol.solve(s.b[:, 0])
        assert st == rs.OK
        b = torch.from_numpy(np.ascontiguousarray(s.b[:, 0])).cuda()
        z, x = torch.empty_like(v), torch.empty_like(b)
        streams = [torch.cuda.Stream() for _ in range(3)]
        torch.cuda.synchronize()
        for rep in range(3):
            z.zero_()
            torch.cuda.synchronize()
            for k in range(6):
                rs.ilu0_apply(sol.M, v[k], z[k], stream=streams[(k + rep) % 3].cuda_stream)
            rs.bicgstab_solve(sol.M, sol.A, b, x, stream=streams[(rep + 1) % 3].cuda_stream)
            torch.cuda.synchronize()
            assert all(np.array_equal(z[k].cpu().numpy(), want[k][0]) for k in range(6))
            assert np.array_equal(x.cpu().numpy(), xw)


@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
@pytest.mark.parametrize("batch", [64, 65])
def test_streamed_factor_stores_equal_the_cached_ones(batch, precision):
    """250 000 rows of all systems and more write their factors with
    non-temporal stores: the member's factors alone, bit for bit."""
    s = make_grid_system(21, 17, 11, seed=12)      # 3 927 rows: 251 328 and 255 255
    scale = 1.0 + np.arange(batch) / 64.0
    nnzb = len(s.colidx)
    with rs.Solver(s.rowptr, s.colidx, s.vals[0] * scale[:, None, None, None], ordering=rs.ORDER_GRAPH_COLOUR,
                   precision=precision) as many:
        many.factor()
        for k in (0, 1, batch - 1):
            got = rs.ilu0_get_factors(many.M, k, s.n, nnzb)
            with rs.Solver(s.rowptr, s.colidx, s.vals * scale[k], ordering=rs.ORDER_GRAPH_COLOUR,
                           precision=precision) as one:
                one.factor()
                want = rs.ilu0_get_factors(one.M, 0, s.n, nnzb)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("ordering", [rs.ORDER_LEVEL_SET, rs.ORDER_GRAPH_COLOUR, rs.ORDER_RCM_LEVEL_SET])
@pytest.mark.parametrize("n", [3, 40, 600])
def test_patterns_without_the_transposed_blocks(n, ordering):
    """A row without upper blocks that a later row's L names: its y counts in
    every form of the sweeps."""
    rng = np.random.default_rng(n)
    mask = np.eye(n, dtype=bool)
    mask[1 + np.arange(n - 1), np.arange(n - 1) // 2] = True      # blocks below the diagonal only
    mask[rng.integers(0, n, n // 3), rng.integers(0, n, n // 3)] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int32)
    rows, cols = np.nonzero(mask)
    vals = rng.uniform(-1, 1, (1, len(cols), 3, 3)) / 4.0
    vals[0, rows == cols] += 6.0 * np.eye(3)
    v = rng.standard_normal((1, n, 3))
    with rs.Solver(rowptr, cols.astype(np.int32), vals, ordering=ordering) as s:
        s.factor()
        perm, _, _ = rs.ilu0_get_schedule(s.M, n)
        prow, pcol, pv = oracle.permute(rowptr, cols.astype(np.int32), vals[0], perm)
        st, _, lu, dinv = oracle.ilu0(prow, pcol, pv)
        want = np.empty((n, 3))
        want[perm] = oracle.apply(prow, pcol, lu, dinv, v[0][perm])
        for tiles in (0, 1):
            rs.ilu0_set_option(s.M, rs.OPT_SWEEP_TILES, tiles)
            z = rs.ilu0_apply(s.M, v)
            assert np.linalg.norm(z[0] - want) <= 1e-12 * np.linalg.norm(want)
        rs.ilu0_set_option(s.M, rs.OPT_SWEEP_TILES, 0)
        got = []
        for graph in (0, 1):
            rs.ilu0_set_option(s.M, rs.OPT_USE_GRAPH, graph)
            x, st, info = s.solve(v, reduction=1e-6)
            assert st == rs.OK
            got.append((x, info[0]["half_steps"]))
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]


@pytest.mark.parametrize("grid", [(5, 4, 3), (21, 16, 8), (23, 17, 11)])
def test_one_and_four_wave_products_give_the_same_sums(grid):
    """The partials of a product's dot products are those of four waves in
    workgroups of one (kept apart, 128 a group) as in workgroups of four."""
    s = make_grid_system(*grid, active_frac=0.9, nnc_frac=0.03, seed=grid[0])
    for ordering in (rs.ORDER_GRAPH_COLOUR, rs.ORDER_LEVEL_SET):
        with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=ordering) as sol:
            sol.factor()
            got = []
            for graph in (0, 1):
                rs.ilu0_set_option(sol.M, rs.OPT_USE_GRAPH, graph)
                for variant in (0, 2, 6, 8):
                    rs.ilu0_set_option(sol.M, rs.OPT_SPMV_VARIANT, variant)
                    x, st, info = sol.solve(s.b[:, 0], reduction=1e-8)
                    got.append((x, st, info[0]["half_steps"], info[0]["final_norm"], info[0]["true_rel_residual"]))
        for g in got[1:]:
            assert np.array_equal(g[0], got[0][0]) and g[1:] == got[0][1:]


def test_lower_blocks_without_updates_leave_the_pivot_alone():
    """A lower block whose transposed block is not stored updates nothing, so
    an infinite one (1e250 times an inverse of 1e100) stays out of its row's
    pivot in the single-launch factorisation too."""
    n = 6
    pairs = sorted({(i, i) for i in range(n)} | {(i, j) for i in range(1, n) for j in (i - 1, i + 1) if 1 <= j < n} | {(5, 0)})
    rowptr = np.searchsorted([i for i, _ in pairs], np.arange(n + 1)).astype(np.int32)
    colidx = np.array([j for _, j in pairs], np.int32)
    rng = np.random.default_rng(3)
    vals = rng.uniform(-1, 1, (1, len(pairs), 3, 3)) / 9.0
    for p, (i, j) in enumerate(pairs):
        if i == j:
            vals[0, p] += 2.0 * np.eye(3)
    vals[0, pairs.index((0, 0))] = np.eye(3) * 1e-100
    vals[0, pairs.index((5, 0))] = 1e250
    want = oracle.ilu0(rowptr, colidx, vals[0])
    assert want[0] == oracle.OK and np.isinf(want[2][pairs.index((5, 0))]).all() and np.isfinite(want[3]).all()
    with rs.Solver(rowptr, colidx, vals, ordering=rs.ORDER_NATURAL) as s:
        st, bad = s.factor()
        assert st == rs.OK and bad[0] == -1
        lu, dinv = rs.ilu0_get_factors(s.M, 0, n, len(pairs))
    assert np.isinf(lu[pairs.index((5, 0))]).all()
    assert rel_block_err(dinv[1:], want[3][1:]) <= 1e-12


def test_single_launch_factorisation_recovers_from_a_wait_that_gives_up():
    """RS_OPT_SPIN_LIMIT bounds the factorisation's waits too: one that gives
    up is RS_HIP_ERROR from the factorisation, or when it was only queued from
    the next solve and ilu0_factor_status, and the next factorisation is sound."""
    s = make_grid_system(17, 13, 9, active_frac=0.85, nnc_frac=0.03, seed=4)
    nnzb = len(s.colidx)
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_LEVEL_SET) as sol:
        sol.factor()
        want, x0 = rs.ilu0_get_factors(sol.M, 0, s.n, nnzb), sol.solve(s.b[:, 0])[0]
        default = rs.ilu0_get_option(sol.M, rs.OPT_SPIN_LIMIT)
        rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, 0)
        with pytest.raises(rs.RsolveError) as e:
            for _ in range(5):
                sol.factor()
        assert e.value.status == rs.HIP_ERROR
        rs.ilu0_set_option(sol.M, rs.OPT_FACTOR_ASYNC, 1)
        gave_up = False
        for _ in range(5):
            rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, 0)
            assert sol.factor()[0] == rs.OK
            rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, default)
            try:
                sol.solve(s.b[:, 0])
            except rs.RsolveError as err:
                assert err.status == rs.HIP_ERROR
                with pytest.raises(rs.RsolveError) as e:
                    rs.ilu0_factor_status(sol.M, 1)
                assert e.value.status == rs.HIP_ERROR
                gave_up = True
                break
        assert gave_up
        sol.factor()
        got = rs.ilu0_get_factors(sol.M, 0, s.n, nnzb)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        x, st, _ = sol.solve(s.b[:, 0])
        assert st == rs.OK and np.array_equal(x, x0) and rs.ilu0_factor_status(sol.M, 1)[0] == rs.OK


@pytest.mark.parametrize("method", ["bicgstab", "gmres"])
def test_polled_reduction_recovers_from_a_wait_that_gives_up(method):
    """A reduction whose polls reach RS_OPT_SPIN_LIMIT makes the solve
    RS_HIP_ERROR; late partials do not reach the next solve."""
    n = 120_000
    vals = np.tile(np.eye(3), (n, 1, 1)) * np.linspace(1.0, 2.0, n)[:, None, None]
    b = np.random.default_rng(1).standard_normal((1, n, 3))
    with rs.Solver(np.arange(n + 1), np.arange(n), vals, ordering=rs.ORDER_GRAPH_COLOUR) as sol:
        rs.ilu0_set_option(sol.M, rs.OPT_FUSE_SPMV, 0)        # separate launches: only reductions wait
        sol.factor()

        def solve():
            x, st, info = sol.solve(b, reduction=1e-6) if method == "bicgstab" else sol.solve_gmres(b, reduction=1e-6)
            return x, st, [(i["status"], i["half_steps"], i["final_norm"], i["true_rel_residual"]) for i in info]

        want = solve()
        assert want[1] == rs.OK
        default = rs.ilu0_get_option(sol.M, rs.OPT_SPIN_LIMIT)
        rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, 0)
        with pytest.raises(rs.RsolveError) as e:
            for _ in range(10):
                solve()
        assert e.value.status == rs.HIP_ERROR
        rs.ilu0_set_option(sol.M, rs.OPT_SPIN_LIMIT, default)
        for _ in range(3):
            got = solve()
            assert np.array_equal(got[0], want[0]) and got[1:] == want[1:]


def test_tuning_knows_the_one_launch_iteration(tmp_path, monkeypatch):
    """Where an iteration runs its applications as one launch the product's
    shape cannot matter, so tuning leaves it; a choice saved by another
    format, or by a handle whose iterations are separate launches, is not
    taken."""
    s = make_grid_system(16, 12, 8, seed=31)
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("RSOLVE_TUNE_CACHE", str(cache))
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_GRAPH_COLOUR) as sol:
        sol.factor()
        shape = rs.ilu0_get_option(sol.M, rs.OPT_SPMV_VARIANT)
        for _ in range(4):
            r = rs.ilu0_autotune(sol.M, sol.A, s.b[:, 0], reps=1)
            assert r["from_cache"] == 0
            if r["reduce_split"] == 0 and r["sweep_tiles"] == 0:
                assert r["spmv_variant"] == shape
            rs.ilu0_set_option(sol.M, rs.OPT_SPMV_VARIANT, shape)
            rs.ilu0_set_option(sol.M, rs.OPT_SWEEP_TILES, 0)
            rs.ilu0_set_option(sol.M, rs.OPT_REDUCE_SPLIT, 0)
            saved = cache.read_text()
            cache.unlink()
        # a line of the format before this one with the split reduction
        import re
        key = re.sub("(fmt=[0-9]+)(,path=[a-z]+)?", "fmt=3", saved.split()[0])
        cache.write_text(f"{key} 0 0 0 256 1 1.0\n")
        assert rs.ilu0_autotune(sol.M, sol.A, s.b[:, 0], reps=1)["from_cache"] == 0
        cache.write_text(saved)
        assert rs.ilu0_autotune(sol.M, sol.A, s.b[:, 0], reps=1)["from_cache"] == 1
        rs.ilu0_set_option(sol.M, rs.OPT_USE_GRAPH, 0)
        assert rs.ilu0_autotune(sol.M, sol.A, s.b[:, 0], reps=1)["from_cache"] == 0


@pytest.mark.parametrize("n", [21, 671, 672, 673, 2687, 2688, 2689, 3381, 5377])
def test_one_wave_products_count_their_groups(n):
    """One-wave products at the edges of their counters (32 workgroups of 21
    rows a counter, four counters a group): the sums of four waves, and the
    counters cleared for the next launch."""
    rowptr, colidx, vals = _pattern(f"chain_{n}")
    b = np.random.default_rng(n).standard_normal((1, n, 3))
    with rs.Solver(rowptr, colidx, vals, ordering=rs.ORDER_GRAPH_COLOUR) as sol:
        rs.ilu0_set_option(sol.M, rs.OPT_USE_GRAPH, 0)        # separate launches
        sol.factor()
        for fuse in (1, 0):
            rs.ilu0_set_option(sol.M, rs.OPT_FUSE_SPMV, fuse)
            got = []
            for variant in (0, 2, 8, 2):
                rs.ilu0_set_option(sol.M, rs.OPT_SPMV_VARIANT, variant)
                x, st, info = sol.solve(b, reduction=1e-9)
                got.append((x, st, info[0]["half_steps"], info[0]["final_norm"], info[0]["true_rel_residual"]))
            assert got[0][1] == rs.OK
            for g in got[1:]:
                assert np.array_equal(g[0], got[0][0]) and g[1:] == got[0][1:]


def test_two_threads_run_one_launch_applications_at_once():
    """Two handles, two streams, two host threads, each with launches whose
    workgroups wait on each other: every solve gives the bits it gives alone
    (captures made before the threads start)."""
    import threading
    torch = pytest.importorskip("torch")
    systems = [make_grid_system(23, 17, 11, active_frac=0.9, nnc_frac=0.03, seed=5), make_grid_system(40, 30, 20, seed=6)]
    sols, want, fails = [], [], []
    try:
        for k, s in enumerate(systems):
            st = torch.cuda.Stream()
            sol = rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_GRAPH_COLOUR, stream=st.cuda_stream)
            sols.append((sol, st, torch.from_numpy(np.ascontiguousarray(s.b[:, 0])).cuda()))
            torch.cuda.synchronize()
            sol.factor()
            x = torch.empty_like(sols[k][2])
            for _ in range(4):
                sol.solve(sols[k][2], x, reduction=1e-6)
            torch.cuda.synchronize()
            want.append(x.cpu().numpy())

        def work(k):
            sol, _, b = sols[k]
            x = torch.empty_like(b)
            for _ in range(40):
                if sol.solve(b, x, reduction=1e-6)[1] != rs.OK or not np.array_equal(x.cpu().numpy(), want[k]):
                    fails.append(k)
                    return

        threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not fails
    finally:
        for sol, _, _ in sols:
            sol.close()


@pytest.mark.parametrize("n", [512, 513])
def test_deep_schedules_keep_separate_launches(n):
    """A chain under reverse Cuthill-McKee has a level a row: up to 512 levels
    an iteration's applications are one launch each, beyond it stays separate
    launches; the bits of graphs off either way."""
    rowptr, colidx, vals = _pattern(f"chain_{n}")
    b = np.random.default_rng(n).standard_normal((1, n, 3))
    with rs.Solver(rowptr, colidx, vals, ordering=rs.ORDER_RCM_LEVEL_SET) as s:
        rs.ilu0_set_option(s.M, rs.OPT_SWEEP_TILES, 0)
        s.factor()
        assert rs.ilu0_get_sweep_levels(s.M)[0] == n
        got = []
        for graph in (0, 1, 1):
            rs.ilu0_set_option(s.M, rs.OPT_USE_GRAPH, graph)
            x, st, info = s.solve(b, reduction=1e-9)
            got.append((x, st, info[0]["half_steps"], info[0]["final_norm"], info[0]["true_rel_residual"]))
    assert got[0][1] == rs.OK
    for g in got[1:]:
        assert np.array_equal(g[0], got[0][0]) and g[1:] == got[0][1:]
