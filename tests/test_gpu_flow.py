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
