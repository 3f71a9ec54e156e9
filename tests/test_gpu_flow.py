"""Launches whose rows wait on each other through the result itself (the
single-launch sweeps): bit for bit the per-level launches, whatever the
number of rows a level holds (one XCD below 1 000, all XCDs above), tiles
that a level fills exactly or not, rows longer than one walk batch, batches,
and inputs that hold NaN, the mark's own bit pattern among them."""

import numpy as np
import pytest

import paper_2309_11488_amd as rs
from synth import make_ensemble, make_grid_system

pytestmark = pytest.mark.gpu

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
