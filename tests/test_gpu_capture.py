"""Entry points under HIP graph capture: what may be captured still may after
queued applications of the same handle, and what refuses a capture leaves the
handle as it was."""

import ctypes as ct

import numpy as np
import pytest

import paper_2309_11488_amd as rs
from synth import make_grid_system

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


class Capture:
    """A raw HIP capture of one stream (through the runtime librsolve is
    bound to); the body may invalidate it."""

    def __init__(self, stream):
        self.hip, self.s = rs.lib(), ct.c_void_p(stream.cuda_stream)
        self.graph, self.exec = ct.c_void_p(), ct.c_void_p()

    def __enter__(self):
        assert self.hip.hipStreamBeginCapture(self.s, 0) == 0     # global mode
        return self

    def __exit__(self, *exc):
        self.status = self.hip.hipStreamEndCapture(self.s, ct.byref(self.graph))
        self.hip.hipGetLastError()

    def replay(self):
        if not self.exec:
            assert self.status == 0
            assert self.hip.hipGraphInstantiate(ct.byref(self.exec), self.graph, None, None, ct.c_size_t(0)) == 0
        assert self.hip.hipGraphLaunch(self.exec, self.s) == 0
        torch.cuda.synchronize()

    def free(self):
        if self.exec:
            self.hip.hipGraphExecDestroy(self.exec)
        if self.graph:
            self.hip.hipGraphDestroy(self.graph)


@pytest.mark.parametrize("call", ["apply", "bicgstab", "gmres"])
def test_a_refused_capture_leaves_the_handle_as_it_was(call):
    """The calls that synchronise refuse a capture; single-launch sweeps
    switched on just before still find their marks afterwards."""
    s = make_grid_system(17, 13, 9, active_frac=0.85, nnc_frac=0.03, seed=8)
    v = torch.randn(1, s.n, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(3)).cuda()
    z = torch.empty_like(v)
    stream = torch.cuda.Stream()
    run = {"apply": lambda sol, st=None: rs.ilu0_apply(sol.M, v, z, stream=st),
           "bicgstab": lambda sol, st=None: rs.bicgstab_solve(sol.M, sol.A, v, z, 1e-8, stream=st),
           "gmres": lambda sol, st=None: rs.gmres_solve(sol.M, sol.A, v, z, 10, 1e-8, stream=st)}[call]
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_LEVEL_SET) as sol:
        sol.factor()
        assert rs.ilu0_get_option(sol.M, rs.OPT_SWEEP_TILES) == 1
        run(sol)
        torch.cuda.synchronize()
        want = z.cpu().numpy()
        rs.ilu0_set_option(sol.M, rs.OPT_SWEEP_TILES, 0)
        rs.ilu0_apply(sol.M, 1e3 * s.b[:, 0])                # per-level sweeps store over the marks
        rs.ilu0_set_option(sol.M, rs.OPT_SWEEP_TILES, 1)
        with Capture(stream) as c:
            with pytest.raises(rs.RsolveError) as e:
                run(sol, stream.cuda_stream)
        assert e.value.status == rs.HIP_ERROR
        c.free()
        for _ in range(2):
            z.zero_()
            torch.cuda.synchronize()
            run(sol)
            torch.cuda.synchronize()
            assert np.array_equal(z.cpu().numpy(), want)
