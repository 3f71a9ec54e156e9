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


@pytest.mark.parametrize("same_stream", [True, False])
@pytest.mark.parametrize("precision", [rs.PREC_FP64, rs.PREC_FP32_FACTORS])
def test_noalloc_application_is_captured_after_queued_applications(precision, same_stream):
    """ilu0_apply on device vectors returns before its work is done; a capture
    of ilu0_apply_noalloc that follows on the handle is accepted and replays
    to the same bits, also after another factorisation's queued application."""
    s = make_grid_system(17, 13, 9, seed=8)
    g = torch.Generator().manual_seed(3)
    v = torch.randn(2, s.n, 3, generator=g, dtype=torch.float64).cuda()
    z = torch.empty_like(v)
    stream = torch.cuda.Stream()
    other = stream if same_stream else torch.cuda.Stream()
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_GRAPH_COLOUR, precision=precision) as sol:
        sol.factor()
        rs.ilu0_apply_noalloc(sol.M, v[0], z[0])            # the workspace exists before the capture
        for rep in range(2):
            sol.factor()
            torch.cuda.synchronize()
            rs.ilu0_apply(sol.M, v[1], z[1], stream=other.cuda_stream)
            with Capture(stream) as c:
                rs.ilu0_apply_noalloc(sol.M, v[0], z[0], stream=stream.cuda_stream)
            torch.cuda.synchronize()
            want = [rs.ilu0_apply(sol.M, v[k].cpu().numpy()[None])[0] for k in range(2)]
            assert np.array_equal(z[1].cpu().numpy(), want[1])
            for _ in range(3):
                z[0].zero_()
                torch.cuda.synchronize()
                c.replay()
                assert np.array_equal(z[0].cpu().numpy(), want[0])
                v[0].mul_(-1.5)                              # eager work and other inputs between the replays
                torch.cuda.synchronize()
                want[0] = rs.ilu0_apply(sol.M, v[0].cpu().numpy()[None])[0]
            c.free()


@pytest.mark.parametrize("same_stream", [True, False])
def test_queued_factorisation_is_captured_after_a_queued_application(same_stream):
    s = make_grid_system(17, 13, 9, seed=8)
    n, nnzb = s.n, len(s.colidx)
    v = torch.randn(s.n, 3, dtype=torch.float64, generator=torch.Generator().manual_seed(3)).cuda()
    z = torch.empty_like(v)
    stream = torch.cuda.Stream()
    vals = [torch.from_numpy(np.ascontiguousarray(s.vals * k)).cuda() for k in (2.0, 1.0)]
    with rs.Solver(s.rowptr, s.colidx, s.vals, ordering=rs.ORDER_LEVEL_SET) as sol:
        sol.factor()
        want = rs.ilu0_get_factors(sol.M, 0, n, nnzb)
        rs.ilu0_set_option(sol.M, rs.OPT_SWEEP_TILES, 0)
        rs.ilu0_set_option(sol.M, rs.OPT_FACTOR_ASYNC, 1)
        rs.bcsr_set_values(sol.A, vals[0])
        sol.factor()
        torch.cuda.synchronize()
        rs.ilu0_apply(sol.M, v, z, stream=stream.cuda_stream if same_stream else None)
        with Capture(stream) as c:
            st, _ = rs.ilu0_factor(sol.M, sol.A, stream=stream.cuda_stream)
        assert st == rs.OK
        rs.bcsr_set_values(sol.A, vals[1])
        for _ in range(3):
            torch.cuda.synchronize()
            c.replay()
            got = rs.ilu0_get_factors(sol.M, 0, n, nnzb)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        c.free()


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
