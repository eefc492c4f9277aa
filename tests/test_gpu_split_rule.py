"""The split schedule where it is chosen automatically, and the sums of its
parts: against the CPU FP64 oracle (FP64 path <= 1e-10 in fixed-iteration
mode, the bar of the other solver tests), around the part counts where the
update adds the parts itself or after a kernel of its own, with blocks of one
and of two 64-value chunks, and at the ends of the iteration (no update, one,
two, to tol) that the host learns of one pass late."""
import sys

import numpy as np
import pytest

from oracle import solver as o_solver
from test_gpu_band import band_chain
from test_gpu_solve import gpu_solve, noisy_problem, rel_err

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture
def ctx(qc_lib):
    yield qc_lib
    qc_lib.set_split(0)


@pytest.mark.parametrize("n_ant", [7, 11])
@pytest.mark.parametrize("parts", [4, 5, 16, 17, 33])
def test_sums_of_parts(ctx, parts, n_ant):
    say(f"sums of {parts} parts, {n_ant} antennas")
    vis, chain = noisy_problem(401, n_ant=n_ant, n_time=4, n_chan=20, kind="diag", t_int=2, f_int=20)
    ref, rst = o_solver.solve_term(vis, chain, 0, tol=-1.0, max_iter=4)
    ctx.set_split(parts)
    got, st = gpu_solve(ctx, vis, chain, 0, tol=-1.0, max_iter=4, prec="fp64")
    assert ctx.last_split_parts() == parts and (st["iters"] == 4).all()
    assert rel_err(got[0].gains, ref[0].gains, "diag") <= 1e-10
    np.testing.assert_allclose(st["chisq_last"], rst["chisq_last"], rtol=1e-10)


@pytest.mark.parametrize("kind,n_ant,n_time,n_chan,f_int", [("diag", 9, 40, 96, 96), ("c2x2", 8, 50, 70, 70),
                                                            ("phase", 12, 30, 130, 65), ("delay", 10, 30, 128, 128)])
def test_automatic_split(ctx, kind, n_ant, n_time, n_chan, f_int):
    say(f"automatic split: {kind}")
    vis, chain = noisy_problem(403, n_ant=n_ant, n_time=n_time, n_chan=n_chan, kind=kind, t_int=n_time, f_int=f_int)
    for k in (0, 1, 2, 5):
        ref, rst = o_solver.solve_term(vis, chain, 0, tol=-1.0, max_iter=k)
        got, st = gpu_solve(ctx, vis, chain, 0, tol=-1.0, max_iter=k, prec="fp64")
        assert ctx.last_split_parts() > 1
        assert (st["iters"] == k).all()
        np.testing.assert_allclose(st["chisq_last"], rst["chisq_last"], rtol=1e-10)
        if kind in ("diag", "c2x2"):
            assert rel_err(got[0].gains, ref[0].gains, kind) <= 1e-10
        else:
            scale = max(np.abs(ref[0].params).max(), 1e-300)
            assert np.abs(got[0].params - ref[0].params).max() <= 1e-10 * scale
    # a solve that stopped at max_iter, then one to tol in the same context
    ref, rst = o_solver.solve_term(vis, chain, 0, tol=1e-6, max_iter=60)
    got, st = gpu_solve(ctx, vis, chain, 0, tol=1e-6, max_iter=60, prec="fp64")
    np.testing.assert_array_equal(st["iters"], rst["iters"])
    np.testing.assert_array_equal(st["converged"], rst["converged"])


def test_automatic_band_split(ctx):
    say("automatic split of one-channel intervals")
    vis, chain = band_chain(405, n_ant=10, n_time=96, n_chan=18)
    chain[1] = chain[1].copy(t_map=np.zeros_like(chain[1].t_map), n_gt=1, gains=chain[1].gains[:1].copy(),
                             gain_flags=None if chain[1].gain_flags is None else chain[1].gain_flags[:1].copy())
    ref, _ = o_solver.solve_term(vis, chain, 1, tol=-1.0, max_iter=3)
    got, st = gpu_solve(ctx, vis, chain, 1, tol=-1.0, max_iter=3, prec="fp64")
    assert ctx.last_split_parts() > 1
    assert (st["iters"] == 3).all()
    assert rel_err(got[1].gains, ref[1].gains, "diag") <= 1e-10
