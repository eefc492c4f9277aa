"""The wavefronts per workgroup that the fused schedule chooses by the number
and size of the intervals (eight where they leave the chip room, one or two
where many small ones wait in line, four otherwise or where the LDS of eight
does not fit): against the CPU FP64 oracle, at the bar of the other solver
tests (FP64 path <= 1e-10 in fixed-iteration mode)."""
import sys

import numpy as np
import pytest

from oracle import solver as o_solver
from test_gpu_solve import gpu_solve, noisy_problem, rel_err

pytestmark = pytest.mark.gpu


# kind, antennas, times, channels, f_int: eight wavefronts (one step, several and a
# remainder), eight whose LDS does not fit, four, two and one
@pytest.mark.parametrize("kind,n_ant,n_time,n_chan,f_int", [
    ("diag", 3, 2, 3, 3), ("c2x2", 9, 2, 37, 19), ("phase", 9, 3, 20, 20), ("c2x2", 141, 1, 2, 2),
    ("diag", 4, 257, 1, 1), ("c2x2", 12, 64, 32, 1), ("diag", 4, 128, 34, 2), ("delay", 5, 2050, 5, 5)])
def test_fused_waves(qc_lib, kind, n_ant, n_time, n_chan, f_int):
    print(f"fused waves: {kind}, {n_ant} antennas, {n_time} x {n_chan}", flush=True)
    sys.stdout.flush()
    vis, chain = noisy_problem(407, n_ant=n_ant, n_time=n_time, n_chan=n_chan, kind=kind, t_int=1, f_int=f_int)
    ref, rst = o_solver.solve_term(vis, chain, 0, tol=-1.0, max_iter=3)
    qc_lib.set_split(1)
    try:
        got, st = gpu_solve(qc_lib, vis, chain, 0, tol=-1.0, max_iter=3, prec="fp64")
    finally:
        qc_lib.set_split(0)
    assert (st["iters"] == 3).all()
    np.testing.assert_allclose(st["chisq_last"], rst["chisq_last"], rtol=1e-10)
    if kind in ("diag", "c2x2"):
        assert rel_err(got[0].gains, ref[0].gains, kind) <= 1e-10
    else:
        assert np.abs(got[0].params - ref[0].params).max() <= 1e-10 * np.abs(ref[0].params).max()
