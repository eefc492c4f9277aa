"""A Levenberg-Marquardt solve of no attempts (max_iter 0: chi^2 only) on the split
schedule leaves the gain flags as they were, also after a solve of the same context
whose blocks did not converge (flag 2)."""
import numpy as np
import pytest

from test_gpu_divergence import gpu, two_cycle

pytestmark = pytest.mark.gpu


def test_no_attempt_leaves_the_flags(qc_lib):
    print("LM of no attempts after a divergent solve", flush=True)
    vis, start = two_cycle()
    qc_lib.set_split(2)
    try:
        got, _ = gpu(qc_lib, vis, start, tol=1e-8, max_iter=10, prec="fp64", damping="full")
        assert (got[0].gain_flags == 2).all()
        got, st = gpu(qc_lib, vis, start, tol=1e-8, max_iter=0, prec="fp64", damping="lm")
        assert qc_lib.last_split_parts() == 2
    finally:
        qc_lib.set_split(0)
    assert (got[0].gain_flags == 0).all() and (st["iters"] == 0).all()
    np.testing.assert_array_equal(got[0].gains, start[0].gains)
