"""MIXED sums of per-antenna blocks over long runs of equal contributions, where
plain FP32 addition rounds every addend the same way and drifts: 8000 equal
addends are off by up to 1e-4 of the sum (measured with NumPy), a compensated sum
or one in FP64 by the rounding of the products alone.  Those are at most eight
roundings of 2^-24 in either block of the update, so 2e-6 of the update bounds it
with a factor of two to spare.  Gains against the CPU FP64 oracle on the same
complex64 values."""
import sys

import numpy as np
import pytest

from helpers import make_term, make_vis, unit_like
from oracle import solver as o_solver
from test_gpu_solve import gpu_solve

pytestmark = pytest.mark.gpu
TOL = 2e-6


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def constant_vis(n_time, rows_per_time, n_chan, n_dir):
    """One baseline, the same values in every row and channel."""
    rng = np.random.default_rng(5)
    vis = make_vis(rng, n_ant=2, n_time=n_time, n_chan=n_chan, n_dir=n_dir)
    n = n_time * rows_per_time
    vis.ant1 = np.zeros(n, np.int32)
    vis.ant2 = np.ones(n, np.int32)
    vis.row_time = np.repeat(np.arange(n_time), rows_per_time).astype(np.int32)
    vis.model = np.zeros((n, n_chan, n_dir, 4), np.complex64)
    for d in range(n_dir):
        vis.model[:, :, d, 0] = 1.1 + 0.3 * d
        vis.model[:, :, d, 3] = 0.9 - 0.2j + 0.1 * d
    vis.data = np.zeros((n, n_chan, 4), np.complex64)
    vis.data[..., 0] = 3.1 + 0.7j
    vis.data[..., 3] = 2.3 - 1.1j
    vis.weight = np.full((n, n_chan, 4), 0.77, np.float32)
    vis.flag = np.zeros((n, n_chan), np.uint8)
    return vis


def check(ctx, vis, chain, act, k):
    kw = dict(tol=-1.0, max_iter=k, damping="half")
    ref, _ = o_solver.solve_term(vis, chain, act, **kw)
    got, _ = gpu_solve(ctx, vis, chain, act, prec="mixed", **kw)
    sel = [0, 3]
    g, w = got[act].gains[..., sel], ref[act].gains[..., sel]
    step = np.abs(w - chain[act].gains[..., sel])
    assert step.min() > 0.1
    err = float((np.abs(g - w) / step).max())
    say(f"  largest error {err:.2e} of the update")
    assert err <= TOL


@pytest.fixture
def ctx(qc_lib):
    yield qc_lib
    qc_lib.set_split(0)
    qc_lib.set_tile(0, 0)


def test_directional_solve_over_a_long_run(ctx):
    """Two gain directions, one wavefront over 8000 rows of one antenna p."""
    say("directional MIXED sums, 8000 rows of one baseline")
    vis = constant_vis(8000, 1, 20, 2)
    rng = np.random.default_rng(7)
    dE = unit_like(make_term(rng, "diag", 8000, 20, 2, n_dir=2, dd=True))
    ctx.set_split(1)
    ctx.set_tile(1, 0)
    check(ctx, vis, [dE], 0, 1)


@pytest.mark.parametrize("rows", [4, 8])
@pytest.mark.parametrize("route", ["single", "chain", "folded chain"])
def test_one_channel_intervals_over_a_long_run(ctx, route, rows):
    """One-channel intervals whose one time repeats a baseline 8000 times, in two
    parts (the pass over 16 or 8 channels per wavefront): a single term, a chain of
    too few updates for the folded model, and one folded."""
    say(f"one-channel MIXED sums, 8000 rows of one time, {route}, {rows} rows per step")
    n_dir = 1 if route == "single" else 2
    vis = constant_vis(1, 8000, 10, n_dir)
    rng = np.random.default_rng(9)
    chain = [unit_like(make_term(rng, "diag", 1, 10, 2, f_int=1, n_dir=n_dir))]
    if route != "single":
        chain.append(unit_like(make_term(rng, "diag", 1, 10, 2, n_dir=n_dir)))
    ctx.set_split(2)
    ctx.set_tile(0, rows)
    check(ctx, vis, chain, 0, 3 if route == "folded chain" else 1)
