"""Solves of a diagonal chain's term over the folded model (the fixed terms and
directions summed once per solve), against the CPU FP64 oracle (FP64 <= 1e-10
in fixed-iteration mode), beside the unfolded route that fewer than three updates
take: fixed terms with and without tables, one and several model directions,
channel counts that the fold takes by rows and flat, non-finite values under
flags, one-channel intervals right of untabulated terms."""
import sys

import numpy as np
import pytest

from helpers import forward_data, make_term, make_vis, rand_c, unit_like
from oracle import solver as o_solver
from test_gpu_solve import gpu_solve, rel_err

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def problem(seed, kinds, n_chan, n_dir, n_ant=7, n_time=6):
    """A chain of (kind, t_int, f_int, direction dependent) terms near the truth,
    the first one at unit gains, 15% flags with NaN data and model under some."""
    rng = np.random.default_rng(seed)
    vis = make_vis(rng, n_ant=n_ant, n_time=n_time, n_chan=n_chan, n_dir=n_dir, freq0=1.0e9, dfreq=2e6, polarised=False)
    chain = []
    for kind, t_int, f_int, dd in kinds:
        t = make_term(rng, kind, n_time, n_chan, n_ant, t_int=t_int, f_int=min(f_int, n_chan), n_dir=n_dir, dd=dd, scale=0.2)
        if kind == "delay":
            t.params = t.params * 0.3
        chain.append(t)
    vis.data = forward_data(vis, chain) + 0.02 * rand_c(rng, *vis.data.shape)
    vis.flag = (rng.random(vis.flag.shape) < 0.15).astype(np.uint8)
    bad = (vis.flag != 0) & (rng.random(vis.flag.shape) < 0.3)
    clean = vis.copy(data=vis.data.copy(), model=vis.model.copy())
    vis.data[bad] = np.nan
    vis.model[bad] = np.nan
    return vis, clean, [unit_like(chain[0])] + chain[1:]


CHAINS = {
    "several_directions": ([("diag", 2, 1000, False)], 3),
    "tables": ([("diag", 2, 1000, False), ("delay", 6, 1000, False), ("diag", 3, 20, True)], 3),
    "three_dd_terms": ([("diag", 1, 1000, False), ("diag", 3, 20, True), ("phase", 2, 30, True), ("diag", 6, 9, True)], 2),
    "one_direction": ([("phase", 2, 1000, False), ("diag", 1, 25, False)], 1),
    "delay": ([("delay", 3, 1000, False), ("diag", 1, 1000, False), ("diag", 2, 40, True)], 4),
    "one_channel": ([("diag", 3, 1, False), ("delay", 6, 1000, False), ("phase", 3, 10, True)], 3),
}


@pytest.mark.parametrize("n_chan", [18, 64, 70])
@pytest.mark.parametrize("name", sorted(CHAINS))
def test_fold_matches_oracle(qc_lib, name, n_chan):
    kinds, n_dir = CHAINS[name]
    vis, clean, chain = problem(sum(map(ord, name)) + n_chan, kinds, n_chan, n_dir)
    for parts in (1, 3):
        for k in (2, 4):
            say(f"fold {name} {n_chan} channels, {parts} parts, {k} updates")
            ref, rst = o_solver.solve_term(clean, chain, 0, tol=-1.0, max_iter=k)
            qc_lib.set_split(parts)
            try:
                got, st = gpu_solve(qc_lib, vis, chain, 0, tol=-1.0, max_iter=k, prec="fp64")
            finally:
                qc_lib.set_split(0)
            assert (st["iters"] == k).all()
            np.testing.assert_allclose(st["chisq_first"], rst["chisq_first"], rtol=1e-10)
            if chain[0].kind == "diag":
                assert rel_err(got[0].gains, ref[0].gains, "diag") <= 1e-10
            else:
                scale = max(np.abs(ref[0].params).max(), 1e-300)
                assert np.abs(got[0].params - ref[0].params).max() <= 1e-10 * scale
