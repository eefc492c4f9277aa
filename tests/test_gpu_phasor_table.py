"""FP64 delay terms on the split schedule read their phasors from a table per
pass; phase-only and amplitude gains are formed once per pass: against the CPU
FP64 oracle (<= 1e-10 of the parameters, fixed iterations), several intervals in
time and frequency of unequal width, both data types, single terms and terms of a
chain, one wavefront chunk and several."""
import sys

import numpy as np
import pytest

from helpers import forward_data, make_term, make_vis, rand_c, unit_like
from oracle import solver as o_solver
from test_gpu_solve import gpu_solve

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("chained", [False, True])
@pytest.mark.parametrize("n_chan,f_int", [(17, 17), (70, 30), (40, 7)])
@pytest.mark.parametrize("kind", ["delay", "delay_offset", "phase", "amplitude"])
def test_parameter_terms_match_oracle(qc_lib, kind, n_chan, f_int, chained, dtype):
    rng = np.random.default_rng(n_chan + len(kind))
    n_ant, n_time = 6, 6
    vis = make_vis(rng, n_ant=n_ant, n_time=n_time, n_chan=n_chan, n_dir=2 if chained else 1, freq0=1.0e9, dfreq=4e6,
                   polarised=False)
    n_dir = vis.model.shape[2]
    truth = [make_term(rng, kind, n_time, n_chan, n_ant, t_int=2, f_int=f_int, n_dir=n_dir, scale=0.2)]
    truth[0].params = truth[0].params * (0.2 if kind.startswith("delay") else 1.0)
    if chained:
        truth.append(make_term(rng, "diag", n_time, n_chan, n_ant, t_int=3, f_int=n_chan, n_dir=n_dir, scale=0.2))
    vis.data = forward_data(vis, truth) + 0.02 * rand_c(rng, *vis.data.shape)
    vis.flag = (rng.random(vis.flag.shape) < 0.1).astype(np.uint8)
    if dtype == "c64":
        vis = vis.copy(data=vis.data.astype(np.complex64), model=vis.model.astype(np.complex64),
                       weight=vis.weight.astype(np.float32))
    start = [unit_like(truth[0])] + truth[1:]
    if kind.startswith("delay"):          # near the truth, as after a delay start
        start[0].params = truth[0].params * (1.0 + 1e-3 * rng.standard_normal(truth[0].params.shape))
    ref, _ = o_solver.solve_term(vis, start, 0, tol=-1.0, max_iter=4)
    scale = np.abs(ref[0].params).reshape(-1, ref[0].params.shape[-1]).max(0)
    for parts in (1, 3):
        say(f"{kind} {n_chan}/{f_int} chained={chained} {dtype} parts={parts}")
        qc_lib.set_split(parts)
        try:
            got, st = gpu_solve(qc_lib, vis, start, 0, tol=-1.0, max_iter=4, prec="fp64")
        finally:
            qc_lib.set_split(0)
        assert (st["iters"] == 4).all()
        assert (np.abs(got[0].params - ref[0].params) <= 1e-10 * np.maximum(scale, 1e-300)).all()
