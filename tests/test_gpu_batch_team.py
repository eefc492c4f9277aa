"""Batched solves whose intervals are shared by teams of workgroups (too large
for one workgroup beside the rest of the batch): against the CPU FP64 oracle
(FP64 <= 1e-10 in fixed-iteration mode, MIXED <= 1e-4 at tol 1e-6, the bars of
the other batch tests), with one and with several groups of parts, a ragged
last group, both term types, divergence flags, and repeated launches bitwise
equal."""
import sys

import numpy as np
import pytest
import torch

from helpers import forward_data, make_term, make_vis
from oracle import solver as o_solver
from test_gpu_batch import rel_err
from test_gpu_solve import noisy_problem

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (antennas, times, channels, kind): about 14, 40, 7 and 5 parts of the first
# three intervals' rows, the last problem too small for a team
SHAPES = [(9, 50, 18, "diag"), (10, 60, 40, "c2x2"), (7, 64, 16, "diag"), (5, 6, 20, "c2x2")]


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def problems(dtype):
    from paper_2412_10072_amd import qc
    host, dev = [], []
    for i, (n_ant, n_time, n_chan, kind) in enumerate(SHAPES):
        vis, chain = noisy_problem(600 + i, n_ant=n_ant, n_time=n_time, n_chan=n_chan, kind=kind, t_int=n_time,
                                   f_int=n_chan, n_wcorr=1 if i == 1 else 4)
        if dtype == "c64":
            vis = vis.copy(data=vis.data.astype(np.complex64), model=vis.model.astype(np.complex64),
                           weight=vis.weight.astype(np.float32))
        host.append((vis, chain[0]))
        dev.append((qc.device_vis(vis, DEV), qc.device_term(chain[0], DEV)))
    return host, dev


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("k", [0, 1, 4])
def test_team_fp64_fixed_iterations(qc_lib, dtype, k):
    from paper_2412_10072_amd import qc
    say(f"batch teams fp64 {dtype}, {k} updates")
    host, dev = problems(dtype)
    b = qc.Batch(qc_lib, dev, tol=-1.0, max_iter=k, prec="fp64")
    b.run()
    qc_lib.sync()
    for (vis, term), (_, t), st in zip(host, dev, b.stats):
        ref, rst = o_solver.solve_term(vis, [term], 0, tol=-1.0, max_iter=k)
        assert rel_err(t.gains.cpu().numpy(), ref[0].gains, term.kind) <= 1e-10
        np.testing.assert_array_equal(st["iters"].cpu().numpy(), rst["iters"])
        np.testing.assert_allclose(st["chisq_first"].cpu().numpy(), rst["chisq_first"], rtol=1e-11)
        np.testing.assert_allclose(st["chisq_last"].cpu().numpy(), rst["chisq_last"], rtol=1e-10)
    b.close()


def test_team_mixed_replays_are_equal(qc_lib):
    from paper_2412_10072_amd import qc
    say("batch teams mixed, replays")
    host, dev = problems("c64")
    init = [t.gains.clone() for _, t in dev]
    b = qc.Batch(qc_lib, dev, tol=1e-6, max_iter=100, prec="mixed")
    outs = []
    for _ in range(4):
        for (_, t), g0 in zip(dev, init):
            t.gains.copy_(g0)
        junk = torch.randn(1 << 20, device=DEV).sum()       # unrelated eager work between the launches
        b.run()
        torch.cuda.synchronize()
        assert torch.isfinite(junk)
        outs.append([t.gains.cpu().numpy() for _, t in dev])
    for o in outs[1:]:
        for x, y in zip(outs[0], o):
            assert np.array_equal(x, y)
    for (vis, term), (_, t), st in zip(host, dev, b.stats):
        ref, _ = o_solver.solve_term(vis, [term], 0, tol=1e-6, max_iter=100)
        assert rel_err(t.gains.cpu().numpy(), ref[0].gains, term.kind) <= 1e-4
        assert st["converged"].cpu().numpy().all()
    b.close()


def test_team_divergence_flags(qc_lib):
    """FULL steps from c times the truth of noise-free data: the scale 2-cycle
    of test_gpu_divergence.two_cycle, in an interval of many parts."""
    from paper_2412_10072_amd import qc
    say("batch teams, divergence flags")
    rng = np.random.default_rng(71)
    vis = make_vis(rng, n_ant=8, n_time=60, n_chan=16, n_dir=1, polarised=False)
    truth = [make_term(rng, "diag", 60, 16, 8, t_int=60, f_int=16)]
    vis.data = forward_data(vis, truth)
    start = o_solver.copy_chain(truth)
    start[0].gains = truth[0].gains * 1.3
    ref, _ = o_solver.solve_term(vis, start, 0, tol=1e-8, max_iter=10, damping="full")
    assert (ref[0].gain_flags == 2).all()
    td = qc.device_term(start[0], DEV)
    b = qc.Batch(qc_lib, [(qc.device_vis(vis, DEV), td)], tol=1e-8, max_iter=10, prec="fp64", damping="full")
    b.run()
    qc_lib.sync()
    np.testing.assert_array_equal(td.gain_flags.cpu().numpy(), ref[0].gain_flags)
    b.close()
