"""Which kernels a solve takes, asserted, and their results against the CPU FP64
oracle (FP64 <= 1e-10 in fixed-iteration mode, MIXED <= 1e-4, the bars of the other
solver tests): the band pass over chains that are not folded (FP64 over complex64,
or fewer than three updates) with no, one and two tabulated direction-dependent terms
and both step shapes, over rows with autocorrelations and repeated baselines; diagonal
chains with one gain direction folded and not folded, in MIXED and FP64; and the
intervals of a batch that teams share."""
import sys

import numpy as np
import pytest

from helpers import forward_data, make_term, make_vis, rand_c, unit_like
from oracle import solver as o_solver
from test_gpu_batch_team import problems
from test_gpu_solve import gpu_solve, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture
def ctx(qc_lib):
    yield qc_lib
    qc_lib.set_split(0)
    qc_lib.set_tile(0, 0)


def irregular(rng, vis):
    """The rows of vis shuffled within each time, two antennas' autocorrelations and
    a baseline given twice in neighbouring rows added."""
    rows = []
    for t in range(vis.n_time):
        idx = np.flatnonzero(vis.row_time == t)
        pairs = [(int(vis.ant1[i]), int(vis.ant2[i])) for i in idx] + [(0, 0), (3, 3)]
        rng.shuffle(pairs)
        k = int(rng.integers(len(pairs)))
        pairs.insert(k, pairs[k])
        rows += [(t, p, q) for p, q in pairs]
    n, n_chan, n_dir = len(rows), vis.n_chan, vis.n_dir
    model = rand_c(rng, n, n_chan, n_dir, 4)
    model[..., 1] = model[..., 2] = 0
    return vis.copy(row_time=np.array([r[0] for r in rows], np.int32), ant1=np.array([r[1] for r in rows], np.int32),
                    ant2=np.array([r[2] for r in rows], np.int32), model=model,
                    weight=rng.uniform(0.5, 2.0, (n, n_chan, 4)), data=np.zeros((n, n_chan, 4), np.complex128),
                    flag=np.zeros((n, n_chan), np.uint8))


def chain_problem(seed, f_int, n_dd, dtype, n_ant=7, n_time=9, n_chan=21, n_dir=3):
    """K (delay), G (diagonal, 3 times x f_int channels, from unit gains) and n_dd
    direction-dependent diagonal terms at the truth, noise and 15% flags."""
    rng = np.random.default_rng(seed)
    vis = irregular(rng, make_vis(rng, n_ant=n_ant, n_time=n_time, n_chan=n_chan, n_dir=n_dir))
    truth = [make_term(rng, "delay", n_time, n_chan, n_ant, t_int=5, f_int=n_chan, n_dir=n_dir),
             make_term(rng, "diag", n_time, n_chan, n_ant, t_int=3, f_int=f_int, n_dir=n_dir, scale=0.3)]
    truth[0].params = truth[0].params * 0.3
    for k in range(n_dd):
        truth.append(make_term(rng, "diag", n_time, n_chan, n_ant, t_int=4 - k, f_int=7 + 3 * k, n_dir=n_dir, dd=True,
                               scale=0.15))
    vis.data = forward_data(vis, truth) + 0.02 * rand_c(rng, *vis.data.shape)
    vis.flag = (rng.random(vis.flag.shape) < 0.15).astype(np.uint8)
    if dtype == "c64":
        vis = vis.copy(data=vis.data.astype(np.complex64), model=vis.model.astype(np.complex64),
                       weight=vis.weight.astype(np.float32))
    return vis, [truth[0], unit_like(truth[1])] + truth[2:]


def solve_and_check(ctx, vis, chain, prec, k, parts, rows=0):
    ref, rst = o_solver.solve_term(vis, chain, 1, tol=-1.0, max_iter=k)
    ctx.set_split(parts)
    ctx.set_tile(0, rows)
    got, st = gpu_solve(ctx, vis, chain, 1, tol=-1.0, max_iter=k, prec=prec)
    assert (st["iters"] == k).all()
    np.testing.assert_array_equal(got[1].gain_flags, ref[1].gain_flags)
    np.testing.assert_allclose(st["chisq_first"], rst["chisq_first"], rtol=1e-11 if prec == "fp64" else 1e-5)
    e = rel_err(got[1].gains, ref[1].gains, "diag")
    say(f"  largest relative difference {e:.2e}")
    assert e <= (1e-10 if prec == "fp64" else 1e-4)


@pytest.mark.parametrize("rows", [4, 8])
@pytest.mark.parametrize("n_dd", [0, 1, 2])
@pytest.mark.parametrize("dtype,prec,k", [("c64", "fp64", 4), ("c128", "fp64", 2), ("c64", "mixed", 2)])
def test_band_pass_over_an_unfolded_chain(ctx, dtype, prec, k, n_dd, rows):
    from paper_2412_10072_amd import qc
    say(f"band pass, {dtype} {prec}, {n_dd} tables, {rows} rows per step")
    vis, chain = chain_problem(700 + n_dd, 1, n_dd, dtype)
    for parts in (2, 5):
        solve_and_check(ctx, vis, chain, prec, k, parts, rows)
        assert ctx.last_route() == qc.ROUTE_SPLIT | qc.ROUTE_BAND


@pytest.mark.parametrize("n_dd", [0, 2])
@pytest.mark.parametrize("dtype,prec", [("c64", "mixed"), ("c128", "fp64"), ("c64", "fp64")])
@pytest.mark.parametrize("f_int", [1, 3, 21])
def test_folded_and_unfolded_chains(ctx, f_int, dtype, prec, n_dd):
    """Fewer than three updates and FP64 over complex64 leave the chain unfolded."""
    from paper_2412_10072_amd import qc
    say(f"chain of intervals of {f_int} channels, {dtype} {prec}, {n_dd} tables")
    vis, chain = chain_problem(710 + n_dd, f_int, n_dd, dtype)
    for k in (2, 4):
        for parts in (1, 3):
            solve_and_check(ctx, vis, chain, prec, k, parts)
            stored = prec == "mixed" or dtype == "c128"         # the model is stored as it is computed
            folded = k >= 3 and stored and (f_int == 21 or (f_int == 1 and parts > 1))
            want = (qc.ROUTE_SPLIT if parts > 1 else 0) | (qc.ROUTE_FOLD if folded else 0)
            if f_int == 1 and parts > 1:
                want |= qc.ROUTE_BAND
            assert ctx.last_route() == want, (k, parts)


@pytest.mark.parametrize("dtype,prec", [("c128", "fp64"), ("c64", "fp64"), ("c64", "mixed")])
def test_team_intervals(qc_lib, dtype, prec):
    """The batch of test_gpu_batch_team: parts of 2048 samples, so the second
    interval (108000 samples, the largest) has seven groups of eight, the last one
    of five, the third one ragged group more than one, and the fourth problem is not
    a team's."""
    from paper_2412_10072_amd import qc
    say(f"team intervals, {dtype} {prec}")
    host, dev = problems(dtype)
    b = qc.Batch(qc_lib, dev, tol=-1.0, max_iter=3, prec=prec)
    assert b.teams() == [53, 16, 11]
    b.run()
    qc_lib.sync()
    for (vis, term), (_, t), st in zip(host, dev, b.stats):
        ref, _ = o_solver.solve_term(vis, [term], 0, tol=-1.0, max_iter=3)
        e = rel_err(t.gains.cpu().numpy(), ref[0].gains, term.kind)
        assert e <= (1e-10 if prec == "fp64" else 1e-4)
        assert (st["iters"].cpu().numpy() == 3).all()
    b.close()


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("n_ant", [35, 36, 86, 171, 256])
def test_band_pass_by_antennas(ctx, n_ant, k):
    """The antenna counts where the step's shape and the LDS limit change (MIXED 4 x 16
    steps to 35, 8 x 8 beyond, over 64 KiB from 171; FP64 to 170), the band pass over
    the chain (2 updates) and over the folded model (3)."""
    from paper_2412_10072_amd import qc
    say(f"band pass, {n_ant} antennas, {k} updates")
    rng = np.random.default_rng(n_ant)
    n_chan, n_dir = 3, 2
    vis = make_vis(rng, n_ant=n_ant, n_time=1, n_chan=n_chan, n_dir=n_dir, polarised=False)
    vis.data = vis.model.sum(axis=2) + 0.1 * rand_c(rng, *vis.data.shape)
    vis = vis.copy(data=vis.data.astype(np.complex64), model=vis.model.astype(np.complex64),
                   weight=vis.weight.astype(np.float32))
    chain = [make_term(rng, "phase", 1, n_chan, n_ant, n_dir=n_dir, scale=0.02),
             unit_like(make_term(rng, "diag", 1, n_chan, n_ant, f_int=1, n_dir=n_dir))]
    solve_and_check(ctx, vis, chain, "mixed", k, 3)
    assert ctx.last_route() == qc.ROUTE_SPLIT | qc.ROUTE_BAND | (qc.ROUTE_FOLD if k >= 3 else 0)
    if k == 2:
        solve_and_check(ctx, vis, chain, "fp64", k, 3)
        assert ctx.last_route() == qc.ROUTE_SPLIT | (qc.ROUTE_BAND if n_ant <= 170 else 0)
