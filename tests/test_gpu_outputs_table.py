"""Outputs whose chain is read from a table, or whose wavefronts run over rows:
corrupted model, residual, corrected data and corrected weights against the
CPU oracle, for channel counts on both sides of a wavefront's 64 (and of the
row form's limit), chains with and without a table, both data types, a masked
direction.  Bars as in test_gpu_solve.test_outputs_match_oracle."""
import sys

import numpy as np
import pytest

from helpers import forward_data, make_term, make_vis, rand_c
from oracle import outputs as o_out
from oracle import robust as o_rob

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def chain_of(rng, name, n_time, n_chan, n_ant, n_dir):
    def t(kind, t_int, f_int, dd=False):
        return make_term(rng, kind, n_time, n_chan, n_ant, t_int=t_int, f_int=f_int, n_dir=n_dir, dd=dd, scale=0.2)
    if name == "per_channel":
        return [t("diag", 1, 1)]
    if name == "per_channel_full":
        return [t("c2x2", 2, 1)]
    if name == "wide":
        return [t("diag", 1, n_chan)]
    if name == "two_full":
        return [t("diag", 1, n_chan), t("c2x2", n_time, 3)]
    if name == "phasor":
        return [t("phase", 1, n_chan)]
    return [t("phase", n_time, n_chan), t("diag", 1, 2), t("diag", 2, 5, dd=True)]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n_chan", [7, 48, 64, 100, 130])
@pytest.mark.parametrize("name", ["per_channel", "per_channel_full", "wide", "two_full", "phasor", "directions"])
def test_outputs_match_oracle(qc_lib, name, n_chan, dtype):
    from paper_2412_10072_amd import qc
    say(f"outputs {name} {n_chan} channels {dtype}")
    rng = np.random.default_rng(n_chan)
    n_ant, n_time = 10, 3
    n_dir = 3 if name == "directions" else 1
    n_wcorr = 1 if n_chan == 48 else 4
    vis = make_vis(rng, n_ant=n_ant, n_time=n_time, n_chan=n_chan, n_dir=n_dir, n_wcorr=n_wcorr)
    chain = chain_of(rng, name, n_time, n_chan, n_ant, n_dir)
    vis.data = forward_data(vis, chain) + 0.05 * rand_c(rng, *vis.data.shape)
    if dtype == "c64":
        vis = vis.copy(data=vis.data.astype(np.complex64), model=vis.model.astype(np.complex64),
                       weight=vis.weight.astype(np.float32))
    tol = 1e-12 if dtype == "c128" else 2e-5
    vis_d = qc.device_vis(vis, DEV)
    chain_d = [qc.device_term(t, DEV) for t in chain]
    scale = np.abs(vis.data).max()
    mask = np.array([1, 0, 1], np.uint8)[:n_dir] if n_dir > 1 else None
    assert np.abs(qc_lib.residual(vis_d, chain_d).cpu().numpy() - o_out.residual(vis, chain)).max() <= tol * scale
    V = qc_lib.apply(vis_d, chain_d, "corrupt", dir_mask=mask).cpu().numpy()
    assert np.abs(V - o_out.corrupt(vis, chain, mask)).max() <= tol * scale
    if name != "directions":
        want = o_out.correct(vis, chain)
        got = qc_lib.apply(vis_d, chain_d, "correct").cpu().numpy()
        assert np.abs(got - want).max() <= tol * np.abs(want).max()
        want = o_rob.corrected_weights(vis, chain)
        got = qc_lib.corrected_weights(vis_d, chain_d).cpu().numpy()
        assert np.abs(got - want).max() <= tol * np.abs(want).max()
    # singular antenna: zeros
    if name == "per_channel_full":
        chain[0].gains[:, :, 2] = 0.0
        got = qc_lib.apply(vis_d, [qc.device_term(chain[0], DEV)], "correct").cpu().numpy()
        hit = (np.asarray(vis.ant1) == 2) | (np.asarray(vis.ant2) == 2)
        assert (got[hit] == 0).all() and np.isfinite(got).all()
    qc_lib.sync()
