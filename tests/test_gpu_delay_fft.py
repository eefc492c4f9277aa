"""The delay start's transforms at every length (an odd and an even number of
radix-2 stages, none a power of two, the longest that fits): the same grid
argmax as the oracle's direct sum, in FP64 on both sides."""
import numpy as np
import pytest

from helpers import forward_data, make_term, make_vis, rand_c
from oracle import delay_init as o_delay

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_chan", [2, 3, 4, 5, 8, 9, 17, 33, 100, 129, 300, 512, 513, 1024])
def test_delay_init_lengths(qc_lib, n_chan):
    from paper_2412_10072_amd import qc
    print(f"delay init, {n_chan} channels", flush=True)
    rng = np.random.default_rng(67)
    vis = make_vis(rng, n_ant=4, n_time=2, n_chan=n_chan, polarised=False, freq0=1.0e9, dfreq=1e9 / n_chan)
    truth = [make_term(rng, "delay", 2, n_chan, 4, t_int=2, f_int=n_chan)]
    vis.data = forward_data(vis, truth) + 0.05 * rand_c(rng, *vis.data.shape)
    ref = o_delay.delay_init(vis, truth, 0, ref_ant=0)
    K = qc.device_term(truth[0], "cuda:0")
    qc_lib.delay_init(qc.device_vis(vis, "cuda:0"), K, ref_ant=0)
    qc_lib.sync()
    assert np.array_equal(K.params.cpu().numpy(), ref[0].params)
