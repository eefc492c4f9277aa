"""The prediction of small skies over groups of rows (one row, two or four to a
wavefront, the directions of a sample turned through the LDS or stored as they
come): at the edges of the groups, of the 64-channel steps and of the
choices, against the CPU FP64 oracle with the tolerance of the other prediction
tests."""
import sys

import numpy as np
import pytest

from oracle import predict as o_pred
from test_gpu_predict import random_sky, run, tolerance, uvw_rows

pytestmark = pytest.mark.gpu


def check(qc_lib, dtype, n_row, n_chan, n_comp, n_dir, spectral, pol, seed=601):
    print(f"predict rows {dtype}: {n_row} x {n_chan}, {n_comp} components, {n_dir} directions", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(seed)
    lm, st, spi, nu0, d = random_sky(rng, n_comp, n_dir, pol=pol)
    sky = (lm, st, spi if spectral else np.zeros_like(spi), nu0, d)
    uvw = uvw_rows(rng, n_row)
    nu = np.linspace(0.9e9, 1.6e9, n_chan)
    got = run(qc_lib, uvw, nu, sky, n_dir, dtype)
    want = o_pred.predict_dft(uvw, nu, *sky, n_dir)
    assert np.abs(got - want).max() <= tolerance(uvw, nu, sky, dtype)
    return got


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n_dir", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("spectral,pol", [(False, False), (True, False), (False, True), (True, True)])
def test_small_skies(qc_lib, dtype, n_dir, spectral, pol):
    for n_row, n_chan in ((1, 1), (9, 63), (7, 65), (2, 130)):
        check(qc_lib, dtype, n_row, n_chan, 3 * n_dir, n_dir, spectral, pol)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n_dir", [1, 3, 5])
def test_rows_in_groups_of_four(qc_lib, dtype, n_dir):
    check(qc_lib, dtype, 16387, 5, 2 * n_dir, n_dir, True, True)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n_comp", [24, 25, 64, 65, 256, 257])
def test_component_counts(qc_lib, dtype, n_comp):
    check(qc_lib, dtype, 11, 67, n_comp, 3, False, True)


def test_unaligned_output(qc_lib):
    import torch
    print("predict rows: unaligned output", flush=True)
    rng = np.random.default_rng(603)
    sky = random_sky(rng, 8, 4)
    uvw, nu = uvw_rows(rng, 10), np.linspace(0.9e9, 1.6e9, 70)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (uvw, nu, *sky)]
    n = 10 * 70 * 4 * 4
    flat = torch.empty(n + 1, dtype=torch.complex64, device="cuda:0")
    whole = qc_lib.predict(*dev, n_dir=4, dtype="c64", out=flat[:n].view(10, 70, 4, 4)).clone()
    off = qc_lib.predict(*dev, n_dir=4, dtype="c64", out=flat[1:].view(10, 70, 4, 4))
    qc_lib.sync()
    assert torch.equal(whole, off)
