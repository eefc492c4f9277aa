"""The matrix kernels of the warm-start network at the edges of their tiles
(16 x 16 and 32 x 32 outputs, 16-deep slices over four wavefronts): sizes below,
at and past them, row lengths that are no multiple of 4 and bases that are not
16-byte aligned (4-byte reads), against float64.  Tolerance: a sum of K products
in FP32, in any order, is within K 2^-24 of the sum of their magnitudes."""
import sys

import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EPS = 2.0 ** -24


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def within(got, want, magnitude, k):
    assert bool(((got.double() - want).abs() <= (k + 2) * EPS * magnitude + 1e-30).all())


@pytest.mark.parametrize("B,I,H,O", [(1, 8, 16, 4), (16, 16, 16, 16), (17, 31, 33, 15), (33, 56, 100, 28),
                                     (5, 513, 18, 257), (700, 64, 256, 60), (256, 512, 256, 256), (1100, 36, 512, 512)])
@pytest.mark.parametrize("shift", [0, 1])
def test_layers_match_float64(qc_lib, B, I, H, O, shift):
    say(f"mlp tiles B={B} I={I} H={H} O={O} shift={shift}")
    g = torch.Generator(device="cpu")
    g.manual_seed(B * 7 + I)
    n = H * I + H + O * H + O

    def rand(*shape):                                 # `shift` floats off a 16-byte boundary
        m = 1
        for x in shape:
            m *= x
        flat = torch.empty(m + 4, dtype=torch.float32, device=DEV)[shift:shift + m]
        flat.copy_(torch.randn(m, generator=g))
        return flat.view(*shape)

    params, x, dy = rand(n), rand(B, I), rand(B, O)
    W1, b1 = params[:H * I].view(H, I), params[H * I:H * I + H]
    W2, b2 = params[H * I + H:n - O].view(O, H), params[n - O:]
    y, pre = qc_lib.mlp_forward(params, x, H, O)
    grad = qc_lib.mlp_backward(params, x, pre, dy, H, O)
    torch.cuda.synchronize()
    d = lambda t: t.double()                          # noqa: E731
    within(pre, d(x) @ d(W1).T + d(b1), d(x).abs() @ d(W1).abs().T + d(b1).abs(), I)
    h = d(pre).clamp(min=0)
    within(y, h @ d(W2).T + d(b2), h @ d(W2).abs().T + d(b2).abs(), H)
    gW1, gb1 = grad[:H * I].view(H, I), grad[H * I:H * I + H]
    gW2, gb2 = grad[H * I + H:n - O].view(O, H), grad[n - O:]
    within(gW2, d(dy).T @ h, d(dy).abs().T @ h, B)
    within(gb2, d(dy).sum(0), d(dy).abs().sum(0), B)
    live = (d(pre) > 0).double()
    dh, dh_mag = (d(dy) @ d(W2)) * live, (d(dy).abs() @ d(W2).abs()) * live
    within(gW1, dh.T @ d(x), dh_mag.T @ d(x).abs(), B + O)
    within(gb1, dh.sum(0), dh_mag.sum(0), B + O)


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 4096, 4100, 70001])
@pytest.mark.parametrize("where", ["own", "y", "t", "shifted"])
def test_mse_in_and_out_of_place(qc_lib, n, where):
    say(f"mse n={n} {where}")
    g = torch.Generator(device="cpu")
    g.manual_seed(n)
    buf = torch.randn(3, n + 4, generator=g).to(DEV)
    k = 1 if where == "shifted" else 0
    y, t = buf[0, k:k + n].clone(), buf[1, k:k + n].clone()
    if where == "shifted":
        hold = torch.empty(n + 4, device=DEV)
        hold[1:1 + n] = y
        y = hold[1:1 + n]
    want, loss64 = 2 * (y - t) / n, ((y.double() - t.double()) ** 2).mean()
    loss = torch.zeros(1, device=DEV)
    dy = {"own": None, "y": y, "t": t, "shifted": None}[where]
    dy = qc_lib.mse_grad(y, t, dy=dy, loss=loss)
    torch.cuda.synchronize()
    assert bool(((dy - want).abs() <= 2 * EPS * want.abs() * 2).all())
    assert abs(float(loss) - float(loss64)) <= 4 * EPS * float(loss64)
