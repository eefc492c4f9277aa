"""Calls on two streams of one context whose kernels overlap: each gives bit for
bit what it gives alone, though both use the context's scratch memory (the outputs'
chain table, the split
solves' state)."""
import sys

import pytest
import torch

from synth.problem import Term, Vis

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def device_problem(seed, n_ant, n_time, n_chan, t_int, f_int, dtype=torch.complex64):
    """Random data and model of one direction and a diagonal term near unit gains,
    made on the device."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    real = torch.float32 if dtype == torch.complex64 else torch.float64
    p, q = torch.triu_indices(n_ant, n_ant, offset=1)
    n = p.numel() * n_time

    def cnormal(*shape, dt=real):
        return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device=DEV, dtype=dt))
    i32 = dict(dtype=torch.int32, device=DEV)
    vis = Vis(data=cnormal(n, n_chan, 4), model=cnormal(n, n_chan, 1, 4),
              weight=torch.rand(n, n_chan, 4, generator=g, device=DEV, dtype=real) + 0.5,
              flag=torch.zeros(n, n_chan, dtype=torch.uint8, device=DEV), ant1=p.repeat(n_time).to(**i32),
              ant2=q.repeat(n_time).to(**i32), row_time=torch.arange(n_time).repeat_interleave(p.numel()).to(**i32),
              chan_freq=1.0e9 + 1.0e6 * torch.arange(n_chan, dtype=torch.float64, device=DEV), n_ant=n_ant, n_time=n_time)
    t_map = (torch.arange(n_time) // t_int).to(**i32)
    f_map = (torch.arange(n_chan) // f_int).to(**i32)
    shape = (int(t_map.max()) + 1, int(f_map.max()) + 1, n_ant, 1)
    gains = torch.zeros(*shape, 4, dtype=torch.complex128, device=DEV)
    gains[..., 0] = 1 + 0.2 * cnormal(*shape, dt=torch.float64)
    gains[..., 3] = 1 + 0.2 * cnormal(*shape, dt=torch.float64)
    term = Term(kind="diag", t_map=t_map, f_map=f_map, d_map=torch.zeros(1, **i32), n_gt=shape[0], n_gf=shape[1],
                n_gdir=1, gains=gains, params=None, gain_flags=torch.zeros(shape, dtype=torch.int8, device=DEV),
                direction_dependent=False, name="G")
    return vis, term


def test_outputs_with_tables_on_two_streams(qc_lib):
    """Residuals through one solution per channel (tabulated) of two problems."""
    say("tabulated residuals on two streams")
    probs = [device_problem(11 + i, 40, 20, 512 - 64 * i, 1, 1) for i in range(2)]
    alone = []
    for vis, term in probs:
        alone.append(qc_lib.residual(vis, [term]))
        torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in probs]
    outs = [torch.empty_like(a) for a in alone]
    torch.cuda.synchronize()
    for _ in range(5):
        for (vis, term), s, out in zip(probs, streams, outs):
            qc_lib.residual(vis, [term], out=out, stream=s)
        torch.cuda.synchronize()
        for a, out in zip(alone, outs):
            assert torch.equal(a, out)
            out.zero_()
        torch.cuda.synchronize()


def test_first_calls_of_a_context_on_a_side_stream():
    """Nothing of the context is in use yet: a solve and a tabulated residual on a
    stream of their own give what they give on the default stream."""
    from paper_2412_10072_amd import qc
    say("first calls on a side stream")
    vis, term = device_problem(31, 24, 20, 64, 1, 1)
    start = term.gains.clone()
    out = []
    for stream in (None, torch.cuda.Stream()):
        ctx = qc.Context(0)
        term.gains.copy_(start)
        torch.cuda.synchronize()
        r = torch.empty_like(vis.data)
        torch.cuda.synchronize()
        ctx.residual(vis, [term], out=r, stream=stream)
        ctx.solve(vis, [term], 0, tol=-1.0, max_iter=2, prec="mixed", stream=stream)
        assert ctx.last_kernel_ms() > 0.0
        torch.cuda.synchronize()
        out.append((r, term.gains.clone()))
        ctx.close()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_split_solves_on_two_streams(qc_lib):
    """Solves that stop at max_iter with their last pass in flight, beside one
    another and beside a residual: unlike sizes, so that every range, block count and
    part differs."""
    say("split solves on two streams")
    probs = [device_problem(21 + i, 24 - 10 * i, 60 - 20 * i, 256 - 192 * i, 60, 128 - 64 * i) for i in range(2)]
    start = [t.gains.clone() for _, t in probs]
    kw = dict(tol=-1.0, prec="mixed")

    def solve(i, k, **more):
        vis, term = probs[i]
        return qc_lib.solve(vis, [term], 0, max_iter=k, **kw, **more)

    def reset():
        torch.cuda.synchronize()
        for (_, t), g in zip(probs, start):
            t.gains.copy_(g)
        torch.cuda.synchronize()
    for k in (1, 3):
        alone = []
        for i in range(2):
            st = solve(i, k)
            assert qc_lib.last_split_parts() > 1
            torch.cuda.synchronize()
            alone.append((probs[i][1].gains.clone(), {n: v.clone() for n, v in st.items()}))
        resid = qc_lib.residual(probs[1][0], [probs[1][1].copy(gains=start[1])])
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(2)]
        out = torch.empty_like(resid)
        for order in ((0, 1), (1, 0)):
            reset()
            got = {i: {n: torch.zeros_like(v) for n, v in alone[i][1].items()} for i in range(2)}
            torch.cuda.synchronize()
            for i in order:
                solve(i, k, stream=streams[i], stats=got[i])
            torch.cuda.synchronize()
            for i in range(2):
                assert torch.equal(probs[i][1].gains, alone[i][0])
                for n, v in got[i].items():
                    assert torch.equal(v, alone[i][1][n]), n
        reset()
        solve(0, k, stream=streams[0], stats=got[0])
        qc_lib.residual(probs[1][0], [probs[1][1]], out=out, stream=streams[1])
        torch.cuda.synchronize()
        assert torch.equal(out, resid) and torch.equal(probs[0][1].gains, alone[0][0])
        reset()
