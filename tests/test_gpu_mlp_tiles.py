"""The decoder kernels where a tile of 32 points, a workgroup's wavefronts or a row of four values ends: batches around those sizes, widths that are
no multiple of four, arrays that are not aligned.  Against the fp64 oracle with the bars of test_gpu_mlp.py (three roundings to fp16: 2e-3 of
the magnitudes)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
from test_gpu_mlp import backward_reference, check, dev, make_case

pytestmark = pytest.mark.gpu


def shifted(t, by):
    """The same values, contiguous, `by` elements behind an aligned address."""
    room = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    room[by:] = t.reshape(-1)
    return room[by:].view(t.shape)


@pytest.mark.parametrize("n_in,n_out,io,N,by", [
    (32, 4, cngp.F16, 31, 0), (32, 4, cngp.F32, 33, 0), (32, 16, cngp.F16, 32, 0),      # a tile and its neighbours
    (24, 8, cngp.F16, 255, 0), (16, 12, cngp.F32, 257, 0), (8, 9, cngp.F16, 513, 0),    # a workgroup of eight wavefronts, two tiles each
    (30, 3, cngp.F16, 1025, 0), (5, 1, cngp.F32, 97, 0), (17, 15, cngp.F16, 64, 0),     # rows read value by value
    (32, 4, cngp.F16, 300, 1), (16, 4, cngp.F32, 65, 1), (32, 16, cngp.F16, 70001, 3),  # unaligned; more tiles than wavefronts
])
def test_mlp_at_the_ends_of_tiles(n_in, n_out, io, N, by):
    y, W1, W2, W3, dout = make_case(4000 + n_in * 50 + n_out + N, N, n_in, n_out, io)
    tdt = torch.float16 if io == cngp.F16 else torch.float32
    W = shifted(dev(np.concatenate([W1.ravel(), W2.ravel(), W3.ravel()]), torch.float16), by)
    yd, dd = shifted(dev(y, tdt), by), shifted(dev(dout, torch.float32), by)
    cfg = cngp.MlpConfig(n_in, n_out, io, flags=cngp.ZERO_GRADS)
    out = shifted(torch.full((N, n_out), float("nan"), device="cuda"), by)
    dy = shifted(torch.full((N, n_in), float("nan"), dtype=tdt, device="cuda"), by)
    gW = torch.full((cfg.weight_count,), float("nan"), device="cuda")
    cngp.mlp_fwd(cfg, yd, W, out)
    cngp.mlp_bwd(cfg, yd, W, dd, dy, gW)
    torch.cuda.synchronize()
    ref, mag, _ = oracle.mlp_fwd(y, W1, W2, W3, want_mag=True)
    check("out", out.cpu().numpy(), ref, mag)
    g, gm, slack, _ = backward_reference(y, W1, W2, W3, dout, io)
    check("dy", dy.float().cpu().numpy(), g["dy"], gm["dy"], slack["dy"])
    for name, t in zip(("dW1", "dW2", "dW3"), cfg.split(gW)):
        check(name, t.cpu().numpy(), g[name], gm[name], slack[name])


@pytest.mark.parametrize("n_in,io", [(32, cngp.F16), (20, cngp.F32), (6, cngp.F16)])
def test_a_point_that_is_not_finite_stays_alone(n_in, io):
    """The last point of a ragged tile is what lanes without a point read instead, a point's first input what columns beyond n_in do."""
    N, n_out = 32 * 5 + 7, 3
    bad = N - 1
    y, W1, W2, W3, dout = make_case(77 + n_in, N, n_in, n_out, io)
    tdt = torch.float16 if io == cngp.F16 else torch.float32
    W = dev(np.concatenate([W1.ravel(), W2.ravel(), W3.ravel()]), torch.float16)
    cfg = cngp.MlpConfig(n_in, n_out, io, flags=cngp.ZERO_GRADS)
    clean, dd = dev(y, tdt), dev(dout, torch.float32)
    dirty = clean.clone()
    dirty[bad] = float("inf")
    dirty[bad, 0] = float("nan")
    keep = [n for n in range(N) if n != bad]
    assert torch.equal(cngp.mlp_fwd(cfg, dirty, W)[keep], cngp.mlp_fwd(cfg, clean, W)[keep])
    assert torch.equal(cngp.mlp_bwd(cfg, dirty, W, dd)[0][keep], cngp.mlp_bwd(cfg, clean, W, dd)[0][keep])
