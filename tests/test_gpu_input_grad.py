"""GPU parity of cngp_encode_bwd_input (gradient of the forward pass with respect to the points) against
the oracle: fp32 arithmetic on exactly representable inputs, so the bar is the fp32 one, relative to the
sum of the magnitudes of the terms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu
DEV = "cuda"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def run(w, fmt, n=None, edge_points=True):
    x = W.make_points(w, n)
    if edge_points:
        x[:4] = [[0.0] * w.d, [1.0] * w.d, [0.5] * w.d, [1.0] + [0.0] * (w.d - 1)]
    D_f = W.make_feature_codebook(w)
    D_f = (D_f.astype(np.float64) * 1e4).astype(D_f.dtype)
    D_c = oracle.bake_probes(W.make_probe_logits(w))
    dy = W.make_upstream_grad(w, x.shape[0])
    D_c_dev = {cngp.IDX_U8: lambda: dev(D_c), cngp.IDX_PACKED4: lambda: cngp.pack4(dev(D_c)),
               cngp.IDX_BITS: lambda: dev(oracle.pack_index_bits(D_c, w.N_p))}[fmt]()
    cfg = cngp.Config.from_workload(w, index_format=fmt)
    gx = torch.full((x.shape[0], w.d), float("nan"), device=DEV)
    cngp.encode_bwd_input(cfg, dev(x), dev(D_f), D_c_dev, dev(dy), gx)
    torch.cuda.synchronize()
    ref, mag = oracle.encode_bwd_input(w, x, D_f, D_c, dy)
    return check_close("dL/dx", gx.cpu().numpy(), ref, mag, fp16_out=False)


@pytest.mark.parametrize("d,N_p,feat,io", [(2, 1, "f32", "f32"), (2, 8, "f16", "f16"), (3, 4, "f32", "f16"),
                                           (3, 16, "f16", "f16"), (3, 16, "f32", "f32"), (3, 2, "f16", "f32")])
@pytest.mark.parametrize("fmt", [cngp.IDX_U8, cngp.IDX_PACKED4, cngp.IDX_BITS])
def test_input_gradient_sweep(d, N_p, feat, io, fmt):
    w = W.custom(cfg=70 + d + N_p, d=d, L=5, N_f=2**11, N_c=2**9, N_p=N_p, N_min=4, N_max=300, N=3000 + 77,
                 feat_dtype=feat, io_dtype=io)
    run(w, fmt)


@pytest.mark.parametrize("N", [1, 63, 255, 256, 257])
def test_input_gradient_small_batches(N):
    """Below one tile the index codebook is read from memory instead of LDS."""
    w = W.custom(cfg=77, d=3, L=4, N_f=2**10, N_c=2**8, N_p=8, N_min=4, N_max=64, N=N)
    run(w, cngp.IDX_U8, edge_points=False)
    run(w, cngp.IDX_BITS, edge_points=False)


def test_input_gradient_index_codebook_too_large_for_lds():
    w = W.custom(cfg=78, d=3, L=2, N_f=2**12, N_c=2**18, N_p=8, N_min=16, N_max=64, N=3000)
    for fmt in (cngp.IDX_U8, cngp.IDX_PACKED4, cngp.IDX_BITS):
        run(w, fmt)


def test_input_gradient_full_size_workloads():
    run(W.WORKLOADS["nerf3d"], cngp.IDX_U8)
    # more than 2^20 points with a 2^16-entry index codebook: the large-tile variant, ragged last tile
    run(W.WORKLOADS["compact3d"], cngp.IDX_BITS, n=2**20 + 1024 + 77)


@pytest.mark.parametrize("feat,N", [("f16", 160 * 1024 - 1), ("f16", 160 * 1024), ("f32", 160 * 1024 + 63), ("f32", 2**19 + 1),
                                    ("f16", 2**19 + 1)])
def test_large_codebook_large_tiles(feat, N):
    """N_c = 2^16: from 160 Ki points workgroups of 1024 lanes with equal shares, one or two points per lane; the last
    size is one point more than a round holds.  Same bits as the same points in small batches (256-lane tiles)."""
    w = W.custom(cfg=71, d=3, L=3, F=2, N_f=2**12, N_c=2**16, N_p=8, N_min=8, N_max=300, N=N, feat_dtype=feat, io_dtype=feat)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    x = dev(W.make_points(w))
    D_f = dev(W.make_feature_codebook(w))
    dy = dev(W.make_upstream_grad(w, N))
    cfg = cngp.Config.from_workload(w)
    D_c = cngp.bake_probes(cfg, dev(W.make_probe_logits(w)))
    whole = cngp.encode_bwd_input(cfg, x, D_f, D_c, dy)
    step = 100_000
    parts = torch.cat([cngp.encode_bwd_input(cfg, x[i:i + step].contiguous(), D_f, D_c, dy[i:i + step].contiguous())
                       for i in range(0, N, step)])
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)


# the shapes that bwd_input_shape picks: 1024-lane workgroups with one or two points a lane, equal shares or full, every format
@pytest.mark.parametrize("d,feat,fmt,N_f,N_c,N", [
    (3, "f16", cngp.IDX_U8, 2**10, 2**16, 160 * 1024 + 1), (3, "f32", cngp.IDX_BITS, 2**18, 2**16, 2**18 + 1),
    (4, "f32", cngp.IDX_PACKED4, 2**18, 2**15, 2**18 + 65), (2, "f16", cngp.IDX_BITS, 2**12, 2**17, 170_003),
    (3, "f16", cngp.IDX_U8, 2**10, 2**13, 2**20 + 5), (2, "f32", cngp.IDX_U8, 2**15, 2**16, 2**20 + 7),
    (3, "f32", cngp.IDX_PACKED4, 2**12, 2**16, 2**20 + 9), (4, "f16", cngp.IDX_PACKED4, 2**12, 2**15, 2**18 + 3)])
def test_every_workgroup_shape_gives_the_bits_of_small_batches(d, feat, fmt, N_f, N_c, N):
    g = torch.Generator(device="cuda").manual_seed(N)
    x = torch.rand((N, d), generator=g, device="cuda")
    x[:2] = torch.tensor([[0.0] * d, [1.0] * d], device="cuda")
    dt = torch.float16 if feat == "f16" else torch.float32
    cfg = cngp.Config(d=d, L=2, F=2, N_f=N_f, N_c=N_c, N_p=8, N_min=16, N_max=200, feat_dtype=cngp.F16 if feat == "f16" else cngp.F32,
                      io_dtype=cngp.F16 if feat == "f16" else cngp.F32, index_format=fmt)
    D_f = (torch.randn((2, N_f, 2), generator=g, device="cuda") * 0.1).to(dt)
    D_c = torch.randint(0, 8, (2, N_c), generator=g, device="cuda", dtype=torch.uint8)
    D_c = cngp.pack4(D_c) if fmt == cngp.IDX_PACKED4 else cngp.pack_bits(D_c, 8) if fmt == cngp.IDX_BITS else D_c
    dy = torch.randn((N, 4), generator=g, device="cuda").to(dt)
    whole = cngp.encode_bwd_input(cfg, x, D_f, D_c, dy)
    parts = torch.cat([cngp.encode_bwd_input(cfg, x[i:i + 100_000].contiguous(), D_f, D_c, dy[i:i + 100_000].contiguous())
                       for i in range(0, N, 100_000)])
    torch.cuda.synchronize()
    assert torch.equal(whole, parts)


def test_four_dimensions_with_packed_probes_against_the_oracle():
    """The sixteen probe bytes of a point are all asked for before one is used."""
    for N_p, feat in ((8, "f16"), (16, "f32"), (1, "f16")):
        run(W.custom(cfg=79, d=4, L=3, N_f=2**12, N_c=2**15, N_p=N_p, N_min=4, N_max=60, N=1500 + 7, feat_dtype=feat, io_dtype=feat), cngp.IDX_PACKED4)
