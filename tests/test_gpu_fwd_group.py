"""The forward with several levels to a workgroup (tables that all fit in LDS: csrc/cngp_fwd_level.h, encode_fwd_group_kernel), bit for bit against
the tile variant, whose arithmetic it repeats: groups of four to sixteen levels, parts with a remainder, every format and type, coordinates
outside the cube, and the calls that keep the level-major copy (rows that no piece of 16 bytes fits, unaligned rows, a permutation, levels not loaded)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W

pytestmark = pytest.mark.gpu
FMT = {"u8": cngp.IDX_U8, "packed4": cngp.IDX_PACKED4, "bits": cngp.IDX_BITS}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def case(d, L, N_f, N_c, N_p, feat, io, fmt, N):
    w = W.custom(cfg=150, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=4, N_max=300, N=N, feat_dtype=feat, io_dtype=io)
    x = W.make_points(w)
    x[: min(3, N)] = np.array([[0.0] * d, [1.0] * d, [1.7] + [0.2] * (d - 1)], dtype=np.float32)[:N]
    D_f = W.make_feature_codebook(w)
    D_f = (D_f.astype(np.float64) * 1e4).astype(D_f.dtype)
    D_c = oracle.bake_probes(W.make_probe_logits(w))
    D_c = {"u8": lambda: dev(D_c), "packed4": lambda: cngp.pack4(dev(D_c)), "bits": lambda: dev(oracle.pack_index_bits(D_c, N_p))}[fmt]()
    return w, (dev(x), dev(D_f), D_c)


def passes(call):
    """Whether the call wrote the level-major copy and turned it into rows."""
    cngp.profile_enable(True)
    cngp.profile_read()
    y = call()
    torch.cuda.synchronize()
    launches = {k: n for k, (t, n) in cngp.profile_read().items() if n}
    cngp.profile_enable(False)
    return y, any("rows" in k for k in launches)


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,feat,io,fmt", [
    (3, 16, 2**8, 2**16, 8, "f16", "f16", "bits"),              # 25 KB a level: four of them
    (3, 16, 2**8, 2**16, 8, "f16", "f32", "u8"),
    (3, 16, 2**12, 2**13, 16, "f32", "f32", "packed4"),
    (2, 12, 2**10, 2**12, 4, "f16", "f16", "u8"),
    (4, 8, 2**9, 2**10, 2, "f32", "f16", "bits"),
    (3, 4, 2**10, 1, 1, "f16", "f32", "bits"),                  # no index codebook at all
    (2, 20, 2**8, 2**12, 8, "f16", "f16", "packed4"),
])
@pytest.mark.parametrize("N", [1, 2049, 70001, 300007])
def test_groups_of_levels_equal_the_tile_variant(d, L, N_f, N_c, N_p, feat, io, fmt, N):
    w, args = case(d, L, N_f, N_c, N_p, feat, io, fmt, N)
    cfg = cngp.Config.from_workload(w, flags=cngp.FWD_LEVEL, index_format=FMT[fmt])
    ws = torch.empty(cngp.fwd_workspace_bytes(cfg, N), dtype=torch.uint8, device="cuda").fill_(0xAB)
    y = torch.full((N + 1, 2 * L), 7.0, dtype=torch.float16 if io == "f16" else torch.float32, device="cuda")
    _, rows = passes(lambda: cngp.encode_fwd(cfg, *args, y[:N], workspace=ws))
    assert not rows and bool((y[N] == 7.0).all())
    want = cngp.encode_fwd(cngp.Config.from_workload(w, flags=cngp.FWD_TILE, index_format=FMT[fmt]), *args)
    assert torch.equal(y[:N], want)


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,feat,io,fmt,N,levels", [      # more than four: from enough points on for a step of each workgroup of one round
    (3, 16, 2**8, 2**12, 8, "f16", "f16", "packed4", 300007, 8),
    (3, 16, 2**8, 2**12, 8, "f16", "f32", "u8", 2**19 + 77, 16),
    (2, 12, 2**10, 2**12, 4, "f16", "f16", "u8", 2**19 + 77, 12),
    (4, 8, 2**9, 2**10, 2, "f32", "f16", "bits", 2**19 + 77, 8),
    (2, 20, 2**8, 2**12, 8, "f16", "f16", "bits", 2**19 + 77, 20),
])
@pytest.mark.parametrize("shift", [0, 4])                       # bytes past a 16-byte boundary where the index codebook begins: 0 is copied in pieces of 16
def test_larger_groups_equal_the_tile_variant(d, L, N_f, N_c, N_p, feat, io, fmt, N, levels, shift):
    w, (x, D_f, D_c) = case(d, L, N_f, N_c, N_p, feat, io, fmt, N)
    moved = torch.empty(D_c.numel() + shift, dtype=torch.uint8, device="cuda")[shift:].view(D_c.shape)
    moved.copy_(D_c)
    assert moved.data_ptr() % 16 == shift
    cfg = cngp.Config.from_workload(w, flags=cngp.FWD_LEVEL, index_format=FMT[fmt])
    assert cngp.fwd_group_levels(cfg, N) == levels
    ws = torch.empty(cngp.fwd_workspace_bytes(cfg, N), dtype=torch.uint8, device="cuda").fill_(0xAB)
    y = torch.full((N + 1, 2 * L), 7.0, dtype=torch.float16 if io == "f16" else torch.float32, device="cuda")
    _, rows = passes(lambda: cngp.encode_fwd(cfg, x, D_f, moved, y[:N], workspace=ws))
    assert not rows and bool((y[N] == 7.0).all()) and bool((ws == 0xAB).all())
    assert torch.equal(y[:N], cngp.encode_fwd(cngp.Config.from_workload(w, flags=cngp.FWD_TILE, index_format=FMT[fmt]), x, D_f, D_c))


@pytest.mark.parametrize("fmt,shift", [("u8", 1), ("packed4", 3), ("bits", 8)])
def test_groups_of_four_with_an_index_codebook_off_a_boundary(fmt, shift):
    N = 5003
    w, (x, D_f, D_c) = case(3, 16, 2**8, 2**12, 8, "f16", "f16", fmt, N)
    moved = torch.empty(D_c.numel() + shift, dtype=torch.uint8, device="cuda")[shift:].view(D_c.shape)
    moved.copy_(D_c)
    level, tile = (cngp.Config.from_workload(w, flags=f, index_format=FMT[fmt]) for f in (cngp.FWD_LEVEL, cngp.FWD_TILE))
    assert cngp.fwd_group_levels(level, N) == 4
    ws = torch.empty(cngp.fwd_workspace_bytes(level, N), dtype=torch.uint8, device="cuda")
    got, rows = passes(lambda: cngp.encode_fwd(level, x, D_f, moved, workspace=ws))
    assert not rows and torch.equal(got, cngp.encode_fwd(tile, x, D_f, D_c))


@pytest.mark.parametrize("L,shift,levels,perm", [(10, 0, None, False), (16, 1, None, False), (16, 0, 9, False), (16, 0, None, True)])
def test_calls_that_keep_the_level_major_copy(L, shift, levels, perm):
    N = 5003
    w, args = case(3, L, 2**8, 2**12, 8, "f16", "f16", "packed4", N)
    level, tile = (cngp.Config.from_workload(w, flags=f, index_format=cngp.IDX_PACKED4) for f in (cngp.FWD_LEVEL, cngp.FWD_TILE))
    ws = torch.empty(cngp.fwd_workspace_bytes(level, N), dtype=torch.uint8, device="cuda")
    y = torch.empty(N * 2 * L + 2, dtype=torch.float16, device="cuda")[2 * shift: 2 * shift + N * 2 * L].view(N, 2 * L)
    if perm:
        order = torch.randperm(N, device="cuda").to(torch.int32)
        got, rows = passes(lambda: cngp.encode_fwd_permuted(level, args[0][order.long()].contiguous(), order, *args[1:], y, workspace=ws))
        want = cngp.encode_fwd(tile, *args)
    elif levels:
        got, rows = passes(lambda: cngp.encode_fwd_partial(level, levels, *args, y, workspace=ws))
        want = cngp.encode_fwd_partial(tile, levels, *args)
    else:
        got, rows = passes(lambda: cngp.encode_fwd(level, *args, y, workspace=ws))
        want = cngp.encode_fwd(tile, *args)
    assert rows and torch.equal(got, want)
