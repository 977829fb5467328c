"""Backward pass whose coarser levels merge the references of neighbouring points per vertex before they are binned
(csrc/cngp_bwd_merge.h), against the oracle and the direct variant: ragged batches, both dimensions, one-pass small tables, chunks
with more vertices than the table has slots, points a table key cannot hold, gradients that are added to, the sparse softmax, wider
features, the fall-back to a smaller workspace, and capture."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu
FLAGS = cngp.ZERO_GRADS | cngp.BWD_BINNED


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def inputs(w, x=None):
    D_f = W.make_feature_codebook(w)
    D_f = (D_f.astype(np.float64) * 1e4).astype(D_f.dtype)
    return W.make_points(w) if x is None else x, D_f, W.make_probe_logits(w), W.make_upstream_grad(w)


def backward(w, args, flags=FLAGS, ws=None, init=float("nan"), **kw):
    cfg = cngp.Config.from_workload(w, flags=flags, **kw)
    ws = cngp.alloc_workspace(cfg, w.N) if ws is None else ws
    if ws is not None:
        ws.fill_(0xAB)                                          # nothing in it is assumed to be zero
    gF, gC = (torch.full(s, init, device="cuda") for s in ((w.L, w.N_f, w.F), (w.L, w.N_c, w.N_p)))
    cngp.profile_enable(True)
    cngp.profile_read()
    cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
    torch.cuda.synchronize()
    names = [k for k, (_, n) in cngp.profile_read().items() if n]
    cngp.profile_enable(False)
    return gF.cpu().numpy(), gC.cpu().numpy(), names


def check(w, args, start=0.0, **kw):
    gF, gC, names = backward(w, args, **kw)
    assert "encode_bwd_merge" in names, names
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args, top_k=kw.get("top_k", 0))
    check_close("grad D_f", gF, gF_ref + start, A_f + abs(start), fp16_out=False)
    check_close("grad Dhat_c", gC, gC_ref + start, A_c + abs(start), fp16_out=False)


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,N_max,feat,io", [
    (3, 196608, 4, 2**13, 2**11, 16, 80, "f16", "f16"),        # the smallest batch that is merged
    (3, 250007, 3, 2**13, 2**10, 8, 60, "f16", "f32"),         # a ragged last round and chunk
    (2, 500009, 4, 2**13, 2**11, 2, 900, "f32", "f16"),
    (2, 2**19 + 1, 6, 2**13, 1, 1, 300, "f32", "f32"),         # plain hashing: no confidence bins
    (3, 2**18, 5, 2**13, 2**10, 4, 40, "f32", "f32"),          # every level but the last
    (3, 200003, 4, 2**18, 2**16, 8, 70, "f16", "f16"),         # one drain workgroup per bin of a merged level: nothing is cleared first
    (3, 200003, 16, 2**8, 2**16, 8, 2048, "f16", "f16"),          # small feature table: both gradients in one pass
])
def test_merged_levels_against_the_oracle(d, N, L, N_f, N_c, N_p, N_max, feat, io):
    w = W.custom(cfg=110, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=8 if L < 16 else 40, N_max=N_max, N=N, feat_dtype=feat, io_dtype=io)
    check(w, inputs(w))


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,N_max", [
    (3, 200003, 4, 2**18, 2**16, 8, 70),                       # one drain workgroup per bin of a merged level: stores where the array is cleared, adds here
    (3, 2**19 + 3, 4, 2**13, 2**10, 4, 70),                    # several
    (2, 400003, 6, 2**13, 1, 1, 300),                          # plain hashing
    (3, 200003, 16, 2**8, 2**16, 8, 2048)])                    # both gradients in one pass
def test_merged_levels_add_onto_the_gradients_that_are_there(d, N, L, N_f, N_c, N_p, N_max):
    w = W.custom(cfg=116, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=8 if L < 16 else 40, N_max=N_max, N=N, feat_dtype="f16", io_dtype="f16")
    check(w, inputs(w), flags=cngp.BWD_BINNED, init=-0.5, start=-0.5)


@pytest.mark.parametrize("L,N_f,N_c,N_p,top_k", [(4, 2**13, 2**11, 16, 3), (4, 2**13, 2**10, 4, 1), (16, 2**8, 2**16, 8, 2)])
def test_merged_levels_with_the_sparse_softmax(L, N_f, N_c, N_p, top_k):
    w = W.custom(cfg=117, d=3, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=8 if L < 16 else 40, N_max=80 if L < 16 else 2048, N=200003,
                 feat_dtype="f16", io_dtype="f16")
    check(w, inputs(w), top_k=top_k)


@pytest.mark.parametrize("F,d,N,N_p,feat,io", [(4, 3, 200003, 8, "f16", "f16"), (4, 2, 400003, 1, "f32", "f32"), (1, 3, 200003, 4, "f32", "f16")])
def test_merged_levels_with_other_feature_widths(F, d, N, N_p, feat, io):
    """A pair of features at a time: dL/dy is then the pair's plane, and the second pass adds to the confidence gradient."""
    w = W.custom(cfg=118, d=d, L=5, F=F, N_f=2**13, N_c=2**11 if N_p > 1 else 1, N_p=N_p, N_min=8, N_max=80, N=N, feat_dtype=feat, io_dtype=io)
    args = inputs(w)
    check(w, args)
    check(w, args, flags=cngp.BWD_BINNED, init=0.25, start=0.25)


def test_more_vertices_than_slots():
    """85 % of the points in one cell, the others spread: where they are, almost every reference is a vertex of its own
    (1024 points, 3700 vertices, 3520 slots), on a level that is merged because of the average."""
    w = W.custom(cfg=111, d=2, L=3, N_f=2**13, N_c=2**10, N_p=4, N_min=600, N_max=1000, N=450001, feat_dtype="f16", io_dtype="f16")
    rng = np.random.default_rng(5)
    x = rng.random((w.N, 2), dtype=np.float32)
    x[rng.random(w.N) < 0.85] = (0.3, 0.7)
    x[:100] = 1.0                                               # the far corner, and the faces
    x[100:300, 0] = 0.0
    check(w, inputs(w, x))


def test_points_outside_the_cube_agree_with_the_direct_variant():
    w = W.custom(cfg=112, d=3, L=2, N_f=2**13, N_c=2**10, N_p=4, N_min=8, N_max=100, N=200001, feat_dtype="f32", io_dtype="f32")
    rng = np.random.default_rng(6)
    x = rng.random((w.N, 3), dtype=np.float32)
    far = rng.random(w.N) < 0.1
    x[far] *= 200.0                                             # coordinates of up to 1600 and 20000: more than ten bits
    args = inputs(w, x)
    gF, gC, names = backward(w, args)
    assert "encode_bwd_merge" in names
    hF, hC, _ = backward(w, args, flags=cngp.ZERO_GRADS | cngp.BWD_DIRECT)
    _, _, A_f, A_c = oracle.encode_bwd(w, np.minimum(x, 1.0), *args[1:])
    # the direct variant adds up in fp32: n references to an entry are off by sqrt(n) 2^-24 of their magnitude, here below 4e-6
    # of the largest entry's
    for g, h, A in ((gF, hF, A_f), (gC, hC, A_c)):
        assert np.abs(g - h).max() <= 4e-6 * np.abs(A).max()


@pytest.mark.parametrize("d,N,last", [
    (3, 200001, (np.inf, np.inf, np.inf)), (3, 200001, (0.95, np.inf, 0.95)), (3, 200001, (np.inf, 3e38, 0.99)), (3, 199681, (0.99, 0.99, np.inf)),
    (2, 400003, (np.inf, np.inf)), (2, 400003, (0.99, np.inf))])
def test_lanes_beyond_a_ragged_chunk_ignore_a_point_at_infinity(d, N, last):
    """The point the idle lanes of the last round repeat is not finite (the last of the order: nobody else is in its cell).  The rows it
    touches are meaningless in every variant, and the same ones; all others are as if it were not there."""
    w = W.custom(cfg=115, d=d, L=3, N_f=2**13, N_c=2**10, N_p=4, N_min=8, N_max=60, N=N, feat_dtype="f16", io_dtype="f16")
    x = np.random.default_rng(7).random((N, d), dtype=np.float32) * np.float32(0.9)
    x[N // 3] = last
    args = inputs(w, x)
    gF, gC, names = backward(w, args)
    assert "encode_bwd_merge" in names
    hF, hC, _ = backward(w, args, flags=cngp.ZERO_GRADS | cngp.BWD_DIRECT)
    _, _, A_f, A_c = oracle.encode_bwd(w, np.where(np.isfinite(x) & (x <= 1.0), x, np.float32(0.5)), *args[1:])
    for g, h, A in ((gF, hF, A_f), (gC, hC, A_c)):
        touched = ~np.isfinite(h)
        assert 0 < touched.sum() < 0.02 * h.size and (touched == ~np.isfinite(g)).all()
        assert np.abs(g - h)[~touched].max() <= 4e-6 * np.abs(A).max()      # the direct variant's fp32 sums, as above


def test_a_smaller_workspace_and_no_pre_reduction_are_not_merged():
    w = W.custom(cfg=113, d=3, L=4, N_f=2**13, N_c=2**11, N_p=8, N_min=16, N_max=200, N=200003, feat_dtype="f16", io_dtype="f16")
    args = inputs(w)
    need = cngp.workspace_bytes(cngp.Config.from_workload(w, flags=FLAGS), w.N)
    small = cngp.workspace_bytes(cngp.Config.from_workload(w, flags=FLAGS, bin_bytes_max=4 << 30), w.N)
    assert small < need
    gF, gC, names = backward(w, args)
    hF, hC, other = backward(w, args, ws=torch.empty(small, dtype=torch.uint8, device="cuda"))
    assert "encode_bwd_merge" in names and "encode_bwd_merge" not in other
    assert "encode_bwd_merge" not in backward(w, args, flags=FLAGS | cngp.BWD_NO_PREREDUCE)[2]
    for g, h in ((gF, hF), (gC, hC)):                           # both sum in fp64 what fp32 products give: a few 2^-24 of the norm
        assert np.linalg.norm(g - h) <= 1e-6 * np.linalg.norm(h)


def test_capture_replays_the_merge():
    w = W.custom(cfg=114, d=3, L=3, N_f=2**13, N_c=2**10, N_p=8, N_min=16, N_max=90, N=200003, feat_dtype="f16", io_dtype="f16")
    args = inputs(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    cfg = cngp.Config.from_workload(w, flags=FLAGS)
    t = [dev(a) for a in args]
    gF, gC = torch.empty((w.L, w.N_f, 2), device="cuda"), torch.empty((w.L, w.N_c, w.N_p), device="cuda")
    ws = cngp.alloc_workspace(cfg, w.N)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cngp.encode_bwd(cfg, *t, gF, gC, workspace=ws)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cngp.encode_bwd(cfg, *t, gF, gC, workspace=ws)
    for _ in range(3):
        gF.fill_(float("nan")); gC.fill_(float("nan")); ws.fill_(0xCD)
        graph.replay()
        torch.cuda.synchronize()
        check_close("grad D_f", gF.cpu().numpy(), gF_ref, A_f, fp16_out=False)
        check_close("grad Dhat_c", gC.cpu().numpy(), gC_ref, A_c, fp16_out=False)
        cngp.encode_bwd(cfg, *t, gF, gC, workspace=ws)          # eager work between the replays
        (gF.sum() + gC.sum()).item()
