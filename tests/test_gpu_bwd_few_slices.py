"""Backward of large batches with tables of a few slices, which is binned where levels are merged or there is no probing, and scanned in a
smaller workspace (csrc/cngp_api.hip, kMinMergedSlices and kMinBinnedPlainScans), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu
SCAN, DRAIN, MERGE, SUMS = "encode_bwd_sliced_points_and_grid", "encode_bwd_bin_drain", "encode_bwd_merge", "encode_bwd_partial_sums"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def run(w, args, room=None, start=None, **kw):
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS if start is None else 0, **kw)
    ws = torch.full((cngp.workspace_bytes(cfg, w.N) if room is None else room,), 0xAB, dtype=torch.uint8, device="cuda")
    gF, gC = (torch.full(s, float("nan") if start is None else start, device="cuda") for s in ((w.L, w.N_f, w.F), (w.L, w.N_c, w.N_p)))
    cngp.profile_enable(True)
    cngp.profile_read()
    try:
        cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
        torch.cuda.synchronize()
        names = {k for k, (_, n) in cngp.profile_read().items() if n}
    finally:
        cngp.profile_enable(False)
    return gF.cpu().numpy(), gC.cpu().numpy(), names


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,N_min,N_max,feat,io,merged", [
    (2, 400003, 16, 2**16, 2**12, 8, 16, 8192, "f16", "f16", True),    # 8 + 2 slices
    (3, 196609, 8, 2**15, 2**13, 8, 36, 250, "f16", "f32", True),      # 4 + 4: the fewest; little more than the fewest points
    (3, 200003, 8, 2**13, 2**16, 4, 30, 300, "f32", "f16", True),      # 1 + 16
    (2, 500009, 8, 2**16, 2**10, 2, 200, 4000, "f16", "f16", True),    # N_p = 2: 8 + 1, six levels a scan would not pre-reduce
    (3, 196613, 12, 2**16, 1, 1, 100, 8192, "f32", "f32", False),      # plain hashing, 8 slices on 12 levels, none that could be merged
    (3, 110003, 8, 2**17, 1, 1, 60, 2048, "f16", "f16", False),        # 16 slices, fewer points
])
def test_tables_of_few_slices_are_binned(d, N, L, N_f, N_c, N_p, N_min, N_max, feat, io, merged):
    w = W.custom(cfg=140, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N, feat_dtype=feat, io_dtype=io)
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)

    def check(gF, gC, start=0.0):
        check_close("grad D_f", gF, gF_ref + start, A_f + abs(start), fp16_out=False)
        check_close("grad Dhat_c", gC, gC_ref + start, A_c + abs(start), fp16_out=False)

    gF, gC, names = run(w, args)
    assert DRAIN in names and SCAN not in names and (MERGE in names) == merged
    check(gF, gC)
    gF, gC, names = run(w, args, start=0.5)
    assert DRAIN in names
    check(gF, gC, 0.5)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=8 << 30)     # (a bound: the scan)
    room = cngp.workspace_bytes(cfg, N)
    assert room < cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS), N)
    gF, gC, names = run(w, args, room=room)
    assert SCAN in names and DRAIN not in names
    check(gF, gC)


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,N_min,N_max", [
    (3, 745393, 8, 2**16, 2**11, 8, 40, 2048),                          # one logit slice: 64 workgroups a bin, a scan of nine chunks at most
    (2, 900001, 6, 2**16, 2**10, 2, 200, 8192),
    (3, 400003, 8, 2**13, 2**16, 4, 40, 600),                           # one feature slice
    (3, 600011, 16, 2**16, 1, 1, 16, 2048),                             # plain hashing: levels enough that a scan would not pre-reduce (96 bins)
])
def test_binning_few_slices_is_no_less_precise_than_scanning_them(d, N, L, N_f, N_c, N_p, N_min, N_max):
    """2-norm error against 64 bits, both gradients: the sums of a bin's workgroups meet in 64 bits, a scan's chunks in 32."""
    w = W.custom(cfg=141, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N, feat_dtype="f16", io_dtype="f16")
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    refs = oracle.encode_bwd(w, *args)[:2]
    room = cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=8 << 30), N)
    binned, scanned = run(w, args), run(w, args, room=room)
    assert MERGE in binned[2] and SUMS in binned[2] and SCAN in scanned[2]
    for got, scan, ref in zip(binned, scanned, refs):
        off, off_scan = (float(np.linalg.norm(g.astype(np.float64) - ref)) for g in (got, scan))
        assert off <= off_scan


def test_sums_of_drain_workgroups_with_the_sparse_softmax_other_widths_and_capture():
    w = W.custom(cfg=142, d=3, L=8, N_f=2**16, N_c=2**11, N_p=8, N_min=30, N_max=300, N=200003, feat_dtype="f16", io_dtype="f16")
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args, top_k=3)
    gF, gC, names = run(w, args, top_k=3)
    assert SUMS in names
    check_close("grad D_f", gF, gF_ref, A_f, fp16_out=False)
    check_close("grad Dhat_c", gC, gC_ref, A_c, fp16_out=False)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, top_k=3)
    t, ws = [dev(a) for a in args], cngp.alloc_workspace(cfg, w.N)
    gF, gC = torch.empty((w.L, w.N_f, 2), device="cuda"), torch.empty((w.L, w.N_c, w.N_p), device="cuda")
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
    w4 = W.custom(cfg=143, d=3, L=8, F=4, N_f=2**16, N_c=2**11, N_p=8, N_min=30, N_max=300, N=200003, feat_dtype="f32", io_dtype="f32")
    D_f = W.make_feature_codebook(w4)
    args = W.make_points(w4), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w4), W.make_upstream_grad(w4)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w4, *args)
    for start in (None, 0.5):
        gF, gC, names = run(w4, args, start=start)
        assert SUMS in names
        check_close("grad D_f", gF, gF_ref + (start or 0.0), A_f + (start or 0.0), fp16_out=False)
        check_close("grad Dhat_c", gC, gC_ref + (start or 0.0), A_c + (start or 0.0), fp16_out=False)
