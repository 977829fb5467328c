"""Replicated-scan backward of batches that would leave CUs without a workgroup: cut into many chunks, whose fp64 sums meet in the workspace
(csrc/cngp_bwd_sliced.h, bwd_partial_sums_kernel), against the oracle: every N_p, one role with a single chunk, several slices, pre-reduced
levels beside it, gradients that are added to, the sparse softmax, wider features, points no chunk size divides, and the room without them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu
NAME = "encode_bwd_partial_sums"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def inputs(w):
    D_f = W.make_feature_codebook(w)
    return W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)


def backward(w, args, init=float("nan"), room=None, **kw):
    cfg = cngp.Config.from_workload(w, **{"flags": cngp.ZERO_GRADS, **kw})
    ws = torch.full((cngp.workspace_bytes(cfg, w.N) if room is None else room,), 0xAB, dtype=torch.uint8, device="cuda")
    gF, gC = (torch.full(s, init, device="cuda") for s in ((w.L, w.N_f, w.F), (w.L, w.N_c, w.N_p)))
    cngp.profile_enable(True)
    cngp.profile_read()
    try:
        cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
        torch.cuda.synchronize()
        launches = cngp.profile_read().get(NAME, (0, 0))[1]
    finally:
        cngp.profile_enable(False)
    return gF.cpu().numpy(), gC.cpu().numpy(), launches


def check(w, args, start=0.0, launched=1, **kw):
    gF, gC, launches = backward(w, args, **kw)
    assert launches == launched
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args, top_k=kw.get("top_k", 0))
    check_close("grad D_f", gF, gF_ref + start, A_f + abs(start), fp16_out=False)
    check_close("grad Dhat_c", gC, gC_ref + start, A_c + abs(start), fp16_out=False)


def workload(d, N, L, N_f, N_c, N_p, N_min, N_max, **kw):
    return W.custom(**{**dict(cfg=130, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N, feat_dtype="f16", io_dtype="f16"), **kw})


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,N_min,N_max,feat,io", [
    (3, 25752, 8, 2**13, 2**11, 16, 16, 512, "f16", "f16"),    # one and two slices
    (3, 8193, 8, 2**13, 2**10, 8, 40, 300, "f32", "f32"),      # just enough references; 512 points and one more chunk
    (2, 60001, 8, 2**13, 2**9, 4, 16, 2048, "f16", "f32"),     # three pre-reduced levels
    (4, 14003, 8, 2**13, 2**13, 2, 16, 64, "f32", "f16"),
    (3, 20011, 8, 2**13, 1, 1, 40, 400, "f16", "f16"),         # plain hashing: no logits
    (3, 12007, 6, 2**15, 2**8, 16, 40, 400, "f16", "f16"),     # four slices and one
    (3, 30011, 2, 2**11, 2**13, 8, 16, 600, "f16", "f16"),     # a small table: the scan is asked for
    (3, 22912, 8, 2**17, 2**13, 8, 16, 2048, "f16", "f16"),    # sixteen slices with one chunk each, which store their rows, and four
])
def test_partial_sums_against_the_oracle(d, N, L, N_f, N_c, N_p, N_min, N_max, feat, io):
    w = workload(d, N, L, N_f, N_c, N_p, N_min, N_max, feat_dtype=feat, io_dtype=io)
    args = inputs(w)
    flags = cngp.BWD_SLICED if L == 2 else 0
    check(w, args, flags=cngp.ZERO_GRADS | flags)
    check(w, args, flags=flags, init=-0.5, start=-0.5)         # adds to what is there


def test_partial_sums_with_the_sparse_softmax_and_other_widths():
    w = workload(3, 25752, 8, 2**13, 2**11, 16, 16, 512)
    check(w, inputs(w), top_k=3)
    w = workload(3, 20011, 8, 2**13, 2**11, 8, 16, 512, F=4)
    check(w, inputs(w), launched=2)


def test_a_workspace_without_the_room_for_partial_sums_is_enough():
    """The scan then runs in the few chunks it had, whose fp32 sums are added with atomics; below that the call is refused."""
    w = workload(3, 60000, 8, 2**13, 2**8, 8, 16, 2048)
    args = inputs(w)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS)
    need, small = cngp.workspace_bytes(cfg, w.N), cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=1 << 20), w.N)
    assert small < need
    check(w, args, launched=0, room=small)
    check(w, args, launched=1, room=need)
    with pytest.raises(cngp.CngpError) as e:
        backward(w, args, room=small // 2 // 256 * 256)
    assert e.value.status == cngp.ERR_WORKSPACE


def test_calls_on_two_streams_add_to_the_same_gradients():
    """Each with a workspace of its own: no sum of either is lost, as where the chunks' sums are added with atomics."""
    w, times = workload(3, 25752, 8, 2**13, 2**11, 16, 16, 512), 8
    args = inputs(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    cfg = cngp.Config.from_workload(w, flags=0)
    t = [dev(a) for a in args]
    gF, gC = torch.zeros((w.L, w.N_f, 2), device="cuda"), torch.zeros((w.L, w.N_c, w.N_p), device="cuda")
    sides = [(torch.cuda.Stream(), cngp.alloc_workspace(cfg, w.N)) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(times):
        for stream, ws in sides:
            with torch.cuda.stream(stream):
                cngp.encode_bwd(cfg, *t, gF, gC, workspace=ws)
    torch.cuda.synchronize()
    check_close("grad D_f", gF.cpu().numpy(), 2 * times * gF_ref, 2 * times * A_f, fp16_out=False)
    check_close("grad Dhat_c", gC.cpu().numpy(), 2 * times * gC_ref, 2 * times * A_c, fp16_out=False)


def test_capture_replays_partial_sums():
    w = workload(3, 25752, 8, 2**13, 2**11, 16, 16, 512)
    args = inputs(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS)
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
