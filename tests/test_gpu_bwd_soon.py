"""Backward of batches below 2^21 references that is binned (csrc/cngp_api.hip, kMinBinnedSoonRefs and the rules beside it): against the oracle, and in the
room of the variants that ran before (scan, atomics)."""
import numpy as np
import pytest

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close
from test_gpu_bwd_few_slices import DRAIN, SCAN, run

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,feat,io", [
    (3, 2053, 16, 2**16, 2**14, 16, "f16", "f16"),      # 8 + 16 slices, many candidates: from 2^18 references, atomics before
    (3, 4507, 16, 2**16, 2**15, 16, "f32", "f32"),      # ... scanned before
    (4, 8209, 8, 2**17, 2**13, 16, "f16", "f32"),       # 16 + 8, d = 4: from 2^20
    (2, 17003, 16, 2**17, 2**15, 8, "f16", "f16"),      # 16 + 16: from 2^20
    (3, 8209, 16, 2**18, 2**16, 8, "f16", "f16"),       # 32 + 32
    (3, 2061, 16, 2**8, 2**14, 16, "f16", "f16"),       # a small feature table, atomics before
    (3, 4099, 8, 2**12, 2**13, 8, "f32", "f32"),
])
def test_short_batches_are_binned(d, N, L, N_f, N_c, N_p, feat, io):
    w = W.custom(cfg=150, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=16, N_max=1024, N=N, feat_dtype=feat, io_dtype=io)
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS)
    before = cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=1 << 20), N)
    assert before < cngp.workspace_bytes(cfg, N)
    for start, room in ((None, None), (0.5, None), (None, before)):
        gF, gC, names = run(w, args, room=room, start=start)
        assert (DRAIN in names) == (room is None), names
        assert room is None or (SCAN in names) == ((N << d) * L >= 2**19), names
        s = start or 0.0
        check_close("grad D_f", gF, gF_ref + s, A_f + s, fp16_out=False)
        check_close("grad Dhat_c", gC, gC_ref + s, A_c + s, fp16_out=False)


@pytest.mark.parametrize("d,N,L,N_f,N_c,N_p,points", [
    (3, 20011, 8, 2**16, 2**14, 16, "nerf_rays"),       # 8 + 16 slices
    (3, 30000, 8, 2**16, 2**14, 16, "uniform"),
    (3, 24860, 8, 2**17, 2**13, 16, "uniform"),         # 16 + 8
    (3, 23413, 6, 2**16, 2**14, 16, "uniform"),
    (3, 61147, 4, 2**18, 2**16, 8, "sdf_shell"),        # 32 + 32
    (2, 61147, 8, 2**17, 2**15, 8, "uniform"),          # 16 + 16
    (4, 15287, 8, 2**17, 2**14, 16, "uniform"),
])
def test_no_further_from_64_bits_than_the_scan(d, N, L, N_f, N_c, N_p, points):
    """Both form an entry's sum in 64 bits and round it once, so their errors are those of that rounding and of the same fp32 terms: alike to the
    scatter of a norm over 10^5 entries and more, below 1 %."""
    w = W.custom(cfg=150, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=16, N_max=2048, N=N, feat_dtype="f16", io_dtype="f32", points=points)
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    refs = oracle.encode_bwd(w, *args, want_abs=False)[:2]
    room = cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=1 << 20), N)
    error = []
    for room in (None, room):
        *grads, names = run(w, args, room=room)
        assert (DRAIN if room is None else SCAN) in names, names
        error.append([float(np.linalg.norm(g - r) / np.linalg.norm(r)) for g, r in zip(grads, refs)])
    print("binned", error[0], "scanned", error[1])
    assert all(b <= s * 1.01 for b, s in zip(*error)), error
