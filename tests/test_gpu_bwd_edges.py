"""Binned backward whose feature-table bins hold edges, two corners a record (csrc/cngp_bwd_binned.h), against the oracle: edges whose ends are
in two slices, ends of weight zero, both scatters, every dimension and number of candidates, and softmax rows that are NaN."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def points(w, rows):
    """A third of them in cells that end a slice (v_0 = rows - 1 or 2 rows - 1 on the finest level), some of those with an end of weight zero."""
    x = W.make_points(w)
    third = x[::3, 0]
    cell = np.arange(third.size) % 2 * rows + rows - 1
    frac = np.where(np.arange(third.size) % 5 == 0, 0.0, 0.25 + 0.5 * third)
    third[:] = ((cell + frac) / w.N_max).astype(np.float32)
    x[1::7, -1] = 1.0                                           # on a face: both ends of an edge weightless
    return x


def run(w, x, Dhat=None):
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS | cngp.BWD_BINNED | cngp.BWD_NO_PREREDUCE)
    D_f = (W.make_feature_codebook(w).astype(np.float64) * 1e4).astype(W.make_feature_codebook(w).dtype)
    args = [x, D_f, W.make_probe_logits(w) if Dhat is None else Dhat, W.make_upstream_grad(w)]
    ws = cngp.alloc_workspace(cfg, w.N)
    ws.fill_(0xAB)
    gF, gC = (torch.full(s, 7.0, device="cuda") for s in ((w.L, w.N_f, 2), (w.L, w.N_c, w.N_p)))
    cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
    return cngp.bwd_plan_info(cfg, w.N), args, gF.cpu().numpy(), gC.cpu().numpy()


@pytest.mark.parametrize("d,N_f,N_c,N_p,feat,io,slices", [
    (3, 2**14, 2**12, 16, "f16", "f16", (2, 4)),                # a wavefront per chunk writes directly
    (2, 2**16, 2**12, 8, "f16", "f32", (8, 2)),
    (3, 2**15, 2**13, 4, "f32", "f16", (4, 2)),
    (4, 2**14, 2**12, 2, "f32", "f32", (2, 1)),
    (3, 2**15, 1, 1, "f16", "f16", (4, 0)),
    (2, 2**19, 2**17, 8, "f16", "f16", (64, 64)),               # in runs
    (3, 2**18, 2**15, 8, "f16", "f32", (32, 16)),
    (4, 2**18, 2**15, 8, "f32", "f16", (32, 16)),
    (3, 2**13, 2**12, 16, "f16", "f16", (1, 4)),                # a single slice: no edge leaves it
])
def test_edges_against_the_oracle(d, N_f, N_c, N_p, feat, io, slices):
    rows = 128 * 1024 // (16 * N_p)
    w = W.custom(cfg=140, d=d, L=3, N_f=N_f, N_c=N_c, N_p=N_p, N_min=24, N_max=2 * rows + 7, N=9001 if d < 4 else 4001, feat_dtype=feat, io_dtype=io)
    plan, args, gF, gC = run(w, points(w, rows))
    assert plan["binned"] == 1 and (plan["slices_f"], plan["slices_c"]) == slices, plan
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    check_close("grad D_f", gF, gF_ref, A_f, fp16_out=False)
    check_close("grad Dhat_c", gC, gC_ref, A_c, fp16_out=False)


def test_nan_rows_reach_the_entries_they_belong_to_and_no_others():
    rows = 128 * 1024 // (16 * 8)
    w = W.custom(cfg=141, d=3, L=2, N_f=2**16, N_c=2**12, N_p=8, N_min=24, N_max=2 * rows + 7, N=3001, feat_dtype="f16", io_dtype="f16")
    x = W.make_points(w)
    x[::3, 0] = ((rows - 1 + 0.5) / w.N_max)                    # ends in two slices; no weight is zero
    Dhat = W.make_probe_logits(w)
    Dhat[:, ::97, 3] = np.nan
    plan, args, gF, gC = run(w, x, Dhat)
    assert plan["binned"] == 1 and plan["slices_f"] == 8, plan
    gF_ref, gC_ref, _, _ = oracle.encode_bwd(w, *args)
    assert np.isnan(gF_ref).any() and not np.isnan(gF_ref).all()
    assert np.array_equal(np.isnan(gF), np.isnan(gF_ref))
    assert not np.isnan(gC[~np.isnan(Dhat).any(axis=2)]).any()          # (a NaN row that no point refers to is NaN too: its Jacobian is)
