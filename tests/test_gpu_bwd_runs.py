"""Binned backward whose scatter writes the records in runs (csrc/cngp_bwd_runs.h: 48 .. 512 bins of a level), against the oracle: the fewest
and the most bins, bins of one table only, every dimension, rounds and chunks with a remainder, pre-reduced and merged levels beside the
hashed ones, points whose references fill single bins, and one bin more than it takes."""
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


def check(w, slices, x=None, flags=cngp.ZERO_GRADS | cngp.BWD_BINNED, **want):
    cfg = cngp.Config.from_workload(w, flags=flags)
    plan = cngp.bwd_plan_info(cfg, w.N)
    assert plan["binned"] == 1 and (plan["slices_f"], plan["slices_c"]) == slices and all(plan[k] == v for k, v in want.items()), plan
    D_f = W.make_feature_codebook(w)
    args = [W.make_points(w) if x is None else x, (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)]
    ws = cngp.alloc_workspace(cfg, w.N)
    ws.fill_(0xAB)                                              # nothing in it is assumed to be zero
    gF, gC = (torch.full(s, float("nan"), device="cuda") for s in ((w.L, w.N_f, 2), (w.L, w.N_c, w.N_p)))
    cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    check_close("grad D_f", gF.cpu().numpy(), gF_ref, A_f, fp16_out=False)
    check_close("grad Dhat_c", gC.cpu().numpy(), gC_ref, A_c, fp16_out=False)


@pytest.mark.parametrize("d,N,N_f,N_c,N_p,slices,merged", [
    (3, 1, 2**18, 2**15, 8, (32, 16), 0),                      # one point; the fewest bins
    (3, 513, 2**18, 2**15, 8, (32, 16), 0),                    # a round and one point
    (2, 1025, 2**19, 2**17, 8, (64, 64), 0),                   # a round of 1024 points and one
    (4, 257, 2**16, 2**16, 16, (8, 64), 0),                    # two lanes per point
    (4, 40007, 2**18, 2**15, 8, (32, 16), 0),
    (3, 50003, 2**19, 1, 1, (64, 0), 0),                       # plain hashing: one table
    (3, 70001, 2**18, 2**11, 8, (32, 1), 0),                   # 33 bins: written directly
    (3, 70001, 2**14, 2**18, 4, (2, 64), 0),                   # two bins of one table
    (3, 60001, 2**21, 2**19, 8, (256, 256), 0),                # the most bins
    (3, 30001, 2**21, 2**20, 8, (256, 512), 0),                # more than that
    (3, 200003, 2**18, 2**15, 8, (32, 16), 3),                 # entries of merged levels
    (2, 400003, 2**19, 2**12, 2, (64, 1), 3),                  # a single bin of one table: written directly
    (2, 400003, 2**21, 1, 1, (256, 0), 0),                     # (plain hashing with three levels is not merged)
])
def test_scatter_in_runs_against_the_oracle(d, N, N_f, N_c, N_p, slices, merged):
    w = W.custom(cfg=120, d=d, L=4, N_f=N_f, N_c=N_c, N_p=N_p, N_min=40, N_max=100 if d < 4 else 60, N=N, feat_dtype="f16", io_dtype="f16")
    check(w, slices, merged_levels=merged)


def test_pre_reduced_levels_beside_runs():
    w = W.custom(cfg=121, d=3, L=5, N_f=2**18, N_c=2**16, N_p=8, N_min=8, N_max=300, N=70001, feat_dtype="f32", io_dtype="f32")
    check(w, (32, 32), dense_levels=3)


@pytest.mark.parametrize("N", [70001, 200003])
def test_runs_of_equal_points_fill_single_bins(N):
    """All references of a wavefront in eight bins of either table, 512 in one at most: the largest rank there is; and points on faces,
    whose weightless corners are not written."""
    w = W.custom(cfg=122, d=3, L=3, N_f=2**18, N_c=2**16, N_p=8, N_min=60, N_max=200, N=N, feat_dtype="f16", io_dtype="f16")
    x = np.full((N, 3), (0.31, 0.62, 0.17), dtype=np.float32)
    x[::3] = (0.0, 0.5, 1.0)
    check(w, (32, 32), x=x)
