"""Backward of small batches with small tables: a level's two gradient tables accumulated in LDS by workgroups of 1024
lanes, against the oracle (Sec. 3, Fig. 3) and beside the variant that adds to memory directly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2312_17241_amd as cngp
import workloads as W
from parity import check_close

pytestmark = pytest.mark.gpu


# one point, one less / more than a workgroup's lane groups, several chunks per level; N_p from 1 to 16; the largest
# tables that are taken (2^13 feature entries at N_p = 1: exactly 128 KB) and the first that are not
@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N,feat,io,top_k", [
    (2, 4, 2**10, 2**8, 4, 1, "f32", "f32", 0), (2, 4, 2**10, 2**8, 4, 255, "f32", "f32", 0), (2, 4, 2**10, 2**8, 4, 4097, "f16", "f32", 0),
    (3, 5, 2**9, 2**6, 16, 65, "f16", "f16", 3), (3, 1, 2**13, 1, 1, 3001, "f32", "f16", 0), (3, 2, 2**13, 2, 2, 1500, "f32", "f32", 0),
    (4, 3, 2**8, 2**7, 8, 1290, "f32", "f32", 0), (2, 32, 2**6, 2**5, 2, 700, "f16", "f32", 1),
    (4, 12, 2**10, 2**9, 16, 100, "f32", "f32", 0), (3, 2, 2**11, 2**8, 16, 1023, "f16", "f16", 0),   # cut into whole wavefronts
    (3, 1, 2**12, 2**11, 2, 513, "f32", "f32", 0), (2, 3, 2**8, 1, 1, 1025, "f32", "f32", 0)])
def test_small_tables_accumulate_in_lds(d, L, N_f, N_c, N_p, N, feat, io, top_k):
    w = W.custom(cfg=80 + d + N_p, d=d, L=L, F=2, N_f=N_f, N_c=N_c, N_p=N_p, N_min=4, N_max=64, N=N, feat_dtype=feat, io_dtype=io)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    x, D_f, Dhat, dy = W.make_points(w), W.make_feature_codebook(w), W.make_probe_logits(w), W.make_upstream_grad(w, N)
    x[0] = 1.0
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, x, D_f, Dhat, dy, top_k=top_k) if top_k else oracle.encode_bwd(w, x, D_f, Dhat, dy)
    for flags in (cngp.ZERO_GRADS, cngp.ZERO_GRADS | cngp.BWD_DIRECT):
        cfg = cngp.Config.from_workload(w, flags=flags, top_k=top_k)
        gF = torch.full((L, N_f, 2), 7.0, device="cuda")
        gC = torch.full((L, N_c, N_p), 7.0, device="cuda")
        cngp.profile_enable(True)
        cngp.profile_read()
        cngp.encode_bwd(cfg, dev(x), dev(D_f), dev(Dhat), dev(dy), gF, gC)
        torch.cuda.synchronize()
        ran = {k for k in cngp.profile_read() if k != "zero"}
        cngp.profile_enable(False)
        # fp64 copies of both tables in 128 KB of LDS
        fits = 8 * (2 * N_f + (N_c * N_p if N_p > 1 else 0)) <= 128 * 1024
        assert ran == {"encode_bwd_small" if fits and not flags & cngp.BWD_DIRECT else "encode_bwd_direct"}
        check_close("grad D_f", gF.cpu().numpy(), gF_ref, A_f, fp16_out=False)
        check_close("grad Dhat_c", gC.cpu().numpy(), gC_ref, A_c, fp16_out=False)
    # without clearing, a second call adds the same gradients once more
    cfg = cngp.Config.from_workload(w, top_k=top_k)
    cngp.encode_bwd(cfg, dev(x), dev(D_f), dev(Dhat), dev(dy), gF, gC)
    torch.cuda.synchronize()
    check_close("grad D_f, twice", gF.cpu().numpy(), 2 * gF_ref, 2 * A_f, fp16_out=False)


# nerf3d's tables and one with few vertices on its coarse levels, on both sides of the choice and of the line above which it
# is always taken; the dense grids of 2^20 references or more as before
@pytest.mark.parametrize("d,L,N_min,N_max,N_f,N,dense", [(3, 16, 16, 2048, 2**16, 20011, False), (3, 16, 16, 2048, 2**16, 80000, True),
                                                       (2, 12, 16, 512, 2**16, 60000, False), (2, 12, 16, 512, 2**16, 2**18 - 1, True),
                                                       (3, 8, 8, 256, 2**18, 2**17 - 1, True), (3, 8, 8, 256, 2**18, 2**17, True), (2, 8, 8, 256, 2**18, 2**18, True)])
def test_binned_batches_pre_reduce_where_it_pays(d, L, N_min, N_max, N_f, N, dense):
    """A batch below a million references per level bins every level or sums the coarse ones per vertex: the same gradients."""
    w = W.custom(cfg=95 + d, d=d, L=L, F=2, N_f=N_f, N_c=2**14, N_p=16, N_min=N_min, N_max=N_max, N=N, feat_dtype="f32", io_dtype="f32")
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")
    args = [dev(a) for a in (W.make_points(w), W.make_feature_codebook(w), W.make_probe_logits(w), W.make_upstream_grad(w, N))]
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS)
    info = cngp.bwd_plan_info(cfg, N)
    assert info["binned"] == 1 and (info["dense_levels"] > 0) == dense
    got = cngp.encode_bwd(cfg, *args, workspace=cngp.alloc_workspace(cfg, N))
    mag = cngp.encode_bwd(cfg, *args[:3], args[3].abs(), workspace=cngp.alloc_workspace(cfg, N))[0]
    ref_cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS | cngp.BWD_DIRECT)
    ref = cngp.encode_bwd(ref_cfg, *args)
    torch.cuda.synchronize()
    # the direct kernel sums in fp32: up to a few thousand terms to an entry, 2^-24 each, of the terms' magnitudes
    assert bool(((got[0] - ref[0]).abs() <= 1e-4 * mag + 1e-12).all())
    assert float((got[0] - ref[0]).norm() / ref[0].norm()) < 1e-5 and float((got[1] - ref[1]).norm() / ref[1].norm()) < 1e-5
