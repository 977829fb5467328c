"""Binned backward on both sides of the batch size from which levels are merged (csrc/cngp_api.hip, kMinMergeRefs), and in a workspace of
the layout without them, against the oracle."""
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


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N_min,N_max,feat,io", [
    (3, 8, 2**17, 2**14, 8, 16, 300, "f16", "f16"),                    # 16 + 8 slices
    (2, 8, 2**13, 2**15, 16, 30, 3000, "f32", "f32"),                  # 1 + 32
    (2, 6, 2**18, 1, 1, 16, 2048, "f16", "f16"),                       # plain hashing, 32
])
@pytest.mark.parametrize("past", [0, 1])
def test_batches_at_the_line(d, L, N_f, N_c, N_p, N_min, N_max, feat, io, past):
    N = ((9 << 17) >> d) - 1 + past
    w = W.custom(cfg=150, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N, feat_dtype=feat, io_dtype=io)
    D_f = W.make_feature_codebook(w)
    args = W.make_points(w), (D_f.astype(np.float64) * 1e4).astype(D_f.dtype), W.make_probe_logits(w), W.make_upstream_grad(w)
    cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS)
    plan = cngp.bwd_plan_info(cfg, N)
    assert plan["binned"] == 1 and (plan["merged_levels"] > 0) == bool(past)
    gF_ref, gC_ref, A_f, A_c = oracle.encode_bwd(w, *args)
    bounded = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS, bin_bytes_max=8 << 30)     # (a bound: nothing is merged for it)
    for room in (cngp.workspace_bytes(cfg, N), cngp.workspace_bytes(bounded, N)):
        ws = torch.full((room,), 0xAB, dtype=torch.uint8, device="cuda")
        gF, gC = (torch.full(s, float("nan"), device="cuda") for s in ((L, N_f, 2), (L, N_c, N_p)))
        cngp.encode_bwd(cfg, *(dev(a) for a in args), gF, gC, workspace=ws)
        check_close("grad D_f", gF.cpu().numpy(), gF_ref, A_f, fp16_out=False)
        check_close("grad Dhat_c", gC.cpu().numpy(), gC_ref, A_c, fp16_out=False)
