"""Which forward calls put several levels into a workgroup (csrc/cngp_fwd_level.h, encode_fwd_group_kernel), and what the plan query says of them.
Host arithmetic only."""
import dataclasses

import pytest

import paper_2312_17241_amd as cngp

FMT = {"u8": cngp.IDX_U8, "packed4": cngp.IDX_PACKED4, "bits": cngp.IDX_BITS}


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,feat,fmt,N,levels", [
    (3, 16, 2**8, 2**16, 8, "f16", "bits", 2**22, 4),           # 25 KB a level
    (3, 16, 2**8, 2**12, 8, "f16", "packed4", 70001, 4), (3, 16, 2**8, 2**12, 8, "f16", "packed4", 300007, 8), (3, 16, 2**8, 2**12, 8, "f16", "packed4", 2**19 + 77, 16),
    (2, 12, 2**10, 2**12, 4, "f16", "u8", 300007, 4), (2, 12, 2**10, 2**12, 4, "f16", "u8", 2**19 + 77, 12),
    (4, 8, 2**9, 2**10, 2, "f32", "bits", 300007, 4), (4, 8, 2**9, 2**10, 2, "f32", "bits", 2**19 + 77, 8),
    (2, 20, 2**8, 2**12, 8, "f16", "packed4", 2**19 + 77, 20),
    (3, 10, 2**8, 2**12, 8, "f16", "packed4", 300007, 0),       # no whole fours
    (3, 16, 2**16, 2**14, 16, "f16", "packed4", 2**22, 0),      # a level's features do not fit
    (3, 16, 2**12, 2**16, 8, "f32", "u8", 2**22, 0),            # four levels' do not
])
def test_levels_to_a_workgroup(d, L, N_f, N_c, N_p, feat, fmt, N, levels):
    cfg = cngp.Config(d=d, L=L, F=2, N_f=N_f, N_c=N_c, N_p=N_p, N_min=4, N_max=300, feat_dtype=cngp.F16 if feat == "f16" else cngp.F32, io_dtype=cngp.F16,
                      index_format=FMT[fmt], flags=0)
    assert cngp.fwd_group_levels(cfg, N) == levels
    plan = cngp.fwd_plan_info(cfg, N)
    assert plan["level_resident"] == 1
    if levels:
        probes = 4 * -(-N_c * (N_p.bit_length() - 1) // 32) + 4 if fmt == "bits" else (N_c + 1) // 2
        assert plan["lds_bytes"] == levels * ((probes + 15) // 16 * 16 + N_f * (4 if feat == "f16" else 8)) <= 160 * 1024
        assert plan["parts"] * (L // levels) >= 224                 # workgroups: a round of 256 CUs, or nearly
    assert cngp.fwd_group_levels(cfg, 0) == 0


def test_refusals():
    cfg = cngp.Config(d=3, L=16, F=2, N_f=2**8, N_c=2**12, N_p=8, N_min=4, N_max=300, feat_dtype=cngp.F16, io_dtype=cngp.F16, index_format=cngp.IDX_U8, flags=0)
    with pytest.raises(RuntimeError):
        cngp.fwd_group_levels(cfg, -1)
    for off in (cngp.FWD_SIMPLE, cngp.FWD_TILE):
        assert cngp.fwd_group_levels(dataclasses.replace(cfg, flags=off), 2**20) == 0
