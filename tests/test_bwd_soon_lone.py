"""Batches from 2^19 references on that are binned although shorter than 2^21: one drain workgroup per bin, as a scan has one rounding per entry; where
that leaves few, long bins they are scanned.  Host arithmetic only."""
import random

import pytest

import paper_2312_17241_amd as cngp
from test_bwd_least_room import config


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N,binned", [
    (3, 8, 2**16, 2**14, 16, 20011, 1), (3, 8, 2**16, 2**14, 16, 23744, 1), (3, 8, 2**16, 2**14, 16, 30000, 1),
    (3, 8, 2**17, 2**13, 16, 24860, 1), (3, 12, 2**17, 2**13, 16, 16462, 1), (4, 8, 2**17, 2**13, 16, 8192, 1),
    (3, 4, 2**16, 2**14, 16, 16384, 1), (3, 4, 2**16, 2**14, 16, 16385, 0), (3, 4, 2**16, 2**14, 16, 60000, 0),       # 4 * 4096 references in a bin
    (3, 6, 2**17, 2**13, 16, 24576, 1), (3, 6, 2**17, 2**13, 16, 24577, 0),
    (3, 4, 2**18, 2**16, 8, 60000, 1), (3, 2, 2**16, 2**14, 16, 120000, 0), (3, 1, 2**16, 2**14, 16, 231072, 0), (3, 1, 2**18, 2**16, 8, 200000, 0),
])
def test_writers_of_a_bin(d, L, N_f, N_c, N_p, N, binned):
    plan = cngp.bwd_plan_info(config(d, L, N_f, N_c, N_p, 2048), N)
    assert plan["binned"] == binned and plan["sliced"] == 1, plan
    assert not binned or (plan["drain_wgs_feat"], plan["drain_wgs_logit"]) == (1, 1), plan
    forced = cngp.bwd_plan_info(config(d, L, N_f, N_c, N_p, 2048, flags=cngp.BWD_BINNED), N)
    assert forced["binned"] == 1


def test_drawn_batches():
    rng, seen = random.Random(5), 0
    for _ in range(4000):
        d, L = rng.choice((2, 3, 3, 4)), rng.randint(1, 20)
        cfg = config(d, L, 2**rng.randint(13, 18), 2**rng.randint(11, 17), 2**rng.randint(1, 4), 2048)
        N = int(2 ** rng.uniform(18, 21) / (L << d))
        plan, refs = cngp.bwd_plan_info(cfg, N), (N << d) * L
        if refs >= 2**19 and refs < 2**21 and plan["binned"]:
            seen += 1
            assert (plan["drain_wgs_feat"], plan["drain_wgs_logit"]) == (1, 1), (cfg, N, plan)
            assert plan["merged_levels"] == 0
    assert seen > 100


def test_a_flag_about_coarse_levels_does_not_change_the_variant():
    rng, seen = random.Random(6), 0
    for _ in range(2000):
        d, L = rng.choice((2, 3, 3, 4)), rng.randint(1, 20)
        sizes = d, L, 2**rng.randint(6, 18), 2**rng.randint(11, 17), 2**rng.randint(1, 4), 2048
        N = int(2 ** rng.uniform(17, 21) / (L << d))
        plain, flagged = (cngp.bwd_plan_info(config(*sizes, flags=f), N) for f in (cngp.ZERO_GRADS, cngp.ZERO_GRADS | cngp.BWD_NO_PREREDUCE))
        seen += plain["binned"]
        assert flagged["binned"] == plain["binned"] and flagged["dense_levels"] == 0, (sizes, N)
    assert seen > 200
