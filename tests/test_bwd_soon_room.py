"""Batches below 2^21 references that are binned: the room that the scan or the atomics took is still enough, a bound on the bins leaves them
unbinned, and no shorter batch needs more than a longer one's workspace.  Without a GPU, as test_bwd_least_room.py."""
import dataclasses

import pytest
import torch

import paper_2312_17241_amd as cngp
from test_bwd_least_room import accepts, config

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="its pointers are made up")


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N,binned", [
    (3, 16, 2**16, 2**14, 16, 2047, 0), (3, 16, 2**16, 2**14, 16, 2048, 1), (3, 16, 2**16, 2**14, 16, 16383, 1),      # many candidates
    (2, 16, 2**17, 2**15, 16, 16383, 0), (2, 16, 2**17, 2**15, 16, 16384, 1),                                          # ... d = 2
    (4, 8, 2**17, 2**13, 16, 8191, 0), (4, 8, 2**17, 2**13, 16, 8192, 1), (3, 16, 2**18, 2**16, 16, 4000, 0),          # ... d = 4, 96 slices
    (3, 16, 2**18, 2**16, 8, 8191, 0), (3, 16, 2**18, 2**16, 8, 8192, 1),
    (3, 16, 2**13, 2**16, 8, 12000, 0), (3, 16, 2**18, 2**11, 16, 14000, 0),                                           # one or two slices of a table
    (3, 16, 2**8, 2**14, 16, 2047, 0), (3, 16, 2**8, 2**14, 16, 2048, 1), (3, 16, 2**8, 2**14, 16, 4096, 0),          # small feature table
    (3, 12, 2**12, 2**16, 8, 3141, 0), (3, 16, 2**11, 2**15, 8, 3176, 1), (3, 16, 2**12, 2**16, 16, 2580, 0),                                                                                # ... 256 slices of the other
])
def test_which_short_batches_are_binned(d, L, N_f, N_c, N_p, N, binned):
    cfg = config(d, L, N_f, N_c, N_p, 1024)
    assert cngp.bwd_plan_info(cfg, N)["binned"] == binned
    bounded = dataclasses.replace(cfg, bin_bytes_max=8 << 30)
    assert cngp.bwd_plan_info(bounded, N)["binned"] == 0
    before = cngp.workspace_bytes(bounded, N)
    assert accepts(cfg, N, before) and before <= cngp.workspace_bytes(cfg, N)
    for longer in (N + 1, 2 * N, 3 * N + 5, 16384, 20011, 300007):
        assert longer < N or accepts(cfg, N, cngp.workspace_bytes(cfg, longer)), longer
