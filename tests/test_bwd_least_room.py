"""The smallest workspace that a backward call accepts, asked without a GPU: the room is looked at before anything is launched, so a call
with enough of it ends at the missing device and one without is refused.  Its pointers are made up, so it does not run where there is a
device.  Plain hashing (N_p = 1) with tables of few slices, and tables of few slices where levels are merged: binned where the room is
there, scanned in what a scan takes."""
import ctypes
import dataclasses

import pytest
import torch

import paper_2312_17241_amd as cngp

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="its pointers are made up")
P = ctypes.c_void_p(1 << 20)


def config(d, L, N_f, N_c, N_p, N_max, **kw):
    return cngp.Config(**{**dict(d=d, L=L, F=2, N_f=N_f, N_c=N_c, N_p=N_p, N_min=16, N_max=N_max, feat_dtype=cngp.F16, io_dtype=cngp.F16,
                                 flags=cngp.ZERO_GRADS), **kw})


def accepts(cfg, N, room):
    return cngp._lib.cngp_encode_bwd(ctypes.byref(cfg.c()), P, N, P, P, P, P, P, P, room, None) != cngp.ERR_WORKSPACE


def accepts_static(cfg, N):
    return cngp._lib.cngp_encode_bwd_static(ctypes.byref(cfg.c()), P, N, P, P, P, P, P, None) != cngp.ERR_WORKSPACE


def scan_bytes(cfg, N):
    """What a replicated scan takes in one launch: flagged, and in the few chunks that a bound on the bins asks for."""
    return cngp.workspace_bytes(dataclasses.replace(cfg, flags=cfg.flags | cngp.BWD_SLICED, bin_bytes_max=1 << 20), N)


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N_max,N", [
    (3, 16, 2**17, 1, 1, 2048, 202209),
    (3, 16, 2**16, 1, 1, 8192, 200831),
    (4, 9, 2**17, 1, 1, 860, 133118),
    (2, 16, 2**17, 1, 1, 4096, 700009),                       # levels merged
    (2, 16, 2**16, 2**12, 8, 8192, 2**20),                    # 8 + 2 slices, levels merged
    (3, 16, 2**17, 1, 1, 2048, 20_000_000),                   # passes
])
@pytest.mark.parametrize("F", [2, 4])
def test_the_room_of_a_scan_is_enough(d, L, N_f, N_c, N_p, N_max, N, F):
    cfg = config(d, L, N_f, N_c, N_p, N_max, F=F)
    room = scan_bytes(cfg, N)
    assert room < cngp.workspace_bytes(cfg, N)                # (binned with the room it asks for)
    assert accepts(cfg, N, room) and not accepts(cfg, N, 4096)
    if room <= cngp.static_scratch_bytes():
        assert accepts_static(cfg, N)


@pytest.mark.parametrize("bound", [1 << 26, 1 << 33])
def test_a_bound_on_the_bins_leaves_few_slices_scanned(bound):
    for args, N in (((3, 16, 2**17, 1, 1, 2048), 202209), ((2, 16, 2**16, 2**12, 8, 8192), 2**20)):
        cfg = config(*args, bin_bytes_max=bound)
        assert cngp.bwd_plan_info(cfg, N)["binned"] == 0 and cngp.workspace_bytes(cfg, N) == scan_bytes(cfg, N)


@pytest.mark.parametrize("N", [17_000_000, 20_000_000, 40_000_000, 190_000_000])
def test_a_workspace_of_a_batch_in_passes_serves_every_shorter_one(N):
    cfg = config(3, 16, 2**17, 1, 1, 2048)
    have = cngp.workspace_bytes(cfg, N)
    for n in (N - 1, N * 7 // 8, N * 3 // 4, 16_000_000, 14_000_000, 12_000_000, 8_400_000, 300_000, 202209, 1000):
        assert n > N or accepts(cfg, n, have), (n, N)


@pytest.mark.parametrize("F", [2, 4])
@pytest.mark.parametrize("args,bound", [((4, 7, 2**18, 2**8, 16, 2048), 0), ((3, 9, 2**9, 2**17, 16, 2048), 0), ((3, 16, 2**16, 2**14, 16, 2048), 0),
                                        ((4, 10, 2**16, 2**16, 16, 2048), 1 << 28), ((3, 6, 2**18, 1, 1, 256), 1 << 28), ((2, 12, 2**18, 2**12, 8, 4096), 1 << 26)])
def test_tables_that_are_always_binned_too(args, bound, F):
    """One more point than fits a pass is taken in two halves, whose workspace is smaller than that of one pass."""
    cfg = config(*args, F=F, bin_bytes_max=bound)
    most = 1                                                  # the longest batch in one pass
    while cngp.bwd_plan_info(cfg, 2 * most)["passes"] == 1:
        most *= 2
    step = most // 2
    while step:
        most += step if cngp.bwd_plan_info(cfg, most + step)["passes"] == 1 else 0
        step //= 2
    for N in (most + 1, most * 3 // 2, 2 * most + 1, 5 * most + 12345):
        have = cngp.workspace_bytes(cfg, N)
        for n in (most // 3, most // 2, most // 2 + 1, most * 3 // 4, most, most + 1, 2 * most, 2 * most + 1, 3 * most, 4 * most, N - 1):
            assert n > N or accepts(cfg, n, have), (n, N)
    assert cngp.workspace_bytes(cfg, most + 1) < cngp.workspace_bytes(cfg, most)
    assert not accepts(cfg, most, cngp.workspace_bytes(cfg, most) // 8) and not accepts(cfg, most, 4096)
