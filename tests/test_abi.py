"""Host-side checks of the C ABI: the library loads, exports every symbol the header declares,
validates arguments before touching the GPU, and computes the level table.  No GPU needed:
no call here reaches a kernel launch.
"""
import ctypes
import dataclasses
import os
import re

import numpy as np
import pytest

import paper_2312_17241_amd as cngp
import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GOLDEN = os.path.join(ROOT, "tests", "golden")


def declared_functions():
    text = open(os.path.join(ROOT, "include", "cngp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(cngp_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = declared_functions()
    assert {"cngp_encode_fwd", "cngp_encode_bwd", "cngp_bake_probes", "cngp_level_resolutions",
            "cngp_workspace_bytes", "cngp_debug_indices"} <= set(names)
    lib = ctypes.CDLL(cngp.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_error_strings():
    assert cngp.version() >= 100
    seen = {cngp.error_string(s) for s in range(0, -6, -1)}
    assert len(seen) == 6 and all(seen)
    assert "unknown" in cngp.error_string(-99)


def base_cfg(**kw):
    return cngp.Config.from_workload(W.WORKLOADS["nerf3d"], **kw)


@pytest.mark.parametrize("nmin,nmax,L,expect", [
    (int(h.split()[0]), int(h.split()[1]), int(h.split()[2]), list(map(int, t.split())))
    for h, t in (ln.split(":") for ln in open(os.path.join(GOLDEN, "level_tables.txt"))
                 if ln.strip() and not ln.startswith("#"))])
def test_level_table_golden(nmin, nmax, L, expect):
    cfg = base_cfg(N_min=nmin, N_max=nmax, L=L)
    assert cngp.level_resolutions(cfg).tolist() == expect


def test_level_table_edge_cases():
    assert cngp.level_resolutions(base_cfg(L=1, N_min=7, N_max=3)).tolist() == [7]
    assert cngp.level_resolutions(base_cfg(L=11, N_min=1, N_max=1024)).tolist() == [2**i for i in range(11)]
    r = cngp.level_resolutions(base_cfg(L=16, N_min=16, N_max=524288))
    assert r[0] == 16 and r[-1] == 524288 and np.all(np.diff(r.astype(np.int64)) > 0)


BAD = [
    dict(d=1), dict(d=5), dict(L=0), dict(L=33), dict(F=0),
    dict(N_f=0), dict(N_f=3000), dict(N_c=0), dict(N_c=100), dict(N_p=0), dict(N_p=3), dict(N_p=32),
    dict(N_p=16, N_f=8), dict(N_min=0), dict(N_max=8), dict(N_max=2**25),
    dict(feat_dtype=2), dict(io_dtype=-1), dict(index_format=3), dict(flags=256), dict(flags=64 | 128), dict(flags=64 | 16), dict(flags=6), dict(flags=34),
    dict(index_format=cngp.IDX_PACKED4, N_c=1, N_p=1), dict(top_k=17), dict(N_p=4, top_k=5),
]


@pytest.mark.parametrize("over", BAD, ids=[str(b) for b in BAD])
def test_invalid_configs_are_rejected_on_the_host(over):
    c = base_cfg(**over).c()
    one = ctypes.c_void_p(256)          # never dereferenced: validation fails first
    lib = cngp._lib
    assert lib.cngp_encode_fwd(ctypes.byref(c), one, 8, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_encode_bwd(ctypes.byref(c), one, 8, one, one, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_bake_probes(ctypes.byref(c), one, one, None) == cngp.ERR_INVALID
    assert lib.cngp_debug_indices(ctypes.byref(c), one, 8, one, one, one, one, one, None) == cngp.ERR_INVALID
    assert cngp.workspace_bytes(base_cfg(**over), 8) == 0


def test_reserved_field_must_be_zero_and_top_k_up_to_the_probing_range_is_valid():
    c = base_cfg().c()
    c.reserved = 1
    assert cngp._lib.cngp_bake_probes(ctypes.byref(c), ctypes.c_void_p(256), ctypes.c_void_p(256), None) == cngp.ERR_INVALID
    for k in (0, 1, base_cfg().N_p):
        assert cngp.workspace_bytes(base_cfg(top_k=k, flags=cngp.BWD_SLICED), 1 << 16) > 0


def test_unsupported_feature_width():
    c = base_cfg(F=3).c()                # 1, 2, 4 and 8 are built; the others are valid in the paper's terms only
    one = ctypes.c_void_p(256)
    assert cngp._lib.cngp_encode_fwd(ctypes.byref(c), one, 8, one, one, one, None, 0, None) == cngp.ERR_UNSUPPORTED
    out = np.zeros(16, np.uint32)        # the level table does not depend on F
    assert cngp._lib.cngp_level_resolutions(ctypes.byref(c), out.ctypes.data_as(ctypes.c_void_p)) == cngp.OK


def test_null_pointers_and_negative_counts():
    c = base_cfg().c()
    one = ctypes.c_void_p(256)
    lib = cngp._lib
    assert lib.cngp_encode_fwd(None, one, 8, one, one, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_fwd(ctypes.byref(c), None, 8, one, one, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_fwd(ctypes.byref(c), one, 8, None, one, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_fwd(ctypes.byref(c), one, 8, one, None, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_fwd(ctypes.byref(c), one, 8, one, one, None, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_fwd(ctypes.byref(c), one, -1, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_encode_fwd(ctypes.byref(c), None, 0, None, None, None, None, 0, None) == cngp.OK   # N == 0
    assert lib.cngp_encode_bwd(ctypes.byref(c), one, 8, one, one, one, None, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_bwd(ctypes.byref(c), one, 8, one, None, one, one, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_bwd(ctypes.byref(c), one, -5, one, one, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_bake_probes(ctypes.byref(c), None, one, None) == cngp.ERR_NULL
    assert lib.cngp_bake_probes(ctypes.byref(c), one, None, None) == cngp.ERR_NULL
    assert lib.cngp_debug_indices(ctypes.byref(c), None, 8, one, one, one, one, one, None) == cngp.ERR_NULL
    assert lib.cngp_debug_indices(ctypes.byref(c), one, 8, None, one, one, one, None, None) == cngp.ERR_NULL
    assert lib.cngp_level_resolutions(ctypes.byref(c), None) == cngp.ERR_NULL
    # encoding + decoder in one call: checked on the host in the same way, with or without a workspace
    b = base_cfg()
    m, m_bad = cngp.MlpConfig(b.L * b.F, 3).c(), cngp.MlpConfig(b.L * b.F - 2, 3).c()
    mp = lambda v: ctypes.cast(ctypes.byref(v), ctypes.c_void_p)
    assert lib.cngp_encode_mlp_fwd(ctypes.byref(c), mp(m), None, 8, one, one, one, one, None, 0, None) == cngp.ERR_NULL
    assert lib.cngp_encode_mlp_fwd(ctypes.byref(c), mp(m), one, 8, one, one, None, one, one, 1 << 20, None) == cngp.ERR_NULL
    assert lib.cngp_encode_mlp_fwd(ctypes.byref(c), mp(m), one, -1, one, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_encode_mlp_fwd(ctypes.byref(c), mp(m_bad), one, 8, one, one, one, one, None, 0, None) == cngp.ERR_INVALID
    assert lib.cngp_encode_mlp_fwd(ctypes.byref(c), mp(m), None, 0, None, None, None, None, None, 0, None) == cngp.OK


def test_adam_step_bake_rejects_bad_arguments():
    """Every check of the optimiser entry point runs on the host before anything is launched."""
    lib = ctypes.CDLL(cngp.LIB_PATH)
    c = base_cfg().c()                                   # nerf3d: fp16 feature storage
    a = ctypes.c_void_p(4096)                            # an aligned, never dereferenced address
    ok = cngp.Adam().c()
    feats = [a, a, a, a, a]
    logits = [a, a, a, a, a]

    def call(cfg, of, oc, f=feats, l=logits):
        ref = lambda o: None if o is None else ctypes.cast(ctypes.byref(o), ctypes.c_void_p)
        return lib.cngp_adam_step_bake(ctypes.byref(cfg), ref(of), ref(oc), *f, *l, None)

    assert call(c, None, None) == cngp.OK                # nothing to do
    for bad in (dict(lr=-1.0), dict(lr=float("nan")), dict(beta1=1.0), dict(beta2=-0.1), dict(eps=0.0),
                dict(step=0), dict(grad_scale=float("inf"))):
        assert call(c, cngp.Adam(**bad).c(), None) == cngp.ERR_INVALID, bad
        assert call(c, None, cngp.Adam(**bad).c()) == cngp.ERR_INVALID, bad
    for i in range(5):
        f = list(feats); f[i] = None
        assert call(c, ok, None, f=f) == cngp.ERR_NULL, i
        l = list(logits); l[i] = None
        assert call(c, None, ok, l=l) == cngp.ERR_NULL, i
    for i in (0, 2, 3, 4):                               # misaligned float arrays
        f = list(feats); f[i] = ctypes.c_void_p(4100)
        assert call(c, ok, None, f=f) == cngp.ERR_INVALID, i
    for i in range(4):
        l = list(logits); l[i] = ctypes.c_void_p(4104)
        assert call(c, None, ok, l=l) == cngp.ERR_INVALID, i
    c32 = base_cfg(feat_dtype=cngp.F32).c()              # fp32 storage: D_f is NULL or the master itself
    assert call(c32, ok, None, f=[a, ctypes.c_void_p(8192), a, a, a]) == cngp.ERR_INVALID
    bad_cfg = base_cfg(N_p=3).c()
    assert call(bad_cfg, ok, ok) == cngp.ERR_INVALID


def test_storage_bytes_match_the_oracle_arithmetic():
    import oracle
    for N_p, N_c, fmt in [(8, 65536, cngp.IDX_BITS), (16, 16384, cngp.IDX_BITS), (2, 4, cngp.IDX_BITS), (1, 64, cngp.IDX_BITS),
                          (4, 8, cngp.IDX_BITS), (8, 1, cngp.IDX_BITS), (16, 16384, cngp.IDX_U8), (16, 16384, cngp.IDX_PACKED4)]:
        w = W.custom(d=3, L=16, N_f=256, N_c=N_c, N_p=N_p, N_min=16, N_max=2048, N=16, feat_dtype="f16")
        got = cngp.storage_bytes(cngp.Config.from_workload(w, index_format=fmt))
        if fmt == cngp.IDX_PACKED4:
            want = {"D_f": 16 * 256 * 2 * 2, "D_c_level": N_c // 2, "D_c": 16 * N_c // 2}
        else:
            want = oracle.storage_bytes(w, index_bits_exact=(fmt == cngp.IDX_BITS))
        assert got == want, (N_p, N_c, fmt)
        assert cngp.Config.from_workload(w, index_format=fmt).index_cols == want["D_c_level"]


def test_backward_plan_is_reported_on_the_host():
    """The plan needs no GPU: benchmark shapes take the LDS-sliced variant with merged coarse levels, pre-reduced ones in a
    bounded workspace, a tiny batch takes global atomics, and the flags override the choice."""
    w = W.WORKLOADS["nerf3d"]
    p = cngp.bwd_plan_info(cngp.Config.from_workload(w), w.N)
    assert p["sliced"] == 1 and p["slices_f"] == 8 and p["slices_c"] == 16 and p["dense_levels"] == 0 and p["merged_levels"] == 6
    pg = cngp.bwd_plan_info(cngp.Config.from_workload(w, bin_bytes_max=4 << 30), w.N)
    assert pg["sliced"] == 1 and 1 <= pg["dense_levels"] <= 6 and pg["merged_levels"] == 0
    assert cngp.workspace_bytes(cngp.Config.from_workload(w), w.N) >= 4 * w.L * w.N_c * w.N_p + 2 * w.N * w.L * w.F
    t = W.WORKLOADS["tiny2d"]
    assert cngp.bwd_plan_info(cngp.Config.from_workload(t), t.N)["sliced"] == 0
    assert cngp.bwd_plan_info(cngp.Config.from_workload(t, flags=cngp.BWD_SLICED), t.N)["sliced"] == 1
    assert cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_DIRECT), w.N)["sliced"] == 0
    assert cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_NO_PREREDUCE), w.N)["dense_levels"] == 0
    pb = cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_BINNED), w.N)
    assert pb["sliced"] == 1 and pb["binned"] == 1 and pb["drain_wgs_feat"] >= 1 and pb["bin_chunks"] == 256
    assert cngp.workspace_bytes(cngp.Config.from_workload(w, flags=cngp.BWD_BINNED), w.N) > 2 * (w.L - pb["dense_levels"]) * w.N * 8 * 4
    assert p["binned"] == 1                               # two dozen slices per level: the library bins by itself
    assert cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_SLICED), w.N)["binned"] == 0
    im = W.WORKLOADS["image2d"]
    pi = cngp.bwd_plan_info(cngp.Config.from_workload(im), im.N)     # ten slices: binned because eleven levels are merged, else a replicated scan
    assert pi["binned"] == 1 and pi["merged_levels"] == 11 and pi["bin_chunks"] >= 1 and pi["drain_wgs_feat"] >= 1
    for scan in (dict(flags=cngp.BWD_SLICED), dict(flags=cngp.BWD_NO_PREREDUCE), dict(bin_bytes_max=8 << 30)):
        ps = cngp.bwd_plan_info(cngp.Config.from_workload(im, **scan), im.N)
        assert ps["binned"] == 0 and ps["merged_levels"] == 0 and ps["sliced"] == 1
    huge = cngp.Config.from_workload(w)                   # 2^25 points: the bins would take 32 GiB: 4 passes of 8 GiB
    ph = cngp.bwd_plan_info(huge, 2**25)
    assert ph["binned"] == 1 and ph["passes"] == 4 and cngp.workspace_bytes(huge, 2**25) < 10 << 30
    assert cngp.workspace_bytes(huge, 2**25) == cngp.workspace_bytes(huge, 2**23)
    pf = cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_BINNED), 2**25)   # on request: in one pass
    assert pf["binned"] == 1 and pf["passes"] == 1
    assert cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_BINNED), 2**29)["passes"] == 3   # 2^31 references at most
    small = cngp.Config.from_workload(w, bin_bytes_max=1 << 30)
    assert cngp.bwd_plan_info(small, w.N)["passes"] == 1 and cngp.bwd_plan_info(small, 2**22)["passes"] == 4
    assert cngp.bwd_plan_info(cngp.Config.from_workload(w, bin_bytes_max=1 << 20), w.N)["binned"] == 0    # too small to bin
    assert p["passes"] == 1 and cngp.bwd_plan_info(cngp.Config.from_workload(w, flags=cngp.BWD_SLICED), 2**25)["passes"] == 1
    # the paper's compressed configurations (small N_f): binned by confidence-table slice only, both gradients in one pass
    for N_f, N_c, N_p, flag in ((2**8, 2**16, 8, 0), (2**12, 2**12, 16, 0), (2**6, 2**10, 4, cngp.BWD_BINNED)):
        small_f = W.custom(d=3, L=16, N_f=N_f, N_c=N_c, N_p=N_p, N_min=16, N_max=2048, N=2**18)
        ps = cngp.bwd_plan_info(cngp.Config.from_workload(small_f, flags=flag), small_f.N)
        assert ps["binned"] == 1 and ps["slices_f"] == 0 and ps["dense_levels"] == 0 and ps["slices_c"] >= 1
    few = W.custom(d=3, L=16, N_f=2**6, N_c=2**10, N_p=4, N_min=16, N_max=2048, N=2**18)      # two slices per level: replicated scan
    assert cngp.bwd_plan_info(cngp.Config.from_workload(few), few.N)["binned"] == 0
    assert cngp.bwd_plan_info(cngp.Config.from_workload(W.custom(d=3, L=16, N_f=2**13, N_c=2**10, N_p=4, N_min=16, N_max=2048, N=2**18)), 2**18)["slices_f"] > 0
    big = W.custom(d=3, L=16, N_f=2**24, N_c=2**24, N_p=2, N_min=16, N_max=2048, N=2**18)
    assert cngp.bwd_plan_info(cngp.Config.from_workload(big), big.N)["sliced"] == 0     # too many slices


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N_min,N_max,N,merged", [
    (2, 16, 2**16, 2**12, 8, 16, 8192, 2**20, 11),             # 8 + 2 slices, seven of sixteen levels that a scan pre-reduces
    (3, 8, 2**16, 2**11, 8, 40, 2048, 745393, 3),              # 8 + 1, none of eight
    (2, 12, 2**16, 2**6, 4, 16, 75, 1411859, 0),               # a scan pre-reduces every level: 174 us, binned 619
    (2, 6, 2**17, 2**6, 4, 16, 65, 394677, 0),                 # the same: 40 us, binned 211
    (3, 14, 2**14, 2**15, 2, 64, 5041, 637972, 0),             # 2 + 4 slices: 775 us, binned 1199
    (2, 8, 2**15, 2**14, 4, 16, 273, 1891700, 0),              # two levels to scan of eight: 422 us, binned 593
    (3, 9, 2**15, 2**14, 2, 64, 1027, 446890, 0),              # 4 + 2: 430 us, binned 562
    (3, 6, 2**15, 2**14, 4, 64, 1024, 548667, 0),              # 4 + 4, two of six levels mergeable: 388 us, binned 496
    (3, 10, 2**13, 2**16, 2, 32, 1024, 1030647, 0),            # 1 + 8: 1088 us, binned 1324
])
def test_tables_of_few_slices_are_binned_only_where_a_scan_has_enough_to_do(d, L, N_f, N_c, N_p, N_min, N_max, N, merged):
    p = cngp.bwd_plan_info(cngp.Config.from_workload(W.custom(cfg=7, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N,
                                                              feat_dtype="f16", io_dtype="f16"), flags=cngp.ZERO_GRADS), N)
    assert p["merged_levels"] == merged and 8 <= p["slices_f"] + p["slices_c"] + 2 < 24


@pytest.mark.parametrize("d,L,N_f,N_c,N_p,N_min,N_max,N,merged", [
    (2, 5, 2**19, 2**15, 4, 64, 256, 347924, 0),               # five levels: 157 us, merged 207
    (3, 7, 2**18, 2**12, 16, 16, 512, 150001, 0),              # seven
    (3, 8, 2**18, 2**12, 16, 16, 512, 150001, 4),
    (3, 12, 2**18, 2**11, 4, 64, 1024, 165000, 0),             # one level of twelve: 345 us, merged 381
    (3, 4, 2**19, 1, 1, 8, 60, 150001, 0), (3, 7, 2**18, 1, 1, 8, 256, 165000, 4),      # plain hashing: four levels are enough
    (2, 5, 2**19, 2**15, 4, 64, 256, 3 * 2**17, 4),            # 3 * 2^19 references a level: any that can be
    (3, 12, 2**18, 2**11, 4, 64, 1024, 3 * 2**16, 2),
])
def test_shorter_batches_are_merged_where_enough_levels_share_the_launches(d, L, N_f, N_c, N_p, N_min, N_max, N, merged):
    p = cngp.bwd_plan_info(cngp.Config.from_workload(W.custom(cfg=7, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N,
                                                              feat_dtype="f16", io_dtype="f16"), flags=cngp.ZERO_GRADS), N)
    assert p["binned"] == 1 and p["merged_levels"] == merged


def test_merged_levels_are_reported_as_what_they_are():
    """Levels are either merged or pre-reduced on their grids: never both, and each under its own name."""
    plan = lambda flags=0, **kw: cngp.bwd_plan_info(cngp.Config.from_workload(W.custom(**kw), flags=cngp.ZERO_GRADS | flags), kw["N"])
    head = dict(d=3, L=16, N_f=2**16, N_c=2**14, N_p=16, N=2**18)
    p = plan(N_min=64, N_max=180, **head)                       # levels of 64 .. 90 cells: from 2.4 references per vertex on
    assert p["merged_levels"] == 6 and p["dense_levels"] == 0 and p["chunks_grid"] == p["grid_slices"] == 0
    assert p["merge_chunks"] * p["merge_chunk_points"] >= 2**18 > (p["merge_chunks"] - 1) * p["merge_chunk_points"]
    assert p["merge_tiles"] == 64 and p["merged_drain_wgs_feat"] >= 1 and p["merged_drain_wgs_logit"] >= 1
    fused = plan(cngp.BWD_BINNED, d=3, L=16, N_f=2**8, N_c=2**16, N_p=8, N_min=40, N_max=2048, N=200003)
    assert fused["merged_levels"] == 3 and fused["slices_f"] == 0 and fused["dense_levels"] == 0
    for other in (plan(cngp.BWD_NO_PREREDUCE, N_min=16, N_max=2048, **head), plan(cngp.BWD_BINNED, N_min=16, N_max=2048, **{**head, "N": 2**17}),
                  plan(cngp.BWD_SLICED, N_min=16, N_max=2048, **head), plan(N_min=16, N_max=2048, **{**head, "N": 2**22})):
        assert [other[k] for k in other if k.startswith("merge")] == [0] * 6
    with pytest.raises(cngp.CngpError):
        cngp.bwd_plan_info(base_cfg(), -1)


@pytest.mark.parametrize("N_f,N_c,N_p", [(2**20, 2**14, 2), (2**20, 1, 1), (2**16, 2**18, 8), (2**11, 2**18, 4), (2**20, 2**20, 2), (2**21, 1, 1), (2**16, 2**14, 16)])
def test_counts_of_merged_levels_stay_in_lds_with_the_others(N_f, N_c, N_p):
    """One workgroup scans a level's counts, [chunk][slice], in up to 36864 words of LDS, and through memory, one dependent load
    after the other, where some level's do not fit: the merged levels' fit where the references' own 256 rows do, or are no more rows."""
    for N in (2**18 + 2**16, 2**19, 2**19 + 1, 2**20, 3 * 2**19 + 77):
        p = cngp.bwd_plan_info(cngp.Config.from_workload(W.custom(d=3, L=16, N_f=N_f, N_c=N_c, N_p=N_p, N_min=16, N_max=2048, N=N), flags=cngp.ZERO_GRADS | cngp.BWD_BINNED), N)
        big = max(p["slices_f"], p["slices_c"])
        assert p["merged_levels"] > 0 and p["merge_chunks"] <= max(36864 // big, 256), (N, p)


def test_binding_rejects_host_tensors_and_wrong_shapes():
    import torch
    cfg = base_cfg()
    x = torch.zeros((4, 3))
    with pytest.raises(TypeError):
        cngp.encode_fwd(cfg, x, x, x, y=x)


def test_product_does_not_import_the_oracle():
    """The product package and its sources never reference the test oracle."""
    pkg = os.path.join(ROOT, "paper_2312_17241_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".h", ".hip", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "import oracle" not in text and "from oracle" not in text and "cngp_oracle" not in text, f
    for f in os.listdir(os.path.join(ROOT, "oracle")):
        if f.endswith((".py", ".c")):
            assert "paper_2312_17241_amd" not in open(os.path.join(ROOT, "oracle", f)).read(), f


def test_backward_plan_layout_stays_inside_the_workspace():
    """For seeded random configurations and batch sizes, on every backward variant: the regions of the workspace the
    kernels index (cngp_bwd_plan_layout computes them from the kernels' own extents, but for those that hold the merged levels'
    arrays, whose extents the next test checks) are 256-byte aligned, do not
    overlap, and end inside cngp_workspace_bytes; the plan's counts are consistent with each other."""
    rng = np.random.default_rng(2024)
    seen = {"direct": 0, "sliced": 0, "binned": 0, "passes": 0, "fused": 0, "merged": 0, "few": 0, "plain": 0, "partial sums": 0}
    for it in range(700):
        d = int(rng.choice([2, 3]))
        N_p = int(2 ** rng.integers(0, 5))
        N_f = int(2 ** rng.integers(max(2, int(np.log2(N_p))), 21))
        N_c = int(2 ** rng.integers(1, 19))
        L = int(rng.integers(1, 17))
        N_min = int(rng.integers(1, 33))
        N_max = int(N_min * 2 ** rng.integers(0, 9))
        N = int(rng.choice([1, 63, 4097, 70001, 2**18, 2**20 + 5, 2**22]))
        flags = int(rng.choice([0, 0, cngp.BWD_SLICED, cngp.BWD_BINNED, cngp.BWD_BINNED | cngp.BWD_NO_PREREDUCE, cngp.BWD_SLICED | cngp.BWD_NO_PREREDUCE]))
        bound = int(rng.choice([0, 0, 1 << 20, 1 << 26, 1 << 30]))
        if it >= 400:                              # tables of a few slices
            N_f, N_c, L, N_min = int(2 ** rng.integers(13, 18)), int(2 ** rng.integers(8, 16)), int(rng.integers(6, 17)), int(rng.integers(16, 65))
            N_max, N, flags, bound = N_min * 64, int(2 ** rng.uniform(14, 21)), 0, 0
        w = W.custom(cfg=7, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_max, N=N,
                     feat_dtype=str(rng.choice(["f16", "f32"])), io_dtype=str(rng.choice(["f16", "f32"])))
        cfg = cngp.Config.from_workload(w, flags=cngp.ZERO_GRADS | flags, bin_bytes_max=bound)
        total = cngp.workspace_bytes(cfg, N)
        plan = cngp.bwd_plan_info(cfg, N)
        regions = cngp.bwd_plan_layout(cfg, N)
        assert (len(regions) == 0) == (plan["sliced"] == 0), (w, plan)
        spans = sorted((o, o + b) for o, b in regions if b > 0)
        for o, e in spans:
            assert o % 256 == 0 and e <= total, (w, plan, o, e, total)
        for (o0, e0), (o1, e1) in zip(spans, spans[1:]):
            assert e0 <= o1, (w, plan, spans)
        assert plan["passes"] >= 1 and 0 <= plan["dense_levels"] <= L
        if plan["binned"]:
            assert plan["sliced"] == 1 and plan["bin_chunks"] >= 1 and plan["drain_wgs_feat"] >= 1
            assert len(regions) == 12
        else:
            assert plan["merged_levels"] == 0 and len(regions) in (0, 3, 5)          # (5: a scan whose chunks leave partial sums of two tables)
        few = plan["binned"] == 1 and not flags & cngp.BWD_BINNED and 0 < plan["slices_f"] and plan["slices_f"] + plan["slices_c"] < 24
        seen["few"] += few and N_p > 1
        seen["plain"] += few and N_p == 1
        seen["partial sums"] += len(regions) == 5
        seen["binned" if plan["binned"] else "sliced" if plan["sliced"] else "direct"] += 1
        seen["passes"] += plan["passes"] > 1
        seen["fused"] += plan["binned"] == 1 and plan["slices_f"] == 0
        seen["merged"] += plan["merged_levels"] > 0
    assert min(seen.values()) >= 5, seen          # the sweep reaches every variant


def test_arrays_of_the_merged_levels_do_not_overlap():
    """Every array of the merge, with the extent its kernels index (computed here from levels, chunks, slices and N), lies inside
    one of the four regions the plan has for them, apart from all others and from every other region."""
    rng = np.random.default_rng(31)
    merged, seen = 0, {"passes": 0, "fused": 0, "plain": 0, "flat": 0, "planes": 0}
    for it in range(400):
        d, N_p = int(rng.choice([2, 3])), int(2 ** rng.integers(0, 5))
        N_f = int(2 ** rng.integers(max(4, int(np.log2(N_p))), 21))
        N = int(2 ** rng.uniform(21 - d, 26))
        L, N_min, N_c = int(rng.integers(2, 17)), int(rng.integers(8, 200)), int(2 ** rng.integers(1, 19))
        N_max = int(N_min * 2 ** rng.integers(1, 9))
        if it % 20 == 0:                                        # (the largest that are merged: few of the levels, in passes)
            d, N_p, N_f, N, L, N_min, N_c, N_max = 3, 4, 2**6, int(rng.integers(27_000_000, 28_000_000)), 5, 15, 2**14, 15360
        cfg = cngp.Config.from_workload(W.custom(cfg=7, d=d, L=L, F=int(rng.choice([2, 2, 4])), N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min,
                                                 N_max=N_max, N=N, feat_dtype="f16", io_dtype=str(rng.choice(["f16", "f32"]))),
                                        flags=cngp.ZERO_GRADS | int(rng.choice([0, cngp.BWD_BINNED])))
        plan, arrays = cngp.bwd_plan_info(cfg, N), cngp.bwd_merge_layout(cfg, N)
        assert (len(arrays) > 0) == (plan["merged_levels"] > 0)
        if not arrays:
            continue
        merged += 1
        n = N if plan["passes"] == 1 else (-(-N // plan["passes"]) + 63) // 64 * 64
        M, chunks, cap, sf, sc = plan["merged_levels"], plan["merge_chunks"], n << d, plan["slices_f"], plan["slices_c"]
        assert chunks * plan["merge_chunk_points"] >= n and 0 < M < L
        assert [b for _, b in arrays] == [M * cap * 16, n * 4, plan["merge_tiles"] * 4096 * 4, 4096 * 4, M * chunks * sf * 4, M * chunks * sc * 4, M * chunks * 4,
                                          M * (sf + 1) * 4 if sf else 0, M * (sc + 1) * 4 if sc else 0, M * cap * 12 if sf else 0, M * cap * 12 if sc else 0]
        regions = cngp.bwd_plan_layout(cfg, N)
        homes, others = [regions[i] for i in (2, 9, 10, 11)], [regions[i] for i in range(12) if i not in (2, 9, 10, 11)]
        for home, own in zip(homes, (arrays[:4], arrays[4:7], arrays[7:9], arrays[9:])):
            assert all(home[0] <= o and o + b <= home[0] + home[1] for o, b in own if b), (cfg, N, home, own)
        spans = sorted((o, o + b) for o, b in arrays + others if b)
        assert all(e0 <= o1 for (_, e0), (o1, _) in zip(spans, spans[1:])) and spans[-1][1] <= cngp.workspace_bytes(cfg, N), (cfg, N, spans)
        assert all(o % 256 == 0 for o, _ in spans)
        for k, v in (("passes", plan["passes"] > 1), ("fused", sf == 0), ("plain", sc == 0), ("flat", d == 2), ("planes", cfg.F == 4)):
            seen[k] += v
    assert merged >= 100 and min(seen.values()) >= 3, (merged, seen)


def test_sums_of_drain_workgroups_fit_where_the_entries_were():
    """Tables of few slices whose levels are merged: what the workgroups of a bin leave, sums of a whole slice each, lies inside the
    region that the merged entries had, which is as large as the larger of the two."""
    rng = np.random.default_rng(77)
    seen = {"sums": 0, "larger": 0, "plain": 0, "atomics": 0, "wide": 0}
    for it in range(600):
        d, N_p = int(rng.choice([2, 3])), int(2 ** rng.integers(0, 5))
        N_f, N_c = int(2 ** rng.integers(13, 18)), int(2 ** rng.integers(1, 15)) if N_p > 1 else 1
        L, N_min, N = int(rng.integers(2, 17)), int(rng.integers(8, 90)), int(2 ** rng.uniform(20.6 - d, 21.5 - d if it % 2 else 21.5))
        cfg = cngp.Config.from_workload(W.custom(cfg=7, d=d, L=L, N_f=N_f, N_c=N_c, N_p=N_p, N_min=N_min, N_max=N_min * 64, N=N, feat_dtype="f16", io_dtype="f16"),
                                        flags=cngp.ZERO_GRADS)
        p = cngp.bwd_plan_info(cfg, N)
        if p["merged_levels"] == 0 or p["slices_f"] == 0 or p["slices_f"] + p["slices_c"] >= 24:
            continue
        M = p["merged_levels"]
        scan = cngp.bwd_plan_info(dataclasses.replace(cfg, bin_bytes_max=8 << 30), N)          # (a bound: the scan)
        tables, wide = [], False
        for role, slices, entries in [("feat", p["slices_f"], N_f * 2)] + ([("logit", p["slices_c"], N_c * N_p)] if N_p > 1 else []):
            pts, vtx = (scan[f"chunks_{role}_{k}"] for k in ("pts", "vtx"))
            least, wgs, merged = min(pts, vtx) if scan["dense_levels"] else pts, p[f"drain_wgs_{role}"], p[f"merged_drain_wgs_{role}"]
            if wgs > pts or merged > least:
                tables.append((slices, entries // slices, wgs, merged))
                wide = wide or least == 1
            else:                           # no more writers than the scan has chunks: the sums are added with atomics, as the scan's are
                seen["atomics"] += 1
        tables = [(s, n * (8 if wide else 4), w, m) for s, n, w, m in tables]
        seen["wide"] += wide
        sums = sum(s * b * n * levels for s, b, wgs, merged in tables for n, levels in ((wgs, L - M), (merged, M)) if n > 1)
        regions = cngp.bwd_plan_layout(cfg, N)
        entries = (M * (N << d) * 16 + 255) // 256 * 256                          # (the order of the points and the cells behind them)
        assert regions[2][1] >= max(sums, entries) and regions[2][0] + regions[2][1] <= regions[3][0]
        seen["sums"] += sums > 0
        seen["larger"] += sums > entries
        seen["plain"] += N_p == 1 and sums > 0
    assert min(seen.values()) >= 3, seen


def test_small_binned_batches_pre_reduce_where_the_coarse_bins_are_uneven():
    """Below 2^20 references per level the plan weighs pre-reducing the coarse levels against binning them: many levels with
    few vertices (d = 2) pre-reduce, three-dimensional batches of ray samples bin everything; a caller who bounds the bins,
    asks for the binned variant or has more references per level always pre-reduces."""
    dense = lambda N, flags=0, **kw: cngp.bwd_plan_info(base_cfg(flags=cngp.ZERO_GRADS | flags, **kw), N)["dense_levels"]
    flat = dict(d=2, L=12, N_max=512)
    assert dense(20011) == 0 and dense(100003) == 0 and dense(2**17) == 4
    assert dense(2**18 - 1, **flat) == 10 and dense(150000, **flat) == 10 and dense(2**18, **flat) == 10
    assert dense(20011, cngp.BWD_BINNED) == 3 and dense(20011, bin_bytes_max=1 << 30) == 3


def test_a_backward_workspace_holds_a_layout_of_every_shorter_batch():
    """The need of a batch that bins every level may pass that of a larger one, which pre-reduces its coarse levels; the
    pre-reduced layout, which cngp_encode_bwd falls back on, does not."""
    dips = 0
    for d, N_max, kw in ((3, 2048, {}), (2, 512, dict(L=12)), (4, 256, dict(L=12)), (3, 4096, dict(N_f=2**18, N_c=2**16, N_p=8))):
        w = W.custom(**{**dict(cfg=9, d=d, L=16, N_f=2**16, N_c=2**14, N_p=16, N_min=16, N_max=N_max, N=1, feat_dtype="f16", io_dtype="f16"), **kw})
        cfg, least = (cngp.Config.from_workload(w, flags=f) for f in (cngp.ZERO_GRADS, cngp.ZERO_GRADS | cngp.BWD_BINNED))
        line = 2**20 >> d
        for N in (line, line + 1, line + line // 8, 2 * line):
            have = cngp.workspace_bytes(cfg, N)
            for n in (line - 1, line * 7 // 8, line // 2 + 1, line // 4):
                dips += cngp.workspace_bytes(cfg, n) > have
                assert cngp.bwd_plan_info(cfg, n)["binned"] == 1
                assert cngp.workspace_bytes(least, n) <= have, (d, N, n)
    assert dips >= 3                              # (the first of these are real)


def test_forward_plan_is_within_the_chip_and_the_workspace():
    """The level-resident forward variant for seeded random configurations: the resident part of a level's feature
    codebook is a whole number of 16-byte pieces, at most the codebook; index codebook and resident part fit 160 KB of
    LDS; the level-major copy it needs fits cngp_workspace_bytes; the flags that force a variant are honoured."""
    rng = np.random.default_rng(77)
    taken = 0
    for it in range(300):
        N_p = int(2 ** rng.integers(0, 5))
        N_f = int(2 ** rng.integers(max(2, int(np.log2(N_p))), 22))
        feat, io = str(rng.choice(["f16", "f32"])), str(rng.choice(["f16", "f32"]))
        w = W.custom(cfg=8, d=int(rng.choice([2, 3, 4])), L=int(rng.integers(1, 17)), N_f=N_f, N_c=int(2 ** rng.integers(0, 21)),
                     N_p=N_p, N_min=4, N_max=256, N=int(rng.choice([1, 500, 4097, 2**17, 2**22 + 3])), feat_dtype=feat, io_dtype=io)
        cfg = cngp.Config.from_workload(w, flags=int(rng.choice([0, 0, cngp.FWD_LEVEL])))
        plan = cngp.fwd_plan_info(cfg, w.N)
        need = cngp.fwd_workspace_bytes(cfg, w.N)
        entry = 2 * (2 if feat == "f16" else 4)
        if plan["level_resident"]:
            taken += 1
            assert 0 < plan["resident_entries"] <= N_f and (plan["resident_entries"] * entry) % 16 == 0, (w, plan)
            assert plan["lds_bytes"] <= 160 * 1024 and plan["lds_bytes"] >= plan["resident_entries"] * entry + (w.N_c + 1) // 2
            assert plan["parts"] >= 1
            assert need == w.N * w.L * 2 * (2 if io == "f16" else 4) <= cngp.workspace_bytes(cfg, w.N)
        else:
            assert need == 0, (w, plan)
        tile = cngp.Config.from_workload(w, flags=cngp.FWD_TILE)
        assert cngp.fwd_plan_info(tile, w.N)["level_resident"] == 0 and cngp.fwd_workspace_bytes(tile, w.N) == 0
    assert taken >= 100


def test_forward_route_says_which_kernel_a_call_runs():
    """One rule decides for the calls and for the query: a single launch up to 2^20 corner lookups (without room for the
    level-major copy up to 2^22, with fewer than eight levels 2^21), the level-resident variant beyond it when the room is there, tiles otherwise; forced variants
    and the error of one that cannot run; widths other than two inside their part of the workspace."""
    cfg = base_cfg()
    route = lambda N, c=cfg, **kw: cngp.fwd_route(c, N, **kw)["variant"]
    for N in (1, 2048, 8192):
        assert route(N) == route(N, workspace_bytes=0) == "lanes"
    assert cngp.fwd_plan_info(cfg, 8192)["level_resident"] == 1 and cngp.fwd_workspace_bytes(cfg, 8192) > 0    # (encode_mlp_fwd's)
    assert route(8193) == "level" and route(8193, workspace_bytes=cngp.fwd_workspace_bytes(cfg, 8193) - 1) == "lanes"
    assert route(2**15, workspace_bytes=0) == "lanes" and route(2**15 + 1, workspace_bytes=0) == "tile"
    few = base_cfg(L=4)                         # tiles, which take one level after the other, are the faster ones sooner with few levels
    assert route(2**16, few, workspace_bytes=0) == "lanes" and route(2**16 + 1, few, workspace_bytes=0) == "tile"
    assert route(2**18, levels_loaded=0) == "tile" and route(2**18, levels_loaded=3) == "level"
    assert route(2000, base_cfg(flags=cngp.FWD_LEVEL)) == "level" and route(2**20, base_cfg(flags=cngp.FWD_SIMPLE)) == "lanes"
    assert route(2000, base_cfg(flags=cngp.FWD_TILE)) == "tile" and route(200, base_cfg(flags=cngp.FWD_TILE)) == "lanes"
    for c, room, status in ((base_cfg(flags=cngp.FWD_LEVEL), 0, cngp.ERR_WORKSPACE),
                            (base_cfg(flags=cngp.FWD_LEVEL, N_c=2**18), 1 << 30, cngp.ERR_UNSUPPORTED), (base_cfg(F=4), 0, cngp.ERR_WORKSPACE)):
        with pytest.raises(cngp.CngpError) as e:
            cngp.fwd_route(c, 3000, workspace_bytes=room)
        assert e.value.status == status
    assert route(2**17, base_cfg(F=4), workspace_bytes=cngp.workspace_bytes(base_cfg(F=4), 2**17)) == "level"
    assert cngp.fwd_route(base_cfg(N_f=2**18, N_max=256), 2**20)["grids"] >= 3 and cngp.fwd_route(base_cfg(N_f=2**8), 2**20)["grids"] == 0


def test_stream_handle_without_torch_internals(monkeypatch):
    """A torch without the two internal calls still gives the binding its stream, through the public one."""
    class Stream:
        cuda_stream = 77
    monkeypatch.setattr("torch.cuda.current_stream", lambda: Stream)
    assert cngp._stream_getter(object())() == 77
    class Internals:
        _cuda_getDevice = staticmethod(lambda: 3)
        _cuda_getCurrentRawStream = staticmethod(lambda device: 100 + device)
    assert cngp._stream_getter(Internals)() == 103


def test_morton_sort_workspace_is_host_arithmetic():
    """Two key columns, one index column, 128 counters per tile of 8192 points, 128 totals; no device is asked."""
    a = lambda v: (v + 255) // 256 * 256
    f = cngp._lib.cngp_morton_sort_workspace_bytes
    for N in (1, 8192, 8193, 2**24, 2**31 - 1):
        tiles = (N + 8191) // 8192
        assert f(3, N) == f(2, N) == f(4, N) == 3 * a(4 * N) + a(128 * 4 * tiles) + a(128 * 4)
    assert f(3, 0) == 0 and f(3, -5) == 0 and f(3, 2**31) == 0 and f(5, 100) == 0 and f(1, 100) == 0
    assert cngp._lib.cngp_morton_sort(3, None, 0, None, None, None, 0, None) == cngp.OK
    assert cngp._lib.cngp_morton_sort(3, None, 10, None, None, None, 0, None) == cngp.ERR_NULL
    assert cngp._lib.cngp_morton_sort(5, None, 10, None, None, None, 0, None) == cngp.ERR_INVALID


def test_host_code_runs_clean_under_sanitizers():
    """csrc/host_check_main.cpp drives validation, level table, storage sizes, the backward plan and its workspace
    layout through the C ABI for 300 seeded random configurations (valid and invalid) in a program whose host side
    is built with AddressSanitizer and UndefinedBehaviorSanitizer.  No kernel is launched.  The first run compiles
    the program (about two minutes); later runs reuse it until a source changes."""
    import subprocess
    from paper_2312_17241_amd.build import build_host_sanitized
    exe = build_host_sanitized()
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "clean" in res.stdout, res.stdout + res.stderr
