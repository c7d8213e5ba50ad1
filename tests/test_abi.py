"""CPU checks of the C-ABI boundary: the library loads, exports every declared symbol, and the
host-side argument validation works without a GPU (no kernels are launched here)."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "spec.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(spec_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def amd():
    import paper_2408_11850_amd as amd
    if not os.path.exists(amd.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    amd.load_library()
    return amd


def test_library_exports_every_declared_symbol(amd):
    names = _declared()
    assert len(names) >= 20 and {"spec_init", "spec_prefill", "spec_draft_step", "spec_verify", "spec_accept",
                                 "spec_rollback_kv"} <= set(names)
    lib = C.CDLL(amd.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(amd.SIGNATURES), set(names) ^ set(amd.SIGNATURES)


def test_argument_validation_without_a_gpu(amd):
    lib = amd.load_library()
    assert lib.spec_packed_bytes(32, 40) == 2 * 2 * 1024            # 2 panels x ceil(40/32) steps x 1 KiB
    assert lib.spec_gemm_workspace_bytes(33, 64, 64) == 0           # M too large
    assert lib.spec_gemm_workspace_bytes(4, 64, 64) >= 4 * 64 * 4
    assert lib.spec_init(None, None, None, None, None, None) == amd.SPEC_E_INVAL
    assert b"null" in lib.spec_last_error()
    assert lib.spec_verify(None, None, 1, None) == amd.SPEC_E_INVAL
    assert lib.spec_rollback_kv(None, 0, 0) == amd.SPEC_E_INVAL
    assert lib.spec_pack_weight(None, None, 16, 8, 0, 1, None) == amd.SPEC_E_INVAL
    # the prompt-sized projection validates before it launches: null operands, bad epilogue, K not a multiple of 32,
    # N not a multiple of 16 (32 for the gate/up epilogue), missing output
    p = C.c_void_p(256)
    assert lib.spec_dense_gemm(p, None, None, p, 4, 64, 64, 0, None) == amd.SPEC_E_INVAL
    assert lib.spec_dense_gemm(p, None, p, p, 4, 64, 64, 3, None) == amd.SPEC_E_INVAL
    assert lib.spec_dense_gemm(p, None, p, p, 4, 64, 48, 0, None) == amd.SPEC_E_INVAL
    assert lib.spec_dense_gemm(p, None, p, p, 4, 40, 64, 0, None) == amd.SPEC_E_INVAL
    assert lib.spec_dense_gemm(None, p, p, p, 4, 48, 64, 2, None) == amd.SPEC_E_INVAL
    assert lib.spec_dense_gemm(None, None, p, p, 4, 64, 64, 1, None) == amd.SPEC_E_INVAL
    assert lib.spec_set_option(None, amd.SPEC_OPT_PREFILL, 1) == amd.SPEC_E_INVAL
    cfg = amd.Config(4, 128, 64, 1.0, 1.0, None, None)
    bad = amd.ModelDesc(2, 256, 4, 3, 64, 688, 1024, 10000.0, 1e-5)     # heads not a multiple of kv heads
    w = amd.Weights()
    out = C.c_void_p()
    assert lib.spec_init(C.byref(cfg), C.byref(bad), C.byref(w), C.byref(bad), C.byref(w), C.byref(out)) == amd.SPEC_E_INVAL
    assert not out.value


def test_binding_refuses_to_run_without_the_library(amd, monkeypatch):
    import paper_2408_11850_amd as pkg
    monkeypatch.setattr(pkg, "_lib", None)
    monkeypatch.setattr(pkg, "LIB_PATH", "/nonexistent/libspec.so")
    with pytest.raises(RuntimeError):
        pkg.load_library()


def test_projection_plan_covers_every_shape_evenly(amd):
    """Host logic of the decode-time projection: the K steps of 32 are dealt to S slices of 8 waves with at most 8
    steps per wave (what a wave's registers hold), every panel belongs to exactly one group, the launch fits the
    workgroup slots, the K split does not depend on the launch mode (so both modes add the same numbers in the same
    order), and the busiest wave has at most ~12 % more than an even share on the benchmark's matrices."""
    lib = amd.load_library()
    out = (C.c_int * 6)()
    shapes = [(10240, 8192), (8192, 8192), (57344, 8192), (8192, 28672), (32000, 8192),          # 70B
              (12288, 4096), (4096, 4096), (22016, 4096), (4096, 11008), (32000, 4096),          # 7B
              (21504, 7168), (7168, 7168), (38400, 7168), (7168, 19200), (32256, 7168),          # 33B
              (2560, 2048), (2048, 2048), (11264, 2048), (2048, 5632), (6144, 2048), (11008, 2048), (2048, 5504),
              (768, 256), (1376, 256), (256, 688), (1024, 256), (16, 8), (48, 40), (2064, 1032)]
    for N, K in shapes:
        plans = {}
        for M in (1, 7, 16, 17, 32):
            for wgs in (1, 2):
                assert lib.spec_gemm_plan_query(M, N, K, wgs, out) == 0, (M, N, K)
                S, spw, Gs, NT, steps, MT = list(out)
                assert NT == N // 16 and steps == (K + 31) // 32 and MT == (2 if M > 16 else 1)
                assert 1 <= spw <= 8 and S * 8 * spw >= steps > (S * 8) * (spw - 1) - 8 * S
                slots = 256 * (1 if MT == 2 else wgs)
                assert 1 <= Gs <= NT and Gs * S <= max(slots, S)
                # even deal of the K steps: wave-slice i of S*8 takes floor((i+1)*steps/(8S)) - floor(i*steps/(8S))
                per = [(i + 1) * steps // (8 * S) - i * steps // (8 * S) for i in range(8 * S)]
                assert sum(per) == steps and max(per) <= spw <= 8
                # panels: group g takes [g*NT//Gs, (g+1)*NT//Gs): a partition with sizes differing by at most one
                sizes = [(g + 1) * NT // Gs - g * NT // Gs for g in range(Gs)]
                assert sum(sizes) == NT and max(sizes) - min(sizes) <= 1
                plans[(M, wgs)] = S
        assert len(set(plans.values())) == 1, (N, K, plans)          # one K split per shape
        if N * K >= 4096 * 4096:                                      # the benchmark's matrices: little imbalance
            lib.spec_gemm_plan_query(1, N, K, 2, out)
            S, spw, Gs, NT, steps, MT = list(out)
            busiest = -(-NT // Gs) * spw
            even = NT * steps / (8 * 512)
            assert busiest <= 1.15 * even, (N, K, S, Gs, busiest, even)
    assert lib.spec_gemm_plan_query(1, 40, 64, 2, out) == amd.SPEC_E_INVAL
    assert lib.spec_gemm_plan_query(1, 64, 64, 3, out) == amd.SPEC_E_INVAL
    assert lib.spec_gemm_plan_query(1, 64, 64, 2, None) == amd.SPEC_E_INVAL


class _ProjPlan(C.Structure):
    _fields_ = [(n, C.c_int) for n in ("M", "N", "K", "steps", "NT", "mode", "units", "RP", "G", "epi")]


class _ProjArgs(C.Structure):       # as csrc/spec_internal.h; all null here
    _fields_ = [("x", C.c_void_p), ("w", C.c_void_p), ("stamp", C.c_void_p), ("ssq", C.c_void_p), ("ssq_w", C.c_int),
                ("eps", C.c_float), ("y", C.c_void_p), ("h", C.c_void_p), ("gain", C.c_void_p), ("xo", C.c_void_p),
                ("ssq_out", C.c_void_p)] + [(n, C.c_int) for n in ("M", "N", "K", "steps", "per", "rem")]


def test_whole_k_projection_plans_have_a_kernel_and_others_are_refused(amd):
    """Host logic of proj.hip: every plan is one that a kernel is built for, its layout, panels at a time and units (and so
    the order of the sums) do not depend on the launch mode, and a plan made for another epilogue or token count is an
    error instead of a launch that does something else or nothing (only refused plans are launched here)."""
    lib = C.CDLL(amd.LIB_PATH)
    make, ok, launch = lib._Z9proj_planiiiii, lib._Z12proj_plan_okRK8ProjPlan, lib._Z11launch_projRK8ProjPlan8ProjArgsP12ihipStream_ti
    make.restype, make.argtypes = _ProjPlan, [C.c_int] * 5
    ok.restype, ok.argtypes = C.c_bool, [C.POINTER(_ProjPlan)]
    launch.restype, launch.argtypes = C.c_int, [C.POINTER(_ProjPlan), _ProjArgs, C.c_void_p, C.c_int]
    STORE, RESID, SWIGLU = 0, 1, 2
    invalid = 1          # hipErrorInvalidValue
    seen = set()
    for N in (32, 2048, 2080, 4096, 4128, 8192, 8224, 12288, 16384, 16416, 24576, 24608, 38400, 49152, 49184, 57344):
        for K in (8, 40, 2048, 2056, 8192):
            for M in (1, 7, 8, 9, 16, 17, 24, 32):
                for epi in (STORE, RESID, SWIGLU):
                    two, one = make(M, N, K, epi, 2), make(M, N, K, epi, 1)
                    for p in (two, one):
                        assert ok(C.byref(p)) and 1 <= p.G <= min(p.units, 512), (M, N, K, epi)
                    order = lambda p: (p.mode, p.RP, p.units, p.steps, p.NT, p.epi)  # noqa: E731
                    assert order(two) == order(one)
                    seen.add((p.mode, p.RP, epi, M > 16))
                    if epi != STORE:       # a stand-alone launch only stores
                        assert launch(C.byref(two), _ProjArgs(), None, 2) == invalid
                    for other in (STORE, RESID, SWIGLU):
                        q = make(M, N, K, epi, 2)
                        q.epi = other
                        if (other == SWIGLU) != (epi == SWIGLU):      # units are panels of one kind only
                            assert not ok(C.byref(q))
                        if not ok(C.byref(q)):
                            assert launch(C.byref(q), _ProjArgs(), None, 0) == invalid
                    if two.mode:                                       # two K steps per load of x: at most 8 tokens
                        q = make(M, N, K, epi, 2)
                        q.M = 9
                        assert launch(C.byref(q), _ProjArgs(), None, 1) == invalid
    assert {s[:2] for s in seen} == {(0, 1), (0, 2), (0, 4), (1, 1), (2, 1), (2, 2)}
    wide = make(32, 57344, 8192, STORE, 2)
    assert wide.RP == 4
    wide.epi = RESID                       # four panels and two row tiles: no residual kernel
    assert launch(C.byref(wide), _ProjArgs(), None, 0) == invalid


def test_forward_tests_reach_every_projection_layout(amd):
    """Layout, panels at a time and ring that proj_plan takes over 1 to 8 tokens for residual adds and SiLU * mul, against
    those of the GPU tests' models; and that the models of the launch mode test share their work out in two ways."""
    from tests.test_gpu_proj import FORWARDS, MODES
    lib = C.CDLL(amd.LIB_PATH)
    make, whole = lib._Z9proj_planiiiii, lib._Z12proj_whole_kiii
    make.restype, make.argtypes = _ProjPlan, [C.c_int] * 5
    whole.restype, whole.argtypes = C.c_bool, [C.c_int] * 3

    def layout(n, k, epi):
        p = make(8, n, k, epi, 2)
        return epi, p.mode, p.RP, p.steps <= 64 and p.RP != 4 and (p.mode, p.RP) != (0, 1)   # the short ring is in use

    grid = range(16, 16400, 208)
    want = {layout(n, k, 1) for n in grid for k in (64, 512, 800, 1024, 1536, 2048, 2304, 2816, 3072, 4096, 6144, 8192, 12288, 28672)
            if whole(8, n, k)}
    want |= {layout(n, k, 2) for n in range(32, 57376, 736) for k in (64, 512, 1024, 1536, 2048, 2304, 3072, 4096, 6144, 8192, 16384)}
    seen = set()
    for d, heads, _, ffn in FORWARDS:
        seen |= {layout(d, k, 1) for k in (heads * 128, ffn) if whole(8, d, k)} | {layout(2 * ffn, d, 2)}
    assert want == seen, (want - seen, seen - want)
    two_ways = set()
    for d, heads, kv, ffn, vocab in MODES:
        for s in (((heads + 2 * kv) * 128, d, 0), (d, heads * 128, 1), (d, ffn, 1), (2 * ffn, d, 2), (vocab, d, 0)):
            two_ways |= {(m, s) for m in (1, 8, 9, 16) if make(m, *s, 1).G != make(m, *s, 2).G}
    for m in (1, 8):
        assert {s[2] for n, s in two_ways if n == m} == {0, 1, 2}
    for m in (9, 16):
        assert {s[2] for n, s in two_ways if n == m} == {0, 2}      # a residual add only at d_model 16384


def test_sums_of_up_to_eight_tokens_run_in_one_order(amd):
    """Layout, panels at a time and units of a projection over 1 to 8 tokens, and whether it runs in K slices, do not depend
    on how many there are: neither do the rows of a forward."""
    import synth
    lib = C.CDLL(amd.LIB_PATH)
    make, whole = lib._Z9proj_planiiiii, lib._Z12proj_whole_kiii
    make.restype, make.argtypes = _ProjPlan, [C.c_int] * 5
    whole.restype, whole.argtypes = C.c_bool, [C.c_int] * 3
    shapes = set()
    for pair in ("tiny", "small", "7b_1b", "33b_1b", "70b_7b"):
        for s in (synth.config(pair).target, synth.config(pair).draft):
            hd = s.n_heads * s.head_dim
            shapes |= {((s.n_heads + 2 * s.n_kv_heads) * s.head_dim, s.d_model, 0), (s.vocab, s.d_model, 0),
                       (s.d_model, hd, 1), (s.d_model, s.d_ffn, 1), (2 * s.d_ffn, s.d_model, 2)}
    widths = (32, 2048, 2080, 4096, 4128, 6144, 8192, 8224, 12288, 16384, 16416, 24576, 24608, 38400, 57344)
    depths = (8, 200, 768, 1024, 1536, 1792, 2048, 3064, 3072, 5120, 6136, 6144, 8192, 8200, 12280, 12288, 28672)
    shapes |= {(n, k, e) for n in widths for k in depths for e in (0, 1, 2) if e != 1 or n <= 16384}
    for n, k, e in sorted(shapes):
        order = {(p.mode, p.RP, p.units) for p in (make(m, n, k, e, 2) for m in range(1, 9))}
        assert len(order) == 1, (n, k, e, order)
        assert len({whole(m, n, k) for m in range(1, 9)}) == 1, (n, k)
