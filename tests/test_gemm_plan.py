"""The choice of tile and reduction split for one bf16 product (host arithmetic, compiled here for the
CPU): which products may be split, and the choices that whole forward passes were timed for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
T128x128, T128x256, T128x320, T256x256, T256x320, T64x64, T64x128 = range(7)
TILE = [(128, 128, 2), (128, 256, 2), (128, 320, 1), (256, 256, 1), (256, 320, 1), (64, 64, 2), (64, 128, 2)]   # rows, columns, workgroups per CU


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "gemm_plan.h"\n'
                   'extern "C" void plan(long M, int N, int K, int glu, int dual, int a_tiled, int can_split, int fix, int* out) {\n'
                   '  const ffsplit::GemmPlan p = ffsplit::gemm_plan(M, N, K, glu, dual, a_tiled, can_split, fix);\n'
                   '  out[0] = p.shape; out[1] = p.split; out[2] = p.fix; }\n'
                   'extern "C" size_t room(long M, int N, int K, int glu, int a_tiled) { return ffsplit::gemm_part_room(M, N, K, glu, a_tiled); }\n'
                   'extern "C" size_t need(long M, int N, int split, int fix) {\n'
                   '  return fix ? ffsplit::gemm_fix_bytes(M, N, split) : ffsplit::gemm_part_bytes(M, N, split); }\n'
                   'extern "C" int limits(int i) { return i ? ffsplit::GEMM_FIX_MAX_SPLIT : ffsplit::FIX_COUNTERS; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2401_04044_amd", "csrc"), str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))
    lib.plan.argtypes = [ctypes.c_long] + [ctypes.c_int] * 7 + [ctypes.POINTER(ctypes.c_int)]
    lib.room.argtypes, lib.room.restype = [ctypes.c_long] + [ctypes.c_int] * 4, ctypes.c_size_t
    lib.need.argtypes, lib.need.restype = [ctypes.c_long] + [ctypes.c_int] * 3, ctypes.c_size_t

    def get(M, N, K, glu=False, dual=False, a_tiled=True, can_split=True):
        return planned(M, N, K, glu, dual, a_tiled, can_split, False)[:2]

    def planned(M, N, K, glu, dual, a_tiled, can_split, fix):
        out = (ctypes.c_int * 3)()
        lib.plan(M, N, K, glu, dual, a_tiled, can_split, fix, out)
        return out[0], out[1], out[2]

    get.with_fix = lambda M, N, K: planned(M, N, K, False, False, True, True, True)
    get.lib = lib
    return get


def test_ranges_added_inside_the_launch_have_counters_and_room(plan):
    """Un-activated products on a tiled operand behind the first, as the forward pass plans them: only 64x64 tiles, at most
    GEMM_FIX_MAX_SPLIT ranges and FIX_COUNTERS tiles, and whatever is split, either way, fits the scratch that a workspace
    of at least as many tokens holds for the product."""
    counters, most = plan.lib.limits(0), plan.lib.limits(1)
    rng = np.random.default_rng(5)
    shapes = [(130, 800, 1728), (423, 32, 1280)] + [(int(2 ** rng.uniform(6, 13.5)), 32 * int(rng.integers(1, 200)), 64 * int(rng.integers(1, 260)))
                                                    for _ in range(20000)]
    seen = 0
    for M, N, K in shapes:
        s, sp, fix = plan.with_fix(M, N, K)
        if fix:
            seen += 1
            assert s == T64x64 and 1 < sp <= most and -(-M // 64) * -(-N // 64) <= counters, (M, N, K)
        if sp > 1:
            assert plan.lib.need(M, N, sp, fix) <= plan.lib.room(M, N, K, False, True) <= plan.lib.room(2 * M, N, K, False, True), (M, N, K)
        s, sp = plan(M, N, K, False, False, True)
        if sp > 1:
            assert plan.lib.need(M, N, sp, 0) <= plan.lib.room(M, N, K, False, True), (M, N, K)
    assert seen > 500


def test_split_products_fill_at_most_one_round_and_only_valid_tiles_are_chosen(plan):
    rng = np.random.default_rng(3)
    for _ in range(3000):
        M, N, K = int(2 ** rng.uniform(0, 17)), 8 * int(rng.integers(1, 4000)), 8 * int(rng.integers(1, 3000))
        glu, a_tiled = bool(rng.integers(0, 2)), bool(rng.integers(0, 2))
        s, sp = plan(M, N, K, glu, False, a_tiled)
        bm, bn, per_cu = TILE[s]
        assert not (glu and s in (T128x320, T256x320, T64x64))
        assert 1 <= sp <= 16
        if sp > 1:
            assert -(-M // bm) * -(-N // bn) * sp <= 256 * per_cu and -(-K // 32) // sp >= 8
        assert plan(M, N, K, glu, False, a_tiled, can_split=False)[1] == 1
        s, sp = plan(M, N, K, True, True, True, can_split=False)
        assert s in (T128x128, T256x256) and sp == 1


# Products of layers timed as a whole on the tiles and numbers of ranges: the tile must be that of the
# shortest pass (or of one within 3 %), the ranges near its number (M, N, K, gated, row-major left
# operand, allowed).
TIMED = [
    (2816, 1664, 4096, True, True, {(T128x256, 1)}),                    # 146 us; in three ranges 166
    (4096, 1152, 4096, True, True, {(T128x256, 1), (T128x128, 1)}),     # 70.1; in three ranges 80.6
    (300, 1152, 4096, True, True, {(T64x128, sp) for sp in (4, 5, 6)}),   # 22.8; 128x128 in nine ranges 25.4
    (300, 512, 8000, False, False, {(T64x64, sp) for sp in range(3, 8)}),   # 42.9; 64x128 in twelve 46.3
    (220, 512, 8000, False, False, {(T64x64, sp) for sp in range(3, 8)}),   # 38.2; 128x128 in sixteen 42.2
    (1500, 3200, 4096, True, True, {(T128x256, 1), (T256x256, 3), (T256x256, 2)}),   # 207; 128x256 in three 216
    (700, 768, 2048, False, True, {(T64x64, 1)}),                       # 53.4
]


@pytest.mark.parametrize("M,N,K,glu,rows,allowed", TIMED)
def test_choice_is_among_the_best_of_the_timed_ones(plan, M, N, K, glu, rows, allowed):
    assert plan(M, N, K, glu, False, not rows) in allowed
    if not rows and not glu:   # (as it is planned behind the first product)
        assert plan.with_fix(M, N, K)[:2] in allowed


def test_device_cases_reach_every_form(plan):
    """The parity cases of test_gpu_gemm_shapes.py run every tile on tiled and on row-major left operands,
    whole and split, gated and not, as far as products of their size choose it."""
    from test_gpu_gemm_shapes import CASES
    seen = set()
    for T, d, f, k, r, act in CASES:
        glu, up = act == "swiglu", lambda v: -(-v // 64) * 64
        n_up, kp, rp, mp = 2 if glu else 1, up(k), up(r), up(f - k)
        for N, K, gated, dual, a_tiled in ((n_up * (kp + rp), d, glu, False, False), (n_up * mp, rp, glu, glu, True),
                                           (rp, mp, False, False, True), (d, kp + rp, False, False, True)):
            s, sp = plan(T, N, K, gated, dual, a_tiled, not dual)
            seen.add((s, "dual" if dual else "gated" if gated else "", "tiled" if a_tiled else "rows", sp > 1))
    want = {(s, "", "tiled", False) for s in (T128x128, T128x256, T128x320, T256x320, T64x64, T64x128)}
    want |= {(s, "", "rows", False) for s in (T128x128, T128x256, T128x320, T256x320, T64x64, T64x128)}
    want |= {(s, "gated", "rows", False) for s in (T128x128, T128x256, T256x256, T64x128)}
    want |= {(T128x128, "dual", "tiled", False), (T256x256, "dual", "tiled", False)}
    want |= {(s, "", a, True) for s in (T128x128, T64x64, T64x128) for a in ("tiled", "rows")}
    want |= {(s, "gated", "rows", True) for s in (T128x128, T64x128)}
    assert want <= seen, want - seen
