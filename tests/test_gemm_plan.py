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
                   'extern "C" void plan(long M, int N, int K, int glu, int dual, int a_tiled, int can_split, int* out) {\n'
                   '  const ffsplit::GemmPlan p = ffsplit::gemm_plan(M, N, K, glu, dual, a_tiled, can_split);\n'
                   '  out[0] = p.shape; out[1] = p.split; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2401_04044_amd", "csrc"), str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))
    lib.plan.argtypes = [ctypes.c_long] + [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_int)]

    def get(M, N, K, glu=False, dual=False, a_tiled=True, can_split=True):
        out = (ctypes.c_int * 2)()
        lib.plan(M, N, K, glu, dual, a_tiled, can_split, out)
        return out[0], out[1]

    return get


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
