"""The coefficients of the factorisation's polar iteration (host arithmetic, compiled here for the
CPU): as a map of singular values the steps must take everything the sketch may start with to 1,
and must not amplify a rounding error, wherever in the range it occurs."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RANKS = sorted(set(range(1, 129)) | set(range(136, 2049, 8)) | {300, 2500, 3001, 4096, 5120, 8191, 8192})


@pytest.fixture(scope="module")
def steps_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("polar")
    src, so = d / "polar.cpp", d / "polar.so"
    src.write_text('#include "polar_steps.h"\n'
                   'extern "C" int steps(int r, float* c) { return ffsplit::polar_steps(r, (float(*)[3])c); }\n'
                   'extern "C" int max_steps() { return ffsplit::POLAR_MAX_STEPS; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2401_04044_amd", "csrc"), str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))

    def get(r):
        c = np.zeros((lib.max_steps(), 3), np.float32)
        return c[:lib.steps(r, c.ctypes.data_as(ctypes.c_void_p))].astype(np.float64)

    return get


def quintic(p, x):
    return x * (p[0] + x * x * (p[1] + x * x * p[2]))


def test_whole_range_converges_with_an_overshoot_at_every_step(steps_of):
    """The range [1 / (1024 r), 1] of the Frobenius norm, widened by 1e-6 of itself (some ten fp32
    roundings) on both sides before every step, ends within 1e-5 of 1; what lies below it stays
    between 0 and 1."""
    wide = 1e-6
    for r in RANKS:
        lo, hi, below = 1.0 / (1024 * r), 1.0, 1.0 / (1024 * r)
        for p in steps_of(r):
            y = quintic(p, np.linspace(lo * (1 - wide), hi * (1 + wide), 3001))
            z = quintic(p, np.linspace(0.0, below * (1 + wide), 301))
            assert y.min() > 0 and z.min() >= 0, r
            lo, hi, below = y.min(), y.max(), z.max()
            assert hi < 2 and below < 2, (r, lo, hi)
        assert 1 - 1e-5 < lo and hi < 1 + 1e-5 and below < 1 + 1e-5, (r, lo, hi, below)


@pytest.mark.parametrize("r", [128, 256, 512])
def test_fp32_iteration_on_dominated_and_deficient_sketches(steps_of, r):
    """The iteration itself in fp32: one singular value carries everything (norm 1, nothing else
    appears), or a chosen share of the Frobenius norm beside r - 1 equal ones (rows
    orthonormal to 1e-5: ten fp32 roundings; at most 9e-7 observed)."""
    rng = np.random.default_rng(r)
    coef = steps_of(r).astype(np.float32)

    def run(X):
        X = X.astype(np.float32)
        for a, b, c in coef:
            S = X @ X.T
            X = (c * (S @ S) + b * S + a * np.eye(r, dtype=np.float32)) @ X
        return X

    X = np.outer(rng.standard_normal(r), rng.standard_normal(2 * r))
    X = run(X / np.linalg.norm(X))
    assert np.isfinite(X).all() and abs(np.linalg.norm(X, 2) - 1) < 1e-5
    U = np.linalg.qr(rng.standard_normal((r, r)))[0]
    V = np.linalg.qr(rng.standard_normal((2 * r, r)))[0].T
    for top in (0.9999, 0.433, 0.43303, 0.43306, 0.4331, 0.12242):
        s = np.full(r, np.sqrt((1 - top * top) / (r - 1)))
        s[0] = top
        X = run((U * s) @ V)
        assert np.abs(X @ X.T - np.eye(r)).max() < 1e-5, top
