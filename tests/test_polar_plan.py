"""The polar iteration with its steps chosen from ||S - I||_F^2 (polar_decide, compiled here for the CPU): as a
map of singular values, over spectra from flat to decaying, deficient and dominated, and in fp32 on matrices."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text('#include "polar_steps.h"\nusing namespace ffsplit;\n'
                   'extern "C" int max_steps(int r) { return polar_plan(r, 2 * r).max_steps; }\n'
                   'extern "C" int is_fixed(int r, int d) { return polar_plan(r, d).fixed; }\n'
                   'extern "C" int fixed_steps(int r) { float c[POLAR_MAX_STEPS][3]; return polar_steps(r, c); }\n'
                   'extern "C" void decide(int r, int step, int* s, float fig, float* c) {\n'
                   '  float k[3]; PolarState t = {s[0], s[1], s[2], s[3], s[4]};\n'
                   '  t = polar_decide(polar_plan(r, 2 * r), step, r, t, fig, k);\n'
                   '  s[0] = t.mode; s[1] = t.grown; s[2] = t.parity; s[3] = t.act; s[4] = t.last;\n'
                   '  for (int i = 0; i < 3; ++i) c[i] = k[i]; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2401_04044_amd", "csrc"), str(src), "-o", str(so)])
    return ctypes.CDLL(str(so))


def iterate(lib, r, apply, first, later):
    """Runs the steps; returns their number."""
    s, c, n = np.zeros(5, np.int32), np.zeros(3, np.float32), 0
    pi, pf = (lambda a: a.ctypes.data_as(ctypes.c_void_p)), ctypes.c_float
    for step in range(lib.max_steps(r)):
        lib.decide(r, step, pi(s), pf(first() if step == 0 else later()), pi(c))
        if not s[3]:
            assert n > 0
            break
        assert s[2] == (step + 1) & 1
        apply(c.astype(np.float64))
        n += 1
    return n


def spectra(r):
    i = np.arange(1, r + 1)
    yield "flat", np.ones(r)
    yield "decay 1/2", i ** -0.5
    yield "decay 1", 1.0 / i
    yield "decay 2", i ** -2.0
    yield "linear", np.linspace(1e-3, 1, r)
    yield "least", np.r_[np.ones(r - 1), 1 / (1000 * np.sqrt(r))]
    yield "half", np.r_[np.ones(r - r // 2), np.full(r // 2, 1e-3)]
    yield "dominated", np.r_[1, np.full(r - 1, 1e-2)]
    yield "dominated far", np.r_[1, np.full(r - 1, 1 / (1020.0 * r))]
    yield "geometric", np.logspace(0, -np.log10(500 * r), r)
    yield "three sizes", np.r_[1, np.full((r - 1) // 2, 1e-2), np.full(r - 1 - (r - 1) // 2, 2e-4)]


@pytest.mark.parametrize("r", [2, 3, 8, 33, 64, 138, 400, 512, 1024, 1380, 5120])
@pytest.mark.parametrize("slack", [1.0, 2.2, 8.0])
def test_every_spectrum_above_the_least_value_converges(lib, r, slack):
    """Whatever lies above 1 / (1024 r) of the norm ends within 1e-6 of 1 (the coefficients are fp32), in no more
    steps than the plan's, with a bound of the largest value up to `slack` too large."""
    for name, x in spectra(r):
        x = x / np.linalg.norm(x)
        state = {"x": np.maximum(x, 1.0 / (1024 * r))}

        def apply(c):
            v = state["x"]
            state["x"] = v * (c[0] + v * v * (c[1] + v * v * c[2])) * (1 + 1e-6 * np.cos(np.arange(r)))
            assert (state["x"] > 0).all() and state["x"].max() < 1.2, (name, state["x"].max())

        n = iterate(lib, r, apply, lambda: min(1.0, slack * state["x"].max()), lambda: float(((1 - state["x"] ** 2) ** 2).sum()))
        assert np.abs(state["x"] - 1).max() < 3e-6, (name, n, np.abs(state["x"] - 1).max())
        assert n <= {"flat": 5, "decay 1/2": 9}.get(name, 99), (name, n)


@pytest.mark.parametrize("kind", ["zero", "rank one", "deficient", "nan"])
def test_what_never_converges_stays_bounded(lib, kind):
    r = 64
    x = {"zero": np.zeros(r), "rank one": np.r_[1.0, np.zeros(r - 1)], "deficient": np.r_[np.ones(r // 2), np.full(r // 2, 1e-9)],
         "nan": np.r_[np.nan, np.ones(r - 1)]}[kind]
    norm = np.linalg.norm(x)
    state = {"x": x / norm if norm > 0 else x}

    def apply(c):
        v = state["x"]
        assert np.isfinite(c).all()
        state["x"] = v * (c[0] + v * v * (c[1] + v * v * c[2]))

    iterate(lib, r, apply, lambda: float(np.max(state["x"])), lambda: float(((1 - state["x"] ** 2) ** 2).sum()))
    if kind != "nan":
        assert np.isfinite(state["x"]).all() and state["x"].min() >= 0 and state["x"].max() < 1.001
        assert np.abs(state["x"][x > 0.5 * x.max()] - 1).max(initial=0) < 1e-5


def test_fp32_iteration_takes_few_steps_and_ends_orthonormal(lib):
    """In fp32 on a Gaussian sketch (four or five steps, where the steps for any spectrum are 12) and on one whose
    columns decay like 1/i: rows orthonormal to 1e-5 (ten fp32 roundings; 1e-6 observed)."""
    rng = np.random.default_rng(1)
    r, d = 128, 600
    for decay, most in ((0.0, 5), (1.0, 9)):
        Z = rng.standard_normal((d, 3 * d)) * (np.arange(1, d + 1) ** -decay)[:, None]
        Y = (np.sign(rng.standard_normal((r, 3 * d))) @ Z.T).astype(np.float32)
        st = {"X": Y / np.float32(np.linalg.norm(Y))}
        st["S"] = st["X"] @ st["X"].T

        def apply(c):
            a, b, q = c.astype(np.float32)
            S = st["S"]
            st["X"] = (q * (S @ S) + b * S + a * np.eye(r, dtype=np.float32)) @ st["X"]
            st["S"] = st["X"] @ st["X"].T

        n = iterate(lib, r, apply, lambda: float(np.sqrt(min(np.abs(st["S"]).sum(1).max(), np.linalg.norm(st["S"])))),
                    lambda: float(((st["S"] - np.eye(r)) ** 2).sum()))
        assert n <= most, n
        assert np.abs(st["S"] - np.eye(r)).max() < 1e-5


@pytest.mark.parametrize("r", [8, 33, 64, 100, 128, 200, 300, 400, 512, 800, 1024, 1380, 2000, 5120])
def test_no_spectrum_takes_many_more_steps_than_the_fixed_ones(lib, r):
    """At most two more than the steps that take any spectrum to 1: a few values that are left far behind when the bulk
    is past 0.5 must not be climbed after one by one (16 steps instead of 13 at rank 512)."""
    least = 1.0 / (1024 * r)
    assert lib.max_steps(r) <= lib.fixed_steps(r) + 2
    rng = np.random.default_rng(r)
    for share in (0.02, 0.1, 0.2, 0.34):
        for low in (least, 3 * least, 30 * least, 1e-2):
            n = max(1, int(share * r))
            x = np.r_[rng.uniform(0.5, 1.0, r - n), np.full(n, low * np.sqrt(r))]
            state = {"x": np.maximum(x / np.linalg.norm(x), least)}

            def apply(c):
                v = state["x"]
                state["x"] = v * (c[0] + v * v * (c[1] + v * v * c[2])) * (1 + 1e-6 * np.cos(np.arange(r)))
                assert (state["x"] > 0).all() and state["x"].max() < 1.2

            iterate(lib, r, apply, lambda: min(1.0, 1.5 * state["x"].max()), lambda: float(((1 - state["x"] ** 2) ** 2).sum()))
            assert np.abs(state["x"] - 1).max() < 3e-6, (share, low, np.abs(state["x"] - 1).max())


@pytest.mark.parametrize("share,decay", [(0.5, 0.0), (0.75, 0.0), (0.9, 0.0), (0.9, 0.5), (0.9, 1.0)])
def test_chosen_steps_are_no_more_than_the_fixed_ones_where_they_are_taken(lib, share, decay):
    """Gaussian sketches of r = share d rows: up to nine tenths of d the steps are chosen, and there are no more of them."""
    rng = np.random.default_rng(7)
    d = 400
    r = int(share * d)
    assert not lib.is_fixed(r, d) and lib.is_fixed(d, d) and lib.is_fixed(int(0.91 * d), d)
    Y = rng.standard_normal((r, d)) * np.arange(1, d + 1) ** -decay
    Y /= np.linalg.norm(Y)
    G = Y @ Y.T
    state = {"x": np.linalg.svd(Y, compute_uv=False)}

    def apply(c):
        v = state["x"]
        state["x"] = v * (c[0] + v * v * (c[1] + v * v * c[2]))

    n = iterate(lib, r, apply, lambda: float(np.sqrt(min(np.abs(G).sum(1).max(), np.linalg.norm(G)))),
                lambda: float(((1 - state["x"] ** 2) ** 2).sum()))
    assert np.abs(state["x"] - 1).max() < 3e-6 and n <= lib.fixed_steps(r), (n, lib.fixed_steps(r))
