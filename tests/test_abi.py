"""The C-ABI library loads, exports every symbol the header declares, and turns
bad arguments into error codes on the host before anything is launched (these
run without a GPU: no call here reaches a kernel launch)."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    txt = open(os.path.join(ROOT, "include", "ffsplit.h")).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return sorted(set(re.findall(r"\b(ffsplit_[a-z_0-9]+)\s*\(", txt)))


def test_library_exports_every_declared_symbol():
    import paper_2401_04044_amd as ff
    syms = declared_symbols()
    assert {"ffsplit_score_neurons", "ffsplit_select_heavy", "ffsplit_build_split", "ffsplit_forward"} <= set(syms)
    for s in syms:
        assert hasattr(ff.lib, s), s


def test_status_strings_and_sizes():
    import paper_2401_04044_amd as ff
    assert ff.status_string(0) == "ok"
    for c in range(-9, 0):
        assert ff.status_string(c) != "unknown status"
    d = ff.make_desc(2048, 8192, "gelu", "bf16", 246, "lowrank", 512)
    sb = ff.split_bytes(d)
    algorithmic = 2 * 2 * (2048 * 246 + 512 * (2048 + 7946))
    assert algorithmic <= sb <= 1.03 * algorithmic        # padding stays small
    assert ff.workspace_bytes(d, ff.WS_FORWARD, 4096) > 0
    assert ff.workspace_bytes(d, ff.WS_FORWARD, 0) >= 0
    d4 = ff.make_desc(4096, 11008, "swiglu", "bf16", 550, "int4", 0, 128)
    assert 79.78e6 <= ff.split_bytes(d4) <= 1.02 * 79.78e6
    # invalid descriptors give size 0
    assert ff.split_bytes(ff.make_desc(2048, 8192, "gelu", "bf16", 9000, "lowrank", 512)) == 0
    assert ff.split_bytes(ff.make_desc(2044, 8192, "gelu", "bf16", 10, "none")) == 0


def test_argument_errors_are_found_on_the_host():
    import paper_2401_04044_amd as ff
    L = ff.lib
    fake = ctypes.c_void_p(0x1000)          # aligned, never dereferenced: every call below fails validation
    odd = ctypes.c_void_p(0x1004)
    tt = ctypes.c_int64(0)
    good = ff.make_desc(64, 256, "gelu", "bf16", 16, "lowrank", 8)
    ref = ctypes.byref
    # NULL descriptor / pointers
    assert L.ffsplit_forward(None, fake, fake, 4, fake, None, None, fake, 1 << 30, None) == -1
    assert L.ffsplit_forward(ref(good), None, fake, 4, fake, None, None, fake, 1 << 30, None) == -1
    assert L.ffsplit_score_neurons(ref(good), fake, 4, None, None, fake, fake, ref(tt), None, 0, fake, 1 << 30, None) == -1
    # bad descriptor fields
    bad = ff.make_desc(64, 256, 7, "bf16", 16, "none")
    assert L.ffsplit_forward(ref(bad), fake, fake, 4, fake, None, None, fake, 1 << 30, None) == -2
    bad = ff.make_desc(64, 256, "gelu", 5, 16, "none")
    assert L.ffsplit_build_split(ref(bad), fake, None, fake, fake, None, fake, fake, 1 << 30, None) == -2
    # bad shapes
    for bad in (ff.make_desc(64, 256, "gelu", "bf16", 257, "none"),
                ff.make_desc(60, 256, "gelu", "bf16", 16, "none"),
                ff.make_desc(64, 256, "gelu", "bf16", 16, "lowrank", 0),
                ff.make_desc(64, 256, "gelu", "bf16", 16, "lowrank", 65),
                ff.make_desc(256, 1024, "swiglu", "bf16", 16, "int4", 0, 96)):
        assert L.ffsplit_forward(ref(bad), fake, fake, 4, fake, None, None, fake, 1 << 30, None) == -3
    assert L.ffsplit_forward(ref(good), fake, fake, -1, fake, None, None, fake, 1 << 30, None) == -3
    assert L.ffsplit_select_heavy(fake, 100, 101, fake, None, None, fake, 1 << 20, None) == -3
    # the entry point without a workspace: beyond its fixed scratch, and the usual argument checks
    assert L.ffsplit_select_heavy_static(fake, 65537, 5, fake, None, None, None) == -9
    assert L.ffsplit_select_heavy_static(fake, 100, 101, fake, None, None, None) == -3
    assert L.ffsplit_select_heavy_static(None, 100, 10, fake, None, None, None) == -1
    assert L.ffsplit_select_heavy_static(odd, 100, 10, fake, None, None, None) == -4
    # int4 needs bf16
    bad = ff.make_desc(256, 1024, "swiglu", "f32", 16, "int4", 0, 128)
    assert L.ffsplit_forward(ref(bad), fake, fake, 4, fake, None, None, fake, 1 << 30, None) == -6
    # alignment
    assert L.ffsplit_forward(ref(good), fake, odd, 4, fake, None, None, fake, 1 << 30, None) == -4
    # workspace too small / missing
    assert L.ffsplit_forward(ref(good), fake, fake, 4, fake, None, None, fake, 16, None) == -5
    assert L.ffsplit_forward(ref(good), fake, fake, 4, fake, None, None, None, 0, None) == -5
    assert L.ffsplit_select_heavy(fake, 100, 10, fake, None, None, fake, 8, None) == -5
    assert L.ffsplit_score_neurons(ref(good), fake, 4, fake, None, fake, fake, ref(tt), None, 0, fake, 16, None) == -5
    # missing factors for a low-rank build
    assert L.ffsplit_build_split(ref(good), fake, None, fake, fake, None, fake, fake, 1 << 30, None) == -1
    # device factorisation: wrong remainder kind, missing outputs, misaligned output, small workspace
    vp6 = ctypes.c_void_p * 6
    outs = vp6(fake, fake, None, None, fake, fake)
    dense = ff.make_desc(64, 256, "gelu", "bf16", 16, "dense")
    assert L.ffsplit_factorize_remainder(ref(dense), fake, None, fake, fake, 1, outs, fake, 1 << 30, None) == -2
    assert L.ffsplit_factorize_remainder(ref(good), fake, None, fake, fake, 1, None, fake, 1 << 30, None) == -1
    assert L.ffsplit_factorize_remainder(ref(good), fake, None, fake, fake, 1, vp6(fake, None, None, None, fake, fake),
                                         fake, 1 << 30, None) == -1
    assert L.ffsplit_factorize_remainder(ref(good), fake, None, fake, fake, 1, vp6(fake, odd, None, None, fake, fake),
                                         fake, 1 << 30, None) == -4
    assert L.ffsplit_factorize_remainder(ref(good), fake, None, fake, fake, 1, outs, fake, 64, None) == -5
    assert ff.workspace_bytes(good, ff.WS_FACTORIZE, 0) > 0 and ff.workspace_bytes(dense, ff.WS_FACTORIZE, 0) == 0
    w3 = ff.make_desc(256, 1024, "swiglu", "bf16", 16, "w3h8", 0, 128)
    assert ff.split_bytes(w3) > 0 and ff.workspace_bytes(w3, ff.WS_FORWARD, 8) > 0
    assert L.ffsplit_forward(ref(ff.make_desc(256, 1024, "swiglu", "f32", 16, "w3h8", 0, 128)), fake, fake, 4, fake, None,
                             None, fake, 1 << 30, None) == -6
    # T = 0 is a valid no-op that launches nothing
    assert L.ffsplit_forward(ref(good), fake, fake, 0, fake, None, None, None, 0, None) == 0
    assert tt.value == 0


def test_argument_errors_of_the_epilogue_norm_stack_and_probe_calls():
    """The calls added around the layer stack validate on the host like the others (no launch here)."""
    import paper_2401_04044_amd as ff
    L = ff.lib
    fake, odd = ctypes.c_void_p(0x1000), ctypes.c_void_p(0x1004)
    ref = ctypes.byref
    good = ff.make_desc(64, 256, "gelu", "bf16", 16, "lowrank", 8)
    gated = ff.make_desc(256, 1024, "swiglu", "bf16", 16, "int4", 0, 128)
    big = 1 << 30

    def epi(b1=None, b2=None, res=None, f32=0):
        e = ff.Epilogue()
        e.b1_packed, e.b2, e.residual, e.y_f32 = b1, b2, res, f32
        return e

    fwd = L.ffsplit_forward_ex
    assert fwd(ref(good), fake, fake, 4, fake, None, None, None, fake, 16, None) == -5            # as ffsplit_forward
    assert fwd(ref(good), fake, fake, 4, fake, None, None, ref(epi(b2=odd)), fake, big, None) == -4
    assert fwd(ref(good), fake, fake, 4, fake, None, None, ref(epi(res=odd)), fake, big, None) == -4
    assert fwd(ref(gated), fake, fake, 4, fake, None, None, ref(epi(b1=fake)), fake, big, None) == -6   # no b1 for gated units
    assert fwd(ref(good), fake, fake, 0, fake, None, None, ref(epi(b2=fake)), None, 0, None) == 0  # T = 0: no-op
    # neuron-bias packing
    assert ff.lib.ffsplit_neuron_bias_floats(ref(good)) == 64 + 256                                 # 16 -> 64, 240 -> 256
    assert L.ffsplit_pack_neuron_bias(ref(good), None, fake, fake, fake, big, None) == -1
    assert L.ffsplit_pack_neuron_bias(ref(good), fake, None, fake, fake, big, None) == -1          # k > 0 needs idx
    assert L.ffsplit_pack_neuron_bias(ref(good), odd, fake, fake, fake, big, None) == -4
    assert L.ffsplit_pack_neuron_bias(ref(good), fake, fake, fake, fake, 8, None) == -5
    # per-token RMS norm
    f32, bf16 = 0, 1
    assert {int(ff.make_desc(64, 256, "gelu", "f32", 0, "none").dtype), int(good.dtype)} == {f32, bf16}
    norm = L.ffsplit_token_rmsnorm
    assert norm(fake, 4, 60, ctypes.c_float(1e-6), bf16, fake, None) == -3                           # d_model % 8
    assert norm(fake, -1, 64, ctypes.c_float(1e-6), bf16, fake, None) == -3
    assert norm(fake, 4, 64, ctypes.c_float(1e-6), 7, fake, None) == -2
    assert norm(None, 4, 64, ctypes.c_float(1e-6), bf16, fake, None) == -1
    assert norm(odd, 4, 64, ctypes.c_float(1e-6), bf16, fake, None) == -4
    assert norm(None, 0, 64, ctypes.c_float(1e-6), bf16, None, None) == 0
    # stack driver
    vp2 = ctypes.c_void_p * 2
    stack = L.ffsplit_stack_forward
    eps = ctypes.c_float(1e-6)
    assert stack(ref(good), -1, vp2(fake, fake), None, None, fake, 4, eps, fake, big, None) == -3
    assert stack(ref(good), 2, None, None, None, fake, 4, eps, fake, big, None) == -1
    assert stack(ref(good), 2, vp2(fake, None), None, None, fake, 4, eps, fake, big, None) == -1   # a missing layer
    assert stack(ref(good), 2, vp2(fake, fake), None, None, odd, 4, eps, fake, big, None) == -4
    assert stack(ref(good), 2, vp2(fake, fake), None, None, fake, 4, eps, fake, 64, None) == -5
    assert stack(ref(good), 0, None, None, None, None, 4, eps, None, 0, None) == 0
    need = ff.workspace_bytes(good, ff.WS_STACK, 4)
    assert need >= ff.workspace_bytes(good, ff.WS_FORWARD, 4) + 4 * 64 * 2
    # probes
    fl = ctypes.c_double(0.0)
    assert L.ffsplit_probe_mfma(0, 10, fake, ref(fl), None) == -3
    assert L.ffsplit_probe_mfma(8, 10, None, ref(fl), None) == -1
    assert L.ffsplit_probe_stream_read(fake, 24, 8, fake, None) == -3                              # bytes % 16
    assert L.ffsplit_probe_stream_read(None, 32, 8, fake, None) == -1
    assert L.ffsplit_probe_stream_read(odd, 32, 8, fake, None) == -4


def test_forward_workspace_serves_every_smaller_batch():
    """ffsplit_workspace_bytes does not shrink as T grows, forward and stack, every remainder kind: a
    buffer sized for the largest batch is accepted for all smaller ones (the calls refuse one that is
    smaller than the figure for their own T)."""
    import numpy as np
    import paper_2401_04044_amd as ff

    def check(desc, ts):
        for call in (ff.WS_FORWARD, ff.WS_STACK):
            got = [ff.workspace_bytes(desc, call, int(t)) for t in ts]
            bad = [(t0, t1, b0, b1) for t0, t1, b0, b1 in zip(ts, ts[1:], got, got[1:]) if b1 < b0]
            assert not bad, (desc.d_model, desc.d_ff, desc.rem_kind, bad[:3])

    every = list(range(1, 4200)) + list(range(4200, 70000, 611))
    for args in ((2048, 8192, "gelu", "bf16", 246, "lowrank", 512), (4096, 11008, "swiglu", "bf16", 550, "lowrank", 1024),
                 (5120, 20480, "gelu", "bf16", 819, "lowrank", 1280), (4096, 11008, "swiglu", "bf16", 550, "dense"),
                 (4096, 11008, "swiglu", "bf16", 550, "int4", 0, 128), (4096, 11008, "swiglu", "bf16", 550, "w3h8", 0, 128),
                 (512, 560, "gelu", "bf16", 40, "lowrank", 500), (768, 3072, "gelu", "f32", 154, "lowrank", 64)):
        check(ff.make_desc(*args), every)
    rng = np.random.default_rng(9)
    for _ in range(150):
        kind = ("lowrank", "dense", "none", "int4", "w3h8")[int(rng.integers(0, 5))]
        d = 128 * int(rng.integers(1, 17)) if kind in ("int4", "w3h8") else 8 * int(rng.integers(1, 300))
        d_ff = int(rng.integers(8, 6000))
        k = int(rng.integers(0, d_ff))
        r = int(rng.integers(1, min(d, d_ff - k) + 1)) if kind == "lowrank" else 0
        desc = ff.make_desc(d, d_ff, "swiglu" if rng.integers(0, 2) else "gelu", "bf16", k, kind, r, 128 if kind in ("int4", "w3h8") else 0)
        check(desc, sorted(set(rng.integers(1, 400, 100)) | set((2.0 ** rng.uniform(6, 17, 200)).astype(int))))


def test_forward_workspace_has_room_for_every_split_product(tmp_path):
    """More than 64 rows of the low-rank chain (bf16): a product whose reduction is split keeps fp32
    partials [split][T][N] in the call's workspace.  The size the library reports must cover the
    intermediates plus the largest of those scratch buffers, for each of the four products (a scratch
    sized for three of them once let the fourth write past the workspace).  The number of ranges is
    taken from the planner itself."""
    import subprocess
    import numpy as np
    import paper_2401_04044_amd as ff

    src, so = tmp_path / "plan.cpp", tmp_path / "plan.so"
    src.write_text('#include "gemm_plan.h"\n'
                   'extern "C" int split_of(long M, int N, int K, int glu, int a_tiled) {\n'
                   '  return ffsplit::gemm_plan(M, N, K, glu, false, a_tiled, true).split; }\n')
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-shared", "-fPIC",
                           "-I" + os.path.join(ROOT, "paper_2401_04044_amd", "csrc"), str(src), "-o", str(so)])
    lib = ctypes.CDLL(str(so))
    lib.split_of.argtypes = [ctypes.c_long] + [ctypes.c_int] * 4

    def up(v, q):
        return (v + q - 1) // q * q

    rng = np.random.default_rng(5)
    seen = 0
    for _ in range(600):
        glu = bool(rng.integers(0, 2))
        d = int(rng.integers(8, 400)) * 8
        d_ff = int(rng.integers(64, 6000))
        k = int(rng.integers(0, d_ff // 2))
        m = d_ff - k
        r = int(rng.integers(1, min(d, m) + 1))
        T = int(rng.integers(65, 1025)) if rng.integers(0, 2) else int(2 ** rng.uniform(10, 14))
        desc = ff.make_desc(d, d_ff, "swiglu" if glu else "gelu", "bf16", k, "lowrank", r)
        n_up = 2 if glu else 1
        kp, rp, mp = up(k, 64), up(r, 64), up(m, 64)
        k4, tp = kp + rp, up(T, 32)
        inter = sum(up(tp * c * 2, 256) for c in (k4, n_up * rp, mp))
        products = [(n_up * k4, d, glu, 0), (rp, mp, 0, 1), (d, k4, 0, 1)]   # G1, G3, G4
        if not glu:
            products.append((mp, rp, 0, 1))                     # G2 (two left operands: never split)
        need = 0
        for N, K, g, tiled in products:
            sp = lib.split_of(T, N, K, g, tiled)
            seen += sp > 1
            need = max(need, sp * T * up(N, 32) * 4 if sp > 1 else 0)
        got = ff.workspace_bytes(desc, ff.WS_FORWARD, T)
        assert got >= inter + need, (d, d_ff, k, r, T, glu, got, inter, need)
    assert seen > 100   # split products among the 2100 drawn
