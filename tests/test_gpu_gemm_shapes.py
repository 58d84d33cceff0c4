"""GPU parity of the bf16 and fp32 product kernels at sizes that reach each tile shape, unit and
reduction split with remainders on every side (rows, columns, reduction depth), against the CPU
oracle.  Bars: the task's (bf16 1e-2 relative Frobenius, 2e-2 worst row; fp32 a thousandth of that)."""
import numpy as np
import pytest
import torch

from oracle import ffsplit_oracle as orc
from gpu_util import dev, host, assert_close, Guarded

pytestmark = pytest.mark.gpu

# T, d_model, d_ff, k, rank, act: tiles (x ranges of the reduction) of the four products; test_gemm_plan.py
# checks that every form is among them
CASES = [
    (65, 72, 97, 39, 17, "gelu"),              # 64x64, 64x64, 64x64, 64x64
    (565, 256, 87, 0, 3, "swiglu"),            # 64x128, 128x128, 64x64, 64x64
    (2911, 200, 6019, 2763, 3, "gelu"),        # 128x320, 128x320, 64x64 x5, 64x64
    (1838, 80, 5539, 1, 3, "gelu"),            # 64x64, 128x256, 64x64 x6, 64x64
    (4080, 136, 2085, 36, 129, "gelu"),        # 64x64, 128x320, 64x64, 64x64
    (1393, 64, 5212, 47, 2, "swiglu"),         # 64x128, 128x128, 64x64 x6, 64x64
    (4889, 440, 3391, 13, 2, "gelu"),          # 64x64, 256x320, 64x64 x3, 64x128
    (5036, 1592, 294, 1, 10, "gelu"),          # 64x64, 64x64, 64x64, 128x320
    (4370, 1968, 146, 3, 67, "gelu"),          # 64x64, 64x64, 64x64, 128x320
    (4717, 1696, 294, 68, 11, "swiglu"),       # 64x128, 128x128, 64x64, 128x320
    (321, 1048, 1500, 70, 130, "gelu"),        # 64x64, 64x64, 64x64, 64x64
    (700, 1544, 2300, 300, 67, "swiglu"),      # 64x128, 128x128, 64x64 x4, 64x64
    (150, 2056, 1200, 33, 300, "gelu"),        # 64x64 x5, 64x64, 64x64, 64x64
    (100, 88, 2282, 114, 40, "swiglu"),        # 64x128, 128x128, 64x64 x5, 64x64
    (5070, 592, 4005, 40, 80, "gelu"),         # 64x64, 128x128, 64x128 x3, 64x128
    (5978, 176, 6112, 305, 78, "gelu"),        # 64x128, 128x256, 128x128 x5, 64x64
    (2641, 3160, 261, 2, 40, "swiglu"),        # 64x128 x3, 128x128, 64x64, 128x320
    (4365, 3816, 105, 1, 40, "gelu"),          # 64x128 x3, 64x64, 64x64, 256x320
    (1887, 144, 4921, 984, 78, "swiglu"),      # 128x128, 256x256, 64x64 x4, 64x64
    (108, 1592, 84, 0, 40, "gelu"),            # 64x64 x5, 64x64, 64x64, 64x64
    (3729, 72, 1210, 968, 40, "gelu"),         # 128x128, 64x64, 64x64, 64x64
    (4039, 72, 1995, 997, 40, "swiglu"),       # 128x256, 128x128, 64x64, 64x64
    (1831, 72, 6306, 5044, 40, "gelu"),        # 128x320, 64x128, 64x64, 64x64 x4
    (5013, 72, 2740, 2192, 40, "gelu"),        # 128x256, 64x128, 64x64, 64x64
    (82, 3784, 3089, 2471, 311, "swiglu"),     # 128x128 x5, 128x128, 64x64, 64x64 x2
    (4562, 80, 7616, 3808, 40, "gelu"),        # 256x320, 256x320, 64x64 x3, 64x128 x3
    (87, 4008, 8069, 6455, 84, "gelu"),        # 128x128 x4, 64x64, 64x64, 64x128 x4
    (5002, 840, 919, 735, 59, "swiglu"),       # 256x256, 128x128, 64x64, 128x128
]


# At most 64 tokens (one launch per product): blocks of 16 tokens, 16- and 32-row units, reductions
# cut across workgroups, depths that end inside a step of 32.
SMALL = [
    (1, 72, 97, 39, 17, "gelu"),             # reduction shorter than the wavefronts' shares
    (16, 264, 2600, 3, 40, "swiglu"),        # pairs and single pieces in one launch
    (17, 1056, 9000, 100, 64, "gelu"),       # third product: 4 units in 8 ranges
    (32, 4128, 300, 20, 9, "gelu"),          # last product on 32-row units
    (5, 1000, 6000, 2300, 900, "swiglu"),    # first product on 32-row units beside pairs
    (33, 544, 4300, 700, 65, "swiglu"),      # third product in 3 ranges
    (49, 776, 4300, 1, 130, "gelu"),         # d_model % 32 = 8; second product on 32-row units
    (64, 2048, 1030, 1028, 1, "gelu"),       # two remainder neurons
]


@pytest.mark.parametrize("T,d,d_ff,k,r,act", CASES + SMALL)
def test_every_tile_shape_matches_oracle(T, d, d_ff, k, r, act):
    import paper_2401_04044_amd as ff
    rng = np.random.default_rng(T)

    def bf(shape, std):   # values exactly representable in bf16
        t = torch.from_numpy((rng.standard_normal(shape) * std).astype(np.float32))
        return t.to(torch.bfloat16).to(torch.float32).numpy()

    glu, m = act == "swiglu", d_ff - k
    X, W1, W2 = bf((T, d), 1.0), bf((d, d_ff), d ** -0.5), bf((d_ff, d), 0.05)
    Wg = bf((d, d_ff), d ** -0.5) if glu else None
    fac = {"P1": bf((d, r), d ** -0.5), "Q1": bf((r, m), r ** -0.5), "P2": bf((m, r), 0.05), "Q2": bf((r, d), 0.5),
           "Pg": bf((d, r), d ** -0.5) if glu else None, "Qg": bf((r, m), r ** -0.5) if glu else None}
    idx = rng.permutation(d_ff)[:k].astype(np.int32)
    desc = ff.make_desc(d, d_ff, act, "bf16", k, "lowrank", r)
    idx_d = torch.from_numpy(idx).cuda()
    split = ff.build_split(desc, dev(W1, "bf16"), dev(Wg, "bf16"), dev(W2, "bf16"), idx_d,
                           {nm: dev(v, "bf16") for nm, v in fac.items()})
    g = Guarded(ff.workspace_bytes(desc, ff.WS_FORWARD, T))
    Y, Yh, Yr = ff.forward(desc, split, dev(X, "bf16"), None, True, g.view)
    g.check("forward")
    want, w1, w2 = orc.forward_split(X, W1, W2, Wg, idx, act, "lowrank", fac)
    name = f"T{T} d{d} f{d_ff} k{k} r{r} {act}"
    assert_close(host(Y), want, "bf16", name + " Y")
    assert_close(host(Yr), w2, "bf16", name + " Y_rem")
    if k:
        assert_close(host(Yh), w1, "bf16", name + " Y_heavy")
    if not glu:
        # the store step with bias, residual and fp32 destination on the same tiles
        b1 = bf((d_ff,), 0.3)
        b2, res = rng.standard_normal(d).astype(np.float32), rng.standard_normal((T, d)).astype(np.float32)
        Y = ff.forward_ex(desc, split, dev(X, "bf16"), b1_packed=ff.pack_neuron_bias(desc, dev(b1, "bf16"), idx_d),
                          b2=torch.from_numpy(b2).cuda(), residual=torch.from_numpy(res).cuda(), y_f32=True,
                          workspace=g.view)
        g.check("forward_ex")
        want = orc.forward_split_biased(X, W1, W2, idx, "lowrank", fac, b1, b2, res)[0]
        assert_close(host(Y), want, "bf16", name + " biased")


# fp32: every tile of gated (one and two left operands) and plain products; depths of half a slab of 16, and
# of fewer slabs than there are k groups (d_model 8 and 72)
F32 = [
    (1, 8, 70, 3, 5, "gelu"),                # 16x16 throughout
    (7, 72, 300, 20, 30, "swiglu"),          # 16x64, two left operands 16x64
    (300, 520, 1300, 100, 130, "swiglu"),    # two left operands 32x64; 16x16, 32x32
    (517, 1032, 1500, 150, 70, "swiglu"),    # 32x64, two left operands 64x128; 16x32, 64x64
    (1000, 264, 2000, 500, 100, "swiglu"),   # 64x128, two left operands 64x128
    (517, 1032, 2500, 400, 300, "gelu"),     # 32x32, 64x64
    (900, 1000, 3000, 600, 200, "gelu"),     # 64x64 first and last product
    (300, 776, 3000, 150, 64, "gelu"),       # 16x32 first product
]


@pytest.mark.parametrize("T,d,d_ff,k,r,act", F32)
def test_every_fp32_tile_matches_oracle(T, d, d_ff, k, r, act):
    import paper_2401_04044_amd as ff
    rng = np.random.default_rng(T + d)
    glu, m = act == "swiglu", d_ff - k

    def f32(shape, std):
        return (rng.standard_normal(shape) * std).astype(np.float32)

    X, W1, W2 = f32((T, d), 1.0), f32((d, d_ff), d ** -0.5), f32((d_ff, d), 0.05)
    Wg = f32((d, d_ff), d ** -0.5) if glu else None
    fac = {"P1": f32((d, r), d ** -0.5), "Q1": f32((r, m), r ** -0.5), "P2": f32((m, r), 0.05), "Q2": f32((r, d), 0.5),
           "Pg": f32((d, r), d ** -0.5) if glu else None, "Qg": f32((r, m), r ** -0.5) if glu else None}
    idx = rng.permutation(d_ff)[:k].astype(np.int32)
    desc = ff.make_desc(d, d_ff, act, "f32", k, "lowrank", r)
    split = ff.build_split(desc, dev(W1, "f32"), dev(Wg, "f32"), dev(W2, "f32"), torch.from_numpy(idx).cuda(),
                           {nm: dev(v, "f32") for nm, v in fac.items()})
    g = Guarded(ff.workspace_bytes(desc, ff.WS_FORWARD, T))
    got = ff.forward(desc, split, dev(X, "f32"), None, True, g.view)
    g.check("forward")
    want = orc.forward_split(X, W1, W2, Wg, idx, act, "lowrank", fac)
    for y, w, nm in zip(got, want, ("Y", "Y_heavy", "Y_rem")):
        assert_close(host(y), w, "f32", f"f32 T{T} d{d} f{d_ff} k{k} r{r} {act} {nm}")
