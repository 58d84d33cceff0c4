"""8-bit heavy / 3-bit remainder with at most 16 tokens (one launch per product): group counts on every side of the
eight wavefronts, odd numbers of 64-neuron blocks, either part empty, the sizes where the kernels change."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import assert_close, desc_for, dev, guarded_forward, host, layer_to_dev
from oracle import ffsplit_oracle as orc
from workloads.configs import C2, C4, reduced

pytestmark = pytest.mark.gpu

CASES = [(C4, 128, 130, 10), (C4, 384, 500, 100), (C4, 1024, 320, 0), (C4, 1152, 300, 300), (C4, 2176, 200, 64),
         (C2, 128, 96, 30), (C2, 896, 700, 129), (C2, 2048, 260, 60), (C4, 4096, 200, 70), (C4, 4224, 150, 20), (C4, 5120, 96, 30),
         (C2, 4224, 100, 30), (C4, 5248, 64, 10)]


@pytest.mark.parametrize("base,d,n,k", CASES, ids=[f"{c[0].act}_d{c[1]}_n{c[2]}_k{c[3]}" for c in CASES])
def test_up_to_16_tokens(base, d, n, k):
    import paper_2401_04044_amd as ff
    cfg = reduced(base, d, n)
    L = wl.make_layer(cfg)
    idx = np.random.default_rng(d).permutation(n)[:k].astype(np.int32)
    Ld = layer_to_dev(L, cfg.dtype)
    desc = desc_for(ff, cfg, "w3h8", k=k)
    split = ff.build_split(desc, Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(idx).cuda())
    for T in (1, 15, 16, 17):
        X = wl.make_tokens(cfg, T)
        got = guarded_forward(ff, desc, split, dev(X, cfg.dtype), want_parts=True)
        torch.cuda.synchronize()
        want = orc.forward_split(X, L["W1"], L["W2"], L["Wg"], idx, cfg.act, "w3h8", group=128)
        for g, w, nm in zip(got, want, ("Y", "Y_heavy", "Y_rem")):
            if np.linalg.norm(w) == 0:
                assert not host(g).any()
            else:
                assert_close(host(g), w, "bf16", f"d{d} n{n} k{k} T={T} {nm}")


# more neurons than quant16_fits allows, and just below; 8-bit parts between a third of a round and a round, with the 3-bit part in
# what is left of it or behind it; two workgroups a CU
SPLITS = [(C2, 128, 16300, 40), (C2, 128, 16500, 40), (C4, 128, 23600, 40), (C4, 128, 8000, 3900), (C2, 1152, 9000, 5800),
          (C4, 1152, 3000, 2900), (C4, 1152, 9000, 1500), (C2, 256, 4200, 4100)]


@pytest.mark.parametrize("base,d,n,k", SPLITS, ids=[f"{c[0].act}_d{c[1]}_n{c[2]}_k{c[3]}" for c in SPLITS])
def test_every_split_of_the_machine(base, d, n, k):
    test_up_to_16_tokens(base, d, n, k)


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_down_product_rounds_the_activations_only(act):
    """fp32 output against fp64 on the split's own weights: the activations are rounded to fp16 once and once more with their scales,
    2^-10 / sqrt(12) x 0.72 each (the mean of 1 / x over a binade), 2.9e-4 together; the codes enter exactly.  (As 1024 + code, with the
    constant subtracted from the sums, activations of one sign put another 2e-4 there.)"""
    import paper_2401_04044_amd as ff
    d, f, k, T = 1024, 12288, 1224, 16
    gen = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *s: (torch.randn(*s, device="cuda", generator=gen) * 0.05).to(torch.bfloat16)
    W1, W2, Wg = rnd(d, f), rnd(f, d), rnd(d, f) if act == "swiglu" else None
    desc = ff.make_desc(d, f, act, "bf16", k, "w3h8", 0, 128)
    split = ff.build_split(desc, W1, Wg, W2, torch.arange(k, dtype=torch.int32, device="cuda"))
    X = rnd(T, d) * 20

    def weights(what):
        q, s = ff.split_export(desc, split, what)
        return host(q).astype(np.float64) * np.repeat(host(s.view(torch.float16)).astype(np.float64), 128, axis=1)

    up, down = np.vstack([weights(3), weights(0)]), np.vstack([weights(5), weights(2)])
    x = host(X).astype(np.float64)
    h = x @ up.T
    if act == "swiglu":
        g = x @ np.vstack([weights(4), weights(1)]).T
        h = h * g / (1 + np.exp(-g))
    else:
        h = torch.nn.functional.gelu(torch.from_numpy(h)).numpy()
    want = h @ down
    got = torch.empty(T, d, device="cuda")
    ff.forward_ex(desc, split, X, got, y_f32=True)
    torch.cuda.synchronize()
    err = np.linalg.norm(host(got).astype(np.float64) - want) / np.linalg.norm(want)
    assert err < 3.1e-4, err
