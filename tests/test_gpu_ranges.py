"""Reductions whose ranges are added inside the launch, by the last workgroup of a tile to arrive: fp32 products of
few 16x16 tiles and bf16 products on 64x64 tiles, at ragged sizes, several calls on one workspace, each like the first."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import assert_close, desc_for, dev, guarded_forward, host, layer_to_dev
from oracle import ffsplit_oracle as orc
from workloads.configs import C2, C3, reduced

pytestmark = pytest.mark.gpu

CASES = [("f32", C2, 264, 3000, 40, 72, (1, 16, 17, 33, 130)), ("f32", C3, 96, 5000, 0, 20, (3, 64)), ("f32", C2, 64, 1100, 500, 64, (5, 40)),
         ("f32", C2, 72, 200, 10, 33, (128, 300)),            # a short reduction in front
         ("bf16", C2, 512, 4000, 100, 200, (65, 129, 300, 511)), ("bf16", C3, 1000, 3000, 70, 250, (66, 200)),
         ("bf16", C2, 256, 6000, 600, 60, (70, 1000))]


@pytest.mark.parametrize("dtype,base,d,n,k,r,Ts", CASES, ids=[f"{c[0]}_{c[1].act}_d{c[2]}_n{c[3]}_r{c[5]}" for c in CASES])
def test_ranges_added_in_the_launch(dtype, base, d, n, k, r, Ts):
    import paper_2401_04044_amd as ff
    cfg = reduced(base, d, n, rank=r)
    cfg = cfg.__class__(**{**cfg.__dict__, "dtype": dtype})
    L = wl.make_layer(cfg)
    idx = np.random.default_rng(n).permutation(n)[:k].astype(np.int32)
    fac = wl.make_factors(cfg, L, idx)
    Ld = layer_to_dev(L, dtype)
    desc = desc_for(ff, cfg, "lowrank", k=k)
    split = ff.build_split(desc, Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(idx).cuda(),
                           {nm: dev(v, dtype) for nm, v in fac.items()})
    for T in Ts:
        X = wl.make_tokens(cfg, T)
        got = guarded_forward(ff, desc, split, dev(X, dtype), want_parts=True)
        ws = torch.full((int(ff.workspace_bytes(desc, ff.WS_FORWARD, T)),), 0xA5, dtype=torch.uint8, device="cuda")
        again = [ff.forward(desc, split, dev(X, dtype), workspace=ws) for _ in range(3)]
        torch.cuda.synchronize()
        want = orc.forward_split(X, L["W1"], L["W2"], L["Wg"], idx, cfg.act, "lowrank", fac)
        for g, w, nm in zip(got, want, ("Y", "Y_heavy", "Y_rem")):
            if np.linalg.norm(w) > 0:
                assert_close(host(g), w, dtype, f"{dtype} d{d} n{n} T={T} {nm}")
        assert all(torch.equal(a, got[0]) for a in again)
