"""The polar iteration on the device where it leaves the steps launched one by one (the work queue), where the
matrices of a layer end at different steps, and on 64x64 tiles of the symmetric products."""
import numpy as np
import pytest
import torch

import workloads as wl
from gpu_util import desc_for, host, layer_to_dev, relf
from oracle import ffsplit_oracle as orc
from workloads.configs import C2, C3, reduced

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ff():
    import paper_2401_04044_amd as m
    return m


CASES = [("r72", reduced(C2, 264, 500, rank=72), (0.0, 1.0, 2.0)), ("r200", reduced(C2, 640, 900, rank=200), (0.0, 1.0, 2.0)),
         ("r800_wide", reduced(C3, 1608, 1700, rank=800), (0.0, 1.0)), ("r800_nearly_square", reduced(C3, 1096, 1300, rank=800), (0.0, 1.0))]


@pytest.mark.parametrize("cfg,decay", [(c, d) for _, c, ds in CASES for d in ds],
                         ids=[f"{n}-{d}" for n, _, ds in CASES for d in ds])
def test_factors_of_decaying_remainders(ff, cfg, decay):
    """W1 flat, W2 with singular values i^-decay: the basis orthonormal and the products those of the oracle in
    fp64 (singular values of the sketch above 1 / (1024 r) of its norm, which i^-2 leaves at rank 800)."""
    cfg = cfg.__class__(**{**cfg.__dict__, "dtype": "f32"})
    L = {k: v.copy() if isinstance(v, np.ndarray) else v for k, v in wl.make_layer(cfg).items()}
    scale = (np.arange(1, cfg.d_model + 1) ** -decay).astype(np.float32)
    L["W2"] = (L["W2"] * scale).astype(np.float32)
    idx, Ld = L["planted"], layer_to_dev(L, "f32")
    fd = ff.factorize_remainder(desc_for(ff, cfg, "lowrank"), Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(idx).cuda(), seed=3)
    torch.cuda.synchronize()
    got = {k: host(v) for k, v in fd.items() if v is not None}
    want = orc.factorize_remainder(L["W1"], L["W2"], L["Wg"], idx, cfg.rank, seed=3)
    eye = np.eye(cfg.rank)
    assert np.abs(got["P1"].T @ got["P1"] - eye).max() < 1e-5
    assert np.abs(got["Q2"] @ got["Q2"].T - eye).max() < 1e-5
    for p, q in (("P1", "Q1"), ("Pg", "Qg"), ("P2", "Q2")):
        if p in want:
            assert relf(got[p] @ got[q], want[p] @ want[q]) < 1e-4, p


@pytest.mark.parametrize("cfg", [reduced(C2, 72, 400, rank=8), reduced(C3, 264, 300, rank=130), reduced(C2, 1032, 2100, rank=72), reduced(C2, 2056, 700, rank=250)],
                         ids=["d72", "d264_gated", "d1032", "d2056"])
def test_projection_of_three_terms_in_one_reduction(ff, cfg):
    """bf16 factors at widths that are no multiple of 64 (the left operand of the projection starts again at the
    padded width): products like the oracle's in fp64 but for two bf16 roundings."""
    L = wl.make_layer(cfg)
    idx, Ld = L["planted"], layer_to_dev(L, "bf16")
    fd = ff.factorize_remainder(desc_for(ff, cfg, "lowrank"), Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(idx).cuda(), seed=9)
    torch.cuda.synchronize()
    got = {k: host(v) for k, v in fd.items() if v is not None}
    want = orc.factorize_remainder(L["W1"], L["W2"], L["Wg"], idx, cfg.rank, seed=9)
    for p, q in (("P1", "Q1"), ("Pg", "Qg"), ("P2", "Q2")):
        if p in want:
            assert relf(got[p] @ got[q], want[p] @ want[q]) < 6e-3, p
