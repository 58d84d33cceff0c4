"""The polar iteration on the device: remainders that decay and so take many steps, matrices of a layer that end at different
steps, and every form that its products are launched in."""
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


# || B B^T - I ||_F / sqrt(r): what a row of B lacks of unit length and of being orthogonal to the others.  Rounding the last sum
# of each element takes a row's length by up to 2^-25; rounding T - I, and the sums of the last X X^T behind it, by as much
# each; the off-diagonal elements add as much again: 4 x 2^-24 = 2.4e-7.  Where the rows' energy lies in few columns (decaying
# remainders) fewer roundings average out: 6 x 2^-24.  At 2048 x 2600 rank 512 the iteration has 1.7e-7 (3.0e-7 with i^-1);
# with one accumulator a tile, a chain of d / 4 terms, it had 6.8e-7.
ORTHONORMAL, ORTHONORMAL_DECAY = 4 * 2.0 ** -24, 6 * 2.0 ** -24


def off_orthonormal(b):
    b = b.astype(np.float64)
    return float(np.linalg.norm(b @ b.T - np.eye(len(b))) / np.sqrt(len(b)))


# every form that the products are launched in: tiles of X X^T of 16, 32 and 64, the other two products together (rank 64,
# rank 128) and apart, the last one on 32x32 and on 64x64 tiles; ranks and widths that no tile divides
FORMS = [(C2, 72, 300, 8), (C3, 264, 400, 33), (C2, 520, 700, 64), (C2, 1032, 1200, 65), (C2, 2056, 2300, 128), (C3, 640, 900, 130),
         (C2, 1024, 1400, 256), (C2, 1000, 1300, 256), (C2, 4104, 2300, 250), (C3, 360, 900, 175), (C2, 8, 40, 1)]


@pytest.mark.parametrize("base,d,n,r", FORMS, ids=[f"{c[0].act}_d{c[1]}_n{c[2]}_r{c[3]}" for c in FORMS])
def test_every_form_of_the_products(ff, base, d, n, r):
    """W1 flat, W2 with singular values i^-3/2 (the matrices of the layer end at different steps): the basis orthonormal, the
    products those of the oracle in fp64, and every call like the first."""
    cfg = reduced(base, d, n, rank=r)
    cfg = cfg.__class__(**{**cfg.__dict__, "dtype": "f32"})
    L = {k: v.copy() if isinstance(v, np.ndarray) else v for k, v in wl.make_layer(cfg).items()}
    L["W2"] = (L["W2"] * (np.arange(1, d + 1) ** -1.5)).astype(np.float32)
    idx, Ld = L["planted"], layer_to_dev(L, "f32")
    desc = desc_for(ff, cfg, "lowrank")
    args = (desc, Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(idx).cuda())
    ws = torch.full((int(ff.workspace_bytes(desc, ff.WS_FACTORIZE, 0)),), 0xA5, dtype=torch.uint8, device="cuda")
    fd = ff.factorize_remainder(*args, seed=3, workspace=ws)
    again = ff.factorize_remainder(*args, seed=3, workspace=ws)
    torch.cuda.synchronize()
    assert all(torch.equal(v, again[k]) for k, v in fd.items() if v is not None)
    got = {k: host(v) for k, v in fd.items() if v is not None}
    want = orc.factorize_remainder(L["W1"], L["W2"], L["Wg"], idx, cfg.rank, seed=3)
    for b, most in ((got["P1"].T, ORTHONORMAL), (got.get("Pg", got["P1"]).T, ORTHONORMAL), (got["Q2"], ORTHONORMAL_DECAY)):
        assert off_orthonormal(b) < most, off_orthonormal(b)
    for p, q in (("P1", "Q1"), ("Pg", "Qg"), ("P2", "Q2")):
        if p in want:
            assert relf(got[p] @ got[q], want[p] @ want[q]) < 1e-4, p


@pytest.mark.parametrize("d,r,decay", [(2048, 512, 0.0), (2048, 512, 1.0), (1608, 800, 0.0), (768, 768, 0.0), (1024, 128, 0.0)])
def test_basis_is_as_orthonormal_as_fp32_sums_allow(ff, d, r, decay):
    cfg = reduced(C2, d, 2600, rank=r)
    cfg = cfg.__class__(**{**cfg.__dict__, "dtype": "f32"})
    L = {k: v.copy() if isinstance(v, np.ndarray) else v for k, v in wl.make_layer(cfg).items()}
    L["W2"] = (L["W2"] * (np.arange(1, d + 1) ** -decay)).astype(np.float32)
    Ld = layer_to_dev(L, "f32")
    fd = ff.factorize_remainder(desc_for(ff, cfg, "lowrank"), Ld["W1"], Ld["Wg"], Ld["W2"], torch.from_numpy(L["planted"]).cuda(), seed=5)
    torch.cuda.synchronize()
    assert off_orthonormal(host(fd["P1"]).T) < ORTHONORMAL
    assert off_orthonormal(host(fd["Q2"])) < (ORTHONORMAL_DECAY if decay else ORTHONORMAL), off_orthonormal(host(fd["Q2"]))


def test_basis_larger_than_four_gib(ff):
    """X of 1104 x 1048608 floats, further than a 32-bit offset reaches from its first element: rows from 1024 on must not be taken
    for the first ones, which would leave their rows' lengths wrong by as much as the steps change them; and sums over 2^20 columns.  These are
    256 sums of 4096: 16 x 2^-25 by 256 roundings of either sign on top of what a short row has."""
    d, n, k, r = 1048608, 1208, 8, 1100
    desc = ff.make_desc(d, n, k=k, rank=r, act="gelu", dtype="f32", rem_kind="lowrank")
    gen = torch.Generator(device="cuda").manual_seed(7)
    W1 = torch.randn(d, n, device="cuda", generator=gen)
    W2 = torch.randn(n, d, device="cuda", generator=gen)
    fd = ff.factorize_remainder(desc, W1, None, W2, torch.arange(k, dtype=torch.int32, device="cuda"), seed=3)
    eye = torch.eye(r, dtype=torch.float64, device="cuda")
    for b in (fd["Q2"], fd["P1"].t()):
        g = torch.zeros(r, r, dtype=torch.float64, device="cuda")
        for c in range(0, d, 65536):
            x = b[:, c:c + 65536].double().contiguous()
            g += x @ x.t().contiguous()
        off = float((g - eye).norm()) / r ** 0.5
        assert off < ORTHONORMAL + 16 * 2.0 ** -25, off
