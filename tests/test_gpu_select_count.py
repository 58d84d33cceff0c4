"""Selection by counting, at the edges of its blocks of 32 elements, of the 8192 keys it holds at a time and of the
sizes that it serves; bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import ffsplit_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 129, 1023, 1025, 8191, 8192, 8193, 8229, 16385, 24575, 24576, 24577])
def test_selection_by_counting(n):
    import paper_2401_04044_amd as ff
    rng = np.random.default_rng(n)
    for scores in (rng.random(n).astype(np.float32), (rng.integers(-3, 3, n) / 4.0).astype(np.float32),
                   np.where(rng.random(n) < 0.3, np.float32(np.inf), rng.choice([-0.0, 0.0, 1e-45, -np.inf], n)).astype(np.float32)):
        sd = torch.from_numpy(scores).cuda()
        for k in sorted({0, 1, n // 30, n // 2, n - 1, n} & set(range(n + 1))):
            idx, perm, flag = ff.select_heavy(sd, k, want_perm=True)
            only = ff.select_heavy(sd, k)[0]
            torch.cuda.synchronize()
            want = orc.select_heavy(scores, k)
            assert np.array_equal(idx.cpu().numpy(), want) and torch.equal(only, idx), (n, k)
            assert np.array_equal(perm.cpu().numpy(), orc.neuron_permutation(want, n)), (n, k)
            assert int(flag.item()) == 0


@pytest.mark.parametrize("n", [1, 1024, 1025, 8192, 8193, 20000, 60001])
def test_nothing_selected(n):
    """k = 0: no index, the identity as permutation, and the flag of a NaN all the same (nothing is ranked)."""
    import paper_2401_04044_amd as ff
    scores = torch.rand(n, device="cuda")
    for nan in (False, True):
        if nan:
            scores[n - 1] = float("nan")
        idx, perm, flag = ff.select_heavy(scores, 0, want_perm=True)
        only = ff.select_heavy(scores, 0)[2]
        torch.cuda.synchronize()
        assert idx.numel() == 0 and torch.equal(perm.cpu(), torch.arange(n, dtype=torch.int32))
        assert int(flag.item()) == int(only.item()) == (-7 if nan else 0)
