"""Training on index-picked batches, at the edges of a tile, a wave and a
block of the gradient kernel: the same parameters and losses, bit for bit, as
single steps on the gathered rows; an index outside the training set is read
as row 0 and reported.
"""
import numpy as np
import pytest

from workloads import surrogate as WS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


def _set(n, seed=1):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(n, 8, generator=g)
    return x.cuda(), (x[:, 0] * 0.5 - 0.1 * x[:, 1]).cuda(), torch.rand(n, generator=g).cuda()


# a tile is 32 cells, a wave takes two, a block four waves, 512 blocks at most
@pytest.mark.parametrize("batch", [1, 31, 33, 64, 255, 257, 32 * 512 * 4 + 5, 2 * 32 * 512 * 4 + 33])
def test_picked_batches_equal_gathered_ones(batch):
    n, steps = 5000, 3
    x, y, w = _set(n)
    idx = torch.randint(0, n, (steps, batch), generator=torch.Generator().manual_seed(batch)).cuda()
    lrs = [1e-3, 2e-3, 5e-4]
    p0 = WS.initial_params(2)
    with M.Mlp(p0) as a, M.Mlp(p0) as b:
        la = a.train_steps(x, y, w, idx, lrs, want_losses=True)
        lb = [b.train_step(x[i].contiguous(), y[i].contiguous(), w[i].contiguous(), lr, want_loss=True)
              for i, lr in zip(idx, lrs)]
        assert la == lb
        assert a.params() == b.params()


@pytest.mark.parametrize("bad", [-1, 1000, 1 << 40])
def test_bad_index_is_reported(bad):
    x, y, w = _set(1000)
    idx = torch.zeros((1, 100), dtype=torch.int64)
    idx[0, 57] = bad
    with M.Mlp(WS.initial_params(2)) as a, M.Mlp(WS.initial_params(2)) as b:
        with pytest.raises(M.MCLyaError) as e:
            a.train_steps(x, y, w, idx.cuda(), [1e-3])
        assert e.value.status == M.MC_LYA_EINVAL
        b.train_steps(x, y, w, torch.zeros((1, 100), dtype=torch.int64).cuda(), [1e-3])
        assert a.params() == b.params()
