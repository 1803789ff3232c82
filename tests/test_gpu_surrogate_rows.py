"""Training reads the rows of the caller's features where they lie: a set that
starts at any float (a slice of a larger buffer) trains to the parameters and
losses of the same set at the start of an allocation, bit for bit.
"""
import pytest

from workloads import surrogate as WS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2312_11448_amd as M  # noqa: E402


@pytest.mark.parametrize("offset", [1, 2, 3])
def test_rows_at_any_float(offset):
    n, steps, batch = 3000, 3, 700
    g = torch.Generator().manual_seed(offset)
    x = torch.randn(n, 8, generator=g).cuda()
    y, w = torch.randn(n, generator=g).cuda(), torch.rand(n, generator=g).cuda()
    idx = torch.randint(0, n, (steps, batch), generator=g).cuda()
    room = torch.zeros(8 * n + 8, device="cuda")
    moved = room[offset:offset + 8 * n].view(n, 8)
    moved.copy_(x)
    assert moved.data_ptr() % 16 == 4 * offset and moved.is_contiguous()
    p0 = WS.initial_params(2)
    with M.Mlp(p0) as a, M.Mlp(p0) as b:
        assert a.gradient(x, y, w) == b.gradient(moved, y, w)
        la = a.train_steps(x, y, w, idx, [1e-3] * steps, want_losses=True)
        lb = b.train_steps(moved, y, w, idx, [1e-3] * steps, want_losses=True)
        assert la == lb and a.params() == b.params()
