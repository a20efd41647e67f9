"""Forward passes that go layer by layer on a network whose training steps run
in one kernel: the same sums in the same order, so the rows of a call of up to
384 rows are those of a larger call, which runs in one kernel, bit for bit;
and they leave nothing behind that a training step would take in."""
import numpy as np
import pytest

from oracle import mlp_oracle as R
from test_gpu_mlp import flat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(768, 768), (700, 590, 640, 530), (514,) * 9, (512,) * 9, (640, 8, 640), (3, 256, 579)],
                         ids=lambda s: f"{len(s) - 1}x{max(s)}in{s[0]}")
def test_rows_of_a_larger_call(sizes):
    import torch
    import paper_1701_02005_amd as P
    p = flat(R.init_params(sizes, seed=1))
    rng = np.random.default_rng(2)
    x = torch.tensor(rng.uniform(-1, 1, (520, sizes[0])), dtype=torch.float32, device="cuda")
    y = torch.tensor(rng.standard_normal((520, sizes[-1])), dtype=torch.float32, device="cuda")
    net, other = P.Mlp(sizes, 520, p), P.Mlp(sizes, 520, p)
    ref = net.forward(x)
    for rows in (384, 1, 33, 64):
        assert torch.equal(net.forward(x[:rows].contiguous()), ref[:rows]), rows
    for rows in (33, 520, 16):
        net.forward(x[:rows].contiguous())
        xr, yr = x[:rows].contiguous(), y[:rows].contiguous()
        assert torch.equal(net.train_step(xr, yr, 1e-3), other.train_step(xr, yr, 1e-3))
        for a, b in zip(net.get_params(), other.get_params()):
            assert np.array_equal(a, b)
