"""The two-launch network kernels at their edges: rows around the 16-row tile
and the 32-row batch padding, fewer rows than an earlier call on the handle,
widths around the 16-column tile, the 16-wave block and the 256-deep load
group, one layer, and a network too wide for a block's LDS (layer by layer).
Against the oracle's BF16 reading, at the bar of the production network's
test: 2^-7 of |ref| + rms(ref)."""
import numpy as np
import pytest

from oracle import mlp_oracle as R
from test_gpu_mlp import flat, unflat

pytestmark = pytest.mark.gpu


def close(got, ref):
    return np.max(np.abs(got - ref) / (np.abs(ref) + np.sqrt(np.mean(ref ** 2)) + 1e-30)) < 2.0 ** -7


@pytest.mark.parametrize("rows", [1, 15, 16, 17, 33, 64])
@pytest.mark.parametrize("sizes", [(3, 5), (3, 16, 17, 7), (40, 288, 31), (3, 256, 256, 579), (4, 768, 7), (4, 800, 7), (5, 1000, 9)],
                         ids=lambda s: "x".join(map(str, s)))
def test_edges(rows, sizes):
    import torch
    import paper_1701_02005_amd as P
    params = R.init_params(sizes, seed=rows)
    rng = np.random.default_rng(rows)
    net = P.Mlp(sizes, 70, flat(params))
    for n in (70, rows):  # (the rows of the first call lie behind those of the second)
        x = rng.uniform(-1, 1, (n, sizes[0]))
        y = rng.standard_normal((n, sizes[-1]))
        xt = torch.tensor(x, dtype=torch.float32, device="cuda")
        yt = torch.tensor(y, dtype=torch.float32, device="cuda")
        loss = net.gradients(xt, yt)
        out = net.forward(xt).cpu().numpy()
    ref, _, _ = R.forward(params, xt.cpu().numpy().astype(np.float64), bf16=True)
    assert close(out, ref)
    loss_ref, grads = R.backward(params, xt.cpu().numpy().astype(np.float64), yt.cpu().numpy().astype(np.float64), bf16=True)
    assert loss == pytest.approx(loss_ref, rel=2.0 ** -7)
    _, g = net.get_params()
    for (gW, gb), (rW, rb) in zip(unflat(g, sizes), grads):
        assert close(gW, rW) and close(gb, rb)
