"""A forward pass whose outputs overlap its inputs in memory (in place, or
shifted against them) gives what it gives in a buffer of its own."""
import ctypes

import numpy as np
import pytest

from oracle import mlp_oracle as R
from test_gpu_mlp import flat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(24, 32, 24), (24, 32, 40), (40, 32, 24), (24, 800, 24)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("rows", [1, 17, 500])
def test_overlapping_output(sizes, rows):
    import torch
    import paper_1701_02005_amd as P
    net = P.Mlp(sizes, rows, flat(R.init_params(sizes, seed=rows)))
    rng = np.random.default_rng(rows)
    x = torch.tensor(rng.uniform(-1, 1, (rows, sizes[0])), dtype=torch.float32, device="cuda")
    ref = net.forward(x)
    nin, nout, room = rows * sizes[0], rows * sizes[-1], rows * 40
    for xo, yo in ((room, room), (room, room - nout // 2), (room, room + nin // 2)):
        buf = torch.zeros(3 * room, dtype=torch.float32, device="cuda")
        buf[xo:xo + nin] = x.ravel()
        rc = net.lib.nspnp_mlp_forward(net._h, ctypes.c_void_p(buf.data_ptr() + 4 * xo), rows,
                                       ctypes.c_void_p(buf.data_ptr() + 4 * yo))
        assert rc == 0
        net.sync()
        assert torch.equal(buf[yo:yo + nout].view(rows, -1), ref), (xo, yo)
