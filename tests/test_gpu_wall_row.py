"""The wall row of v holds 0 whatever the solves above it hold: also in a run
that has produced a value that is not finite, under every Crank-Nicolson method
and with implicit x/z."""
import dataclasses

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("imp", [0, 1])
@pytest.mark.parametrize("rows,cnslab", [(8, 0), (8, 16), (40, 32), (322, 0)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_wall_row_of_a_bad_run(precision, rows, cnslab, imp, value):
    import torch
    import paper_1701_02005_amd as P
    s = P.Solver(dataclasses.replace(P.configs.couette_small(precision=precision), nx=16, ny=rows + 1, nz=12,
                                     implicit_xz=imp, u_noise=0.05))
    s.set_tiles(cnslab=cnslab)
    s.step(1)
    u = s.get_field("u")
    u[4, 3, 5] = value
    s.set_field("u", u)
    s.step(1)
    v = s.get_field("v")
    assert torch.isnan(v[1:]).any() and torch.equal(v[0], torch.zeros_like(v[0]))
