"""Above 320 rows no path reads the pivot pairs of the lane-split mode solves:
they take no room in the workspace, and members of an ensemble that tall give
what runs of their own give, bit for bit."""
import dataclasses

import pytest


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_no_room_for_unread_pivots(precision):
    import paper_1701_02005_amd as P
    base = dataclasses.replace(P.configs.couette_small(precision=precision), nx=64, nz=64)
    low, tall = (P.workspace_bytes(dataclasses.replace(base, ny=rows + 1)) for rows in (320, 321))
    pivots = 2 * 33 * 64 * 320 * 16
    assert low - pivots < tall < low - pivots + low / 300  # (a row more: 1 / 320 and tables)


@pytest.mark.gpu
@pytest.mark.parametrize("imp", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_members_equal_runs(precision, imp):
    import torch
    import paper_1701_02005_amd as P
    base = dataclasses.replace(P.configs.couette_small(precision=precision), nx=12, ny=322, nz=6, implicit_xz=imp, u_noise=0.05)
    cfgs = [dataclasses.replace(base, seed=m, re=300.0 + 50 * m) for m in range(3)]
    e = P.Ensemble(cfgs)
    e.step(4)
    for m, c in enumerate(cfgs):
        s = P.Solver(c)
        s.step(4)
        for k in ("u", "v", "w", "cp", "cm", "phi", "p"):
            assert torch.equal(e.get_field(m, k), s.get_field(k)), (m, k)
