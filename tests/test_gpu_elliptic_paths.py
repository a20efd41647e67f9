"""The elliptic solve on the paths that its sizes choose: whole-plane
transforms (planes of up to two blocks per CU's LDS) and their limit, radices
2, 3, 4 and 8 in either direction, lines of 64 to 512 points (1, 2 or 4 a wave),
groups of 16, 32 and 64 lanes per mode, and,
for caller-owned right-hand sides and above 320 rows, slabs of rows in
registers at the edges of every slab height.  Against the oracle.  Bar: the
wall-normal operator's condition number, about 1e6 on 512 stretched rows,
times the unit roundoff, 1e-10 (the whole-step parity bar)."""
import dataclasses

import numpy as np
import pytest

from inputs import random_field

pytestmark = pytest.mark.gpu


def config(P, nx, ny, nz):
    return dataclasses.replace(P.configs.couette_small(), nx=nx, ny=ny, nz=nz, dt=0.0, cfl=0.5, u_noise=0.05, seed=3)


def check_solve(P, O, cfg):
    import torch
    o = O.Oracle(**cfg.oracle_kwargs())
    s = P.Solver(cfg)
    for kind in (0, 1):
        rhs = random_field(o.shape, 5 + kind)
        if kind == 0:
            vol = o.dn[:, None, None] * np.ones(o.shape)
            rhs -= np.sum(rhs * vol) / np.sum(vol)
        ref = o.poisson(kind, rhs)
        t = torch.tensor(rhs, dtype=torch.float64, device="cuda")
        for out in (s.poisson_solve(kind, t), P.poisson_solve_noalloc(cfg, kind, t)):
            err = np.max(np.abs(out.cpu().numpy() - ref)) / np.max(np.abs(ref))
            assert err < 1e-10, (kind, err)


@pytest.mark.parametrize("nx,nz", [(4, 4), (6, 4), (4, 54), (16, 12), (48, 48), (64, 64), (36, 108), (64, 72), (128, 32), (256, 18), (512, 4),
                                   (4, 512), (768, 4), (256, 54), (512, 54), (54, 256), (36, 512), (1024, 6),
                                   (64, 162), (162, 64), (64, 256), (256, 64), (128, 108), (108, 128), (128, 128)])
def test_plane_transforms(oracle_mod, nx, nz):
    import paper_1701_02005_amd as P
    check_solve(P, oracle_mod, config(P, nx, 9, nz))


@pytest.mark.parametrize("rows", [4, 16, 17, 32, 33, 64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512])
def test_rows_in_registers(oracle_mod, rows):
    import paper_1701_02005_amd as P
    check_solve(P, oracle_mod, config(P, 18, rows + 1, 6))  # 60 modes: a block and a part


@pytest.mark.parametrize("rows", [15, 16, 17, 31, 32, 33, 320, 321])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_runs_across_the_row_limits(oracle_mod, rows, precision):
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(config(P, 12, rows + 1, 18), precision=precision)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(6)
    s = P.Solver(cfg)
    s.step(6)
    for k in ("u", "v", "w", "cp", "cm", "phi", "p") if precision == "fp64" else ("u", "cp", "cm"):
        a, b = s.get_field(k).cpu().numpy(), o.field(k)
        err = np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)
        assert err < (1e-10 if precision == "fp64" else 1e-5), (k, err)


# Members of an ensemble large enough for the columns in registers (up to 64
# rows, a partial group of members and of modes) against runs of their own,
# which stay lane-split: the same operations in the same order.
@pytest.mark.parametrize("rows", [4, 7, 8, 9, 15, 16, 17, 32, 33, 48, 49, 63, 64, 65])
def test_columns_of_an_ensemble(rows):
    import numpy as np
    import paper_1701_02005_amd as P
    base = config(P, 96, rows + 1, 54)  # 2646 modes: 165 tiles of 16 and a part
    cfgs = [dataclasses.replace(base, seed=3 + m, re=300.0 + 50.0 * m, u_noise=0.05) for m in range(7)]
    e = P.Ensemble(cfgs)
    e.step(2)
    e.sync()
    for m in (0, 3, 4, 6):
        s = P.Solver(cfgs[m])
        s.step(2)
        for k in ("u", "v", "w", "cp", "cm", "phi", "p"):
            a, b = e.get_field(m, k).cpu().numpy(), s.get_field(k).cpu().numpy()
            assert np.array_equal(a, b), (m, k, np.max(np.abs(a - b)))
