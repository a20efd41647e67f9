"""The periodic x-lines of the three-direction form where a wave takes many
lines in turn (up to 16, two or four at a time, a partial last group and a
partial last wave) and its lanes hold 1 to 6 points, with whole and partial
lanes.  FP64 against the oracle at the whole-step bar of 1e-10, mixed against
it at 1e-5 (n 2^-24 over n = 3 substeps, O(1) fields)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(6, 206, 64), (72, 138, 96), (162, 138, 96), (256, 103, 48), (324, 69, 54)])
def test_many_lines_a_wave(oracle_mod, nx, ny, nz):
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(), nx=nx, ny=ny, nz=nz, dt=0.0, cfl=0.5, seed=nx, u_noise=0.05,
                              implicit_xz=1)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(3)
    for prec, names, bar in (("fp64", ("u", "v", "w", "cp", "cm", "phi", "p"), 1e-10), ("mixed", ("u", "cp", "cm"), 1e-5)):
        g = P.Solver(dataclasses.replace(cfg, precision=prec))
        g.step(3)
        for k in names:
            a, b = g.get_field(k).cpu().numpy(), o.field(k)
            err = np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)
            assert err < bar, (prec, k, err)
