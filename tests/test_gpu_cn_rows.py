"""The Crank-Nicolson solve at the row counts where its method and its split
of the rows change: lane scans (FP64 up to 320 rows) and slabs of rows in
registers, the edges of each slab height (4, 8, 16, 24 rows per thread, and 16
with 32-column blocks above 384 rows), whole and partial last slabs, planes
below and not a multiple of a block's columns; the plain and the
three-direction form.  FP64 against the oracle at the whole-step bar of
1e-10; mixed against it at 1e-5 (n 2^-24 over n = 6 substeps, O(1) fields)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [4, 31, 32, 33, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 384, 385, 512])
@pytest.mark.parametrize("nx,nz,imp", [(6, 4, 0), (12, 18, 1)], ids=["24cols", "216cols-implicit"])
def test_rows(oracle_mod, rows, nx, nz, imp):
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(), nx=nx, ny=rows + 1, nz=nz, dt=0.0, cfl=0.5, seed=rows,
                              u_noise=0.05, implicit_xz=imp)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(6)
    for prec, names, bar in (("fp64", ("u", "v", "w", "cp", "cm", "phi", "p"), 1e-10), ("mixed", ("u", "cp", "cm"), 1e-5)):
        g = P.Solver(dataclasses.replace(cfg, precision=prec))
        g.step(6)
        for k in names:
            a, b = g.get_field(k).cpu().numpy(), o.field(k)
            err = np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)
            assert err < bar, (prec, k, err)


# The x-lines of the three-direction form: points per lane 1 to 16, whole and
# partial lanes, lines that are no multiple of a wave's, at the same bar.
@pytest.mark.parametrize("nx", [4, 54, 64, 72, 128, 162, 192, 216, 256, 288, 486, 512, 648, 768, 972, 1024])
def test_periodic_x_lines(oracle_mod, nx):
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(), nx=nx, ny=10, nz=6, dt=0.0, cfl=0.5, seed=nx, u_noise=0.05,
                              implicit_xz=1)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(3)
    g = P.Solver(cfg)
    g.step(3)
    for k in ("u", "v", "w", "cp", "cm", "phi", "p"):
        a, b = g.get_field(k).cpu().numpy(), o.field(k)
        assert np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300) < 1e-10, k
