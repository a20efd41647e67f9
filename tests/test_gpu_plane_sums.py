"""The plane reductions at the edges of their split of a row into blocks (one
block for small planes, partial last blocks, many rows): wall stresses, ion
fluxes and contents, kinetic energy, minima and the energy budget against the
oracle after 3 substeps, at the 1e-10 of whole-step parity (fluxes and budget
relative to their largest value)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("face", [0, 2])
@pytest.mark.parametrize("nx,ny,nz", [(4, 5, 6), (16, 17, 32), (36, 9, 32), (54, 40, 96), (12, 513, 6), (288, 9, 12), (1024, 6, 4)])
def test_against_oracle(oracle_mod, nx, ny, nz, face):
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(), nx=nx, ny=ny, nz=nz, dt=0.0, cfl=0.5, u_noise=0.05, seed=8,
                              migration_face=face)
    g = P.Solver(cfg)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    g.step(3)
    o.run(3)
    assert np.allclose(g.wall_shear_stress(), o.wall_shear(), rtol=1e-10, atol=0)
    jp, jm, mp, mm = g.ion_flux()
    ojp, ojm, omp, omm = o.ion_flux()
    scale = max(np.max(np.abs(ojp)), np.max(np.abs(ojm)))
    assert np.max(np.abs(np.array(jp) - ojp)) < 1e-10 * scale and np.max(np.abs(np.array(jm) - ojm)) < 1e-10 * scale
    assert abs(mp - omp) < 1e-12 * omp and abs(mm - omm) < 1e-12 * omm
    d = g.diagnostics()
    cp, cm = o.field("cp"), o.field("cm")
    assert abs(d["ke"] - o.kinetic_energy()) < 1e-12 * o.kinetic_energy() and d["max_div"] < 1e-11
    for name, ref in (("min_cp", cp.min()), ("min_cm", cm.min()), ("max_csum", (cp + cm).max())):
        assert abs(d[name] - ref) < 1e-10 * abs(ref), name
    got, ref = list(g.energy_budget().values()), o.energy_terms()
    assert np.max(np.abs(np.array(got) - ref)) < 1e-10 * np.max(np.abs(ref))
