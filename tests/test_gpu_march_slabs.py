"""Row marches over long slabs: on planes whose column tiles alone fill the chip
a block of the explicit kernel marches up to the rows it is given, and the
limiter's pass 32, with what they carry from row to row (the two-row ring, the
ions of two rows below, the window of five rows).  256 x 256 columns, 65 rows:
slabs of 1, 5, 16 and 32 rows (whole and partial) agree bit for bit, and the
mixed form's limited flux inside the explicit kernel with its pass; 33 rows
with the limiter against the oracle, FP64 at the whole-step bar of 1e-10,
mixed at 1e-5 (n 2^-24 over n = 3 substeps, O(1) fields)."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FIELDS = ("u", "v", "w", "cp", "cm", "phi", "p")


def config(P, rows, **kw):
    return dataclasses.replace(P.configs.couette_small(), nx=256, ny=rows + 1, nz=256, dt=0.0, cfl=0.5, u_noise=0.2,
                               c_noise=0.2, seed=9, **kw)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("face", [0, 2])
def test_rows_per_block(face, precision):
    import torch
    import paper_1701_02005_amd as P
    cfg = config(P, 65, migration_face=face, precision=precision)
    shapes = [dict(slab=1), dict(slab=5), dict(slab=16), dict(slab=32)]
    if precision == "mixed" and face == 2:
        shapes.append(dict(expl=64))  # the limiter in a pass of its own
    ref = None
    for shape in shapes:
        s = P.Solver(cfg)
        s.set_tiles(**shape)
        s.step(4)
        got = [s.get_field(k) for k in FIELDS]
        del s
        ref = ref or got
        assert all(torch.equal(a, b) for a, b in zip(got, ref)), shape


def test_limited_slabs_against_the_oracle(oracle_mod):
    import paper_1701_02005_amd as P
    cfg = config(P, 33, migration_face=2)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(3)
    for prec, names, bar in (("fp64", FIELDS, 1e-10), ("mixed", ("u", "cp", "cm"), 1e-5)):
        s = P.Solver(dataclasses.replace(cfg, precision=prec))
        s.step(3)
        for k in names:
            a, b = s.get_field(k).cpu().numpy(), o.field(k)
            err = np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300)
            assert err < bar, (prec, k, err)
