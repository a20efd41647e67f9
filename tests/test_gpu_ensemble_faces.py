"""Members that differ in the face values of the ions: each gives what a run
of its own gives, bit for bit, whichever of them comes first."""
import dataclasses

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("faces", [(0, 2, 1, 2), (2, 0, 2, 1)], ids=str)
def test_members_with_other_face_values(faces, precision):
    import torch
    import paper_1701_02005_amd as P
    base = dataclasses.replace(P.configs.couette_small(precision=precision), nx=24, ny=17, nz=18, vhat=30.0, debye=0.1,
                               u_noise=0.2, c_noise=0.2)
    cfgs = [dataclasses.replace(base, migration_face=f, seed=m) for m, f in enumerate(faces)]
    e = P.Ensemble(cfgs)
    e.capture(3)
    e.step(6)
    for m, c in enumerate(cfgs):
        s = P.Solver(c)
        s.step(6)
        for k in ("u", "v", "w", "cp", "cm", "phi", "p"):
            assert torch.equal(e.get_field(m, k), s.get_field(k)), (m, k)
