"""The row marches (explicit kernel, limited advection, projection correction)
take fewer rows per block on small grids: whatever the rows per block, one to
a whole column, the results are the same bit for bit."""
import dataclasses

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("face", [0, 2])
@pytest.mark.parametrize("nx,ny,nz", [(16, 17, 12), (48, 27, 36), (6, 65, 4), (96, 33, 64)])
def test_rows_per_block_are_bitwise_neutral(nx, ny, nz, face, precision):
    import torch
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(precision=precision), nx=nx, ny=ny, nz=nz, dt=0.0, cfl=0.5,
                              u_noise=0.05, migration_face=face, seed=4)
    fields = []
    for slab in (None, 1, 5, 512):
        s = P.Solver(cfg)
        if slab:
            s.set_tiles(slab=slab)
        s.step(6)
        fields.append([s.get_field(k) for k in ("u", "v", "w", "cp", "cm", "phi", "p")])
    for other in fields[1:]:
        for a, b in zip(fields[0], other):
            assert torch.equal(a, b)


# The mixed form's limited flux inside the explicit kernel (its three tiles)
# and, with 64 threads a block on lines of 64 and 48, in a pass of its own.
@pytest.mark.parametrize("nx,ny,nz", [(64, 5, 4), (48, 6, 6), (64, 33, 18), (48, 18, 12), (96, 9, 8), (128, 12, 6)])
def test_limited_flux_in_the_explicit_kernel(nx, ny, nz):
    import torch
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(precision="mixed"), nx=nx, ny=ny, nz=nz, dt=0.0, cfl=0.5,
                              u_noise=0.2, c_noise=0.2, migration_face=2, seed=6)
    fields = []
    for threads in (256, 64):
        s = P.Solver(cfg)
        s.set_tiles(expl=threads)
        s.step(6)
        fields.append([s.get_field(k) for k in ("u", "v", "w", "cp", "cm", "phi", "p")])
    for a, b in zip(*fields):
        assert torch.equal(a, b)
