"""The Crank-Nicolson lane scans' tiles of 16 and 32 columns, on planes with
enough columns that the number of threads is read (1944 columns: a part of a
tile of 16 and of 32), for 1 to 5 rows per lane, 16 and 32 lanes a column and
tiles above 64 KB of LDS: every number of threads gives the same bit for bit,
and the 32-column tiles agree with the oracle at the whole-step bar of 1e-10."""
import dataclasses

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
FIELDS = ("u", "v", "w", "cp", "cm", "phi", "p")


@pytest.mark.parametrize("imp", [0, 1], ids=["plain", "implicit"])
@pytest.mark.parametrize("rows", [15, 31, 64, 65, 129, 193, 257, 320])
def test_threads(oracle_mod, rows, imp):
    import torch
    import paper_1701_02005_amd as P
    cfg = dataclasses.replace(P.configs.couette_small(), nx=54, ny=rows + 1, nz=36, dt=0.0, cfl=0.5, seed=rows,
                              u_noise=0.05, implicit_xz=imp)
    o = oracle_mod.Oracle(**cfg.oracle_kwargs())
    o.init(cfg.seed, cfg.u_noise, cfg.c_noise)
    o.run(3)
    ref = None
    for threads in (512, 64, 128, 256):
        s = P.Solver(cfg)
        s.set_tiles(cn=threads)
        s.step(3)
        got = [s.get_field(k) for k in FIELDS]
        if ref is None:
            for k, a in zip(FIELDS, got):
                b = o.field(k)
                assert np.max(np.abs(a.cpu().numpy() - b)) / max(np.max(np.abs(b)), 1e-300) < 1e-10, k
        ref = ref or got
        assert all(torch.equal(a, b) for a, b in zip(got, ref)), threads
