"""The tuner tries the shapes that a kernel reads at the sizes at hand and no
others: its trials, two of the start and two per candidate (the default again
where another beat it), show in the substeps that it took."""
import dataclasses

import pytest

pytestmark = pytest.mark.gpu

# candidates besides the default: explicit threads 2, correction threads 1 and
# slab rows 3 always; CN threads 3; x and z transform points 2 each; mode tiles
# 3 and the fused marches 1; CN methods 2
CASES = {
    # whole planes, a plane of few columns
    "planes": (dict(nx=16, ny=17, nz=12), 2 + 1 + 3 + 4 + 2),
    # a wave per line both ways; the mixed form's CN solve has no tiles of threads
    "lines": (dict(nx=256, ny=9, nz=64, precision="mixed"), 2 + 1 + 3 + 4 + 2),
    # transforms in LDS tiles; above 320 rows no mode tiles, above 384 one CN method
    "tall": (dict(nx=96, ny=386, nz=54), 2 + 1 + 3 + 2 + 2 + 1),
    # every shape
    "all": (dict(nx=72, ny=65, nz=72), 2 + 1 + 3 + 3 + 2 + 2 + 4 + 2),
}


@pytest.mark.parametrize("case", CASES)
def test_trials(case):
    import paper_1701_02005_amd as P
    sizes, candidates = CASES[case]
    s = P.Solver(dataclasses.replace(P.configs.couette_small(), dt=1e-5, **sizes))
    tiles, default = s.autotune(None, 3), P.Solver(dataclasses.replace(P.configs.couette_small(), **sizes)).tiles()
    read = {"planes": ("thomas", "cnslab"), "lines": ("thomas", "cnslab"), "tall": ("fftx", "fftz", "thomas"),
            "all": ("cn", "fftx", "fftz", "thomas", "cnslab")}[case] + ("expl", "corr", "slab")
    trials = s.clock()[3] // 3
    assert 2 * (1 + candidates) <= trials <= 2 * (1 + candidates + len(read))
    assert all(tiles[k] == default[k] for k in tiles if k not in read)


def test_limited_runs_have_shapes_of_their_own(tmp_path):
    """The mixed form's limited flux is formed in the explicit kernel on some
    tiles and in a pass of its own on others: shapes tuned without it are not
    taken over."""
    import paper_1701_02005_amd as P
    cache = tmp_path / "shapes.txt"
    base = dataclasses.replace(P.configs.couette_small(precision="mixed"), nx=64, ny=9, nz=8)
    for face, lines in ((0, 1), (1, 1), (2, 2), (2, 2)):
        P.Solver(dataclasses.replace(base, migration_face=face)).autotune(str(cache), 3)
        keys = [line.split()[0] for line in cache.read_text().splitlines()]
        assert len(keys) == lines == len(set(keys)), (face, keys)
