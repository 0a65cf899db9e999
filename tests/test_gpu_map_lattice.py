"""Mixed maps on fine and far pixel lattices, where |e|^2 + |p|^2 comes close to
what a single-precision sum holds exactly: the squared distances of the matrix
cores split |p|^2 into 4096 sh + sl, whose first part may exceed it.  Against the
oracle at the mixed bound, and bit for bit between the tile widths, the narrowest
of which forms its distances without the matrix cores.  The pitch is a power of
two, so that pixel coordinates over pitch are what is written here."""
import json

import numpy as np
import pytest

from gpu_util import assert_close, oracle_scan

pytestmark = pytest.mark.gpu

PITCH = 2.0 ** -30
# (probes a side, pixel spacing, first pixel, pixels a side, kappa): grids at the bound
# with sh > 0, the far corner of the probes in the map, a negative corner
GRIDS = [(33, 1 / 64, 30.0, 63, 0.1), (33, 1 / 32, 83.0, 54, 2.0), (64, 1 / 16, 168.0, 26, 2.0),
         (64, 1 / 32, 62.0, 64, 0.1), (40, 1 / 16, -175.0, 40, 10.0), (33, 1 / 32, 0.0, 70, 0.5)]


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: f"{g[0]}-{g[1]}-{g[2]}")
def test_map_lattice(ora, tmp_path, grid):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd
    from paper_2507_00294_amd import workloads as wl

    side, px, x0, n, kappa = grid
    spec = wl.ScanSpec(side, side, "random", PITCH, 1e-6, 0.5 * PITCH, kappa * PITCH ** 2 / 1e-6,
                       1.0, seed=side)
    g = (x0 * PITCH, x0 * PITCH, px * PITCH, px * PITCH, n, n)
    V = spec.n_visits
    times = [t * spec.tau_v for t in (3, V / 3 + 0.25, V)]
    scan = dd.Scan(**spec.kwargs())
    shapes = {"arch": "gfx950", "arrival_mixed": {"R": 4, "RN": 2, "K": 2048},
              "arrival_fp64": {"R": 2, "RN": 2, "K": 1024}, "map_mixed": {"R": 4, "K": 4096},
              "map_fp64": {"R": 1}}
    path = tmp_path / "tune.json"
    got = {}
    try:
        for R in (1, 2, 4):
            path.write_text(json.dumps(dict(shapes, map_mixed={"R": R, "K": 4096})))
            dd.tune_load(str(path))
            got[R] = scan.damage_map(*g, times, "mixed").cpu().numpy()
    finally:
        path.write_text(json.dumps(shapes))
        dd.tune_load(str(path))
    assert_close(got[4], oracle_scan(ora, spec, scan).psi_map(*g, times), spec, "mixed", str(grid))
    for R in (1, 2):
        assert np.array_equal(got[R], got[4]), f"{grid}, R {R}"
