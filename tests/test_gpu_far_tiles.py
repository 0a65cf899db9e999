"""The mixed arrival query's far region (distances as 4x4 matrix-core blocks,
lags slanted over a block's columns): visit counts around its tiles (64 R
visits, R = 2 and 4), ranges with short lag chunks, and probes over the whole
2048x2048 lattice, against the oracle at the mixed bound and bit for bit
between the whole query, the batch and a repeat."""

import numpy as np
import pytest

from gpu_util import assert_close, oracle_scan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [2, 4])
def test_far_tiles(ora, tmp_path, R):
    import json

    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd
    from paper_2507_00294_amd import workloads as wl

    shapes = {"arch": "gfx950", "arrival_mixed": {"R": R, "RN": 2, "K": 2048},
              "arrival_fp64": {"R": 2, "RN": 2, "K": 1024}, "map_mixed": {"R": 4, "K": 4096},
              "map_fp64": {"R": 1}}
    default = dict(shapes, arrival_mixed={"R": 4, "RN": 2, "K": 2048})
    rng = np.random.default_rng(3)
    specs = [wl.ScanSpec(40, 40, "explicit", 1e-9, 1e-6, 0.5e-9, D, 1.0,
                         visits=[int(v) for v in rng.integers(0, 1600, n)])
             for n, D in ((63, 1e-11), (64, 1e-11), (127, 3e-12), (129, 1e-11), (255, 1e-12),
                          (256, 1e-12), (257, 3e-11), (515, 1e-10), (1021, 1e-11))]
    corners = [0, 2047, 2047 * 2048, 2048 * 2048 - 1]
    specs.append(wl.ScanSpec(2048, 2048, "explicit", 1e-9, 1e-6, 0.5e-9, 1e-8, 1.0,
                             visits=corners + [int(v) for v in rng.integers(0, 2048 ** 2, 600)] +
                             corners))
    path = tmp_path / "tune.json"
    path.write_text(json.dumps(shapes))
    dd.tune_load(str(path))
    try:
        scans = [dd.Scan(**s.kwargs()) for s in specs]
        outs = dd.batch_solve(scans, dd.Q_ARRIVAL, "mixed")
        for spec, s, o in zip(specs, scans, outs):
            got = s.arrival("mixed").cpu().numpy()
            assert_close(got, oracle_scan(ora, spec, s).psi_arrival(), spec, "mixed",
                         f"{spec.n_visits} visits, R {R}")
            assert np.array_equal(o.cpu().numpy(), got)
            assert np.array_equal(s.arrival("mixed").cpu().numpy(), got)
            V = spec.n_visits
            rng_ = s.arrival_range(V // 3, V, "mixed").cpu().numpy()
            assert_close(rng_, got[V // 3:], spec, "mixed", f"range of {V}, R {R}")
    finally:
        path.write_text(json.dumps(default))
        dd.tune_load(str(path))


# (scan side, pixel spacing in pitches, first pixel, w, h): one row; lattices whose
# pixel coordinates are half-precision values and, with 12 bits, are not; negative
# coordinates; far and near bands with remainders of four lags
GRIDS = [(5, 0.5, 0.0, 37, 1), (12, 1 / 256, 0.0, 61, 45), (15, 1 / 256, 15 - 60 / 256, 70, 66),
         (24, 0.25, -8.0, 130, 50), (33, 1.0, 3.0, 9, 31)]


@pytest.mark.parametrize("R", [1, 2, 4])
def test_map_tiles(ora, tmp_path, R):
    import json

    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd
    from paper_2507_00294_amd import workloads as wl

    shapes = {"arch": "gfx950", "arrival_mixed": {"R": 4, "RN": 2, "K": 2048},
              "arrival_fp64": {"R": 2, "RN": 2, "K": 1024}, "map_mixed": {"R": 4, "K": 4096},
              "map_fp64": {"R": 1}}
    path = tmp_path / "tune.json"

    def maps(width):
        path.write_text(json.dumps(dict(shapes, map_mixed={"R": width, "K": 4096})))
        dd.tune_load(str(path))
        out = []
        for side, px, x0, w, h in GRIDS:
            spec = wl.ScanSpec(side, side, "random", 1e-9, 1e-6, 0.5e-9, 5e-13, 1.0, seed=side)
            grid = (x0 * 1e-9, x0 * 1e-9, px * 1e-9, px * 1e-9, w, h)
            V = spec.n_visits
            times = [t * spec.tau_v for t in (0.5, 3, 1 + V // 3, V - 0.25, V, 2 * V + 0.5)]
            scan = dd.Scan(**spec.kwargs())
            out.append((spec, scan, grid, times,
                        scan.damage_map(*grid, times, "mixed").cpu().numpy()))
        return out

    try:
        widest = maps(4)
        for (spec, scan, grid, times, got), ref in zip(maps(R), widest):
            want = oracle_scan(ora, spec, scan).psi_map(*grid, times)
            assert_close(got, want, spec, "mixed", f"{spec.nx} {grid}, R {R}")
            assert np.array_equal(got, ref[4]), f"{spec.nx} {grid}, R {R}"
    finally:
        path.write_text(json.dumps(shapes))
        dd.tune_load(str(path))
