"""The values of the mixed arrival query do not depend on how its far sums are
laid out over lanes and launches: whole queries, ranges and batches against
values recorded from the form that summed a group's lags from registers, for
both tile widths, every visit order and every form of the far series.

Tolerance: the terms and their FP32 sums over a group of lags are the same
operations with the same roundings; only the order of the FP64 sums may differ,
up to 1e4 additions of positive terms, 1e4 * 1.1e-16 = 1.1e-12 relative."""
import json
import pathlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GOLDEN = json.loads((pathlib.Path(__file__).parent / "golden/mixed_arrival.json").read_text())
RTOL = 1.1e-12


@pytest.mark.parametrize("R", [4, 2])
def test_recorded_sums(tmp_path, R):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd

    shapes = {"arch": "gfx950", "arrival_mixed": {"R": R, "RN": 2, "K": 2048},
              "arrival_fp64": {"R": 2, "RN": 2, "K": 1024}, "map_mixed": {"R": 4, "K": 4096},
              "map_fp64": {"R": 1}}
    path = tmp_path / "tune.json"
    path.write_text(json.dumps(shapes))
    dd.tune_load(str(path))
    try:
        scans = [dd.Scan(**c["scan"]) for c in GOLDEN["cases"]]
        batch = dd.batch_solve(scans, dd.Q_ARRIVAL, "mixed")
        for c, s, b in zip(GOLDEN["cases"], scans, batch):
            at = np.array(c["visits"])
            want = np.array([float.fromhex(v) for v in c[f"R{R}"]])
            for what, got in (("query", s.arrival("mixed")), ("batch", b)):
                np.testing.assert_allclose(got.cpu().numpy()[at], want, rtol=RTOL, atol=0,
                                           err_msg=f"{what} {c['scan']}")
            j0 = s.num_visits // 2 + 3
            part = s.arrival_range(j0, s.num_visits, "mixed").cpu().numpy()
            want = np.array([float.fromhex(v) for v in c[f"range{R}"]])
            np.testing.assert_allclose(part[at[at >= j0] - j0], want, rtol=RTOL, atol=0,
                                       err_msg=f"range {c['scan']}")
    finally:
        path.write_text(json.dumps(dict(shapes, arrival_mixed={"R": 4, "RN": 2, "K": 2048})))
        dd.tune_load(str(path))
