"""FP64 maps of few rows or columns, whose pixels go 64 in a row instead of in
square tiles: shapes around the tile, of scans and of visit lists, against the
oracle at the FP64 bound, with the same map a second time bit for bit."""
import numpy as np
import pytest

from gpu_util import assert_close, oracle_scan

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (63, 1), (65, 1), (1, 200), (130, 2), (2, 67), (3, 99), (1000, 1), (40, 5)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_lines(ora, shape):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd
    from paper_2507_00294_amd import workloads as wl

    w, h = shape
    for D in (2e-15, 4e-13, 3e-11):
        spec = wl.ScanSpec(17, 13, "random", 1e-9, 1e-6, 0.5e-9, D, 1.0, seed=w)
        grid = (-1.3e-9, 2.1e-9, 20e-9 / w, 11e-9 / h, w, h)
        times = [t * spec.tau_v for t in (0.0, 0.6, 1, 2.25, 100, 221, 500)]
        scan = dd.Scan(**spec.kwargs())
        got = scan.damage_map(*grid, times).cpu().numpy()
        ref = oracle_scan(ora, spec, scan).psi_map(*grid, times)
        assert_close(got, ref, spec, "fp64", f"scan {shape} D {D}")
        assert np.array_equal(scan.damage_map(*grid, times).cpu().numpy(), got)
        ids = scan.visits()
        n = len(ids)
        vis = dd.Visits((ids % 17) * 1e-9, (ids // 17) * 1e-9, np.arange(n) * spec.tau_v,
                        np.full(n, spec.tau_v), sigma_m=0.5e-9, D_m2s=D, Q0_us=1.0)
        assert_close(vis.damage_map(*grid, times).cpu().numpy(), ref, spec, "fp64",
                     f"list {shape} D {D}")
