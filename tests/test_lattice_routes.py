"""Host check (not a GPU test) of which FP64 arrival queries run as sums over rasters:
those whose table is worth it, and none whose launch a grid cannot hold."""
import fake_hip
import pytest

# nx, ny, order, stride, frames, runs as sums
CASES = [(64, 64, "raster", 1, 1, True), (1, 2048, "raster", 1, 1, True),
         (64, 64, "interleaved", 8, 1, True), (64, 256, "interleaved", 8, 1, True),
         (256, 256, "interleaved", 8, 1, True), (128, 1024, "interleaved", 8, 1, True),
         (8, 1024, "interleaved", 8, 1, False), (8, 2048, "interleaved", 8, 1, False),
         (32, 2048, "interleaved", 8, 1, False), (6, 2048, "interleaved", 6, 1, False),
         (1, 256, "multiframe", 1, 1024, True), (1, 2048, "multiframe", 1, 64, True),
         (1, 16, "multiframe", 1, 2 ** 20, False)]

CODE = r"""
nx, ny, order, stride, frames, sums = %r
s = scan(nx, ny, order, stride=stride, frames=frames)
out = buf(s.num_visits)
ok(lib.dd_damage_at_probe_arrival(s.handle, 0, ptr(out), 1, None))
names = [name for name, _, _ in launches()]
assert any("k_lat_terms" in n for n in names) == sums, names
assert any("k_arrival" in n for n in names) != sums, names
"""


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_route(tmp_path, case):
    fake_hip.run(tmp_path, CODE % (case,))
