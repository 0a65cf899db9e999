"""Host check (not a GPU test): the device scratch of a batch of FP64 final maps is
bounded, whatever the number of scans, beside what the scans themselves hold."""
import fake_hip

CODE = r"""
def peak(n):
    scans = [scan(128, 128, "raster", D_m2s=1e-13 * (k + 1)) for k in range(n)]
    outs = [buf(128 * 128) for _ in range(n)]
    for s in scans:  # the scans' own tables
        ok(lib.dd_damage_at_probe_arrival(s.handle, 0, ptr(outs[0]), 1, None))
    launches()
    fake.fake_peak(1)
    base = fake.fake_peak(0)
    hs = (C.c_void_p * n)(*[s.handle.value for s in scans])
    ps = (C.c_void_p * n)(*[o.ctypes.data for o in outs])
    ok(lib.dd_batch_solve(hs, n, 2, 0, ps, 1, None))
    maps = [(name, x, y) for name, x, y in launches() if "gauss_map" in name]
    assert sum(x for _, x, _ in maps) == n, maps
    return fake.fake_peak(1) - base
small, large = peak(16), peak(96)
print(small, large)
# at most 2^25 partial sums, and the call's tables
assert large < 8 * 2 ** 25 + 2 ** 24, (small, large)
"""


def test_fp64_maps(tmp_path):
    print(fake_hip.run(tmp_path, CODE))
