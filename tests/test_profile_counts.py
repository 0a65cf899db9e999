"""Host check (not a GPU test): the kernel statistics count the pairs of the near
band and of the far region apart, also where one launch sums both: the ranges of a
scan together count what they evaluate, every (evaluation point, earlier visit) pair
once, and the near band's share is neither nothing nor everything."""
import fake_hip

CODE = r"""
s = scan(64, 64, "random", seed=1)
V = 64 * 64
out = buf(V)
for p in (0, 1):
    for j0, j1 in ((0, V), (V - 1024, V), (1024, 2048)):
        ok(lib.dd_profiling(1))
        ok(lib.dd_damage_at_probe_arrival_range(s.handle, j0, j1, p, ptr(out), 1, None))
        ok(lib.dd_profiling(0))
        near, far = dd.KernelStats(), dd.KernelStats()
        ok(lib.dd_profile_read(b"arrival_near", C.byref(near), 1))
        ok(lib.dd_profile_read(b"arrival_far", C.byref(far), 1))
        want = sum(range(j0, j1))  # whole tiles of visits
        assert abs(near.pairs + far.pairs - want) <= 0.01 * want + 64 * V, (
            p, j0, j1, near.pairs, far.pairs, want)
        assert near.pairs > 0 and near.flops > 0 and far.pairs > 0 and far.flops > 0, (p, j0, j1)
"""


def test_counts(tmp_path):
    fake_hip.run(tmp_path, CODE)
