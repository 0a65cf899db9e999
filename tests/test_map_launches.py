"""Host check (not a GPU test): a mixed map call runs its far and its near-band
items in one launch, so that a small call takes as long as the longer of them."""
import fake_hip

CODE = r"""
for side, w, h, n_t in ((8, 16, 16, 1), (40, 64, 64, 7), (128, 16, 16, 1), (64, 128, 128, 64)):
    s = scan(side, side, "random", seed=1)
    g, out = dd.Grid(0, 0, 5e-10, 5e-10, w, h), buf(n_t * w * h)
    t = (C.c_double * n_t)(*[side * side * 1e-6 * (k + 1) / n_t for k in range(n_t)])
    launches()
    ok(lib.dd_damage_map(s.handle, C.byref(g), t, n_t, 1, ptr(out), 1, None))
    names = [name for name, _, _ in launches() if name.startswith("k_map")]
    assert len(names) == 1, names
"""


def test_one_launch(tmp_path):
    fake_hip.run(tmp_path, CODE)
