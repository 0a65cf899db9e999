"""Host check (not a GPU test) of the tiles of FP64 maps: whatever the shape of the
maps, the tiles of a call that fills the chip hold at most a few times its pixels
(or are one tile a map), read off the kernel that is launched."""
import fake_hip
import pytest

SHAPES = [(4096, 1), (1, 4096), (100000, 1), (2048, 2), (2, 2048), (3, 700), (512, 8), (8, 512),
          (300, 20), (8, 8), (64, 64), (128, 128), (97, 101), (1000, 1000)]

CODE = r"""
import re
w, h = %r
def padded(F):
    return 128 * -(-w * h // 128) if F == 0 else (16 * F) ** 2 * -(-w // (16 * F)) * -(-h // (16 * F))
def check(what):
    F = {int(re.search(r"k_gauss_mapILi(\d)E", name).group(1)) for name, _, _ in launches()
         if "k_gauss_map" in name}
    assert len(F) == 1, (what, F)
    assert padded(max(F)) <= max(6 * w * h, 256), (what, F)
s = scan(64, 64, "random", seed=1)
n = 4096
i = np.arange(n)
v = dd.Visits((i %% 64) * 1e-9, (i // 64) * 1e-9, i * 1e-6, np.full(n, 1e-6))
g = dd.Grid(0, 0, 64e-9 / w, 64e-9 / h, w, h)
for n_t in (4 if w * h > 50000 else 64,):
    t, out = (C.c_double * n_t)(*[(k + 1) * 64e-6 for k in range(n_t)]), buf(n_t * w * h)
    ok(lib.dd_damage_map(s.handle, C.byref(g), t, n_t, 0, ptr(out), 1, None))
    check(("scan", n_t))
    ok(lib.dd_visits_map(v._h, C.byref(g), t, n_t, 0, ptr(out), 1, None))
    check(("visits", n_t))
"""


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_tiles_fit(tmp_path, shape):
    fake_hip.run(tmp_path, CODE % (shape,))


RECENT = r"""
import re
side, w, h, n_t, tiles, least = %r
s = scan(side, side, "random", seed=1)
V = side * side
g, out = dd.Grid(0, 0, 1e-9, 1e-9, w, h), buf(n_t * w * h)
t = (C.c_double * n_t)(*[V * 1e-6 * (k + 1) / n_t for k in range(n_t)])
ok(lib.dd_damage_map(s.handle, C.byref(g), t, n_t, 0, ptr(out), 1, None))
blocks = [(x, y) for name, x, y in launches() if "k_gauss_map" in name]
assert len(blocks) == 1 and blocks[0][0] == n_t, blocks
# chunks of 2, 2, 4, .. 32 recent visits beside those of older ones
assert 4 * blocks[0][1] / tiles >= least, blocks
"""


@pytest.mark.parametrize("case", [(64, 33, 33, 256, 1, 69), (64, 48, 48, 256, 1, 69),
                                  (128, 33, 33, 256, 1, 38), (64, 128, 128, 512, 4, 10),
                                  (64, 100, 30, 16, 4, 69), (16, 64, 64, 256, 4, 9)],
                         ids=lambda c: "-".join(map(str, c)))
def test_recent_visits_split(tmp_path, case):
    """The most recent visits take most nodes: they are spread over waves in every
    call whose maps alone do not fill the chip many times over."""
    fake_hip.run(tmp_path, RECENT % (case,))
