"""Host check (not a GPU test): a mixed arrival query whose items all run at once
sums its near band and its far region in one launch, so that it takes as long as
the longer of them; a large one, whose far region fills the chip by itself, in two."""
import fake_hip

CODE = r"""
for nx, ny, one in ((2, 2, True), (9, 7, True), (16, 16, True), (200, 200, True),
                    (400, 400, False)):
    s = scan(nx, ny, "random", seed=1)
    out = buf(nx * ny)
    launches()
    ok(lib.dd_damage_at_probe_arrival(s.handle, 1, ptr(out), 1, None))
    names = [name for name, _, _ in launches() if name.startswith("k_arrival")]
    assert len(names) == (1 if one else 2), (nx, ny, names)
"""


def test_launches(tmp_path):
    fake_hip.run(tmp_path, CODE)
