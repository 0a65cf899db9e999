"""Host check (not a GPU test): one thread queries scans on one device and then on
another, and back, as a program with a device per scan does."""
import fake_hip
import pytest

CODE = r"""
g, t, out = dd.Grid(0, 0, 1e-9, 1e-9, 64, 64), (C.c_double * 1)(1e-3), buf(64 * 64)
calls = {
    "map": lambda h: lib.dd_damage_map(h, C.byref(g), t, 1, 0, ptr(out), 1, None),
    "sweep": lambda h: lib.dd_damage_sweep(h, C.byref(g), 0.0, 1e-3, 1, 0, ptr(out), 1, None),
    "range": lambda h: lib.dd_damage_at_probe_arrival_range(h, 900, 1024, 1, ptr(out), 1, None),
}
call = calls["%s"]
scans = [scan(32, 32, "random", seed=k) for k in range(2)]
for dev in (0, 1, 0, 1):
    fake.fake_set_device(dev)
    for _ in range(2):
        ok(call(scans[dev].handle))
"""


@pytest.mark.parametrize("call", ["map", "sweep", "range"])
def test_two_devices(tmp_path, call):
    fake_hip.run(tmp_path, CODE % call)


UNET = r"""
u = C.c_void_p()
ok(lib.dd_unet_create(C.c_uint64(3), C.byref(u)))
n = lib.dd_unet_num_params(u)
m, step = np.zeros(n, np.float32), C.c_int64()
for dev in (0, 1, 0):
    fake.fake_set_device(dev)
    p = np.zeros(n, np.float32)
    ok(lib.dd_unet_params(u, ptr(p), None))
    assert p.any()
    ok(lib.dd_unet_grads(u, ptr(m)))
    ok(lib.dd_unet_adam_state(u, ptr(m), None, C.byref(step), None, None, None))
"""


def test_network_reads_from_another_device(tmp_path):
    fake_hip.run(tmp_path, UNET)
