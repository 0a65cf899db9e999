"""Host check (not a GPU test): events that outlive a call (a scan's, a thread's
scratch) are last recorded on a stream that still exists when they are waited for,
also after a prediction, whose judge runs on a stream of the library's own, the
network's destruction and an autotune run."""
import fake_hip

SETUP = r"""
scans = [scan(64, 64, "random", seed=k, sigma_m=0.5e-9, D_m2s=2.5e-13) for k in range(3)]
h = (C.c_void_p * 3)(*[s.handle.value for s in scans])
out = [buf(4096) for _ in scans]
outs = (C.c_void_p * 3)(*[a.ctypes.data for a in out])
g, t = dd.Grid(0, 0, 1e-9, 1e-9, 64, 64), (C.c_double * 1)(1e-3)


def all_calls(s):
    ok(lib.dd_batch_solve(h, 3, 2, 1, outs, 1, None))
    for p in (0, 1):
        ok(lib.dd_damage_map(s.handle, C.byref(g), t, 1, p, ptr(out[0]), 1, None))
        ok(lib.dd_damage_at_probe_arrival_range(s.handle, 4000, 4096, p, ptr(out[0]), 1, None))
"""
PREDICT = r"""
for _ in range(2):
    u, psi, used = C.c_void_p(), buf(3 * 4096), np.zeros(3, np.int32)
    ok(lib.dd_unet_create(C.c_uint64(3), C.byref(u)))
    launches()
    ok(lib.dd_unet_predict(u, h, 3, C.c_double(0.02), 1, ptr(psi),
                           used.ctypes.data_as(C.POINTER(C.c_int32)), None))
    assert any("k_spot" in name for name, _, _ in launches())  # judged
    lib.dd_unet_destroy(u)
    all_calls(scans[1])
    scans[1].close()
    scans[1] = scan(64, 64, "random", seed=9)
    h[1] = scans[1].handle.value
"""
TUNE = r"""
ok(lib.dd_autotune(b"tune.json"))
all_calls(scans[0])
"""


def test_prediction_then_other_calls(tmp_path):
    fake_hip.run(tmp_path, SETUP + PREDICT)


def test_autotune_then_other_calls(tmp_path):
    fake_hip.run(tmp_path, SETUP + TUNE)
