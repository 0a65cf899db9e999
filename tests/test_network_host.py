"""Host check (not a GPU test) of the network's training pass: buffers, tables and
launches for batches that grow, shrink and grow, with the gradients read back.  Its
host arithmetic is what the sanitizer build checks."""
import fake_hip

CODE = r"""
u = C.c_void_p()
ok(lib.dd_unet_create(C.c_uint64(3), C.byref(u)))
g = np.zeros(lib.dd_unet_num_params(u), np.float32)
for B in (3, 1, 48, 7):
    x, y = np.zeros(B * 4096 * dd.CHANNELS, np.float32), np.zeros(B * 4096, np.float32)
    ok(lib.dd_unet_forward(u, B, ptr(x), ptr(y), 1, None))
    launches()
    ok(lib.dd_unet_backward(u, ptr(x), ptr(y), None))
    names = [name for name, _, _ in launches()]
    assert sum("k_act_bwd" in n for n in names) == 14 and sum("k_wgrad" in n for n in names) == 14
    assert sum("k_sum_parts" in n for n in names) == 1
    ok(lib.dd_unet_grads(u, ptr(g)))
lib.dd_unet_destroy(u)
"""


def test_training_pass(tmp_path):
    fake_hip.run(tmp_path, CODE)
