"""Training batches whose pixel counts do not fill the weight gradient's tiles or
share them unevenly: 1 to 7 maps (the 8x8 level has 64 to 448 pixels against
256-pixel tiles), and a batch after a larger one.  Every gradient group
against the BF16-emulating reference at the bounds of the element-wise parity
test (FP32 accumulation and rare BF16 roundings to the other side), and
bitwise the same on a second pass."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
TOL_G, TOL_G_NORM = 1e-2, 5e-3


@pytest.mark.parametrize("batches", [(1,), (2,), (3,), (5,), (7, 3)])
def test_ragged_batches(batches):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd
    from oracle import unet_ref as R

    rng = np.random.default_rng(sum(batches))
    net = dd.UNet(3)
    p = net.params()
    p[-33:] = rng.normal(0, 0.3, 33)
    net.set_params(p)
    for B in batches:
        x = rng.random((B, 64, 64, dd.CHANNELS)).astype(np.float32)
        dy = (rng.uniform(0.5, 1.5, (B, 64, 64)) / (B * 4096)).astype(np.float32)
        xg, dyg = torch.tensor(x, device="cuda"), torch.tensor(dy, device="cuda")
        grads = []
        for _ in range(2):
            net.forward(xg, train=True)
            net.backward(dyg)
            grads.append(net.grads())
        assert np.array_equal(*grads)
    pt = torch.tensor(p.astype(np.float64))
    _, state = R.forward_bf16(pt, torch.tensor(x, dtype=torch.float64))
    ref = R.backward_bf16(pt, state, torch.tensor(dy, dtype=torch.float64)).numpy()
    got = grads[0].astype(np.float64)
    for name, s in R.layer_slices():
        d = got[s] - ref[s]
        assert np.abs(d).max() <= TOL_G * np.abs(ref[s]).max(), name
        assert np.linalg.norm(d) <= TOL_G_NORM * np.linalg.norm(ref[s]), name
