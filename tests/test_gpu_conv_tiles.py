"""The convolutions' two tiles (64 pixels below 256 blocks of the large tile,
256 above) add up in the same order: a map's network output is the same to the
bit in batches on either side of each level's switch (32x32 at 64 maps, 16x16
at 128, 8x8 at 253) and in a ragged batch."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("train", [False, True])
def test_batch_size_changes_no_bit(train):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd

    rng = np.random.default_rng(5)
    net = dd.UNet(4)
    p = net.params()
    p[-33:] = rng.normal(0, 0.3, 33)
    net.set_params(p)
    x = torch.tensor(rng.random((256, 64, 64, dd.CHANNELS)).astype(np.float32), device="cuda")
    full = net.forward(x, train=train).cpu().numpy()
    assert np.isfinite(full).all() and full.std() > 0
    for B in (1, 3, 63, 64, 127, 128, 252, 253):
        got = net.forward(x[256 - B:].contiguous(), train=train).cpu().numpy()
        assert np.array_equal(got, full[256 - B:]), B
