"""The one-block-per-map renderer decides most log-scale pixels in single
precision and the close ones in double: values on, next to and between the bin and
level boundaries, over ranges from 1.0003 to 10^600 and for any level count, give
the general kernel's image (an output one byte off alignment goes there)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lo,hi", [(1.0, 1.0003), (3.0, 3.3), (0.7, 700.0), (1e-7, 1e5),
                                   (1e-280, 1e20), (1e-300, 1e300), (1e300, 1.7e308)])
def test_decisions_equal_the_general_kernel(lo, hi):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd

    rng = np.random.default_rng(1)
    ratio = np.log(hi) - np.log(lo)
    for levels in (0, 1, 6, 7, 256):
        k = rng.integers(0, 257, 4096) / 256.0
        if levels:
            k[::2] = rng.integers(0, levels + 1, 2048) / levels
        off = rng.choice([0, 1e-15, 1e-12, 1e-9, 1e-7, 1e-6, 1e-5, 1e-4, 3e-3], 4096)
        t = k + off * rng.choice([-1, 1], 4096)
        with np.errstate(over="ignore"):
            v = np.exp(np.log(lo) + t * ratio).reshape(4, 32, 32)
        v[0, 0, :5] = lo, hi, np.nan, np.inf, 0.0
        for w in (32, 31):  # packed and byte-wise level tests
            psi = torch.tensor(np.ascontiguousarray(v[:, :, :w]), device="cuda")
            if w == 31:
                psi = psi[:, :28].contiguous()
            n, h, _ = psi.shape
            fast = dd.render_maps(psi, lo=lo, hi=hi, levels=levels)
            buf = torch.empty(3 * n * h * w + 1, dtype=torch.uint8, device="cuda")
            slow = dd.render_maps(psi, out=buf[1:].view(n, h, w, 3), lo=lo, hi=hi, levels=levels)
            assert torch.equal(fast, slow), (levels, w)
