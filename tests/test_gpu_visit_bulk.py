"""FP64 visit-list arrival, one pair per list, at the edges of its forms against
the binary128 bracket of Eqs. 1-4: delta = db / (2 bm) and X = x delta around the
bulk polynomial's bounds (2^-9 and 2^-5), the visit still on, x up to the cull, and
the E1 differences around x = 2.5 and beyond."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIGMA, D = 0.5e-9, 2.5e-13
TH4 = 4 * D / SIGMA ** 2


def _pairs():
    tau = 1e-6
    out = []
    for delta in (2.0 ** -8, 2.0 ** -9 * 1.001, 2.0 ** -9 * 0.999, 2.0 ** -10, 2.0 ** -14):
        bm = TH4 * tau / (2 * delta)
        lag = (bm - 2) / TH4 + tau / 2
        for X in (0.0, 1e-6, 2.0 ** -6, 2.0 ** -5 * 0.999, 2.0 ** -5 * 1.001, 0.1, 0.6):
            x = X / delta
            if x < 740:
                out.append((math.sqrt(x * bm) * SIGMA, lag, tau))
    for lag in (0.3e-6, 1e-6, 1.5e-6, 4e-6):  # on at the query, or just ended
        b1 = 2 + TH4 * lag
        for x1 in (1e-9, 0.3, 2.4, 2.6, 11.0, 101.0, 700.0):
            out.append((math.sqrt(x1 * b1) * SIGMA, lag, tau))
    return out


def test_pairs_against_binary128(ora):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_00294_amd as dd

    pairs = _pairs()
    lists = [dd.Visits([0.0, r], [0.0, 0.0], [0.0, lag], [tau, tau], sigma_m=SIGMA, D_m2s=D)
             for r, lag, tau in pairs]
    outs = dd.visits_batch_arrival(lists, "fp64")
    pref = 1.0 / (4 * math.pi * D)
    for (r, lag, tau), o in zip(pairs, outs):
        o = np.asarray(o.cpu())
        ref = ora.phi_bracket_q(r * r, lag, tau, SIGMA, D)
        x = r * r / SIGMA ** 2 / (2 + TH4 * lag)
        # the forms' 4e-14 (exponential 2e-14, E1 1e-14) and the exponent's rounding
        # errors, a few units of 1.1e-16 of x (2x for a difference of E1 values)
        assert o[0] == 0.0
        assert abs(o[1] / (pref * ref) - 1) <= 4e-14 + 1e-15 * x, (r, lag, o[1] / (pref * ref) - 1)
