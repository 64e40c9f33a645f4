"""The window transform treats every row alike: a window with one nonzero row in W / 4
steps has the same diffraction pattern, bit for bit, whichever row that is.

One active beam at zero angle has the coefficient 1, so the window is the S-matrix plane
times one factor. The column transform of a single row y0 = m W / 4 multiplies by exact
quarter turns and its later stages meet one nonzero input with the twiddle 1, so
|Psi(ky, kx)|^2 is |G(kx)|^2 of the row transform for every ky, without rounding.
"""
import numpy as np
import pytest

import _gpu as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,f", [(128, 8), (192, 8), (128, 4), (576, 16), (192, 4), (128, 2),
                                 (576, 8), (384, 4), (256, 2), (576, 4), (384, 2), (512, 2)])
def test_pattern_does_not_depend_on_the_row(n, f):
    import torch
    from paper_1702_01904_amd import Plan
    w, ns = n // (2 * f), n // 2
    plan = Plan(n, 0.1 * n, 80.0, np.full(2, 2.0))
    alpha = 0.4e3 * f * plan.wavelength / (0.1 * n)  # less than one beam spacing
    amax = plan.alpha_max_default(alpha, f)
    o = dict(alpha_mrad=alpha)
    assert plan.active_beam_count(f, amax, o) == 1
    zero = [tuple(b) for b in plan.beams(f, amax)].index((0, 0))
    rng = np.random.default_rng([n, f, 3])
    row = rng.standard_normal((ns, 2)).astype(np.float32)
    xy = np.array([[1.23, 2.34]])
    top = (int(np.floor(xy[0, 1] / 0.2 + 0.5)) - w // 2) % ns  # S-pixels are 0.2 A
    base = None
    for m in range(4 if w % 4 == 0 else 2):
        y0 = m * w // (4 if w % 4 == 0 else 2)
        S = np.zeros((plan.beam_count(f, amax), ns, ns, 2), dtype=np.float32)
        S[zero, (top + y0) % ns] = row
        C = G.probe_cbed(plan, f, amax, torch.view_as_complex(torch.from_numpy(S)).to(G.device()),
                         xy, o)[0]
        base = C[0] if base is None else base
        assert np.count_nonzero(base) == w
        assert np.array_equal(C, np.broadcast_to(base, (w, w))), y0
