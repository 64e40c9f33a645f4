"""Multislice of few probes (passes through LDS) and of many (step passes): detector sums
of every grid against the FP64 oracle on both sides of the line between them.

Tolerance: rounding of the wave as in test_slice_steps_gpu (7e-7 after three slices),
twice that in the intensity; rounded transform constants take up to 3e-7 of the intensity
per slice; the sum, 2.3e-6, gated at four times.
"""
import numpy as np
import pytest

import oracle as O

import _gpu as G
from test_slice_steps_gpu import _inputs

pytestmark = pytest.mark.gpu

TOL = 1e-5
EDGES = [(0.0, 12.0), (12.0, 25.0), (25.0, 60.0)]


# most probes of the LDS passes on each grid (0: none)
@pytest.mark.parametrize("n,most", [(128, 32), (192, 64), (256, 0), (384, 48), (512, 48), (576, 6),
                                    (768, 16), (1152, 2), (1536, 1), (2048, 0)])
def test_both_sides_of_the_line(n, most):
    d = _inputs(n, 3 if n < 1152 else 2, 31)
    plan = G.make_plan(d)
    optics = dict(alpha_mrad=20.0, C1_A=30.0, C3_A=0.0)
    rng = np.random.default_rng([n, 7])
    xy = rng.uniform(0.0, 0.1 * n, (most + 1, 2))
    some = sorted({0, most // 2, max(most - 1, 0)})
    ref = O.multislice_stem(d["phase"], d["thickness"], d["cell"], 80.0, optics, xy[some], EDGES)
    for count in sorted({1, most, most + 1} - {0}):
        pick = [i for i, k in enumerate(some) if k < count]
        idx = [some[i] for i in pick]
        D = G.multislice_outputs(plan, xy[:count], optics, EDGES)
        assert np.all(np.isfinite(D))
        e = np.linalg.norm(D[idx] - ref[pick]) / np.linalg.norm(ref[pick])
        assert e <= TOL, (n, count, e)
        # which passes run is decided for the call, not for a workspace's chunks
        least = G.multislice_outputs(plan, xy[:count], optics, EDGES, ws_bytes=0)
        assert np.array_equal(D, least), (n, count)
