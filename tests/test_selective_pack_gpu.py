"""Selective packs of up to 2048 probes: the same bits as with everything packed."""
import numpy as np
import pytest

from test_window_sum_gpu import _case, _near, _run

pytestmark = pytest.mark.gpu


def _pack_mib(plan, f, amax, alpha, prec):
    n_act = plan.active_beam_count(f, amax, dict(alpha_mrad=alpha))
    pad = 16 if prec == "fp32" else 32
    word = 8 if prec == "fp32" else 4
    return (plan.n // 2) ** 2 * (8.0 * n_act + word * (-(-n_act // pad) * pad)) / 2 ** 20


# S sides 96, 192, 288 and 576 (tiles of 64 pixels that cross rows and that do not)
@pytest.mark.parametrize("prec", ["fp32", "fp16"])
@pytest.mark.parametrize("n,f,alpha", [(192, 1, 45.0), (384, 3, 45.0), (576, 6, 30.0),
                                       (1152, 12, 30.0)])
def test_selective_pack_of_many_probes(n, f, alpha, prec):
    """One probe to 2048 (several steps of the window test, several beam blocks per
    workgroup) packed by the tiles their windows meet, against the same probes in a fill of
    more than 2048, which packs everything."""
    plan, amax, S = _case(n, f, alpha)
    plan.set_probe_precision(prec)
    assert _pack_mib(plan, f, amax, alpha, prec) >= 24 + 700 * 3 / 64
    rng = np.random.default_rng([n, f, 5])
    # a patch round the corner and a stripe: most tiles are met by a few probes or none
    stripe = np.stack([rng.uniform(0.0, 0.1 * n, 350), np.full(350, 0.043 * n)], axis=1)
    xy = np.concatenate([_near(n, 350, rng), stripe])
    many = np.concatenate([xy, np.repeat(xy[:1], 2049 - len(xy), axis=0)])
    full = _run(plan, f, amax, S, many, alpha)
    assert np.array_equal(full[len(xy):], np.broadcast_to(full[0], (2049 - len(xy), 3)))
    for count in (1, 255, 257, 700):
        assert np.array_equal(_run(plan, f, amax, S, xy[:count], alpha), full[:count]), count
    assert np.array_equal(_run(plan, f, amax, S, many[:2048], alpha), full[:2048])
