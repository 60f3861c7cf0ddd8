"""The FP32 training step's products in three BF16 parts hold FP32's 24 bits, against the FP64 step (itself held to
the oracle).

Ragged shapes to the FP32 bars of the training tests and, over the whole gradient, to a relative norm of
1.5e-6: the FP32 step is off by 3e-7 to 6e-7 (1.4e-6 for seven atoms whose terms cancel), and one of the six
products left out would be an RMS error of 2^-18.6 (2.5e-6) of each of some ten products in a row."""

import numpy as np
import pytest

from tests.test_gpu_train import _case, _check, _gpu

pytestmark = pytest.mark.gpu


def flat(g):
    return np.concatenate([v.reshape(-1) for v in g.values()])


@pytest.mark.parametrize("sizes,F,K,L", [((2,), 64, 32, 1), ((5, 9), 64, 16, 2), ((31, 17, 8), 64, 32, 0),
                                         ((3, 4), 128, 32, 1), ((40, 23, 11), 128, 32, 2), ((33,), 128, 16, 1)])
def test_ragged_shapes_to_the_fp32_bars(dev, sizes, F, K, L):
    pos, z, batch, S, E_ref, F_ref, blob = _case(sizes, F, K, L, 21)
    pos = pos.astype(np.float32).astype(np.float64)
    loss_ref, _, _, ref, _ = _gpu(dev, blob, pos, z, batch, None, S, E_ref, F_ref, "fp64")
    loss, _, _, got, _ = _gpu(dev, blob, pos, z, batch, None, S, E_ref, F_ref, "fp32")
    off = np.linalg.norm(flat(got) - flat(ref)) / np.linalg.norm(flat(ref))
    print(f"relative norm {off:.2e}", flush=True)
    _check(f"{sizes} F={F} K={K} L={L}", "fp32", loss, got, loss_ref, ref)
    assert off <= 1.5e-6


@pytest.mark.parametrize("F,L", [(64, 0), (128, 1)])
def test_infinities_stay_what_they_are(dev, F, L):
    """An infinite target: every gradient entry is infinite (of either sign), NaN or finite where the FP64 step's is."""
    pos, z, batch, S, E_ref, F_ref, blob = _case((5, 9), F, 32, L, 24)
    pos = pos.astype(np.float32).astype(np.float64)
    E_ref = np.array(E_ref)
    E_ref[1] = np.inf
    ref, got = (_gpu(dev, blob, pos, z, batch, None, S, E_ref, F_ref, p)[3] for p in ("fp64", "fp32"))
    assert np.isinf(ref["out.Wh"]).any()
    for k in ref:
        for kind in (np.isnan, np.isposinf, np.isneginf):
            assert np.array_equal(kind(got[k]), kind(ref[k])), (k, kind.__name__)
