"""The FP32 training step's products in three BF16 parts hold FP32's 24 bits, against the FP64 step (itself held to
the oracle).

Ragged shapes to the FP32 bars of the training tests and, over the whole gradient, to a relative norm of
1.5e-6: the FP32 step is off by 3e-7 to 6e-7 (1.4e-6 for seven atoms whose terms cancel), and one of the six
products left out would be an RMS error of 2^-18.6 (2.5e-6) of each of some ten products in a row."""

import time

import numpy as np
import pytest
import torch

from paper_2402_17660_amd import TensorNet
from tests.test_gpu_train import _case, _check, _gpu, _molecules
from tests.util import small_blob

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


def test_steps_with_nan_take_no_longer(dev):
    """NaN and infinite targets: only sums of operands without a NaN are formed again, so the step takes about the time
    of a finite one (within a factor of 3; with all of them formed again it was 18 and more)."""
    pos, z, batch = _molecules(tuple(range(24, 120, 6)), 25)
    S = int(batch[-1]) + 1
    rng = np.random.default_rng(26)
    E_ref, F_ref = rng.normal(size=S), rng.normal(size=pos.shape)
    model = TensorNet(small_blob(F=128, K=32, L=3, seed=27), dev)
    t = lambda a, dt: torch.tensor(a, dtype=dt, device=dev)

    def ms(E, F):
        args = (t(pos, torch.float32), t(z, torch.int32), t(batch, torch.int32), S, t(E, torch.float64),
                t(F, torch.float64))
        out = []
        for _ in range(5):
            torch.cuda.synchronize()
            start = time.perf_counter()
            model.train_grad(*args, precision="fp32", check=False)
            torch.cuda.synchronize()
            out.append(time.perf_counter() - start)
        return 1e3 * sorted(out)[1]

    finite = ms(E_ref, F_ref)
    E_inf, E_nan, F_nan = E_ref.copy(), E_ref.copy(), np.full_like(F_ref, np.nan)
    E_inf[3], E_nan[3] = np.inf, np.nan
    for name, E, F in (("infinite energy", E_inf, F_ref), ("NaN energy", E_nan, F_ref), ("NaN forces", E_ref, F_nan)):
        took = ms(E, F)
        print(f"{name}: {took:.2f} ms, finite {finite:.2f} ms", flush=True)
        assert took <= 3 * finite, name
