"""The FP32 path holds weights and operands in FP32's 24 bits at least, whatever else their matrix holds.

The last bit: with every weight of the pair products and channel mixings one unit in the last place larger, the
forces change as the FP64 oracle's do.  The weights' bits are chosen so that two FP16 numbers cannot
hold that unit (23 bits, round to nearest: both sets would become the same), and they are FP32 numbers
themselves.  The change is 2e-7 of the forces and the path's own roundings may be 2e-6 of them: over the 4800
components of 8 boxes the slope of the one change against the other is then off by up to 2e-6 * sqrt(2) /
2e-7 / sqrt(4800) = 0.2; the bar is 0.5.

Matrices of wide range: channels scaled by powers of two against the matrices that read them.  FP32 loses
nothing by such a scale, so the bounds of the model tests hold as they are (energy 1e-6, forces 1e-5)."""

import numpy as np
import pytest

from oracle import TensorNetOracle
from paper_2402_17660_amd import TensorNet
from synth import make_weights, write_blob
from tests.test_gpu_model import assert_close, gpu_ef
from tests.util import oracle_energy_forces_r21, random_box

pytestmark = pytest.mark.gpu
R_C = 4.5


def box(n, seed):
    pos, z, H = random_box(n, seed, (n / 0.1) ** (1.0 / 3.0))
    return pos.astype(np.float32), z, np.zeros(n, np.int32), H


def last_bits(w, unit):
    """The weights of the pair products and channel mixings as FP32 numbers whose bits past the eleventh are
    01xxxxxxxxx0u, u the unit in the last place: the remainder of an FP16 number that is too large to hold u."""
    out = dict(w)
    for k, v in w.items():
        if k in ("emb.W0", "emb.WI", "emb.WA", "emb.WS") or (k.startswith("layer") and ".W" in k):
            b = v.astype(np.float32).view(np.uint32)
            out[k] = ((b & ~np.uint32(0x1803)) | np.uint32(0x0800 + unit)).view(np.float32).astype(np.float64)
    return out


@pytest.mark.parametrize("F,L", [(64, 2), (128, 2)])
def test_last_bit_of_the_weights(dev, F, L):
    n, ref, got = 200, [], []
    for seed in range(8):
        w = make_weights(F, 32, L, 100, seed=900 + seed)
        pos, z, batch, H = box(n, 950 + seed)
        pair = [write_blob(last_bits(w, u), F, 32, L, 100, R_C) for u in (0, 1)]
        r = [TensorNetOracle(b).energy_forces(pos, z, batch, H, 1)[1] for b in pair]
        g = [gpu_ef(dev, TensorNet(b, dev), pos, z, batch, H, 1, "fp32", "fused", max_pairs=32 * n)[1] for b in pair]
        ref.append((r[1] - r[0]) / np.linalg.norm(r[0]))
        got.append((g[1] - g[0]) / np.linalg.norm(r[0]))
    ref, got = np.array(ref), np.array(got)
    slope = float((ref * got).sum() / (ref * ref).sum())
    print(f"F={F} L={L}: change of the forces {np.sqrt((ref ** 2).sum() / 8):.2e}, slope {slope:.3f}", flush=True)
    assert abs(slope - 1.0) <= 0.5


def small_embedding_channels(w, F, e):   # half of the embedding map's channels, against the mixing's columns
    for part in range(3):
        c = part * F + np.arange(0, F, 2)
        w["emb.W0"][c] *= 2.0 ** -e
        w["emb.b0"][c] *= 2.0 ** -e
        w["emb.W" + "IAS"[part]][:, ::2] *= 2.0 ** e


def small_filter_channels(w, F, e):   # half of the filter's second layer, against the third's columns
    w["layer0.Wb"][::2] *= 2.0 ** -e
    w["layer0.bb"][::2] *= 2.0 ** -e
    w["layer0.Wc"][:, ::2] *= 2.0 ** e


def small_product_channels(w, F, e):   # half of a layer's Y, with it the product's square, against W2's columns
    for part in "IAS":
        w["layer0.W1" + part][::2] *= 2.0 ** -(e // 2)
        w["layer0.W2" + part][:, ::2] *= 2.0 ** (e // 2 * 2)


@pytest.mark.parametrize("path", ["fused", "molecule"])
@pytest.mark.parametrize("change", [small_embedding_channels, small_filter_channels, small_product_channels])
@pytest.mark.parametrize("F,e", [(64, 24), (128, 24)])
def test_matrices_of_wide_range(dev, F, e, change, path):
    w = make_weights(F, 32, 2, 100, seed=77)
    change(w, F, e)
    blob = write_blob(w, F, 32, 2, 100, R_C)
    pos, z, batch, H = box(200, 78)
    if path == "molecule":
        H = None
    E_ref, F_ref, total = oracle_energy_forces_r21(TensorNetOracle(blob), pos, z, batch, H, 1)
    E, Fv = gpu_ef(dev, TensorNet(blob, dev), pos, z, batch, H, 1, "fp32", path, max_pairs=32 * 200)
    assert_close(E, Fv, E_ref, F_ref, "fp32", f"{change.__name__} F={F} 2^{e} {path}", total)
