"""The FP32 pair tiles' edges: fewer pairs than a row block, whole blocks, one pair past them, and many tiles of one
workgroup in sequence (the molecule path), for every basis size and tile shape: forces against the FP64 oracle with
the FP32 bound of the model tests, forces and energies bit for bit between the shapes and the two paths.  (No
bound on these energies themselves: of a few atoms whose energies cancel, FP32 arithmetic of either kind is off by
up to 7e-6 of the tests' scale.)"""

import numpy as np
import pytest

from oracle import TensorNetOracle
from paper_2402_17660_amd import TensorNet
from tests.test_gpu_model import gpu_ef
from tests.util import random_molecule, rel_rms, small_blob

pytestmark = pytest.mark.gpu


def dimers(count, seed):
    """`count` systems of two atoms within reach of each other: as many pairs."""
    rng = np.random.default_rng(seed)
    u = rng.normal(size=(count, 3))
    u *= (rng.uniform(0.9, 4.0, size=count) / np.linalg.norm(u, axis=1))[:, None]
    pos = np.stack([-0.5 * u, 0.5 * u], 1).reshape(-1, 3).astype(np.float32)
    return pos, np.array([1, 6, 7, 8], np.int32)[rng.integers(0, 4, size=2 * count)], np.repeat(np.arange(count, dtype=np.int32), 2)


@pytest.mark.parametrize("F", [64, 128])
@pytest.mark.parametrize("K,count", [(16, 1), (32, 15), (32, 16), (48, 17), (64, 33), (32, 49)])
def test_few_pairs(dev, F, K, count):
    pos, z, batch = dimers(count, 60 + count)
    blob = small_blob(F=F, K=K, L=2, seed=61)
    _, F_ref = TensorNetOracle(blob).energy_forces(pos, z, batch, None, count)
    m = TensorNet(blob, dev)
    first = None
    for v in range(TensorNet.pair_variant_count("fp32")):
        m.set_pair_variant("fp32", v, v)
        E, Fv = gpu_ef(dev, m, pos, z, batch, None, count, "fp32", "fused", max_pairs=count)
        if first is None:
            first = (E, Fv)
            assert np.isfinite(E).all() and rel_rms(Fv, F_ref) <= 1e-5
        assert np.array_equal(E, first[0]) and np.array_equal(Fv, first[1]), v
    if K == 32:
        E, Fv = gpu_ef(dev, m, pos, z, batch, None, count, "fp32", "molecule", max_pairs=64 * count)
        assert np.array_equal(E, first[0]) and np.array_equal(Fv, first[1])


@pytest.mark.parametrize("F", [64, 128])
def test_many_tiles_of_a_molecule(dev, F):
    """Molecules of one to some thirty tiles, whose workgroup runs them one after the other."""
    sizes = [2, 9, 20, 40, 60, 90]
    parts = [random_molecule(n, 640 + n) for n in sizes]
    pos = np.concatenate([p for p, _ in parts]).astype(np.float32)
    z = np.concatenate([q for _, q in parts])
    batch = np.repeat(np.arange(len(sizes), dtype=np.int32), sizes)
    blob = small_blob(F=F, K=32, L=2, seed=62)
    _, F_ref = TensorNetOracle(blob).energy_forces(pos, z, batch, None, len(sizes))
    m = TensorNet(blob, dev)
    E, Fv = gpu_ef(dev, m, pos, z, batch, None, len(sizes), "fp32", "molecule", max_pairs=32 * len(pos))
    assert np.isfinite(E).all() and rel_rms(Fv, F_ref) <= 1e-5
    Ef, Ff = gpu_ef(dev, m, pos, z, batch, None, len(sizes), "fp32", "fused", max_pairs=32 * len(pos))
    assert np.array_equal(E, Ef) and np.array_equal(Fv, Ff)
