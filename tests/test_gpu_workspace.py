"""The FP32 paths' workspace holds the arrays that they use and no others: what one more atom takes (at the same
pair budget) is the sum of its rows, counted here from the paths' steps, to 1 % (alignment)."""

import pytest

from paper_2402_17660_amd import TensorNet
from tests.util import small_blob

pytestmark = pytest.mark.gpu


def row_bytes(F, L, forces):
    feature = 2 + (L + 1) + 4 * L        # Xr, T0; X; Y, M, Pb, D
    # LayerNorm and MLP of the embedding (xhat, out, F -> 2F twice, 3F twice), of the output (xhat, out, F twice, F/2)
    island = (1 + 1 + 2 + 2 + 3 + 3) + (3 + 3 + 1 + 1 + 0.5)
    if forces:
        feature += L + 3                 # dM; dX, dY, dXr
        island += 3 + 2 + 1 + 0.5 + 1 + 3
    return 9 * F * 4 * feature + 8 * F * island


@pytest.mark.parametrize("forces", [False, True])
@pytest.mark.parametrize("F,L", [(64, 2), (128, 0), (128, 3)])
@pytest.mark.parametrize("path", ["fused", "molecule"])
def test_bytes_per_atom(dev, path, F, L, forces):
    m = TensorNet(small_blob(F=F, K=32, L=L, seed=5), dev)
    size = lambda n: m.workspace_bytes(n, 1, 4096, precision="fp32", path=path, forces=forces)
    per_atom = (size(3000) - size(1000)) / 2000
    want = row_bytes(F, L, forces)
    if path == "molecule":
        want += 8 * F / 2   # the last layer's pre-activation
    print(f"{path} F={F} L={L} forces={forces}: {per_atom:.0f} bytes per atom, rows {want:.0f}", flush=True)
    assert abs(per_atom - want) <= 0.01 * want
