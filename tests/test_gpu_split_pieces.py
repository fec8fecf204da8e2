"""The split-bf16 product's loads ahead (csrc/matvec_bf16.hip) against the
complex64 product of the same operator: near blocks in pieces of three or four
contraction steps with remainders, single-term blocks, far blocks of row clusters
around the 64-row limit with odd and even numbers of column tiles, more frequency
tiles than a workgroup has waves, and both numbers of tiles per wave."""
import numpy as np
import pytest
import torch

import paper_2505_00715_amd as g
from synth import freq, mesh
from tests._gpu_common import from_dev, make_ctx, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [32, 64])
@pytest.mark.parametrize("triangles,leaf,L", [(1500, 12, 40), (1500, 40, 33), (1200, 64, 290), (3000, 90, 32)])
def test_split_product_loads_ahead(triangles, leaf, L, cols):
    xyz, tri = mesh.fin_housing(triangles)
    ctx = make_ctx(xyz, tri, 343.0, freq.bdf2_circle(L, 1e-4, 0.7), leaf, 1.0)
    ctx.set_tuning(product_cols_per_wave=cols)
    ctx.aca3d(1e-5, 1e-5, 64, g.C64)
    X = torch.randn((L, ctx.n), dtype=torch.complex64, device="cuda", generator=torch.Generator("cuda").manual_seed(L))
    Y, Z = torch.full_like(X, float("nan")), torch.empty_like(X)
    ctx.compressed_matvec(g.PER_FREQUENCY, g.C64, X, Z)
    ctx.compressed_matvec(g.PER_FREQUENCY, g.C64_SPLIT_BF16, X, Y)
    # the split perturbs every stored operator value by at most 2^-18 of itself;
    # a block's terms, whose fibers are bounded by about 1, cancel in part (a
    # factor of 2 of their sum of moduli over the block itself)
    err = max(rel(from_dev(Y[k]), from_dev(Z[k])) for k in range(L))
    assert np.isfinite(err) and err < 2 * 2.0 ** -18 + 1e-6
