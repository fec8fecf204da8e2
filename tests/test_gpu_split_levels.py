"""The split-bf16 product's work items (csrc/matvec_bf16.hip) against the
complex64 product of the same operator: leaves of two depths (near blocks of a
cluster and of its sons), near blocks wider than the pieces of the right-hand
side held in registers, block lists cut into several items, and frequency counts
that leave column tiles partly empty."""
import numpy as np
import pytest
import torch

import paper_2505_00715_amd as g
from synth import freq, mesh
from tests._gpu_common import from_dev, make_ctx, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("triangles,leaf,L", [(1500, 20, 5), (1500, 20, 70), (1500, 200, 33), (1000, 7, 32)])
def test_split_product_equals_float_product(triangles, leaf, L):
    xyz, tri = mesh.fin_housing(triangles)
    ctx = make_ctx(xyz, tri, 343.0, freq.bdf2_circle(L, 1e-4, 0.7), leaf, 1.0)
    if (triangles, leaf) == (1500, 20):
        blocks = ctx.get_tree()[1]
        rows = {(int(b[0]), int(b[1])) for b in blocks if b[4] == 0}
        assert any(a != c and a[0] <= c[0] and c[1] <= a[1] for a in rows for c in rows)   # nested near rows
    ctx.aca3d(1e-5, 1e-5, 64, g.C64)
    X = torch.randn((L, ctx.n), dtype=torch.complex64, device="cuda", generator=torch.Generator("cuda").manual_seed(L))
    Y, Z = torch.full_like(X, float("nan")), torch.empty_like(X)
    ctx.compressed_matvec(g.PER_FREQUENCY, g.C64, X, Z)
    ctx.compressed_matvec(g.PER_FREQUENCY, g.C64_SPLIT_BF16, X, Y)
    # the split perturbs every stored operator value by at most 2^-18 of itself;
    # a block's terms, whose fibers are bounded by about 1, cancel in part (a
    # factor of 2 of their sum of moduli over the block itself)
    for k in range(L):
        assert rel(from_dev(Y[k]), from_dev(Z[k])) < 2 * 2.0 ** -18 + 1e-6, k
