"""The weighted sum of many narrow blocks at few frequencies (csrc/matvec3d.hip,
one wave and two terms at a time) against the per-frequency product's column sum:
clusters wider than a piece of columns, odd numbers of terms, row counts above and
below a wave, frequency counts around a piece and on both sides of the rule's
line, with and without conjugate partners."""
import pytest
import torch

import paper_2505_00715_amd as g
from synth import freq, mesh
from tests._gpu_common import from_dev, make_ctx, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("triangles,leaf,L,sym", [(4000, 7, 1, True), (4000, 7, 5, False), (3000, 6, 33, True),
                                                  (3000, 15, 20, True)])
def test_weighted_sum_of_narrow_blocks(triangles, leaf, L, sym):
    xyz, tri = mesh.fin_housing(triangles)
    ctx = make_ctx(xyz, tri, 343.0, freq.bdf2_circle(L, 1e-4, 0.7), leaf, 1.0, sym=sym)
    blocks = ctx.get_tree()[1]
    assert len(blocks) > 2048   # the first three at most 260 near columns times frequencies, the last above
    for prec, dt, bound in ((g.C128, torch.complex128, 1e-12), (g.C64, torch.complex64, 1e-5)):
        ctx.aca3d(1e-6, 1e-6, 64, prec)
        X = torch.randn((L, ctx.n), dtype=dt, device="cuda", generator=torch.Generator("cuda").manual_seed(L))
        y, Y = torch.empty(ctx.n, dtype=dt, device="cuda"), torch.empty_like(X)
        ctx.compressed_matvec(g.WEIGHTED_SUM, prec, X, y)
        ctx.compressed_matvec(g.PER_FREQUENCY, prec, X, Y)
        # rounding of sums of L n terms of random sign
        assert rel(from_dev(y), from_dev(Y).sum(0)) < bound
