"""Products whose kernels take a block in pieces: the weighted sum (pieces of
columns, terms and frequencies) against the sum of the per-frequency product's
columns, and the FMM-based product (row tiles and pieces of the contraction by
order) against the complex128 one."""
import numpy as np
import pytest
import torch

import paper_2505_00715_amd as g
from synth import freq, mesh
from tests._gpu_common import from_dev, make_ctx, rel

pytestmark = pytest.mark.gpu


def _vec(L, n, dtype):
    return torch.randn((L, n), dtype=dtype, device="cuda", generator=torch.Generator("cuda").manual_seed(L))


# leaves above 128 and 256 rows (pieces of columns, row loops), more than 8 terms
# per block (1e-9), frequency counts around 64 and without conjugate partners
@pytest.mark.parametrize("triangles,leaf,L,sym,tol", [(1500, 300, 70, True, 1e-6), (1500, 20, 65, True, 1e-9),
                                                      (1000, 40, 5, False, 1e-6)])
def test_weighted_sum_is_the_sum_of_columns(triangles, leaf, L, sym, tol):
    xyz, tri = mesh.fin_housing(triangles)
    ctx = make_ctx(xyz, tri, 343.0, freq.bdf2_circle(L, 1e-4, 0.7), leaf, 1.0, sym=sym)
    for prec, dt, bound in ((g.C128, torch.complex128, 1e-12), (g.C64, torch.complex64, 1e-5)):
        st = ctx.aca3d(tol, tol, 64, prec)
        if tol < 1e-8 and prec == g.C128:
            assert st.rank_max > 8
        X = _vec(L, ctx.n, dt)
        y, Y = torch.empty(ctx.n, dtype=dt, device="cuda"), torch.empty_like(X)
        ctx.compressed_matvec(g.WEIGHTED_SUM, prec, X, y)
        ctx.compressed_matvec(g.PER_FREQUENCY, prec, X, Y)
        # rounding of sums of L n terms of random sign
        assert rel(from_dev(y), from_dev(Y).sum(0)) < bound


@pytest.mark.parametrize("order", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("L", [5, 40])
def test_fmm_product_float_against_double(order, L):
    xyz, tri = mesh.icosphere(3)
    ctx = make_ctx(xyz, tri, 1.0, freq.bdf2_circle(L, 0.05, 0.6), 40, 1.0)
    X = _vec(L, ctx.n, torch.complex128)
    out = []
    for prec, dt in ((g.C128, torch.complex128), (g.C64, torch.complex64)):
        ctx.fmm3d(order, 1e-5, 64, prec)
        Y = torch.full((L, ctx.n), float("nan"), dtype=dt, device="cuda")
        out.append(from_dev(ctx.fmm3d_matvec(X.to(dt), Y)))
    # both compressed to 1e-5 along the frequencies (20 tol per tensor, as in the
    # FMM's own tests), plus float rounding
    assert rel(out[1], out[0]) < 20 * 1e-5
