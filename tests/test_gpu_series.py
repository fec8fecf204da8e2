"""Dense entries of one pair at many frequencies (csrc/series.h): the near and
self tiers in one bin, in several and point by point, the far tier's degrees,
few and many frequencies, partial workgroups; single and double layer, both
precisions, against the float64 oracle entry by entry."""
import numpy as np
import pytest
import torch

import paper_2505_00715_amd as g
from oracle import dlp, entries
from oracle.geometry import Panels
from synth import mesh
from tests._gpu_common import from_dev, make_ctx

pytestmark = pytest.mark.gpu

XYZ, TRI = mesh.icosphere(2)
PAN = Panels(XYZ, TRI)


# |s|: near bins of one to six (float), up to twelve (double) and beyond; 1200 goes point by point
@pytest.mark.parametrize("scale", [0.5, 6.0, 40.0, 1200.0])
@pytest.mark.parametrize("nf", [3, 4, 65])
@pytest.mark.parametrize("layer", [False, True])
def test_entries_at_many_frequencies(scale, nf, layer):
    rng = np.random.default_rng(int(scale) + nf)
    # |Re s| small enough that no entry underflows in float (distances up to 2)
    s = scale * np.exp(1j * rng.uniform(-1.5, 1.5, nf)) * rng.uniform(0.2, 1.0, nf)
    s = np.minimum(s.real, 30.0) + 1j * s.imag
    ctx = make_ctx(XYZ, TRI, 1.0, s, 16, 1.0, sym=False)
    rows, cols = np.arange(5, 42), np.concatenate([np.arange(0, 50), [319, 300, 5]])
    block = (dlp if layer else entries).block
    ref = block(PAN, rows, cols, s, 1.0)
    # sum of the moduli of an entry's quadrature terms, which its rounding is
    # relative to (at large |s| the terms cancel): the entry at Re s, the double
    # layer's times |1 + s r| <= 1 + 2 |s|
    mod = np.abs(block(PAN, rows, cols, s.real, 1.0)) * (1 + 2 * np.abs(s) if layer else np.ones(nf))[:, None, None]
    d2 = ((PAN.centroid[rows][:, None] - PAN.centroid[cols][None]) ** 2).sum(-1)
    close = (d2 < 4.0 * PAN.h2[cols][None]) | (rows[:, None] == cols[None])
    for prec, dt in ((g.C128, torch.complex128), (g.C64, torch.complex64)):
        out = torch.full((nf, len(cols), len(rows)), float("nan"), dtype=dt, device="cuda")
        (ctx.assemble_dlp_slices if layer else ctx.assemble_slices)(rows, cols, np.arange(nf), prec, out)
        err = np.abs(from_dev(out).transpose(0, 2, 1) - ref)
        # phases |s| r carry a rounding of |s| r 2^-53 each (r <= 2); the double
        # layer's d . n_y cancels to the rounding of the coordinates
        f64 = 4e-15 * (1 + 2 * np.abs(s))[:, None, None] * mod
        if layer:
            f64 = f64 + 1e-14 * mod.max((1, 2), keepdims=True)
        if prec == g.C128:
            assert (err <= f64).all(), (err / f64).max()
            continue
        # float64 values rounded once (near, self); float exponentials of exactly
        # reduced arguments (far, from four frequencies on): a few float roundings;
        # below that single float entries, whose phases round at |s| r 2^-24
        tol = np.where(close, 1.3e-7, 1e-6 if nf >= 4 else 1e-6 + 4e-7 * np.abs(s).max())
        assert (err <= tol * mod + f64 + 1e-30).all(), (err / (tol * mod + f64 + 1e-30)).max()
