"""Matched-filter planes of images whose rows are whole cache lines of the plane,
cut into strips of equal width for narrow stamps (R <= 2): around one, two and
three strips; and the widest stamps (R = 11 at an FWHM of 8 px).  The tolerance
is that of FP32 sums: each plane value is a sum of at most (2R + 1) + (2R + 1)
products in two passes, so its error is below 2 (2R + 3) 2^-24 of the sum of the
products' magnitudes (positive weights: |D| in the place of D), plus one rounding
of the scale."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(16, 9), (112, 40), (208, 33), (224, 31), (240, 17), (256, 130), (288, 16), (448, 20), (480, 7), (496, 5),
          (512, 64), (752, 12)]


@pytest.mark.parametrize("dtype", ["float32", "float16"])
@pytest.mark.parametrize("R,fwhm", [(1, 0.7), (2, 1.5), (6, 4.6), (7, 5.4), (11, 8.0)])
def test_planes_of_equal_strips_match_oracle(R, fwhm, dtype):
    import torch
    import paper_2503_08854_amd as dt
    assert math.ceil(3 * fwhm / (2 * math.sqrt(2 * math.log(2)))) == R
    rng = np.random.default_rng(R)
    ctx = dt.Context(0)
    host, exps = [], []
    for k, (w, h) in enumerate(SHAPES):
        d, v = rng.standard_normal((h, w)).astype(dtype), rng.uniform(0.5, 2.0, (h, w)).astype(dtype)
        d[rng.random((h, w)) < 0.02] = np.nan
        host.append((d, v))
        exps.append(dict(t=float(k), obs=[1.0, 0.0, 0.0], crval=[10.0, 5.0], crpix=[1.0, 1.0],
                         cd=[-5e-5, 0.0, 0.0, 5e-5], width=w, height=h, fwhm=fwhm))
    patch = dt.Patch(ctx, exps, [torch.from_numpy(d).cuda() for d, _ in host],
                     [torch.from_numpy(v).cuda() for _, v in host])
    tol = (2 * (2 * R + 3) + 4) * 2.0 ** -24
    for k, (d, v) in enumerate(host):
        got = patch.plane(k).cpu().numpy().astype(np.float64)
        psi, phi = oracle.planes(d, v, fwhm)
        mag, _ = oracle.planes(np.abs(d), v, fwhm)
        assert (np.abs(got[..., 0] - psi) <= tol * mag + 1e-30).all(), SHAPES[k]
        assert (np.abs(got[..., 1] - phi) <= tol * phi + 1e-30).all(), SHAPES[k]
    patch.close()
    ctx.close()
