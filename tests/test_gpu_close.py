"""The checkpoint walk's test of a predicted position for objects 0.04 to 0.07
AU away: its allowance for FP32 rounding is small against the image, so that
few samples that miss are solved, and none that lands is dropped.

All exposures lie within 0.01 days, where the prediction's own error is below a
pixel.  The allowance is 2^-23 of 2 |r| + |o| + 7 |p| + 13 (T |v| + T^2 |h|) + 8 T
vobs (sums of sizes; |r| <= 1.07, |o| = 1, |p| <= 0.07, |v|, vobs <= 0.018 AU/day,
T = 12 days; a sum of sizes is at most sqrt(3) lengths): below 1.4e-6 AU, 36 px
at 0.04 AU.  So at most (64 + 2 x 36 + 4)^2 of the field's pixels can be queued
for every 64^2 that land, less than 4.9 times as many; 1.5 times that is allowed
for the orbits' uneven density."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

ARCSEC = np.pi / 180 / 3600
EPS = np.radians(84381.448 / 3600)


def _equatorial(v):
    return np.array([v[0], np.cos(EPS) * v[1] - np.sin(EPS) * v[2], np.sin(EPS) * v[1] + np.cos(EPS) * v[2]])


def test_rounding_allowance_of_close_objects():
    import torch
    import paper_2503_08854_amd as dt
    c = synth.unit(np.array([1.0, 0.0, 0.01]))
    east = synth.unit(np.cross([0.0, 0.0, 1.0], c))
    half = 1024 * 0.2 * ARCSEC
    field = dict(obs=[1.0, 0.0, 0.0], center=c.tolist(), east=east.tolist(), north=np.cross(c, east).tolist(),
                 half_w=half, half_h=half)
    n, t0, side = 400000, 100.0, 64
    q = _equatorial(c)
    crval = [float(np.degrees(np.arctan2(q[1], q[0])) % 360), float(np.degrees(np.arcsin(q[2])))]
    scale = 0.2 / 3600
    exps = [dict(t=t0 + dt_, obs=[1.0, 0.0172 * dt_, 0.0], crval=crval, crpix=[side / 2 + 0.5, side / 2 + 0.5],
                 cd=[-scale, 0.0, 0.0, scale], width=side, height=side, fwhm=2.5)
            for dt_ in (-0.005, -0.002, 0.0, 0.003, 0.005)]
    ctx = dt.Context(0)
    D = [torch.randn(side, side, device="cuda") for _ in exps]
    V = [torch.ones(side, side, device="cuda") for _ in exps]
    patch = dt.Patch(ctx, exps, D, V)
    el = synth.candidate_orbits(field, n, 5, (1.042, 1.068), (0.0, 0.002), (0.0, 3.0))
    orb = dt.OrbitSet(el, t0)
    ctx.count_work(True)  # counted launches run the checkpoint walk
    nv = dt.stack(patch, orb)[2].cpu().numpy()
    w = ctx.work()
    ctx.count_work(False)
    exact = dt.debug_samples(patch, orb, np.arange(20000))["flags"].cpu().numpy()
    np.testing.assert_array_equal(nv[:20000], ((exact & 4) != 0).sum(1))
    landed = int(nv.sum())
    assert landed > 500
    assert w["switched_waves"] == 0 and w["queued_solves"] >= landed
    assert w["queued_solves"] <= 1.5 * 4.9 * landed, (w["queued_solves"], landed)
    patch.close()
    ctx.close()
