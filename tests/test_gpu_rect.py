"""The checkpoint walk's FP32 test of a predicted position against the image
rectangle: it may only drop samples that the exact walk shows to miss.  Images
of one pixel to wide fields, rotated, sheared and mirrored frames, a tangent
point far off the image, near, main-belt, distant and absurdly distant orbits:
valid counts equal those of the exact per-sample table, and S/N and flux are
the bits of the stack that uses no prediction."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

N = 6000


def _frames(shape, frame):
    g = synth.load_geometry("batched_small")["patches"][6]
    exps = sorted(synth.exposures_of(g), key=lambda x: abs(x["t"] - g["t0"]))[:60]
    out = []
    for i, x in enumerate(exps):
        W, H = shape if shape else (x["width"], x["height"])
        cd = np.array(x["cd"], float).reshape(2, 2)
        crpix = np.array(x["crpix"], float) - [0.5 * (x["width"] - W), 0.5 * (x["height"] - H)]
        c, s = np.cos(0.4 + 0.1 * i), np.sin(0.4 + 0.1 * i)
        if frame == "rotated":
            cd = cd @ np.array([[c, -s], [s, c]])
        elif frame == "sheared":
            cd = cd @ np.array([[-3.0, 1.0], [0.2, 0.5]])
        elif frame == "wide":       # the field's half-angle passes 10 degrees
            cd = cd * (0.2 / (abs(cd).max() * max(W, H) / 2) * 60.0)
        elif frame == "off":        # the tangent point lies ten image widths off the image
            crpix = crpix + [10.0 * W, -7.0 * H]
            # keep the image on the same sky: shift the tangent point's coordinates along
            d = cd @ np.array([10.0 * W, -7.0 * H])
            x = dict(x, crval=[x["crval"][0] + d[0] / np.cos(np.radians(x["crval"][1])), x["crval"][1] + d[1]])
        out.append(dict(x, width=W, height=H, cd=cd.reshape(np.shape(x["cd"])).tolist(), crpix=crpix.tolist()))
    return g, out


ORBITS = {"belt": ((2.0, 3.4), (0.0, 0.3)), "near": ((0.7, 1.4), (0.0, 0.7)), "distant": ((40.0, 2000.0), (0.0, 0.3)),
          "absurd": ((1e14, 1e17), (0.0, 0.1))}


@pytest.mark.parametrize("shape,frame,orbits", [
    (None, "plain", "belt"), (None, "plain", "near"), (None, "plain", "distant"), (None, "plain", "absurd"),
    (None, "rotated", "belt"), (None, "sheared", "belt"), (None, "wide", "belt"), (None, "wide", "near"),
    (None, "off", "belt"), (None, "off", "distant"), ((1, 1), "plain", "belt"), ((1, 64), "rotated", "belt"),
    ((37, 5), "sheared", "distant"), ((64, 64), "rotated", "near")])
def test_no_landing_sample_is_dropped(shape, frame, orbits):
    import torch
    import paper_2503_08854_amd as dt
    ctx = dt.Context(0)
    g, exps = _frames(shape, frame)
    D, V = synth.noise_images(exps, 5, 0.0, "f32", "cuda")
    patch = dt.Patch(ctx, exps, D, V)
    a, e = ORBITS[orbits]
    el = synth.candidate_orbits(g["grid_field"], N, 3, a, e, (0.0, 20.0))
    rng = np.random.default_rng(1)
    el[::7, 5] += rng.normal(0.0, 3e-4, el[::7].shape[0])   # some just off the fields
    o = dt.OrbitSet(el, g["t0"])
    plain = [x.view(torch.int32).cpu().numpy() for x in dt.stack(patch, o)]      # small: no prediction
    ctx.count_work(True)                                                        # counted: the checkpoint walk
    out = dt.stack(patch, o)
    w = ctx.work()
    ctx.count_work(False)
    walk = [x.view(torch.int32).cpu().numpy() for x in out]
    exact = dt.debug_samples(patch, o, np.arange(N))["flags"].cpu().numpy()
    valid = ((exact & 4) != 0).sum(1)
    live = walk[2] >= 0
    np.testing.assert_array_equal(walk[2][live], valid[live])
    for x, y in zip(walk, plain):
        np.testing.assert_array_equal(x, y)
    assert w["predicted"] > 0
    if shape is None and orbits != "absurd":
        assert (valid > 0).sum() > 20
    patch.close()
    ctx.close()
