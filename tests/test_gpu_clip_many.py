"""Outlier trimming of many candidates (four to a wavefront) against calls of few
(one to a wavefront): the same bits for every candidate, at the call sizes and
exposure counts where the route changes, with ids and orbits outside the
domain among them."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_exp", [1, 17, 128, 129])
def test_many_candidates_equal_few(n_exp):
    import torch
    import paper_2503_08854_amd as dt
    g = synth.load_geometry("batched_small")["patches"][6]
    exps = sorted(synth.exposures_of(g), key=lambda x: abs(x["t"] - g["t0"]))[:30]
    exps = [dict(x, t=x["t"] + 1e-3 * r) for r in range(5) for x in exps][:n_exp]
    ctx = dt.Context(0)
    D, V = synth.noise_images(exps, 5, 0.02, "f32", "cuda")
    for d in D:
        d[::40, ::30] = 80.0  # artifacts to trim
    patch = dt.Patch(ctx, exps, D, V)
    n = 9000
    el = synth.candidate_orbits(g["grid_field"], n, 3, g["grid"]["a"], g["grid"]["e"], g["grid"]["inc_deg"])
    el[::97, 1] = 1.5
    orb = dt.OrbitSet(el, g["t0"])
    ids = torch.arange(n, device="cuda")
    ids[5::1001] = -1
    ids[6::1001] = n
    bits = lambda out: [x.view(torch.int32).cpu().numpy() for x in out]  # noqa: E731
    few = [np.concatenate(p) for p in zip(*(bits(dt.clip_candidates(patch, orb, part)) for part in ids.split(3000)))]
    assert (few[2] > 0).any() and (few[2] == 0).any()
    if n_exp > 1:
        plain = dt.stack(patch, orb)[2].cpu().numpy()
        assert (few[2] < np.maximum(plain, 0)).any()  # something was trimmed
    for m in (8191, 8192, 8193, 8195, n):
        for a, b in zip(bits(dt.clip_candidates(patch, orb, ids[:m])), few):
            np.testing.assert_array_equal(a, b[:m])
    patch.close()
    ctx.close()
