"""Small stacks (a workgroup of wavefronts shares 64 orbits, each walking a
range of the exposures) against the one-wavefront walk: an orbit's S/N, flux
and valid count are the same bits whether it is stacked in a small call or in
one too large to be cut, at the sizes where the rule changes, for few and many
exposures, orbits outside the domain, exposures without an observer speed
bound and generated orbits."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

BIG = 49153  # the smallest call that is never cut


def _patch(ctx, n_exp, shared_epoch=False):
    import torch
    import paper_2503_08854_amd as dt
    g = synth.load_geometry("batched_small")["patches"][6]  # 90 exposures over 200 days
    exps = sorted(synth.exposures_of(g), key=lambda x: abs(x["t"] - g["t0"]))  # where the orbits are in the field first
    reps = -(-n_exp // len(exps))
    exps = [dict(x, t=x["t"] + 1e-3 * r) for r in range(reps) for x in exps][:n_exp]
    if shared_epoch:  # two observers at one epoch: no speed bound
        exps[-1] = dict(exps[-1], t=exps[0]["t"], obs=[v + 1e-5 for v in exps[0]["obs"]])
    D, V = synth.noise_images(exps, 5, 0.02, "f16", "cuda")
    return dt.Patch(ctx, exps, D, V), g


def _bits(out, n):
    import torch
    return [x[:n].view(torch.int32).cpu().numpy() for x in out]


@pytest.mark.parametrize("n_exp,shared", [(1, False), (2, False), (7, False), (9, True), (90, False), (104, False),
                                          (304, False), (312, False)])
def test_small_stack_equals_large(n_exp, shared):
    import torch
    import paper_2503_08854_amd as dt
    ctx = dt.Context(0)
    patch, g = _patch(ctx, n_exp, shared)
    el = synth.candidate_orbits(g["grid_field"], BIG, 3, g["grid"]["a"], g["grid"]["e"], g["grid"]["inc_deg"])
    el[::97, 1] = 1.5
    el[::89, 0] = np.nan
    ref = _bits(dt.stack(patch, dt.OrbitSet(el, g["t0"])), BIG)
    assert (ref[2] > 0).any() and (ref[2] == -1).any()
    for n in (1, 63, 65, 16384, 16385, 32769, 49152):
        got = _bits(dt.stack(patch, dt.OrbitSet(el[:n], g["t0"])), n)
        for a, b in zip(got, ref):
            np.testing.assert_array_equal(a, b[:n])
    ctx.count_work(True)  # counted launches run the checkpoint walk
    got = _bits(dt.stack(patch, dt.OrbitSet(el[:500], g["t0"])), 500)
    for a, b in zip(got, ref):
        np.testing.assert_array_equal(a, b[:500])
    patch.close()
    ctx.close()


@pytest.mark.parametrize("n_exp", [3, 90])
def test_small_generated_stack_equals_stored(n_exp):
    import torch
    import paper_2503_08854_amd as dt
    ctx = dt.Context(0)
    patch, g = _patch(ctx, n_exp)
    # a range of semi-major axes inside the observer's orbit: many draws miss
    for a_rng in ((0.8, 3.5), (0.3, 1.1)):
        S = dt.orbit_sampler(g["grid_field"], g["t0"], a_rng, (0.0, 0.6), (0.0, 30.0), 11)
        el = dt.generate_orbits(ctx, S, 5, BIG)
        ref = _bits(dt.stack(patch, dt.OrbitSet(el, g["t0"])), BIG)
        for n in (1, 65, 16384, 16385, 49152):
            got = _bits(dt.stack_generated(patch, S, 5, n), n)
            np.testing.assert_array_equal(got[2], ref[2][:n])
            for a, b in zip(got[:2], ref[:2]):
                np.testing.assert_array_equal(a, b[:n])
    patch.close()
    ctx.close()
