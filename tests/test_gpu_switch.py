"""Where wavefronts of the checkpoint walk give their orbits up depends on the
size of the planes: on both sides of each line, stored, generated and listed
orbits that land often and seldom get the bits of the stack that uses no
prediction (a call small enough to be cut over a workgroup), and some
wavefronts do give up."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SIDE = 2048  # 32 MiB of planes an exposure
LINES = [256 << 20, 10 ** 9, 3 * 10 ** 9]  # bytes: between 7 and 8, 29 and 30, 89 and 90 exposures


@pytest.mark.parametrize("n_exp,above", [(7, 0), (8, 1), (29, 1), (30, 2), (89, 2), (90, 3)])
def test_stack_on_both_sides_of_the_lines(n_exp, above):
    import torch
    import paper_2503_08854_amd as dt
    g = synth.load_geometry("batched_small")["patches"][6]  # 90 exposures over 200 days
    exps = sorted(synth.exposures_of(g), key=lambda x: abs(x["t"] - g["t0"]))[:3]  # within a day of the orbits' epoch, repeated
    exps = [dict(x, t=x["t"] + 1e-3 * r) for r in range(30) for x in exps][:n_exp]
    exps = [dict(x, crpix=[x["crpix"][0] + 0.5 * (SIDE - x["width"]), x["crpix"][1] + 0.5 * (SIDE - x["height"])],
                 width=SIDE, height=SIDE) for x in exps]
    assert sum(8 * SIDE * SIDE * n_exp >= x for x in LINES) == above
    ctx = dt.Context(0)
    images = [torch.randn(SIDE, SIDE, device="cuda").half() for _ in range(4)]
    one = torch.ones(SIDE, SIDE, device="cuda").half()
    patch = dt.Patch(ctx, exps, [images[k % 4] for k in range(n_exp)], [one] * n_exp)
    n, m = 60000, 12000
    bits = lambda out, k: [x[:k].view(torch.int32).cpu().numpy() for x in out]  # noqa: E731
    field = dict(g["grid_field"])
    switched = 0
    for wide in (0.3, 1.0, 12.0):  # orbits that land in most images, in some, and seldom
        f = dict(field, half_w=field["half_w"] * wide, half_h=field["half_h"] * wide)
        el = synth.candidate_orbits(f, n, 3, g["grid"]["a"], g["grid"]["e"], g["grid"]["inc_deg"])
        ctx.count_work(True)
        big = bits(dt.stack(patch, dt.OrbitSet(el, g["t0"])), n)
        switched += ctx.work()["switched_waves"]
        ctx.count_work(False)
        small = bits(dt.stack(patch, dt.OrbitSet(el[:m], g["t0"])), m)
        assert (small[2] > 0).any()
        for a, b in zip(big, small):
            np.testing.assert_array_equal(a[:m], b)
        # a list long enough for the checkpoint walk: every orbit three times
        ids = torch.arange(n, device="cuda").repeat(3)
        out = dt.stack_ids(patch, dt.OrbitSet(el, g["t0"]), ids, torch.tensor([3 * n], device="cuda"))
        for a, b in zip(bits(out, n), big):
            np.testing.assert_array_equal(a, b)
        S = dt.orbit_sampler(f, g["t0"], g["grid"]["a"], g["grid"]["e"], g["grid"]["inc_deg"], 11)
        gen = bits(dt.stack_generated(patch, S, 7, n), n)
        for a, b in zip(gen, bits(dt.stack_generated(patch, S, 7, m), m)):
            np.testing.assert_array_equal(a[:m], b)
    assert switched > 0
    patch.close()
    ctx.close()
