"""The scorer's training kernel at the edges of its work split: one cell, a
workgroup's second slot empty, one more cell than there are slots, and batches
whose 1152-deep layer is summed in four, two and one parts (MI355X)."""
import numpy as np
import pytest

from oracle import nn_ref as nn
from test_gpu_learned import _bf16, _grad_bf16_model, _rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scorer():
    import paper_2503_08854_amd as dt
    sc = dt.Scorer(dt.Context(0), max_batch=32768, seed=3)
    p = nn.unflatten(sc.params().double().cpu().numpy())
    for k in p:
        p[k] = _bf16(p[k])
    rng = np.random.default_rng(5)
    for k in p:
        if k.startswith("b"):   # non-zero biases
            p[k] = rng.standard_normal(p[k].shape).astype(np.float32).astype(np.float64) * 0.125
    import torch
    th = nn.flatten(p).astype(np.float32)
    sc.set_params(torch.from_numpy(th).cuda())
    return sc, th.astype(np.float64)


def _batch(B, seed=11):
    import torch
    rng = np.random.default_rng(seed)
    X, F = _bf16(rng.standard_normal((B, 21, 21))), _bf16(rng.standard_normal((B, 16)))
    Y = (rng.random(B) < 0.5).astype(np.float64)
    return X, F, Y, (torch.from_numpy(X).to(torch.bfloat16).cuda(), torch.from_numpy(F).to(torch.bfloat16).cuda(),
                     torch.from_numpy(Y).float().cuda())


# 256 workgroups of two cells: 256 | 257 fills the second slot, 512 | 513 starts a second pass
@pytest.mark.parametrize("B", [1, 2, 255, 256, 257, 512, 513])
def test_gradient_and_logits_over_batch_sizes(scorer, B):
    sc, th = scorer
    X, F, Y, (Xt, Ft, Yt) = _batch(B)
    z = sc.forward(Xt, Ft).cpu().numpy()
    # a cell's logit does not depend on its place in the batch: the same products in the same order
    for i in sorted({0, B // 2, B - 1}):
        one = sc.forward(Xt[i:i + 1].contiguous(), Ft[i:i + 1].contiguous()).cpu().numpy()
        np.testing.assert_array_equal(one, z[i:i + 1])
    assert _rel(z, nn.forward(th, X, F)) < 1e-2
    loss, g = sc.grad(Xt, Ft, Yt)
    assert float(loss.cpu()[0]) == pytest.approx(nn.bce_with_logits(z.astype(np.float64), Y), rel=1e-5)
    got, want = nn.unflatten(g.double().cpu().numpy()), nn.unflatten(_grad_bf16_model(th, X, F, Y))
    errs = {k: _rel(got[k], want[k]) for k in got}
    assert all(v < 3e-2 for v in errs.values()), errs   # the bound of the model comparison at B = 32
    again = sc.grad(Xt, Ft, Yt)[1]
    np.testing.assert_array_equal(again.cpu().numpy(), g.cpu().numpy())   # sums in a fixed order


# 16 321 cells and more sum the 1152-deep layer in two parts, 32 705 and more in one
@pytest.mark.parametrize("B", [16320, 16321, 32704, 32705, 32768])
def test_gradient_of_a_repeated_batch(scorer, B):
    import torch
    sc, th = scorer
    n = 51
    X, F, Y, (Xt, Ft, Yt) = _batch(n, seed=B)
    i = torch.arange(B, device="cuda") % n
    z = sc.forward(Xt[i].contiguous(), Ft[i].contiguous())
    assert torch.equal(z, z[:n][i])
    # logits of another split differ by FP32 rounding and the BF16 roundings it moves
    z0 = sc.forward(Xt, Ft).cpu().numpy()
    assert _rel(z[:n].cpu().numpy(), z0) < 2e-3
    g = nn.unflatten(sc.grad(Xt[i].contiguous(), Ft[i].contiguous(), Yt[i].contiguous())[1].double().cpu().numpy())
    k = np.arange(B) % n
    count = np.bincount(k, minlength=n)
    # the reference gradient of each cell on its own, weighted by how often the batch holds it
    want = sum(c * _grad_bf16_model(th, X[j:j + 1], F[j:j + 1], Y[j:j + 1]) for j, c in enumerate(count)) / B
    want = nn.unflatten(want)
    errs = {k: _rel(g[k], want[k]) for k in g}
    assert all(v < 3e-2 for v in errs.values()), errs


def test_step_refreshes_every_copy_of_the_weights(scorer):
    import paper_2503_08854_amd as dt
    _, th = scorer
    X, F, Y, (Xt, Ft, Yt) = _batch(300, seed=4)
    sc = dt.Scorer(dt.Context(0), max_batch=300, seed=9)
    other = dt.Scorer(dt.Context(0), max_batch=300, seed=1)
    for _ in range(3):
        sc.train_step(Xt, Ft, Yt, 1e-2)
    other.set_params(sc.params())
    for f in ("forward", "infer"):
        np.testing.assert_array_equal(getattr(sc, f)(Xt, Ft).cpu().numpy(), getattr(other, f)(Xt, Ft).cpu().numpy())
    np.testing.assert_array_equal(sc.grad(Xt, Ft, Yt)[1].cpu().numpy(), other.grad(Xt, Ft, Yt)[1].cpu().numpy())


# 16 cells per group, 256 groups at a time
@pytest.mark.parametrize("B", [1, 15, 16, 17, 4096, 4097, 4111, 16321])
def test_inference_equals_the_training_forward(scorer, B):
    """A batch whose 1152-deep layer is summed in two halves takes the same products in the same order as the
    inference kernel: equal to the last bit, whole batches, slices of them and row lists alike."""
    import torch
    sc, _ = scorer
    n = 16321
    _, _, _, (Xt, Ft, _) = _batch(257, seed=7)
    i = torch.arange(n, device="cuda") * 11 % 257
    Xn, Fn = Xt[i].contiguous(), Ft[i].contiguous()
    z = sc.forward(Xn, Fn)
    assert torch.equal(sc.infer(Xn[:B].contiguous(), Fn[:B].contiguous()), z[:B])
    rows = torch.randperm(n, generator=torch.Generator().manual_seed(B))[:B].cuda()
    out = torch.full((n,), -7.0, device="cuda")
    sc.infer_rows(Xn, Fn, rows, out=out)
    want = torch.full((n,), -7.0, device="cuda")
    want[rows] = z[rows]
    assert torch.equal(out, want)
