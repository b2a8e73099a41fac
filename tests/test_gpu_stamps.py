"""Cell stamps at the edges of the kernel's work split: batches of four usable
exposures, 64 exposures per packing round, and exposure lists whose track
points take less LDS than the 441 node sums (MI355X)."""
import numpy as np
import pytest

import oracle
from test_gpu_learned import _lattice_stamps_oracle, cells  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_exp", [1, 3, 4, 5, 63, 64, 65, 70, 71, 1024])
def test_stamps_over_exposure_counts(cells, n_exp):  # noqa: F811
    import torch
    import paper_2503_08854_amd as dt
    c = cells
    cg = c["g"]["cell_grid"]
    have = len(c["exps"])
    pick = [i % have for i in range(n_exp)]
    exps = [c["exps"][i] for i in pick]
    Dt, Vt = c["keep"]
    patch = dt.Patch(c["ctx"], exps, [Dt[i] for i in pick], [Vt[i] for i in pick])
    reps_el = c["el"][::cg["cell_size"]][:12]
    out = dt.cell_stamps(patch, dt.OrbitSet(reps_el, c["g"]["t0"]), cg["da"], cg["dm"])
    torch.cuda.synchronize()
    st = out["stamps"].cpu().numpy()
    one = [oracle.planes(d, v, x["fwhm"]) for d, v, x in zip(c["D"], c["V"], c["exps"])]
    want, band = _lattice_stamps_oracle(dict(c, exps=exps), reps_el, cg["da"], cg["dm"], planes=[one[i] for i in pick])
    err = np.abs(st - want) / np.maximum(1.0, np.abs(want))
    assert np.all(err[~band] < 1e-4), err[~band].max()   # the bound of the stamps' other oracle comparisons
    assert (~band).sum() >= 6
    ft = out["feats"].cpu().numpy()
    for r in range(len(reps_el)):
        row, col = divmod(int(np.argmax(st[r])), 21)   # the first node holding the maximum
        assert ft[r, 11] == np.float32((col - 10) / 10.0) and ft[r, 12] == np.float32((row - 10) / 10.0)
    patch.close()
