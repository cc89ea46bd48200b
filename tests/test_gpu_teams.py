"""Teams of slabs that take several instances in turn: waits that run out, the
tall slabs with every option (needs an MI355X)."""
import copy

import numpy as np
import pytest
import torch

from paper_2303_08123_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


@pytest.mark.parametrize("spin_limit", [-1, 0, 1, 4, 32])
@pytest.mark.parametrize("L,n", [(256, 150), (160, 300)])
def test_waits_that_run_out_spoil_no_other_instance(gga, model_dict, L, n, spin_limit):
    """More instances than teams, with so small a limit that some waits run out
    (all of them: -1).  Every instance is right or negative (its fitness NaN), and
    negative only if it has an exchange, i.e. two steps or more; a refused protocol
    keeps its -1; the next call with the usual limit is right."""
    print(f"run-out L={L} n={n} spin_limit={spin_limit}", flush=True)
    md = copy.deepcopy(model_dict)
    md["kappa"] = [4.0e-3, 2.0e-3, 2.0e-3]
    dose, gap, nfrac = workloads.random_protocols(n, 4, seed=L, kmin=1)
    nfrac[n // 2] = 5                                          # refused
    horizon = np.random.default_rng(n).integers(0, 7, n).astype(np.int32)
    dd = _dev(dose, gap, nfrac)
    cfg = gga.make_cfg(L, 0, 1, seed=9, dose_cap=100.0)
    lattice = np.full(n, L, np.int32)
    run = lambda: [x.cpu().numpy() for x in gga.simulate_uneven(md, cfg, *dd, lattice, horizon)]
    ref = run()
    try:
        gga.set_team_options(True, spin_limit)
        live, fit = run()
    finally:
        gga.set_team_options(True)
    valid = np.arange(n) != n // 2
    lost = (live[:, 0] < 0) & valid
    print(f"{lost.sum()} of {(valid & (horizon >= 2)).sum()} ran out", flush=True)
    assert np.array_equal(live[~lost], ref[0][~lost]) and np.array_equal(fit[~lost], ref[1][~lost], equal_nan=True)
    assert np.all(horizon[lost] >= 2) and np.isnan(fit[lost]).all()
    if spin_limit < 0:
        assert np.array_equal(lost, valid & (horizon >= 2))
    for a, b in zip(run(), ref):
        assert np.array_equal(a, b, equal_nan=True)
