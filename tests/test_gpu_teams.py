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


@pytest.mark.parametrize("half_hour", [False, True])
@pytest.mark.parametrize("L,variant,low", [(160, 18, 19), (160, 22, 19), (192, 20, 21), (192, 24, 21), (224, 16, 15), (256, 6, 5)])
def test_tall_slabs_with_every_option(gga, model_dict, L, variant, low, half_hour):
    """The tall team kernels with the oxygen effect, mitotic death and incomplete
    repair, with fractions at hours or at half-hours, several instances per team:
    bit for bit the results of slabs of 64 rows, one launch per step."""
    print(f"tall slabs L={L} variant={variant} half_hour={half_hour}", flush=True)
    md = copy.deepcopy(model_dict)
    md.update(kappa=[4.0e-3, 2.0e-3, 2.0e-3], oer_max=3.0, oer_k=0.1, mitotic_death=1, repair_half_time=3.0, T_min=2)
    n, K, H = 140, 4, 12
    rng = np.random.default_rng(L + variant)
    dose = rng.choice([1.0, 2.0, 3.0], (n, K)).astype(np.float32)
    gap = rng.integers(1, 5, (n, K)).astype(np.int32) * (1 if half_hour else 2)
    nfrac = rng.integers(0, K + 1, n).astype(np.int32)
    nfrac[3] = K + 1                                           # refused
    horizon = rng.integers(0, H + 1, n).astype(np.int32)
    dd = _dev(dose, gap, nfrac)
    cfg = gga.make_cfg(L, H, 1, seed=5, dose_cap=100.0, half_hour=half_hour)
    lattice = np.full(n, L, np.int32)
    out = []
    try:
        for v, teams in ((variant, True), (low, False)):
            gga.set_variant(L, v)
            gga.set_team_options(teams)
            uneven = gga.simulate_uneven(md, cfg, *dd, lattice, horizon)
            out.append([x.cpu().numpy() for x in (*uneven, *gga.simulate(md, cfg, *dd, traj=True))])
    finally:
        gga.set_team_options(True)
        gga.clear_variant(L)
    for a, b in zip(*out):
        assert np.array_equal(a, b, equal_nan=True)
    final = out[0][2][np.arange(n) != 3]
    assert len(np.unique(final)) > 10 and (final > 0).all()    # fractions, marks and divisions told on the counts
