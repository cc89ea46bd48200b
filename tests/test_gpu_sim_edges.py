"""Edges of the simulation kernels: odd and single sub-steps, fields that reach
the clamp and fields that cannot, tall slabs, and teams that take several
instances in turn at every slab height (needs an MI355X)."""
import copy

import numpy as np
import pytest
import torch

from oracle import sim
from oracle.model import Params
from paper_2303_08123_amd import workloads
from parity_helpers import compare_cells, field_units, from_field_units, oracle_step_detail, to_field_units

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def high_uptake(md):
    d = copy.deepcopy(md)
    d["kappa"] = [4.0e-3, 2.0e-3, 2.0e-3]
    return d


@pytest.mark.parametrize("L,variant,substeps,low", [
    (64, 0, 1, True), (64, 7, 3, False), (64, 8, 2, True), (96, 9, 5, True), (128, 2, 1, False), (128, 3, 11, True),
    (160, 18, 3, True), (160, 22, 10, False), (192, 20, 7, True), (224, 16, 9, True), (256, 5, 1, True),
    (256, 6, 13, True), (256, 6, 16, False)])
def test_one_step_of_drawn_states_matches_the_oracle(gga, model_dict, L, variant, substeps, low):
    """One step from drawn fields and cells.  `low`: O and G between 0 and a few
    uptakes, so that many sites reach the clamp; else fields that stay clear of
    it.  A sub-step rounds each value by at most 8 units of 2^-24 of the largest
    magnitude (constants included) and passes errors on without enlarging them;
    the same bound widens the window of the counted sites."""
    print(f"drawn state L={L} variant={variant} substeps={substeps} low={low}", flush=True)
    md = high_uptake(model_dict)
    prm = Params.from_dict(md)
    seed, n = 17, 3
    rng = np.random.default_rng(L + substeps)
    g, rho = field_units(prm)
    top = np.array([6 * prm.kappa[0], 6 * prm.kappa[1], prm.ghost[2] + 0.5]) if low else np.array(prm.ghost) + 0.2
    bottom = np.array([0.0, 0.0, prm.ghost[2]]) if low else 0.7 * np.array(prm.ghost)
    phys = bottom[:, None, None] + (top - bottom)[:, None, None] * rng.random((3, L, L))
    fields = to_field_units(phys, prm)
    start = from_field_units(fields, prm)
    state = rng.choice(4, (L, L), p=[0.6, 0.25, 0.1, 0.05])
    state[: L // 4] = 0                                        # rows without a cell
    cells = np.where(state > 0, state | (rng.integers(0, 256, (L, L)) << 2), 0).astype(np.uint16)
    cells[state == 3] = 3
    cfg = gga.make_cfg(L, n + 1, 1, seed=seed, dose_cap=20.0, substeps=substeps)
    protos = _dev(np.array([[2.5]], np.float32), np.array([[n]], np.int32), np.array([0], np.int32))
    f_d, c_d = _dev(fields[None], cells.view(np.int16)[None])
    gga.state_run_variant(md, cfg, variant, *protos, n, 1, f_d, c_d)
    got = f_d.cpu().numpy()[0].astype(np.float64)
    bound = (8 * substeps + 2) * 2.0 ** -24 * np.abs(fields).max()
    f_ref, c_ref, counted = oracle_step_detail(start, cells.astype(np.int64), n, None, 0, 0, seed, prm, substeps,
                                               abs_window=2 * bound * np.abs(rho).max())
    if low:                                                    # sites are clamped by the first sub-step
        first = oracle_step_detail(start, cells.astype(np.int64), n, None, 0, 0, seed, prm, 1)[0]
        assert (first[0] == 0).any()
    assert np.abs(got - (f_ref - g) / rho).max() <= bound
    assert counted.mean() < 0.1
    bad, _ = compare_cells(c_d.cpu().numpy().view(np.uint16)[0], c_ref, counted)
    assert bad == 0


@pytest.mark.parametrize("L,n,substeps", [
    (160, 1, 10), (160, 70, 10), (160, 131, 10), (192, 65, 10), (192, 90, 10), (192, 300, 10), (224, 49, 10), (224, 67, 10),
    (256, 41, 10), (256, 66, 10), (256, 150, 10), (160, 5, 17), (192, 90, 24), (224, 9, 18), (256, 50, 23), (256, 9, 1)])
def test_teams_in_turns_equal_one_launch_per_step(gga, model_dict, L, n, substeps):
    """Counts of instances on both sides of the slab heights' limits, few
    sub-steps and so many that the halo rows come field by field, with mixed
    horizons (none among them) and invalid protocols: teams that take several
    instances in turn give the per-step form's results bit for bit, as do the
    uniform batch's."""
    print(f"teams in turns L={L} n={n} substeps={substeps}", flush=True)
    md = high_uptake(model_dict)
    K = 4
    dose, gap, nfrac = workloads.random_protocols(n, K, seed=L + n, kmin=1)
    nfrac[n // 2] = K + 1                                      # refused
    horizon = np.random.default_rng(n).integers(0, 7, n).astype(np.int32)
    dd = _dev(dose, gap, nfrac)
    lattice = np.full(n, L, np.int32)
    out = {}
    try:
        for teams in (True, False):
            gga.set_team_options(teams)
            cfg = gga.make_cfg(L, 3, 1, seed=9, dose_cap=100.0, substeps=substeps)
            uneven = gga.simulate_uneven(md, cfg, *dd, lattice, horizon)
            even = gga.simulate(md, cfg, *dd, traj=True)
            out[teams] = [x.cpu().numpy() for x in (*uneven, *even)]
    finally:
        gga.set_team_options(True)
    for a, b in zip(out[True], out[False]):
        assert np.array_equal(a, b, equal_nan=True)
    valid = np.arange(n) != n // 2
    assert np.all(out[True][0][valid] > 0) and np.all(out[True][0][~valid] == -1)


@pytest.mark.parametrize("n", [257, 300, 700])
def test_many_small_instances_equal_few(gga, model_dict, n):
    """More 64 x 64 instances than compute units run in another geometry: the
    same results as in batches of at most one instance per compute unit."""
    md = high_uptake(model_dict)
    dose, gap, nfrac = workloads.random_protocols(n, 4, seed=n, kmin=1)
    cfg = gga.make_cfg(64, 30, 1, seed=3, dose_cap=100.0)
    live, fit, traj = gga.simulate(md, cfg, *_dev(dose, gap, nfrac), traj=True)
    few = [x.cpu().numpy() for x in gga.simulate(md, cfg, *_dev(dose[:200], gap[:200], nfrac[:200]), traj=True)]
    for a, b in zip((live, fit, traj), few):
        assert np.array_equal(a.cpu().numpy()[:200], b)
    assert (live.cpu().numpy() > 0).all()
