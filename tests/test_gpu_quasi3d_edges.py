"""Edges of the quasi-3D sub-steps: every window geometry (one instance, and more
instances than compute units), lattices that fill a window, exceed it by a
site or leave most of it empty, odd pitches, single and odd sub-steps and
more than one launch takes, fields that reach the clamp (needs an MI355X)."""
import copy

import numpy as np
import pytest
import torch

from oracle.model import Params
from parity_helpers import compare_cells, field_units, from_field_units, oracle_step_detail, to_field_units

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


@pytest.mark.parametrize("L,n,substeps", [
    (8, 1, 10), (8, 257, 64), (33, 2, 3), (63, 300, 10), (64, 1, 17), (64, 257, 10), (65, 1, 10), (65, 64, 10), (65, 65, 9),
    (97, 300, 10), (127, 1, 16), (127, 260, 20), (128, 1, 10), (128, 28, 16), (128, 29, 10), (128, 3, 33), (129, 3, 10),
    (129, 260, 10), (161, 90, 1), (225, 30, 16), (300, 1, 21), (511, 1, 10)])
def test_one_step_of_drawn_states_matches_the_oracle(gga, model_dict, L, n, substeps):
    """One slot per site: one step of the 2D model from drawn fields (O and G
    between 0 and a few uptakes) and cells.  A sub-step rounds each value by at
    most 8 units of 2^-24 of the largest magnitude and passes errors on without
    enlarging them; the same bound widens the window of the counted sites.  All
    instances start from the same fields and cells; the first and last are
    compared with the oracle, the fields of the others with the first's."""
    print(f"quasi-3D drawn state L={L} n={n} substeps={substeps}", flush=True)
    md = copy.deepcopy(model_dict)
    md["kappa"] = [4.0e-3, 2.0e-3, 2.0e-3]
    prm = Params.from_dict(md)
    seed, step = 23, 3
    rng = np.random.default_rng(L + substeps)
    g, rho = field_units(prm)
    top = np.array([6 * prm.kappa[0], 6 * prm.kappa[1], prm.ghost[2] + 0.5])
    fields = to_field_units(top[:, None, None] * rng.random((3, L, L)), prm)
    start = from_field_units(fields, prm)
    state = rng.choice(4, (L, L), p=[0.6, 0.25, 0.1, 0.05])
    state[: L // 3] = 0
    cells = np.where(state > 0, state | (rng.integers(0, 256, (L, L)) << 2), 0).astype(np.uint16)
    cells[state == 3] = 3
    cfg = gga.make_cfg(L, step + 1, 1, seed=seed, dose_cap=20.0, substeps=substeps)
    protos = _dev(np.zeros((n, 1), np.float32), np.zeros((n, 1), np.int32), np.zeros(n, np.int32))
    f_d = torch.from_numpy(fields).cuda()[None].repeat(n, 1, 1, 1)
    c_d = torch.from_numpy(cells.view(np.int16)).cuda()[None, None].repeat(n, 1, 1, 1)
    gga.q3_run(md, cfg, 1, *protos, step, 1, f_d, c_d)
    assert torch.equal(f_d, f_d[:1].expand_as(f_d))
    got = f_d[0].cpu().numpy().astype(np.float64)
    bound = (8 * substeps + 2) * 2.0 ** -24 * np.abs(fields).max()
    for p in {0, n - 1}:
        f_ref, c_ref, counted = oracle_step_detail(start, cells.astype(np.int64), step, None, p, 0, seed, prm, substeps,
                                                   abs_window=2 * bound * np.abs(rho).max())
        assert np.abs(got - (f_ref - g) / rho).max() <= bound
        bad, _ = compare_cells(c_d[p, 0].cpu().numpy().view(np.uint16), c_ref, counted)
        assert bad == 0 and counted.mean() < 0.1
