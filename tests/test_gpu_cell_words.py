"""Cell words against the oracle: ages past the word's 8 bits, stray bits of a
caller's words, marks without mitotic death, and thresholds that are no number
(needs an MI355X)."""
import copy

import numpy as np
import pytest
import torch

from oracle import protocol, sim
from oracle.model import Params
from parity_helpers import compare_cells, oracle_certain_prefix, oracle_step_detail, to_field_units

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def with_options(md, **kw):
    d = copy.deepcopy(md)
    d.update(kw)
    return d


OXYGEN_MITOTIC = {"oer_max": 3.0, "oer_k": 0.1, "mitotic_death": 1}


@pytest.mark.parametrize("options", [{}, OXYGEN_MITOTIC], ids=["plain", "oxygen_mitotic"])
@pytest.mark.parametrize("A0", [256, 257, 300, 1000, 9000, 70000])
def test_seeded_ages_saturate_at_255(gga, model_dict, A0, options):
    """Ages drawn from 0 .. A0-1 saturate at 255, the word's largest: the live
    counts of a resident side, of slabs as teams and one launch per step, and of
    quasi-3D with one slot equal the oracle's, with a fraction in the first hour
    (its classes read the seeded ages) and one later."""
    print(f"seeded ages A0={A0} {options}", flush=True)
    md = with_options(model_dict, A0=A0, **options)
    prm = Params.from_dict(md)
    H, seed = 10, 3
    dose, gap, nfrac = np.array([[2.0, 2.0]] * 2, np.float32), np.array([[0, 5], [4, 5]], np.int32), np.array([2, 2], np.int32)
    dd = _dev(dose, gap, nfrac)
    runs = {}
    for L in (64, 160):
        cfg = gga.make_cfg(L, H, 1, seed=seed, dose_cap=100.0)
        runs[L, "simulate"] = gga.simulate(md, cfg, *dd, traj=True)[2]
        if L == 64:
            runs[L, "quasi-3D"] = gga.simulate_q3(md, cfg, 1, *dd, traj=True)[2]
            cells = gga.state_init(md, cfg, 1)[1].cpu().numpy().view(np.uint16)[0]
            assert np.array_equal(cells, sim.init_state(prm, L, 0, 0, seed)[1])
        else:
            try:
                gga.set_team_options(False)
                runs[L, "per step"] = gga.simulate(md, cfg, *dd, traj=True)[2]
            finally:
                gga.set_team_options(True)
    for L in (64, 160):
        for p in range(2):
            ev = protocol.events(dose[p], gap[p], 2, H, prm)
            ref, certain = oracle_certain_prefix(prm, L, H, 10, ev, p, 0, seed)
            assert certain == H, (L, p, certain)
            for (side, form), traj in runs.items():
                assert side != L or np.array_equal(traj[p, 0].cpu().numpy(), ref), (L, form, p)


def drawn_words(rng, L, prm):
    """Words of every state and age in a sparse lattice, and fields that keep
    cells cycling in its upper half and starving in its lower one."""
    state = rng.choice(4, (L, L), p=[0.6, 0.2, 0.1, 0.1])
    cells = np.where(state > 0, state | (rng.integers(0, 256, (L, L)) << 2), 0)
    fields = np.empty((3, L, L))
    for f in range(3):
        fields[f] = prm.init[f]
    fields[0, L // 2:] = 0.5 * (prm.th_Od + prm.th_Oq)
    return fields, cells


def one_step(gga, md, L, variant, fields, cells, n, seed):
    """The words after step n of the given state, and the oracle's with its
    counted sites."""
    prm = Params.from_dict(md)
    cfg = gga.make_cfg(L, n + 1, 1, seed=seed, dose_cap=20.0)
    protos = _dev(np.zeros((1, 1), np.float32), np.zeros((1, 1), np.int32), np.zeros(1, np.int32))
    units = to_field_units(fields, prm)
    f_d, c_d = _dev(units[None], cells.astype(np.uint16).view(np.int16)[None])
    gga.state_run_variant(md, cfg, variant, *protos, n, 1, f_d, c_d)
    _, ref, counted = oracle_step_detail(fields, cells, n, None, 0, 0, seed, prm, 10)
    return c_d.cpu().numpy().view(np.uint16)[0], ref, counted


@pytest.mark.parametrize("L,variant", [(64, 0), (64, 7), (96, 9), (128, 2), (128, 4), (160, 22), (256, 6)])
@pytest.mark.parametrize("options", [{}, {"oer_max": 3.0, "oer_k": 0.1}], ids=["plain", "oxygen"])
def test_stray_bits_of_a_callers_words_are_not_read(gga, model_dict, L, variant, options):
    """Bits 10-13 and 15 of a caller's words mean nothing: one step gives the
    oracle's words, which hold state, age and mark only."""
    print(f"stray bits L={L} variant={variant} {options}", flush=True)
    md = with_options(model_dict, **options)
    rng = np.random.default_rng(L + variant)
    fields, cells = drawn_words(rng, L, Params.from_dict(md))
    stray = rng.integers(0, 2, (L, L)) * (rng.integers(0, 16, (L, L)) << 10 | rng.integers(0, 2, (L, L)) << 15)
    got, ref, counted = one_step(gga, md, L, variant, fields, cells | stray, 3, 11)
    assert compare_cells(got, ref, counted)[0] == 0 and counted.mean() < 0.1


@pytest.mark.parametrize("L,variant", [(64, 0), (64, 7), (96, 9), (128, 2), (128, 4), (160, 22), (256, 6)])
@pytest.mark.parametrize("options", [{}, {"oer_max": 3.0, "oer_k": 0.1}], ids=["plain", "oxygen"])
def test_marks_are_kept_without_mitotic_death(gga, model_dict, L, variant, options):
    """Live cells marked for mitotic death keep the mark in a step without it,
    cycling, starving or dividing (a daughter has none); dead ones drop it.
    Their words equal the oracle's, which has marked cells divide like others."""
    print(f"marks without mitotic death L={L} variant={variant} {options}", flush=True)
    md = with_options(model_dict, **options)
    rng = np.random.default_rng(L + variant)
    fields, cells = drawn_words(rng, L, Params.from_dict(md))
    cells |= np.where(cells & 3, rng.integers(0, 2, (L, L)) << 14, 0)
    got, ref, counted = one_step(gga, md, L, variant, fields, cells, 3, 11)
    for state, age in ((1, 1), (1, 0), (2, 1)):               # cycling cells, parents and starving cells with a mark
        assert ((ref >> 14 == 1) & (ref & 3 == state) & ((ref >> 2 & 255 > 0) == age)).sum() > 10, (state, age)
    assert compare_cells(got, ref, counted)[0] == 0 and counted.mean() < 0.1


@pytest.mark.parametrize("L", [64, 96, 128, 160, 256])
@pytest.mark.parametrize("theta", ["theta_O_quiesce", "theta_G_quiesce", "theta_O_death", "theta_G_death", "theta_H_death"])
def test_a_threshold_that_is_no_number_is_passed_everywhere(gga, model_dict, L, theta):
    """With a NaN threshold every cell counts as beyond it, whatever the other
    cells of its wave: all die in the first step, or all turn quiescent and none
    divides."""
    print(f"NaN threshold {theta} L={L}", flush=True)
    md = with_options(model_dict, **{theta: float("nan")})
    protos = _dev(np.zeros((1, 1), np.float32), np.zeros((1, 1), np.int32), np.zeros(1, np.int32))
    traj = gga.simulate(md, gga.make_cfg(L, 20, 2, seed=1), *protos, traj=True)[2].cpu().numpy()
    assert np.all(traj == (113 if "quiesce" in theta else 0))
