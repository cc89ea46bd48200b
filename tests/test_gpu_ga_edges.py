"""Device ranking and breeding at the edges of their lane groups (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import ga as oga

pytestmark = pytest.mark.gpu

ALPHA = dict(dose_quantum=0.5, dose_q=[1, 2, 3, 5], gaps=[6, 12, 24, 60], kmin=1, kmax=64, cap=40.0)


# group widths 16, 32 and 64 at, below and above their limits; populations below
# one workgroup, ragged, and of several workgroups; everything elite; parents
# far over the cap (many guard steps)
@pytest.mark.parametrize("N,K,elite,k,cap", [
    (2, 1, 0, 1, 40.0), (15, 2, 15, 4, 40.0), (64, 16, 1, 4, 40.0), (65, 17, 0, 3, 40.0), (257, 32, 7, 9, 24.0),
    (33, 33, 2, 64, 40.0), (130, 64, 3, 4, 40.0), (1021, 5, 101, 4, 6.0),
])
def test_breed_edges_match_oracle(N, K, elite, k, cap):
    import paper_2303_08123_amd as gga
    rng = np.random.default_rng(N * 100 + K)
    alpha = dict(ALPHA, cap=cap)
    dose = rng.choice([0.5, 1.0, 1.5, 2.5], size=(N, K)).astype(np.float32)
    gap = rng.choice(alpha["gaps"], size=(N, K)).astype(np.int32)
    # ties, both zeros, infinities and NaN
    fitness = rng.choice(np.array([0.0, -0.0, 1.5, -2.0, 1e30, np.inf, -np.inf, np.nan, 3e-42], np.float32), size=N)
    cfg = gga.make_ga(n_elite=elite, tournament_k=k, p_cross=0.8, p_mut=0.3, seed=0xFEDCBA987, crossover="two_point",
                      mutation=("gene", "swap", "raise"))
    al = gga.make_alphabet(alpha["dose_quantum"], alpha["dose_q"], alpha["gaps"], 1, K, cap)
    g_t = torch.tensor([11], dtype=torch.int32, device="cuda")
    order, pos, nd, ng = gga.ga_breed(cfg, al, torch.from_numpy(fitness).cuda(), torch.from_numpy(dose).cuda(),
                                      torch.from_numpy(gap).cuda(), g_t)
    r_order, r_pos = oga.rank_order(fitness)
    assert np.array_equal(order.cpu().numpy(), r_order) and np.array_equal(pos.cpu().numpy(), r_pos)
    rd, rg = oga.next_generation(dose, gap, fitness, 11, 0xFEDCBA987, alpha, elite, k, 0.8, 0.3, crossover="two_point",
                                 mutation=("gene", "swap", "raise"))
    assert np.array_equal(nd.cpu().numpy(), rd) and np.array_equal(ng.cpu().numpy(), rg)
