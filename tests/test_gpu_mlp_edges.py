"""Edges of the surrogate's kernels: batch sizes around each workgroup size's
limits, every protocol length, small and ragged training batches (needs an
MI355X).  Predictions of 300 rows
(16 protocols per workgroup) and 16,600 (64) are compared with the float64
oracle elsewhere; a protocol's sums do not depend on the batch, so the other
sizes have to agree with those bit for bit."""
import numpy as np
import pytest
import torch

import mlp_bounds as mb
from paper_2303_08123_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


@pytest.mark.parametrize("K", [1, 10, 40, 43])
def test_a_protocol_predicts_the_same_in_every_batch(gga, K):
    net = gga.mlp_net(seed=11)
    most = 16500
    dose, gap, nfrac = workloads.random_protocols(most, K, seed=K, kmin=0)
    dd = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (dose, gap, nfrac)]
    whole = gga.mlp_predict(net, *dd)
    small = torch.cat([gga.mlp_predict(net, *(x[k:k + 300].contiguous() for x in dd)) for k in range(0, most, 300)])
    assert torch.equal(whole, small)
    for B in (1, 15, 16, 17, 31, 33, 63, 65, 4095, 4096, 4097, 4129, 8191, 8192, 8193, 8257):
        assert torch.equal(gga.mlp_predict(net, *(x[:B].contiguous() for x in dd)), whole[:B]), B


@pytest.mark.parametrize("B", [1, 5, 33, 130, 1023, 1024, 2050])
def test_gradients_at_edges_match_the_oracle_pass_by_pass(gga, B):
    """One and a few rows (most chunks of the sums empty), ragged splits and
    k-steps, one split and two: every stored tensor and gradient against the
    oracle's arithmetic on the kernels' own inputs of that pass."""
    net = gga.mlp_net(seed=5)
    dose, gap, nfrac = workloads.random_protocols(B, 10, seed=2, kmin=1)
    target = np.random.default_rng(9).normal(0.0, 1.0, size=B).astype(np.float32)
    dd = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (dose, gap, nfrac)]
    work = gga.mlp_work(B)
    loss = gga.mlp_grad(net, *dd, torch.from_numpy(target).cuda(), work=work).item()
    grads = gga.mlp_split(gga.mlp_block(net, "g").cpu().numpy().astype(np.float64))
    v = {k: x.float().cpu().numpy().astype(np.float64) for k, x in gga.mlp_work_views(work, B).items()}
    params = gga.mlp_split(gga.mlp_block(net, "p").cpu().numpy().astype(np.float64))
    params = [mb.bf16(x) if i in (0, 2, 4) else x for i, x in enumerate(params)]
    mb.check_passes(v, grads, params, target.astype(np.float64), loss, z3_kept=B < 1024)


@pytest.mark.parametrize("M,N,K,ta,tb", [(70, 128, 32, False, True), (70, 128, 64, False, True), (1, 64, 128, False, True),
                                         (70, 128, 192, False, True), (129, 64, 384, False, True), (64, 128, 1, True, False),
                                         (128, 64, 127, True, False), (64, 64, 129, True, False)])
def test_products_at_edges_of_the_k_steps(gga, M, N, K, ta, tb):
    """Operands along K (steps of 32, 64 and 128) and across it (steps of 128
    with a remainder) against float64: products of bf16 values are exact in
    fp32, so 1e-5 of the absolute sum covers the accumulation."""
    gen = torch.Generator().manual_seed(M + N + K)
    A = torch.randn(M, K, generator=gen).to(torch.bfloat16)
    B = torch.randn(K, N, generator=gen).to(torch.bfloat16)
    C = gga.mlp_gemm((A.t().contiguous() if ta else A).cuda(), (B.t().contiguous() if tb else B).cuda(), a_trans=ta,
                     b_trans=tb).cpu().numpy().astype(np.float64)
    A64, B64 = A.double().numpy(), B.double().numpy()
    assert np.all(np.abs(C - A64 @ B64) <= 1e-5 * (np.abs(A64) @ np.abs(B64)) + 1e-30)
