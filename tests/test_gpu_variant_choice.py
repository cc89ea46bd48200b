"""A kernel variant that was set is the kernel that runs, whatever the batch;
the defaults suit the number of instances (needs an MI355X)."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gga():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2303_08123_amd as g
    return g


def protocols(n):
    return [torch.zeros((n, 1), device="cuda"), torch.zeros((n, 1), dtype=torch.int32, device="cuda"),
            torch.zeros(n, dtype=torch.int32, device="cuda")]


class KernelNode(ctypes.Structure):       # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint * 3), ("args", ctypes.c_void_p), ("shared", ctypes.c_uint)]


def threads_of_launch(call):
    """Threads per workgroup of the first kernel that `call` launches (recorded, not run)."""
    hip = ctypes.CDLL("libamdhip64.so")
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    g = ctypes.c_void_p(graph.raw_cuda_graph())
    n = ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0 and n.value > 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(g, nodes, ctypes.byref(n)) == 0
    for node in nodes:
        kind = ctypes.c_int(-1)
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0
        if kind.value == 0:               # hipGraphNodeTypeKernel
            params = KernelNode()
            assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(params)) == 0
            return params.block[0]
    raise AssertionError("no kernel in the graph")


@pytest.mark.parametrize("beyond", [False, True])
def test_resident_variants_on_64(gga, model_dict, beyond):
    """At most and more than one instance per compute unit: a variant that was set
    runs as named (4x1 in 16 waves, 8x1 in 8, 16x1 in 4), by gga_simulate and by
    state_run_variant; the default takes eight waves only beyond."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = cus + 1 if beyond else cus
    print(f"resident variants, {n} instances", flush=True)
    cfg = gga.make_cfg(64, 2, 1, seed=1)
    protos = protocols(n)
    out = (torch.empty((n, 1), dtype=torch.int32, device="cuda"), torch.empty(n, device="cuda"), None)
    fields = torch.zeros((n, 3, 64, 64), device="cuda")
    cells = torch.zeros((n, 64, 64), dtype=torch.int16, device="cuda")
    simulate = lambda: gga.simulate(model_dict, cfg, *protos, out=out)
    assert threads_of_launch(simulate) == (512 if beyond else 1024)
    for v, threads in ((0, 1024), (7, 512), (8, 256)):
        assert threads_of_launch(lambda: gga.state_run_variant(model_dict, cfg, v, *protos, 0, 1, fields, cells)) == threads
        gga.set_variant(64, v)
        assert threads_of_launch(simulate) == threads
    gga.clear_variant(64)
    assert threads_of_launch(simulate) == (512 if beyond else 1024)


def step_counts(gga, md, L, n):
    """Step counts that the teams of an n-instance call published: teams x slabs."""
    cfg = gga.make_cfg(L, 3, 1, seed=1)
    ws = gga.workspace(cfg, n)
    ws.zero_()
    gga.simulate(md, cfg, *protocols(n), ws=ws)
    # the workspace ends with the counts (128 x 16 of them) and two buffers of the teams' states
    state = gga._align256(L * L * 14 * min(n, 128))
    end = ws.numel() - 2 * state
    return int(torch.count_nonzero(ws[end - 128 * 16 * 4:end].view(torch.int32)))


@pytest.mark.parametrize("L,variant,slabs", [
    (160, 11, 3), (160, 12, 4), (160, 18, 2), (160, 19, 4), (160, 22, 3), (192, 13, 4), (192, 14, 5), (192, 20, 2),
    (192, 21, 5), (192, 23, 4), (192, 24, 3), (224, 15, 5), (224, 16, 4), (256, 5, 6), (256, 6, 4)])
def test_team_variants_that_were_set(gga, model_dict, L, variant, slabs):
    """One instance by a variant that was set: as many slabs as its rows make,
    each of which published its steps."""
    print(f"teams of variant {variant} on {L}", flush=True)
    gga.set_variant(L, variant)
    try:
        assert step_counts(gga, model_dict, L, 1) == slabs
    finally:
        gga.clear_variant(L)


@pytest.mark.parametrize("L,one,many", [(160, 4, 2), (192, 4, 2), (224, 5, 4), (256, 6, 4)])
def test_team_heights_of_the_defaults(gga, model_dict, L, one, many):
    """Without a choice one instance runs in low slabs, so many that the device
    holds few teams at once in high ones (slabs per instance as given)."""
    print(f"default teams on {L}", flush=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert step_counts(gga, model_dict, L, 1) == one
    held = 8 * (cus // (8 * many))                           # one workgroup per compute unit
    assert step_counts(gga, model_dict, L, 4 * held) == min(held, 128) * many
