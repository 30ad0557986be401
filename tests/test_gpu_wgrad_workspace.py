"""Where the weight gradient of a small layer takes its workspace from: the caller, torch's allocator for the length of
the call, the pool of a graph under capture, or nowhere (a capture that torch knows nothing of, no memory left)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, dev_f16_bits, host_bits
from test_gpu_wgrad import _bracket, _check_f16, _problem

pytestmark = pytest.mark.gpu

TOKENS, OUT, IN = 4096, 512, 512           # 16 small tiles of 64 stages: split whatever the other shapes cost


@pytest.fixture(scope="module")
def problem():
    dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(TOKENS, OUT, IN, "bernoulli10", 17)
    want = oracle.wgrad_compress(dy, x, TOKENS, OUT, IN, idx)
    lo, hi = _bracket(dy, x, TOKENS, OUT, IN, idx)
    args = (d_dy, d_x, d_idx, d_seg)

    def gather(**kw):
        gc = torch.full((idx.shape[0],), float("nan"), device=DEV)
        samo.samo_wgrad_gather(*args, 1.0, gc, **kw)
        return gc

    def check(gc, what):
        _check_f16(host_bits(gc.half()), lo, hi, want, what)
    gc = torch.empty(idx.shape[0], device=DEV)
    need = samo.samo_wgrad_workspace_bytes([args + (gc,)])
    assert need >= 2 * 4 * idx.shape[0]
    return args, gather, check, need


def test_given_withheld_and_missing_workspaces(problem, monkeypatch):
    args, gather, check, need = problem
    default, given = gather(), gather(workspace=torch.empty(need, dtype=torch.uint8, device=DEV))
    refused = gather(workspace=torch.empty(0, dtype=torch.uint8, device=DEV))
    short = gather(workspace=torch.empty(need - 16, dtype=torch.uint8, device=DEV))
    check(given, "given")
    check(refused, "refused")
    assert torch.equal(default, given) and torch.equal(refused, short)
    with pytest.raises(TypeError):
        gather(workspace=torch.empty(need, device=DEV))
    real = torch.empty

    def no_scratch(*a, dtype=None, **kw):
        if dtype == torch.uint8:
            raise torch.OutOfMemoryError("no memory")
        return real(*a, dtype=dtype, **kw)
    monkeypatch.setattr(torch, "empty", no_scratch)
    assert torch.equal(gather(), refused)
    gc16 = torch.zeros(refused.numel(), dtype=torch.float16, device=DEV)
    samo.samo_wgrad_gather_fp16_batched([args + (gc16,)])
    assert torch.equal(gc16.float(), refused)


def test_torch_graph_replays_the_eager_bits(problem):
    args, gather, _, _ = problem
    d_dy = args[0].clone()
    gc, eager = torch.empty_like(gather()), gather()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        assert samo._capture_scratch(4096) is not None              # the graph's own pool
        samo.samo_wgrad_gather(d_dy, *args[1:], 1.0, gc)
    for step in range(4):
        d_dy.copy_(dev_f16_bits(si.output_grads_fp16(TOKENS, OUT, 90 + step)).view(TOKENS, OUT))
        samo.samo_wgrad_gather(d_dy, *args[1:], 1.0, eager)
        noise = [torch.full((1 << 20,), step + 1, dtype=torch.uint8, device=DEV) for _ in range(4)]
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(gc, eager), step
        assert all(bool((n == step + 1).all()) for n in noise)


def test_capture_begun_outside_torch_borrows_no_memory(problem):
    """The graph is launched long after the call has returned: its kernels must not write to memory that the
    allocator has given to somebody else since."""
    args, gather, check, need = problem
    with open("/proc/self/maps") as maps:
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    graph, instance = ctypes.c_void_p(), ctypes.c_void_p()
    side = torch.cuda.Stream()
    unsplit = gather(workspace=torch.empty(0, dtype=torch.uint8, device=DEV))
    gc, own = torch.empty_like(unsplit), torch.empty(need, dtype=torch.uint8, device=DEV)
    given = torch.empty_like(unsplit)
    with torch.cuda.stream(side):
        split = gather()                                    # leaves a block of the workspace's size in the allocator
        torch.cuda.synchronize()
        stream = ctypes.c_void_p(side.cuda_stream)
        assert hip.hipStreamBeginCapture(stream, 1) == 0
        samo.samo_wgrad_gather(*args, 1.0, gc)
        samo.samo_wgrad_gather(*args, 1.0, given, workspace=own)
        assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
        assert hip.hipGraphInstantiate(ctypes.byref(instance), graph, None, None, ctypes.c_size_t(0)) == 0
        victims = [torch.full((need,), 0xA5, dtype=torch.uint8, device=DEV) for _ in range(4)]
        for _ in range(3):
            gc.fill_(float("nan"))
            given.fill_(float("nan"))
            assert hip.hipGraphLaunch(instance, stream) == 0
            torch.cuda.synchronize()
            assert all(bool((v == 0xA5).all()) for v in victims), "wrote to memory that is not the call's any more"
            assert torch.equal(gc, unsplit) and torch.equal(given, split)
    check(gc, "captured")
    hip.hipGraphExecDestroy(instance)
    hip.hipGraphDestroy(graph)
