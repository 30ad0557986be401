"""Unpruned layers in launches long enough for one wave a tile, and for a late last request, against the same elements stepped in short launches (two waves a tile, or the
kernel of short launches): the same bits, over the ragged end of the layer too, beside small layers and pruned ones."""
import pytest
import torch

import paper_2302_05045_amd as samo
from gpu_util import DEV

pytestmark = pytest.mark.gpu
LONG, LONGEST = 25_010 * 1024, 45_010 * 1024            # more workgroups than the lines between the three, by themselves


def _fill(layers, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    for L in layers:
        L.p.copy_(torch.randn(L.p.numel(), generator=gen, device=DEV))
        L.m.copy_(torch.randn(L.m.numel(), generator=gen, device=DEV) * 1e-3)
        if L.v is not None:
            L.v.copy_(torch.rand(L.v.numel(), generator=gen, device=DEV) * 1e-6)
        g = torch.randn(L.n, generator=gen, device=DEV).half()
        L.g.copy_(g)
        if L.gc16 is not None:
            L.gc16.copy_(g)
        L.w.fill_(float("nan"))


def _step(plan, op):
    if op == "adam":
        plan.samo_fused_step_batched(1.0 / 1024, samo.adam_cfg(3, lr=1e-3))
    elif op == "sgd":
        plan.samo_fused_sgd_step_batched(1.0 / 1024, samo.sgd_cfg(1e-3, 0.9))
    elif op == "c16":
        plan.samo_adam_expand_batched(1.0 / 1024, samo.adam_cfg(3, lr=1e-3))
    else:
        plan.samo_decompress_batched()


@pytest.mark.parametrize("op", ["adam", "sgd", "c16", "expand"])
@pytest.mark.parametrize("n", [LONG, LONG + 8, LONG + 515, LONG + 1019, LONGEST + 4, LONGEST + 515])
def test_long_launches_give_the_bits_of_short_ones(n, op):
    extra = n % 1024
    sizes = [(777, 777, True), (n, n, True), (1024, 1024, True)]
    kw = dict(bucket_gc16=True) if op == "c16" else {}
    layers = samo.alloc_model(sizes, DEV, **kw)
    _fill(layers, 3 + extra)
    before = [{k: getattr(L, k).clone() for k in ("p", "m", "v") if getattr(L, k) is not None} for L in layers]
    _step(samo.Plan(layers), op)
    for L, old in zip(layers, before):
        for first in range(0, L.n, 4 << 20):
            n = min(4 << 20, L.n - first)
            part = samo.alloc_model([(n, n, True)], DEV, **kw)
            S = part[0]
            for k, x in old.items():
                getattr(S, k).copy_(x[first:first + n])
            if op == "c16":
                S.gc16.copy_(L.gc16[first:first + n])
            else:
                S.g.copy_(L.g[first:first + n])
            _step(samo.Plan(part), op)
            for k in ("p", "m", "v", "w"):
                if getattr(S, k) is not None:
                    a, b = getattr(L, k)[first:first + n], getattr(S, k)[:n]
                    assert torch.equal(a.view(torch.int16 if k == "w" else torch.int32), b.view(torch.int16 if k == "w" else torch.int32)), (k, first)


@pytest.mark.parametrize("op", ["adam", "sgd"])
@pytest.mark.parametrize("n", [4096, 4099, 4100, 4611, 5117, 5120])
def test_two_records_a_workgroup_give_the_bits_of_one(n, op):
    """The kernel of short launches takes two segments of an unpruned layer as one tile, ragged ends among them."""
    got = []
    for tiles in (samo.KNOB_DEFAULT, 0):
        layers = samo.alloc_model([(n, n, True)] * 750, DEV)
        _fill(layers[:20], n)
        samo.samo_debug_set(samo.KNOB_STAGED_TILES, tiles)
        try:
            _step(samo.Plan(layers), op)
            torch.cuda.synchronize()
        finally:
            samo.samo_debug_set(samo.KNOB_STAGED_TILES)
        got.append([(L.p, L.m, L.w) + (() if L.v is None else (L.v,)) for L in layers[:20]])
    for a, b in zip(*got):
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int16), y.view(torch.int16))
