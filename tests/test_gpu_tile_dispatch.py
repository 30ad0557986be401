"""The tile kernels reach a plan's layers by global or by flat accesses, by what the model keeps; a layer by itself always the same
way.  Either way the same arithmetic: a plan of one layer gives the bits of the single-layer entries, at kept fractions on both sides
of every line of the rule.  The short launches' kernel is switched off, it would take these sizes."""
import pytest
import torch

import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, INV

pytestmark = pytest.mark.gpu


def _layer(n, keep):
    gen = torch.Generator(device=DEV).manual_seed(n)
    rand = lambda k: torch.rand(k, generator=gen, device=DEV)
    mask = (rand(n) < keep).to(torch.uint8)
    ix = samo.samo_build_index(mask)
    return dict(n=n, idx=ix.idx, seg_ptr=ix.seg_ptr, p=rand(ix.nnz) - 0.5, m=rand(ix.nnz) - 0.5, v=rand(ix.nnz),
                w=torch.full((n,), float("nan"), dtype=torch.float16, device=DEV), g=((rand(n) - 0.5) * 1024).half())


def _copy(s):
    return {k: x.clone() if isinstance(x, torch.Tensor) and k in "pmvw" else x for k, x in s.items()}


def _plan(s):
    return samo.Plan([samo.Layer(s["n"], s["idx"], s["seg_ptr"], s["p"], s["m"], s["v"], s["w"], s["g"], None, None)])


def _same(a, b, names):
    for name in names:
        bits = torch.int16 if name == "w" else torch.int32
        assert torch.equal(a[name].view(bits), b[name].view(bits)), name


KEEPS = [0., .02, .03, .05, .06, .08, .15, .3, .95, 1.]


@pytest.mark.parametrize("opt", ["adam", "sgd"])
@pytest.mark.parametrize("keep", KEEPS)
def test_a_plans_step_has_the_bits_of_the_layers(keep, opt):
    a = _layer(300_007, keep)
    b = _copy(a)
    plan = _plan(a)
    samo.samo_debug_set(samo.KNOB_STAGED_TILES, 0)
    try:
        for t in (1, 2):
            if opt == "adam":
                cfg = samo.adam_cfg(t, **si.ADAM)
                plan.samo_fused_step_batched(INV, cfg)
                samo.samo_fused_step(b["g"], b["w"], b["idx"], b["seg_ptr"], b["p"], b["m"], b["v"], INV, cfg)
            else:
                cfg = samo.sgd_cfg(1e-3, 0.9)
                plan.samo_fused_sgd_step_batched(INV, cfg)
                samo.samo_fused_sgd_step(b["g"], b["w"], b["idx"], b["seg_ptr"], b["p"], b["m"], INV, cfg)
    finally:
        samo.samo_debug_set(samo.KNOB_STAGED_TILES)
    _same(a, b, "pmvw")


@pytest.mark.parametrize("keep", KEEPS)
def test_a_plans_expansion_has_the_bits_of_the_layers(keep):
    a = _layer(200_003, keep)
    b = _copy(a)
    _plan(a).samo_decompress_batched()
    samo.samo_decompress(b["p"], b["idx"], b["seg_ptr"], b["w"])
    _same(a, b, "w")
    want = torch.zeros(a["n"], dtype=torch.float16, device=DEV)
    want[a["idx"].long()] = a["p"].half()
    assert torch.equal(a["w"].view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("n,keep", [(200_000_003, .03), (200_000_003, .2), (1003, .03), (1_000_001, .5)])
def test_long_accumulating_gathers_have_the_bits_of_short_ones(n, keep):
    """Beyond the last-level cache the old message is read before or after the gather, by what is kept: the same one
    rounded addition."""
    gen = torch.Generator(device=DEV).manual_seed(n)
    ix = samo.samo_build_index((torch.rand(n, generator=gen, device=DEV) < keep).to(torch.uint8))
    g = torch.randn(n, generator=gen, device=DEV).half()
    old = torch.randn(ix.nnz, generator=gen, device=DEV).half()
    got = old.clone()
    samo.samo_gather_grads_fp16(g, ix.idx, got, accumulate=True)
    want = old + g[ix.idx.long()]
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
