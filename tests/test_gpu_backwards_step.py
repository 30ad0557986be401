"""A long step under a guard takes its tiles from the last one back: the same bits as the step without a guard, where the coefficient is 1."""
import pytest
import torch

import paper_2302_05045_amd as samo
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opt", ["adam", "sgd"])
def test_guarded_long_step_gives_the_bits_of_the_unguarded_one(opt):
    gen = torch.Generator(device=DEV).manual_seed(2)
    sizes, masks = [], []
    for n, keep in ((150_000_001, 0.1), (5000, None), (60_000_000, 0.2), (1500, 0.5)):       # some 55,000 tiles
        masks.append(None if keep is None else (torch.rand(n, generator=gen, device=DEV) < keep).to(torch.uint8))
        sizes.append((n, n if keep is None else int(masks[-1].sum()), keep is None))
    layers = samo.alloc_model(sizes, DEV)
    count = torch.empty(1, dtype=torch.int64, device=DEV)
    for L, mask in zip(layers, masks):
        if mask is not None:
            samo.samo_build_index_into(mask, L.idx, L.seg_ptr, count)
        L.g.copy_(torch.randn(L.n, generator=gen, device=DEV))
    plan = samo.Plan(layers)
    stats = samo.GradStats(plan)
    plan.samo_grad_stats_batched(0, 1e-3, stats)
    got = []
    for guard in (None, stats.guard(1e30, True)):
        seed = torch.Generator(device=DEV).manual_seed(4)
        for L in layers:
            L.p.copy_(torch.randn(L.p.numel(), generator=seed, device=DEV))
            L.m.zero_()
            if L.v is not None:
                L.v.zero_()
            L.w.fill_(float("nan"))
        if opt == "adam":
            plan.samo_fused_step_batched(1e-3, samo.adam_cfg(2, lr=1e-3), *([guard] if guard else []))
        else:
            plan.samo_fused_sgd_step_batched(1e-3, samo.sgd_cfg(1e-3, 0.9), *([guard] if guard else []))
        got.append([(L.p.clone(), L.m.clone(), L.w.clone()) for L in layers])
    for a, b in zip(*got):
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int16), y.view(torch.int16))
