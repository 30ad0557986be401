"""Weight gradients in tiles of 256 rows and 128, 160 or 192 columns, against the oracle's rounding bracket: layers
narrower than a tile, one column past a tile, several tiles with a ragged last one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, host_bits
from test_gpu_wgrad import _bracket, _check_f16, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[128, 160, 192])
def cols(request):
    samo.samo_debug_set(samo.KNOB_WGRAD_COLS, request.param)
    yield request.param
    samo.samo_debug_set(samo.KNOB_WGRAD_COLS)


@pytest.mark.parametrize("kind", ["bernoulli10", "bernoulli50", "edges", "dense_idx"])
@pytest.mark.parametrize("tokens,out_f,in_f", [(1, 8, 8), (33, 264, 136), (96, 256, 160), (97, 8, 168), (130, 520, 384),
                                               (161, 136, 392), (300, 264, 520)])
def test_narrow_tiles_match_the_oracle(tokens, out_f, in_f, kind, cols):
    dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, kind, 11 + tokens)
    nnz = idx.shape[0]
    want = oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx)
    lo, hi = _bracket(dy, x, tokens, out_f, in_f, idx)
    gc16 = torch.full((nnz + 8,), float("nan"), dtype=torch.float16, device=DEV)
    samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz])
    inv = np.float32(1.0 / si.LOSS_SCALE)
    gc = torch.full((nnz + 8,), float("nan"), dtype=torch.float32, device=DEV)
    samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, float(inv), gc[:nnz])
    torch.cuda.synchronize()
    bits16 = host_bits(gc16[:nnz])
    _check_f16(bits16, lo, hi, want, "gc16")
    assert torch.isnan(gc16[nnz:]).all() and torch.isnan(gc[nnz:]).all(), "wrote past the compressed gradient"
    assert np.array_equal(gc[:nnz].cpu().numpy().view(np.uint32), (bits16.view(np.float16).astype(np.float32) * inv).view(np.uint32))
    # a second micro-batch: one correctly rounded half addition to what is there
    samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], accumulate=True)
    torch.cuda.synchronize()
    twice = (bits16.view(np.float16) + bits16.view(np.float16)).astype(np.float16)
    assert np.array_equal(host_bits(gc16[:nnz]), twice.view(np.uint16))
    assert torch.isnan(gc16[nnz:]).all()


@pytest.mark.parametrize("tokens,out_f,in_f", [(65, 3000, 3080), (97, 2600, 2248), (33, 3592, 3048)])
def test_layers_that_the_rule_gives_narrow_tiles(tokens, out_f, in_f):
    """Less than a round of large tiles, so that 160, 128 and 192 columns fill the device better (a layer of such a size, in
    64 bits on the GPU: the bracket of the exact sums by the bound of tokens fp32 additions)."""
    gen = torch.Generator(device=DEV).manual_seed(tokens)
    dy = torch.randn(tokens, out_f, generator=gen, device=DEV).half()
    x = torch.randn(tokens, in_f, generator=gen, device=DEV).half()
    ix = samo.samo_build_index((torch.rand(out_f * in_f, generator=gen, device=DEV) < 0.1).to(torch.uint8))
    at = ix.idx.long()
    exact = (dy.double().t().contiguous() @ x.double()).view(-1)[at]
    slack = (tokens + 2) * 2.0 ** -23 * (dy.double().abs().t().contiguous() @ x.double().abs()).view(-1)[at]
    got = torch.full((ix.nnz,), float("nan"), dtype=torch.float16, device=DEV)
    samo.samo_wgrad_gather_fp16(dy, x, ix.idx, ix.seg_ptr, got)
    as_half = lambda v: torch.from_numpy(v.cpu().numpy().astype(np.float16)).to(DEV)          # one rounding
    assert bool(((got >= as_half(exact - slack)) & (got <= as_half(exact + slack))).all())
    first = got.clone()
    samo.samo_wgrad_gather_fp16(dy, x, ix.idx, ix.seg_ptr, got, accumulate=True)
    assert torch.equal(got, first + first)


def test_narrow_tiles_of_several_layers(cols):
    jobs, wants = [], []
    for tokens, out_f, in_f, kind in ((65, 264, 200, "bernoulli10"), (40, 24, 520, "dense_idx"), (129, 520, 136, "bernoulli50")):
        dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, kind, 3 + tokens)
        gc16 = torch.full((idx.shape[0],), float("nan"), dtype=torch.float16, device=DEV)
        jobs.append((d_dy, d_x, d_idx, d_seg, gc16))
        wants.append((oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx), *_bracket(dy, x, tokens, out_f, in_f, idx)))
    samo.samo_wgrad_gather_fp16_batched(jobs)
    torch.cuda.synchronize()
    for k, (job, (want, lo, hi)) in enumerate(zip(jobs, wants)):
        _check_f16(host_bits(job[4]), lo, hi, want, "job %d" % k)
