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
