"""The two main loops of the weight-gradient kernels (wave groups in step in short calls, half a stage apart in longer
ones) against the oracle's rounding bracket, at the token counts around the line of either tile shape: 704 of the
128 x 128 tile (stages of 64), 192 of the 256 x 256 tile (stages of 32), with and without a partial last stage."""
import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
from gpu_util import DEV, host_bits
from test_gpu_wgrad import _bracket, _check_f16, _problem

pytestmark = pytest.mark.gpu

CASES = [(128, t) for t in (640, 703, 704, 705, 768, 769, 961)] + [(256, t) for t in (63, 160, 191, 192, 193, 224, 225, 257)]


@pytest.mark.parametrize("kind", ["bernoulli10", "edges"])
@pytest.mark.parametrize("out_f,in_f", [(8, 136), (136, 264), (264, 40)])
@pytest.mark.parametrize("tile,tokens", CASES)
def test_both_loops_match_the_oracle(tile, tokens, out_f, in_f, kind):
    dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, kind, 5 + tokens)
    nnz = idx.shape[0]
    want = oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx)
    lo, hi = _bracket(dy, x, tokens, out_f, in_f, idx)
    none = torch.empty(0, dtype=torch.uint8, device=DEV)
    samo.samo_debug_set(samo.KNOB_WGRAD_TILE, tile)
    try:
        gc16 = torch.full((nnz + 8,), float("nan"), dtype=torch.float16, device=DEV)
        samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], workspace=none)
        gc = torch.full((nnz + 8,), float("nan"), device=DEV)
        samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, 1.0, gc[:nnz], workspace=none)
        torch.cuda.synchronize()
    finally:
        samo.samo_debug_set(samo.KNOB_WGRAD_TILE)
    _check_f16(host_bits(gc16[:nnz]), lo, hi, want, "gc16")
    assert torch.isnan(gc16[nnz:]).all() and torch.isnan(gc[nnz:]).all(), "wrote past the compressed gradient"
    assert np.array_equal(gc[:nnz].cpu().numpy(), gc16[:nnz].float().cpu().numpy())


@pytest.mark.parametrize("tile,tokens", [(128, (770, 0, 70, 1)), (128, (704, 0, 63, 640)), (256, (257, 0, 31, 97)), (256, (192, 0, 33, 1))])
def test_layers_of_different_length_share_a_loop(tile, tokens):
    """The longest layer of a call picks the loop; the others go through it with few stages or none."""
    jobs, wants = [], []
    for t, (out_f, in_f, kind) in zip(tokens, ((136, 264, "bernoulli10"), (16, 24, "bernoulli50"), (24, 520, "dense_idx"), (264, 40, "rows"))):
        dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(max(t, 1), out_f, in_f, kind, 5 + t)
        dy, x, d_dy, d_x = dy[:t * out_f], x[:t * in_f], d_dy[:t], d_x[:t]
        jobs.append((d_dy, d_x, d_idx, d_seg, torch.full((idx.shape[0],), float("nan"), dtype=torch.float16, device=DEV)))
        wants.append((oracle.wgrad_compress(dy, x, t, out_f, in_f, idx), *_bracket(dy, x, t, out_f, in_f, idx)))
    samo.samo_debug_set(samo.KNOB_WGRAD_TILE, tile)
    try:
        samo.samo_wgrad_gather_fp16_batched(jobs, workspace=torch.empty(0, dtype=torch.uint8, device=DEV))
        torch.cuda.synchronize()
    finally:
        samo.samo_debug_set(samo.KNOB_WGRAD_TILE)
    for k, (job, (want, lo, hi)) in enumerate(zip(jobs, wants)):
        _check_f16(host_bits(job[4]), lo, hi, want, "job %d" % k)
