"""Weight gradients whose tokens are split over several workgroups per tile (a call with a workspace): every split
count and both tile shapes against the oracle's rounding bracket, at stage counts that divide evenly, leave a
short last split, or leave splits without tokens."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, host_bits
from test_gpu_wgrad import _bracket, _check_f16, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[(128, 2), (128, 5), (256, 2), (256, 7)])
def split(request):
    samo.samo_debug_set(samo.KNOB_WGRAD_TILE, request.param[0])
    samo.samo_debug_set(samo.KNOB_WGRAD_SPLIT, request.param[1])
    yield request.param
    samo.samo_debug_set(samo.KNOB_WGRAD_TILE)
    samo.samo_debug_set(samo.KNOB_WGRAD_SPLIT)


@pytest.mark.parametrize("kind", ["bernoulli10", "rows", "edges", "dense_idx"])
@pytest.mark.parametrize("tokens,out_f,in_f", [(65, 8, 16), (129, 136, 264), (256, 264, 128), (421, 264, 520), (64, 520, 24)])
def test_split_weight_gradient_matches_the_oracle(tokens, out_f, in_f, kind, split):
    dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, kind, 77 + tokens)
    nnz = idx.shape[0]
    want = oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx)
    lo, hi = _bracket(dy, x, tokens, out_f, in_f, idx)
    gc16 = torch.full((nnz + 8,), float("nan"), dtype=torch.float16, device=DEV)
    samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz])
    torch.cuda.synchronize()
    _check_f16(host_bits(gc16[:nnz]), lo, hi, want, "gc16")
    assert torch.isnan(gc16[nnz:]).all(), "wrote past the compressed gradient"
    inv = np.float32(1.0 / si.LOSS_SCALE)
    gc = torch.full((nnz + 8,), float("nan"), dtype=torch.float32, device=DEV)
    samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, float(inv), gc[:nnz])
    again = torch.empty_like(gc[:nnz])
    samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, float(inv), again)
    torch.cuda.synchronize()
    bits16 = host_bits(gc16[:nnz])
    assert np.array_equal(gc[:nnz].cpu().numpy().view(np.uint32), (bits16.view(np.float16).astype(np.float32) * inv).view(np.uint32))
    assert torch.isnan(gc[nnz:]).all()
    assert torch.equal(gc[:nnz], again), "not deterministic"
    # a second micro-batch: one correctly rounded half addition to what is there
    samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], accumulate=True)
    torch.cuda.synchronize()
    twice = (bits16.view(np.float16) + bits16.view(np.float16)).astype(np.float16)
    assert np.array_equal(host_bits(gc16[:nnz]), twice.view(np.uint16))


def test_split_layers_of_different_length_in_one_call(split):
    jobs, wants = [], []
    for tokens, out_f, in_f, kind in ((300, 136, 264, "bernoulli10"), (0, 16, 24, "bernoulli50"), (70, 24, 520, "dense_idx")):
        dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, kind, 5 + tokens)
        gc16 = torch.full((idx.shape[0],), float("nan"), dtype=torch.float16, device=DEV)
        jobs.append((d_dy, d_x, d_idx, d_seg, gc16))
        wants.append((oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx), *_bracket(dy, x, tokens, out_f, in_f, idx)))
    samo.samo_wgrad_gather_fp16_batched(jobs)
    torch.cuda.synchronize()
    for k, (job, (want, lo, hi)) in enumerate(zip(jobs, wants)):
        _check_f16(host_bits(job[4]), lo, hi, want, "job %d" % k)


def test_the_rule_splits_small_layers_and_a_short_workspace_does_not():
    L, size = samo.lib(), ctypes.c_size_t()

    def need(tokens, out_f, in_f, nnz):
        job = (samo.WgradJob * 1)(samo.WgradJob(4096, 4096, tokens, out_f, in_f, 4096, 4096, nnz, 4096))
        assert L.samo_wgrad_workspace_bytes(1, job, ctypes.byref(size)) == samo.SAMO_OK
        return size.value
    assert need(8192, 512, 512, 26214) >= 2 * 4 * 26214            # 16 small tiles, 128 stages
    assert need(2048, 1024, 4096, 419430) == 0                     # 256 small tiles: the device is full
    assert need(2048, 2560, 10240, 2621440) == 0                   # more than half a round of large tiles
    assert need(100, 512, 512, 26214) == 0                         # too short to share
    # a split has to beat the tiles that the call would take without it, narrow ones here
    for tokens, out_f, in_f in ((512, 2560, 2240), (300, 2560, 2560), (1024, 2048, 4096), (700, 12000, 512), (512, 512, 9000)):
        assert need(tokens, out_f, in_f, out_f * in_f // 10) == 0, (tokens, out_f, in_f)
    assert need(4096, 2560, 2560, 655360) >= 2 * 4 * 655360
    assert 2 * samo._MOST_SPLIT_TILES >= torch.cuda.get_device_properties(0).multi_processor_count   # the binding's shortcut loses no split
    for tokens in (300, 2048, 8192, 1 << 20):
        assert need(tokens, 256, 256 * (samo._MOST_SPLIT_TILES + 1), 1000) == 0
    for forced, tokens, splits in ((1 << 30, 1 << 30, 64), (65, 1 << 20, 64), (63, 1 << 20, 63), (1 << 30, 100, 4)):
        samo.samo_debug_set(samo.KNOB_WGRAD_SPLIT, forced)
        try:
            assert need(tokens, 512, 512, 26240) == splits * 26240 * 4
        finally:
            samo.samo_debug_set(samo.KNOB_WGRAD_SPLIT)
    tokens, out_f, in_f = 1024, 512, 512
    dy, x, idx, d_dy, d_x, d_idx, d_seg = _problem(tokens, out_f, in_f, "bernoulli10", 9)
    nnz = idx.shape[0]
    want = need(tokens, out_f, in_f, nnz)
    assert want > 0
    stream = torch.cuda.current_stream().cuda_stream
    ws = torch.full((want,), 0xA5, dtype=torch.uint8, device=DEV)
    outs = []
    for given in (None, want - 1, want):
        gc = torch.empty(nnz, dtype=torch.float32, device=DEV)
        job = (samo.WgradJob * 1)(samo.WgradJob(d_dy.data_ptr(), d_x.data_ptr(), tokens, out_f, in_f, d_idx.data_ptr(), d_seg.data_ptr(), nnz, gc.data_ptr()))
        assert L.samo_wgrad_gather_batched_ws(1, job, 1.0, ws.data_ptr() if given else None, given or 0, stream) == samo.SAMO_OK
        torch.cuda.synchronize()
        assert bool((ws == 0xA5).all()) == (given != want)
        outs.append(gc)
    assert torch.equal(outs[0], outs[1])
    lo, hi = _bracket(dy, x, tokens, out_f, in_f, idx)
    _check_f16(host_bits(outs[2].half()), lo, hi, oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx), "split")
