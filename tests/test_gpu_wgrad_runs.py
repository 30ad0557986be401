"""The weight gradient's epilogue where the search for a tile row's run of kept entries can go wrong: layers with fewer entries than
a look reads, segments whose kept elements sit at one end (the guess misses on either side), runs longer than the entries requested ahead,
runs that end with a tile, a segment or the index."""
import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, dev_f16_bits, dev_i32, host_bits, ref_seg_ptr
from test_gpu_wgrad import _bracket, _check_f16

pytestmark = pytest.mark.gpu


def _kept(kind, out_f, in_f):
    m = np.zeros((out_f, in_f), np.uint8)
    flat = m.reshape(-1)
    if kind.startswith("first"):                       # the first k elements of the layer alone
        flat[:int(kind[5:])] = 1
    elif kind.startswith("last"):
        flat[flat.size - int(kind[4:]):] = 1
    elif kind == "heads":                              # the first 200 of every segment: guesses too early
        flat[np.arange(flat.size) % 1024 < 200] = 1
    elif kind == "tails":                              # the last 200: guesses too late
        flat[np.arange(flat.size) % 1024 >= 824] = 1
    elif kind == "full_rows":                          # every third row whole, the others two elements at tile edges
        m[::3] = 1
        m[1::3, ::128] = 1
    elif kind == "columns":                            # whole columns around the tiles' edges
        for c in (0, 127, 128, 255, 256, in_f - 1):
            if c < in_f:
                m[:, c] = 1
    elif kind == "uneven":                             # every seventh row ten times denser, in segments of several rows
        m[:] = np.random.default_rng(3).random(m.shape) < np.where(np.arange(out_f) % 7 == 3, 0.6, 0.06)[:, None]
    elif kind == "runs33":                             # 33 and 65 entries in a row of a tile: one past a step, one past two
        m[::2, 10:43] = 1
        m[1::2, 20:85] = 1
    else:
        raise KeyError(kind)
    return flat


# The epilogue's shapes, as (knob, value) pairs, and token counts: of the 128 x 128 tile both loops, the longer of which reads old values late, of the
# 256 x 256 tile too, the tiles of 256 rows between, four workgroups to a compute unit, and the sums of a split.
SHAPES = {
    "128": ([("WGRAD_TILE", 128)], 37), "128 long": ([("WGRAD_TILE", 128)], 705), "256": ([("WGRAD_TILE", 256)], 37),
    "256 long": ([("WGRAD_TILE", 256)], 257), "256x128": ([("WGRAD_COLS", 128)], 37), "256x160": ([("WGRAD_COLS", 160)], 37),
    "256x192": ([("WGRAD_COLS", 192)], 37), "resident": ([("WGRAD_TILE", 512)], 37),
    "split 128": ([("WGRAD_TILE", 128), ("WGRAD_SPLIT", 2)], 130), "split 256": ([("WGRAD_TILE", 256), ("WGRAD_SPLIT", 3)], 130),
}


@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("out_f,in_f", [(16, 136), (264, 520), (40, 1032)])
@pytest.mark.parametrize("kind", ["first1", "first31", "first32", "first33", "last1", "last31", "last33", "heads", "tails",
                                  "full_rows", "columns", "uneven", "runs33"])
def test_runs_are_found(kind, out_f, in_f, shape):
    knobs, tokens = SHAPES[shape]
    seed = 4
    dy, x = si.output_grads_fp16(tokens, out_f, seed), si.activations_fp16(tokens, in_f, seed)
    idx = oracle.build_index(_kept(kind, out_f, in_f))
    nnz = idx.shape[0]
    d_dy, d_x = dev_f16_bits(dy).view(tokens, out_f), dev_f16_bits(x).view(tokens, in_f)
    d_idx, d_seg = dev_i32(idx), dev_i32(ref_seg_ptr(idx, out_f * in_f))
    want = oracle.wgrad_compress(dy, x, tokens, out_f, in_f, idx)
    lo, hi = _bracket(dy, x, tokens, out_f, in_f, idx)
    gc16 = torch.full((nnz + 8,), float("nan"), dtype=torch.float16, device=DEV)
    gc = torch.full((nnz + 8,), float("nan"), device=DEV)
    kw = {} if "split" in shape else dict(workspace=torch.empty(0, dtype=torch.uint8, device=DEV))
    for name, value in knobs:
        samo.samo_debug_set(getattr(samo, "KNOB_" + name), value)
    try:
        samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], **kw)
        samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, 1.0, gc[:nnz], **kw)
        torch.cuda.synchronize()
        bits = host_bits(gc16[:nnz])
        samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], accumulate=True, **kw)
        torch.cuda.synchronize()
    finally:
        for name, _ in knobs:
            samo.samo_debug_set(getattr(samo, "KNOB_" + name))
    _check_f16(bits, lo, hi, want, kind)
    assert np.array_equal(gc[:nnz].cpu().numpy(), bits.view(np.float16).astype(np.float32))
    assert np.array_equal(host_bits(gc16[:nnz]), (bits.view(np.float16) + bits.view(np.float16)).astype(np.float16).view(np.uint16))
    assert torch.isnan(gc16[nnz:]).all() and torch.isnan(gc[nnz:]).all(), "wrote past the compressed gradient"


@pytest.mark.parametrize("tile,cols", [(128, None), (256, None), (512, None), (None, 128), (None, 160), (None, 192)])
def test_the_widest_layer(tile, cols):
    """8 x 2^24, the rows of a tile behind its last one among them: nothing is stored behind the index's entries."""
    out_f, in_f = 8, 1 << 24
    rng = np.random.default_rng(6)
    dy, x = rng.standard_normal((1, out_f)).astype(np.float16), rng.standard_normal((1, in_f)).astype(np.float16)
    ends = (np.arange(out_f)[:, None] * in_f + np.concatenate([np.arange(70), in_f - 1 - np.arange(70)])[None]).reshape(-1)
    idx = np.unique(np.concatenate([ends, rng.integers(0, out_f * in_f, 20_000)])).astype(np.int32)
    nnz = idx.shape[0]
    want = (dy[0].astype(np.float32)[idx // in_f] * x[0].astype(np.float32)[idx % in_f]).astype(np.float16)       # the product is exact in fp32
    d_dy, d_x, d_idx, d_seg = torch.from_numpy(dy).to(DEV), torch.from_numpy(x).to(DEV), dev_i32(idx), dev_i32(ref_seg_ptr(idx, out_f * in_f))
    gc16 = torch.full((nnz + 256,), float("nan"), dtype=torch.float16, device=DEV)
    gc = torch.full((nnz + 256,), float("nan"), device=DEV)
    none = torch.empty(0, dtype=torch.uint8, device=DEV)
    if tile:
        samo.samo_debug_set(samo.KNOB_WGRAD_TILE, tile)
    if cols:
        samo.samo_debug_set(samo.KNOB_WGRAD_COLS, cols)
    try:
        samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], workspace=none)
        samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, 1.0, gc[:nnz], workspace=none)
        torch.cuda.synchronize()
        bits = host_bits(gc16[:nnz])
        samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16[:nnz], accumulate=True, workspace=none)
        torch.cuda.synchronize()
    finally:
        samo.samo_debug_set(samo.KNOB_WGRAD_TILE)
        samo.samo_debug_set(samo.KNOB_WGRAD_COLS)
    assert torch.isnan(gc16[nnz:]).all() and torch.isnan(gc[nnz:]).all(), "wrote past the compressed gradient"
    assert np.array_equal(bits, want.view(np.uint16)) and np.array_equal(gc[:nnz].cpu().numpy(), want.astype(np.float32))
    assert np.array_equal(host_bits(gc16[:nnz]), (want + want).view(np.uint16))


@pytest.mark.parametrize("tile", [128, 256, 512])
@pytest.mark.parametrize("keep", [0.002, 0.1, 0.5])
@pytest.mark.parametrize("out_f,in_f", [(16, 136), (264, 520), (40, 1032)])
def test_an_index_shorter_than_its_buffer(out_f, in_f, keep, tile):
    """A layer pruned again with fewer elements kept, in the place of its old index: the entries behind the ones that seg_ptr counts are not
    looked at, and the gradient behind them is left as it was."""
    tokens = 37
    dy, x = si.output_grads_fp16(tokens, out_f, 4), si.activations_fp16(tokens, in_f, 4)
    n = out_f * in_f
    idx = oracle.build_index(si.bernoulli_mask(n, keep, 9))
    nnz = idx.shape[0]
    d_dy, d_x, d_seg = dev_f16_bits(dy).view(tokens, out_f), dev_f16_bits(x).view(tokens, in_f), dev_i32(ref_seg_ptr(idx, n))
    none = torch.empty(0, dtype=torch.uint8, device=DEV)

    def gather(d_idx):
        gc16 = torch.full((d_idx.numel(),), float("nan"), dtype=torch.float16, device=DEV)
        gc = torch.full((d_idx.numel(),), float("nan"), device=DEV)
        samo.samo_debug_set(samo.KNOB_WGRAD_TILE, tile)
        try:
            samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16, workspace=none)
            samo.samo_wgrad_gather_fp16(d_dy, d_x, d_idx, d_seg, gc16, accumulate=True, workspace=none)
            samo.samo_wgrad_gather(d_dy, d_x, d_idx, d_seg, 1.0, gc, workspace=none)
            torch.cuda.synchronize()
        finally:
            samo.samo_debug_set(samo.KNOB_WGRAD_TILE)
        return gc16, gc
    want = gather(dev_i32(idx))
    for tail in (np.arange(n - n // 4, n, 2), np.zeros(70), np.arange(300) * (n // 300)):
        got = gather(dev_i32(np.concatenate([idx, tail.astype(np.int32)])))
        for a, b in zip(got, want):
            assert torch.equal(a[:nnz], b) and torch.isnan(a[nnz:]).all()
