"""Index built in two calls that read the mask once: the counting call leaves a flag bit per element, the
fill call makes the positions from the bits and seg_ptr.  Against the oracle and against the one-call
build, at the edges of a flag word (32), a pair of segments (2048), a group of eight segments and a
workgroup's share of four groups, with pairs that hold more than 1024 kept elements (stored in two halves)
and with less room than there are kept elements."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, dev_u8, ref_seg_ptr

pytestmark = pytest.mark.gpu

SIZES = [1, 31, 32, 33, 1024, 1025, 2047, 2048, 2049, 8191, 8192, 8193, 32768, 32769, 5 * 32768 + 4097]


def _two_calls(masks, caps, between=None):
    k = len(masks)
    seg = [torch.full((samo.samo_seg_ptr_len(m.numel()),), -7, dtype=torch.int32, device=DEV) for m in masks]
    sizes = [samo.samo_index_flags_bytes(m.numel()) for m in masks]
    flags = [torch.full((s + 1024,), 0xA5, dtype=torch.uint8, device=DEV) for s in sizes]
    idx = [torch.full((c + 8,), -1, dtype=torch.int32, device=DEV) for c in caps]
    nnz = torch.full((k,), -5, dtype=torch.int64, device=DEV)
    jobs = (samo.IndexJob * k)()
    for i, m in enumerate(masks):
        jobs[i] = samo.IndexJob(m.data_ptr(), m.numel(), idx[i].data_ptr(), caps[i], seg[i].data_ptr(), nnz.data_ptr() + 8 * i)
    ptrs = (ctypes.c_void_p * k)(*[f.data_ptr() for f in flags])
    stream = torch.cuda.current_stream().cuda_stream
    assert samo.lib().samo_count_flags_batched(jobs, ptrs, k, stream) == samo.SAMO_OK
    torch.cuda.synchronize()
    assert all((i == -1).all() for i in idx), "counting wrote positions"
    for s, f in zip(sizes, flags):
        assert (f[s:] == 0xA5).all(), "flag bits past their buffer"
    if between is not None:
        between(nnz)
    assert samo.lib().samo_fill_index_batched(jobs, ptrs, k, stream) == samo.SAMO_OK
    torch.cuda.synchronize()
    return seg, idx, nnz.cpu().tolist()


@pytest.mark.parametrize("passes", [1, 2, 4])
def test_two_call_build_matches_the_oracle_and_the_one_call_build(passes):
    masks = []
    for n in SIZES:
        for name in ("all_one", "all_zero", "last_only", "every_65"):
            masks.append(si.edge_masks(n)[name])
        for keep in (0.1, 0.45, 0.55, 0.97):
            masks.append(si.bernoulli_mask(n, keep, n))
    refs = [oracle.build_index(m) for m in masks]
    dev = [dev_u8(m) for m in masks]
    samo.samo_debug_set(samo.KNOB_INDEX_PASSES, passes)
    try:
        seg, idx, nnz = _two_calls(dev, [r.shape[0] for r in refs])
        one = samo.samo_build_index_many(dev)
        again = [torch.full((r.shape[0],), -1, dtype=torch.int32, device=DEV) for r in refs]
        seg1 = [torch.empty_like(s) for s in seg]
        samo.samo_build_index_batched(dev, again, seg1, torch.empty(len(dev), dtype=torch.int64, device=DEV))
        torch.cuda.synchronize()
    finally:
        samo.samo_debug_set(samo.KNOB_INDEX_PASSES)
    for i, (m, r) in enumerate(zip(masks, refs)):
        assert nnz[i] == r.shape[0] == one[i].nnz
        assert np.array_equal(seg[i].cpu().numpy(), ref_seg_ptr(r, m.shape[0])), i
        assert np.array_equal(idx[i][:r.shape[0]].cpu().numpy(), r), i
        assert (idx[i][r.shape[0]:] == -1).all(), "wrote past the capacity"
        assert torch.equal(one[i].idx, idx[i][:r.shape[0]]) and torch.equal(one[i].seg_ptr, seg[i])
        assert torch.equal(again[i], idx[i][:r.shape[0]]) and torch.equal(seg1[i], seg[i])


@pytest.mark.parametrize("n,keep,cap", [(40000, 0.1, 1), (40000, 0.9, 1500), (40000, 0.9, 20001), (70000, 0.3, 0)])
def test_fill_stops_at_the_capacity(n, keep, cap):
    mask = si.bernoulli_mask(n, keep, 3)
    ref = oracle.build_index(mask)
    seg, idx, nnz = _two_calls([dev_u8(mask)], [cap])
    assert nnz[0] == ref.shape[0]
    assert np.array_equal(idx[0][:cap].cpu().numpy(), ref[:cap])
    assert (idx[0][cap:] == -1).all()


def test_fill_after_a_count_that_gave_up_writes_nothing():
    """Such a count reports -1.  The report alone is planted here (seg_ptr stays the valid one): the other job is filled."""
    masks = [si.bernoulli_mask(n, 0.3, n) for n in (50000, 50001)]
    refs = [oracle.build_index(m) for m in masks]

    def give_up(nnz):
        nnz[0] = -1
    seg, idx, nnz = _two_calls([dev_u8(m) for m in masks], [r.shape[0] for r in refs], give_up)
    assert nnz == [-1, refs[1].shape[0]]
    assert (idx[0] == -1).all()
    assert np.array_equal(idx[1][:refs[1].shape[0]].cpu().numpy(), refs[1])


def test_build_without_memory_for_the_flag_bits(monkeypatch):
    masks = [si.bernoulli_mask(n, keep, n) for n, keep in ((70001, 0.1), (1, 1.0), (33000, 0.9), (2048, 0.0))]
    real = torch.empty

    def no_scratch(*a, dtype=None, **kw):
        if dtype == torch.uint8:
            raise torch.OutOfMemoryError("no memory")
        return real(*a, dtype=dtype, **kw)
    dev = [dev_u8(m) for m in masks]
    monkeypatch.setattr(torch, "empty", no_scratch)
    built = samo.samo_build_index_many(dev) + [samo.samo_build_index(dev[0])]
    for m, ix in zip(masks + masks[:1], built):
        ref = oracle.build_index(m)
        assert ix.nnz == ref.shape[0] and np.array_equal(ix.idx.cpu().numpy(), ref)
        assert np.array_equal(ix.seg_ptr.cpu().numpy(), ref_seg_ptr(ref, m.shape[0]))
