"""Counting in two launches without a chain: counts within blocks of 64 segments, then the blocks' offsets, where a
workgroup owns 32 blocks and sums the totals of all those before its own, 1024 to a look.  Sizes around a group of eight
segments, a block, a workgroup's blocks and a look; with and without flag bits; the fill's three ways of collecting positions
(a group of 8192 elements that keeps up to 1024, up to 1024 in either half, more) at the densities where they meet.  Whole
numbers, compared exactly."""
import numpy as np
import pytest
import torch

import oracle
import paper_2302_05045_amd as samo
import samo_inputs as si
from gpu_util import DEV, dev_u8, ref_seg_ptr

pytestmark = pytest.mark.gpu

SEG = samo.SEG_ELEMS
BLOCK = 64 * SEG
OFFSETS = 32 * BLOCK


@pytest.mark.parametrize("n", [1, 8 * SEG - 1, 8 * SEG + 1, BLOCK - 1, BLOCK, BLOCK + 1, OFFSETS - SEG, OFFSETS, OFFSETS + 1,
                               5 * OFFSETS + 3 * BLOCK + 17])
def test_counts_and_offsets_match_the_oracle(n):
    for mask in (si.edge_masks(n)["all_one"], si.edge_masks(n)["last_only"], si.bernoulli_mask(n, 0.1, n)):
        ref = oracle.build_index(mask)
        want = ref_seg_ptr(ref, n)
        seg = torch.full((samo.samo_seg_ptr_len(n) + 8,), -7, dtype=torch.int32, device=DEV)
        nnz = torch.full((1,), -5, dtype=torch.int64, device=DEV)
        samo.samo_count_nonzero(dev_u8(mask), seg, nnz)
        assert nnz.item() == ref.shape[0]
        got = seg.cpu().numpy()
        assert np.array_equal(got[:want.shape[0]], want)
        assert (got[want.shape[0]:] == -7).all(), "wrote past the table"
        ix = samo.samo_build_index(dev_u8(mask))
        assert np.array_equal(ix.idx.cpu().numpy(), ref) and np.array_equal(ix.seg_ptr.cpu().numpy(), want)


def test_offsets_over_more_than_one_look():
    """1100 blocks: the last workgroup's sum takes two looks of 1024 totals unless a running total is nearer."""
    n = 1100 * BLOCK + 5
    mask = torch.zeros(n, dtype=torch.uint8, device=DEV)
    at = torch.arange(0, n, 777, device=DEV)
    mask[at] = 1
    ix = samo.samo_build_index(mask)
    assert ix.nnz == at.numel() and torch.equal(ix.idx.long(), at)
    starts = torch.arange(ix.seg_ptr.numel(), device=DEV) * SEG
    assert torch.equal(ix.seg_ptr.long(), torch.searchsorted(at, starts.clamp(max=n)))


@pytest.mark.parametrize("keep", [0.1, 0.124, 0.126, 0.2, 0.249, 0.251, 0.6])
@pytest.mark.parametrize("first", [0, 1, 2, 3])
def test_fill_where_the_ways_of_collecting_positions_meet(keep, first):
    """`first` kept elements in a segment of their own shift every later run against the 16-byte vectors of idx."""
    n = 21 * 8 * SEG + 333
    mask = si.bernoulli_mask(n, keep, int(1000 * keep))
    mask[:8 * SEG] = 0
    mask[:first] = 1
    mask[9 * 8 * SEG: 9 * 8 * SEG + 4 * SEG] = 1                # half a group full, the other half as it was
    ref = oracle.build_index(mask)
    ix = samo.samo_build_index(dev_u8(mask))
    assert np.array_equal(ix.idx.cpu().numpy(), ref)
    assert np.array_equal(ix.seg_ptr.cpu().numpy(), ref_seg_ptr(ref, n))
