"""The index build whose counts are polled in page-locked memory: the counts there, masks counted in two launches, other work ahead of
the build for longer than it polls, several threads on streams of their own, a stream under capture, launches that fail."""
import ctypes
import threading

import pytest
import torch

import paper_2302_05045_amd as samo
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _mask(n, keep, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return (torch.rand(n, generator=gen, device=DEV) < keep).to(torch.uint8)


def _check(mask, ix):
    want = mask.nonzero().view(-1).to(torch.int32)
    assert ix.nnz == want.numel() and torch.equal(ix.idx, want)
    ends = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), mask.long().cumsum(0)])
    at = torch.clamp(torch.arange(ix.seg_ptr.numel(), device=DEV) * samo.SEG_ELEMS, max=mask.numel())
    assert torch.equal(ix.seg_ptr, ends[at].to(torch.int32))


@pytest.mark.parametrize("sizes", [(0,), (1,), (1023, 0, 1025), (65536, 65537, 7)])
def test_counts_in_page_locked_memory(sizes):
    masks = [_mask(n, 0.3, 3 + n) for n in sizes]
    k = len(masks)
    counts = torch.full((k + 1,), -7, dtype=torch.int64, pin_memory=True)
    nnz = torch.full((k,), -7, dtype=torch.int64, device=DEV)
    seg_ptrs = [torch.empty(samo.samo_seg_ptr_len(n), dtype=torch.int32, device=DEV) for n in sizes]
    flags = [torch.empty(max(samo._flag_bytes(n), 16), dtype=torch.uint8, device=DEV) for n in sizes]
    jobs, ptrs = (samo.IndexJob * k)(), (ctypes.c_void_p * k)()
    for i, m in enumerate(masks):
        jobs[i] = samo.IndexJob(m.data_ptr() if sizes[i] else None, sizes[i], None, 0, seg_ptrs[i].data_ptr(), nnz.data_ptr() + 8 * i)
        ptrs[i] = flags[i].data_ptr()
    stream = torch.cuda.current_stream().cuda_stream
    entry = samo.lib().samo_count_flags_mirrored_batched
    assert entry(jobs, ptrs, None, k, stream) == samo.SAMO_ERR_NULL
    assert entry(jobs, ptrs, counts.data_ptr() + 4, k, stream) == samo.SAMO_ERR_ALIGN
    assert entry(jobs, ptrs, counts.data_ptr(), k, stream) == samo.SAMO_OK
    torch.cuda.synchronize()
    assert counts.tolist() == [int(m.sum()) for m in masks] + [-7] and counts[:k].tolist() == nnz.tolist()


@pytest.mark.parametrize("sizes", [((1 << 26) + 5,), (1 << 25, 1 << 25), (5, 1 << 26, 1000), (40_000_001, 30_000_000, 0, 77)])
def test_masks_counted_in_two_launches(sizes):
    masks = [_mask(n, 0.1, 5 + i) for i, n in enumerate(sizes)]
    for m, ix in zip(masks, samo.samo_build_index_many(m for m in masks)):             # any iterable of masks
        _check(m, ix)


def test_work_ahead_for_longer_than_the_host_polls():
    masks = [_mask(n, 0.2, 9) for n in (5000, 70_000)]
    torch.cuda._sleep(50_000_000)                     # some tens of milliseconds
    for m, ix in zip(masks, samo.samo_build_index_many(masks)):
        _check(m, ix)


def test_threads_on_streams_of_their_own():
    masks = [_mask(100_000 + 1000 * i, 0.1 + 0.02 * i, i) for i in range(6)]
    torch.cuda.synchronize()
    found, failed = [None] * 6, []

    def build(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    found[i] = samo.samo_build_index(masks[i])
                torch.cuda.current_stream().synchronize()
        except Exception as e:                        # noqa: BLE001
            failed.append(e)

    threads = [threading.Thread(target=build, args=(i,)) for i in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    for m, ix in zip(masks, found):
        _check(m, ix)


MIRRORED = ctypes.CFUNCTYPE(ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p)


def _mirrored_through(entry):
    """The address of the entry's callback, which calls entry(real entry, arguments); the callback object keeps it alive."""
    real = ctypes.cast(samo._entry_address("samo_count_flags_mirrored_batched"), MIRRORED)
    callback = MIRRORED(lambda *a: entry(real, a))
    return callback, ctypes.cast(callback, ctypes.c_void_p).value


def test_build_under_capture_is_refused_and_captures_no_page_locked_memory(monkeypatch):
    """Nothing runs on a stream under capture, so the read-back of the counts is refused there.  The capture itself goes on, and its graph
    can be launched: what it holds must not write to page-locked memory that has gone back to its cache."""
    with open("/proc/self/maps") as maps:
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    calls = []
    callback, address = _mirrored_through(lambda real, a: (calls.append(a[2]), real(*a))[1])
    entry_address = samo._entry_address
    monkeypatch.setattr(samo, "_entry_address", lambda name: address if name == "samo_count_flags_mirrored_batched" else entry_address(name))
    mask = _mask(70_000, 0.2, 9)
    side, graph = torch.cuda.Stream(), ctypes.c_void_p()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        _check(mask, samo.samo_build_index(mask))                    # the allocators hold what the next call needs
        assert len(calls) == 1
        torch.cuda.synchronize()
        stream = ctypes.c_void_p(side.cuda_stream)
        assert hip.hipStreamBeginCapture(stream, 1) == 0
        try:
            with pytest.raises(RuntimeError):
                samo.samo_build_index(mask)
        finally:
            hip.hipStreamEndCapture(stream, ctypes.byref(graph))
            if graph.value:
                hip.hipGraphDestroy(graph)
        assert len(calls) == 1, "page-locked memory of a call that has returned is written by the captured launch"
        hip.hipGetLastError()
        torch.cuda.synchronize()
        for _ in range(3):
            _check(mask, samo.samo_build_index(mask))
        assert len(calls) == 4
    del callback


@pytest.mark.parametrize("fails", [0, 1])
def test_a_launch_that_fails(fails):
    """The counts of the launches before it are waited for: the page-locked memory goes back to its cache with the call."""
    seen = []

    def entry(real, a):
        seen.append((a[2], a[3]))
        return real(*a) if len(seen) != fails + 1 else samo.SAMO_ERR_HIP
    callback, address = _mirrored_through(entry)
    masks = [_mask(n, 0.1, 4) for n in ((1 << 25) + 3, 5000, 1 << 25)]          # counted in two launches
    torch.cuda.synchronize()
    torch.cuda._sleep(50_000_000)                     # for longer than the host polls
    status = samo._marshal.build_indices(masks, samo._stream, samo._scratch, samo._entry_address("samo_count_flags_batched"),
                                         samo._entry_address("samo_fill_index_batched"), address, samo._entry_address("hipStreamIsCapturing"))
    assert status == samo.SAMO_ERR_HIP and len(seen) == fails + 1
    for counts, num_jobs in seen[:fails]:
        found = list((ctypes.c_int64 * num_jobs).from_address(counts))
        assert found == [int(m.sum()) for m in masks[:num_jobs]]
    torch.cuda.synchronize()
    for m, ix in zip(masks, samo.samo_build_index_many(masks)):
        _check(m, ix)
    del callback
