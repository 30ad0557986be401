"""Tensor arguments of the binding on the GPU: native and Python checks give the same pointers and refusals."""
import pytest
import torch

import paper_2302_05045_amd as samo
from gpu_util import DEV

pytestmark = pytest.mark.gpu


def _outcome(fn, *args):
    try:
        return fn(*args)
    except (TypeError, ValueError) as e:
        return type(e), str(e)


def test_native_and_python_marshalling_agree():
    from paper_2302_05045_amd import _marshal

    class Sub(torch.Tensor):
        pass
    base = torch.zeros(64, device=DEV)
    vectors = [base, base[4:], base[::2], base.view(8, 8), base[:0], base.half(), base.as_subclass(Sub),
               torch.nn.Parameter(base), base[1:2], base.view(8, 8)[:, 1], torch.zeros((), device=DEV)]
    for t in vectors:
        for dtype in (torch.float32, torch.float16):
            for more in ((), (None,), (0,), (60,), (64,), (65,)):
                assert _outcome(_marshal.vector, t, dtype, "t", *more) == _outcome(samo._dev_python, t, dtype, "t", *more)
    half = base.half()
    for t in (half.view(8, 8), half.view(8, 8).t(), half.view(4, 16)[:, :8], half, half.view(8, 8)[:0], base.view(8, 8),
              half.view(1, 64), half.view(8, 8).as_subclass(Sub)):
        assert _outcome(_marshal.matrix, t, "m") == _outcome(samo._dev_matrix_python, t, "m")


def test_the_stream_is_the_current_one():
    side = torch.cuda.Stream()
    assert samo._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert samo._stream() == side.cuda_stream
    assert samo._stream() == torch.cuda.current_stream().cuda_stream


def test_native_and_python_index_builds_agree(monkeypatch):
    """The loops over the masks exist twice; the native ones launch the fill in several parts (the first from 32 M elements on)."""
    from paper_2302_05045_amd import _marshal

    class Sub(torch.Tensor):
        pass
    gen = torch.Generator(device=DEV).manual_seed(3)
    bern = lambda n, keep: (torch.rand(n, generator=gen, device=DEV) < keep).to(torch.uint8)
    small = [bern(n, 0.3) for n in (1, 0, 1024, 70001)]
    large = [bern(n, 0.05) for n in (20_000_003, 1000, 20_000_001, 0, 40_000_000, 17, 50_000_000, 3000)]
    wide = bern(4096, 0.5)
    calls = [small, large, [wide[1:]], [wide[::2]], [wide.view(64, 64)], [wide.float()], small + [wide.as_subclass(Sub)],
             [wide.cpu()], small + [None], tuple(small), [torch.nn.Parameter(wide, requires_grad=False)]]

    def outcome(masks):
        try:
            return samo.samo_build_index_many(masks)
        except (TypeError, ValueError, AttributeError, samo.SamoError) as e:
            return type(e), str(e)
    native = [outcome(c) for c in calls]
    assert isinstance(_marshal.build_indices(small, samo._stream, samo._scratch, samo._entry_address("samo_count_flags_batched"),
                                             samo._entry_address("samo_fill_index_batched")), list)
    monkeypatch.setattr(samo, "_marshal", None)
    for masks, got in zip(calls, native):
        want = outcome(masks)
        if isinstance(want, tuple):
            assert got == want
            continue
        for a, b in zip(got, want):
            assert type(a) is samo.Index and a.nnz == b.nnz and a.n == b.n
            assert torch.equal(a.idx, b.idx) and torch.equal(a.seg_ptr, b.seg_ptr)
            assert a.idx.dtype == b.idx.dtype and a.seg_ptr.dtype == b.seg_ptr.dtype


def test_index_builds_on_a_side_stream_beside_work_on_the_current_one():
    """The fill is launched in parts and the flag words are given back while it still reads them, in stream order: scratch memory, counts
    and indices belong to the stream that is current, and what other streams allocate meanwhile is not theirs."""
    gen = torch.Generator(device=DEV).manual_seed(5)
    sizes = (20_000_003, 1000, 20_000_001, 0, 40_000_000, 17, 50_000_000, 3000)
    masks = [(torch.rand(n, generator=gen, device=DEV) < 0.05).to(torch.uint8) for n in sizes]
    want = samo.samo_build_index_many(masks)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    flag_bytes = sum(samo._flag_bytes(n) for n in sizes)
    for _ in range(3):
        with torch.cuda.stream(side):
            got = samo.samo_build_index_many(masks)
            torch.full((flag_bytes,), 0xff, dtype=torch.uint8, device=DEV)      # the flag words' memory, next in the stream
        for _ in range(4):
            torch.full((flag_bytes,), 0xff, dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        for a, b in zip(got, want):
            assert a.nnz == b.nnz and torch.equal(a.idx, b.idx) and torch.equal(a.seg_ptr, b.seg_ptr)
