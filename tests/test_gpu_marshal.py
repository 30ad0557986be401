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
