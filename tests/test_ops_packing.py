"""Host side of the wrappers: the packed argument block has the layout of the C structure, and the
tensor checks refuse what they refused (on CPU tensors posing as device ones)."""

import ctypes

import pytest
import torch

from paper_2609_32415_amd import _lib as L
from paper_2609_32415_amd import ops


def test_packed_arguments_equal_the_structure():
    quads = [tuple(1000 * i + k + 1 for k in range(4)) for i in range(11)]
    segs = (3, 64, 128, 200, *([0] * 13), 0b101)
    flat = [*sum(quads[:8], ()), 77, *sum(quads[8:10], ()), 1, 2, 3, 4, 5, *segs, 6, *quads[10], 7]
    t = [L.ra_tensor(*q) for q in quads]
    want = L.ra_attn_args(*t[:8], 77, t[8], t[9], 1, 2, 3, 4, 5, 3, (ctypes.c_int32 * L.RA_MAX_SEG)(64, 128, 200),
                          0b101, 6, t[10], 7)
    assert L.ARGS_PACK.pack(*flat) == bytes(want)
    assert L.DESC_PACK.pack(1, 2, 128, 300, 400, 0, 0.25, 1, 2) == bytes(
        L.ra_attn_desc(1, 2, 128, 300, 400, 0, 0.25, 1, 2))


class _Posing(torch.Tensor):
    is_cuda = True


def _t(*shape, dtype=torch.bfloat16):
    return torch.zeros(shape, dtype=dtype).as_subclass(_Posing)


def test_views_of_every_layout():
    x = _t(2, 3, 5, 64)
    assert ops._quad("x", x, torch.bfloat16, (2, 3, 5, 64)) == (x.data_ptr(), 960, 320, 64)
    y = _t(2, 5, 3, 64).transpose(1, 2)
    assert ops._quad("y", y, torch.bfloat16, x.shape) == (y.data_ptr(), 960, 64, 192)
    z = _t(2, 3, 9, 64)[:, 1:, 2:7]
    assert ops._quad("z", z, None, (2, 2, 5, 64)) == (z.data_ptr(), 1728, 576, 64)
    assert ops._quad("e", _t(2, 3, 0, 64), torch.bfloat16, (2, 3, 0, 64)) == (0, 0, 0, 0)
    assert ops._quad("n", None, torch.bfloat16, (2, 3, 0, 64)) == (0, 0, 0, 0)


@pytest.mark.parametrize("bad,text", [
    (lambda: torch.zeros(2, 3, 5, 64, dtype=torch.bfloat16), "GPU tensor"),
    (lambda: _t(3, 5, 64), "B, H, S, d"),
    (lambda: _t(2, 3, 6, 64), "shape"),
    (lambda: _t(2, 3, 64, 5).transpose(2, 3), "contiguous"),
    (lambda: _t(2, 3, 5, 64, dtype=torch.float32), "dtype"),
])
def test_refused_tensors(bad, text):
    with pytest.raises(ValueError, match=text):
        ops._quad("x", bad(), torch.bfloat16, (2, 3, 5, 64))
