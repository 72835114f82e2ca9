"""The packed argument structs of the torch-facing wrapper hold what the ctypes
structures hold when they are filled field by field, over the forms that
either takes: strides, missing pointers, numpy scalars, and values that only
ctypes takes (integers it wraps, floats it rounds to infinity)."""
import ctypes

import numpy as np
import pytest

from paper_2607_04443_amd import ws


class FakeRows:
    """Shape, strides and address of a device tensor (packing reads no more)."""
    is_cuda = True

    def __init__(self, tokens, strides, ptr, dtype=None):
        self.shape, self._strides, self._ptr = (tokens, 5, 128), strides, ptr
        self.dtype = ws.torch.bfloat16 if dtype is None else dtype

    def stride(self, d=None):
        return self._strides if d is None else self._strides[d]

    def data_ptr(self):
        return self._ptr


A, B = FakeRows(7, (640, 128, 1), 2 ** 47 - 256), FakeRows(7, (640, 128, 1), 4096)
WIDE = FakeRows(7, (2 ** 33, 2 ** 31 + 128, 1), 512)
UNITS = [0, -1, 2 ** 31 - 1, -2 ** 31, 2 ** 32 + 5, np.int64(3)]
EPS = [1e-6, 0.0, 1, 1e39, np.float32(1e-5), float("inf")]


def _query(c, mode, pos, gamma, eps, scale):
    c.mode, c.positions, c.gamma = mode, pos and pos.data_ptr(), gamma and gamma.data_ptr()
    c.eps, c.softmax_scale = eps, scale


@pytest.mark.parametrize("pos,gamma", [(None, None), (A, B), (None, WIDE)])
@pytest.mark.parametrize("unit,eps", list(zip(UNITS, EPS)))
def test_packed_structs_equal_field_by_field(unit, eps, pos, gamma):
    it = ws.ws_append_item()
    it.k, it.v, it.tok_stride, it.head_stride = A.data_ptr(), B.data_ptr(), 640, 128
    d = it.desc
    d.unit, d.kind, d.n_tokens, d.mode = unit, 2, 7, 1
    d.positions, d.gamma, d.eps = pos and pos.data_ptr(), gamma and gamma.data_ptr(), eps
    assert ws.Cache._item(unit, 2, A, B, 1, pos, gamma, eps) == bytes(it)

    q = ws.ws_query_item()
    q.q, q.tok_stride, q.head_stride, q.n_q = WIDE.data_ptr(), 2 ** 33, 2 ** 31 + 128, 7
    _query(q.desc, unit, pos, gamma, eps, 0.5)
    q.q_out, q.out_tok_stride, q.out_head_stride = B.data_ptr(), 640, 128
    assert ws.Cache._query_item(WIDE, B, unit, pos, gamma, eps, 0.5) == bytes(q)
    assert bytes(ws._query_desc(unit, pos, gamma, eps, 0.5)) == bytes(q.desc)

    c = ws.ws_attn_call()
    c.q, c.q_tok_stride, c.q_head_stride, c.n_q = A.data_ptr(), 640, 128, 7
    _query(c.desc, 2, pos, gamma, eps, 0.0)
    c.mask = ws.mask_spec(9, -4, (ws.WS_KIND_COND, ws.WS_KIND_AUDIO))
    c.out, c.out_tok_stride, c.out_head_stride = WIDE.data_ptr(), 2 ** 33, 2 ** 31 + 128
    assert bytes(ws.Cache._call(A, WIDE, c.mask, 2, pos, gamma, eps)) == bytes(c)


def test_refused_arguments_stay_refused():
    for bad in (FakeRows(7, (640, 128, 2), 64), FakeRows(7, (640, 1), 64), FakeRows(7, (640, 128, 1), 64, ws.torch.float32)):
        with pytest.raises(ValueError):
            ws.Cache._item(0, 1, A, bad)
        with pytest.raises(ValueError):
            ws.Cache._call(bad, A, ws.mask_spec(0))
    with pytest.raises(ValueError, match="share"):
        ws.Cache._item(0, 1, A, WIDE)
    with pytest.raises(ValueError, match="same shape"):
        ws.Cache._query_item(A, FakeRows(8, (640, 128, 1), 64))
    for kwargs in (dict(unit=1.5), dict(eps="x"), dict(mode=None)):
        with pytest.raises(TypeError):
            ws.Cache._item(**{**dict(unit=0, kind=1, k=A, v=B), **kwargs})
    with pytest.raises(TypeError):
        ws.Cache._call(A, B, 12)
    assert ctypes.sizeof(ws.ws_attn_call * 0) == len((ws.ws_append_item * 0).from_buffer_copy(b"")) == 0
