"""The encoder at the edges of its column blocks (128 columns filled at a time,
512 counted), and of the 16-bit counting lanes (tiles of 32767 rows and
more): bit-exact against the oracle's encoders, with and without a mask, in
the three layouts, into buffers that hold other bytes beforehand."""
import ctypes

import numpy as np
import pytest

import paper_2608_01536_amd as celty
import workloads
from oracle import layouts, rlc


@pytest.mark.parametrize("M,K,R", [(70, 127, 33), (70, 128, 33), (70, 129, 70), (40, 511, 16), (40, 512, 16),
                                   (40, 641, 40), (32767, 3, 32767), (32768, 3, 32768), (33000, 2, 40000),
                                   (33000, 2, 16376)])
@pytest.mark.parametrize("ws", [0, 50, 97])
@pytest.mark.parametrize("masked", [True, False])
def test_encoder_blocks(M, K, R, ws, masked):
    p = workloads.random_small(M + 7 * K + R + ws, M, K, ws=ws, as_=50, zero_weights=5)
    W = p.W if masked else np.where(p.mask != 0, p.W, np.float16(0))
    mask = p.mask if masked else None
    want = rlc.encode_matrix(W, mask, R)
    T = want.T
    gptr = np.full(T * K + 1, 0xA5A5A5A5, np.uint32)
    values = celty._aligned_empty(8 * want.n_groups, np.uint16)
    runs = celty._aligned_empty(want.n_groups, np.uint32)
    colmax = celty._aligned_empty(K, np.uint16)
    for a in (values, runs, colmax):
        a.view(np.uint8)[:] = 0xA5
    Wb = np.ascontiguousarray(W).view(np.uint16)
    out = celty.celty_rlc_csc()
    st = celty._encode(Wb.ctypes.data, K, None if mask is None else mask.ctypes.data, K, M, K, R, celty.LAYOUT_RLC,
                       gptr.ctypes.data, values.ctypes.data, runs.ctypes.data, colmax.ctypes.data, want.n_groups,
                       ctypes.byref(out), 0)
    assert st == celty.CELTY_OK
    assert (out.n_nnz, out.n_pad) == (want.n_nnz, want.n_pad)
    assert celty.celty_encode_plan(W, mask, R) == (want.n_groups, want.n_nnz, want.n_pad)
    for got, ref in ((gptr, want.gptr), (values, want.values), (runs, want.runs), (colmax, want.colmax)):
        assert np.array_equal(got, ref)
    if M > 1000:
        return
    il = celty.celty_encode(W, mask, R, layout=celty.LAYOUT_INTERLEAVED)
    ref = layouts.encode_interleaved(W, mask, R)
    assert np.array_equal(il.values, ref.values) and np.array_equal(il.runs, ref.runs)
    r16 = celty.celty_encode(W, mask, R, layout=celty.LAYOUT_ROWS16)
    ref = layouts.encode_rows16(W, mask, R)
    assert np.array_equal(r16.gptr, ref.gptr) and np.array_equal(r16.values, ref.values)
    assert np.array_equal(r16.runs.view(np.uint16), ref.rows)
