"""GPU tests of the row-dot dense kernel (dense_kernel = 2): the kernel asked for is the one that runs, at the sizes where its
units end, on every batch tile, in groups, and refused where it was."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth

pytestmark = pytest.mark.gpu


def _row_dots(W, x):
    """The kernel's own order in fp32: 64 partial sums per row, chunk c of 8 columns in sum c % 64, ascending, fused
    multiply-adds; then a butterfly over the 64.  (An fp64 sum of an exact product and an fp32 number, rounded once.)"""
    rows, d = W.shape
    n = -(-d // 512) * 512
    Wp, xp = np.zeros((rows, n)), np.zeros(n)
    Wp[:, :d], xp[:d] = W, x
    p = (Wp * xp).reshape(rows, n // 512, 64, 8)
    acc = np.zeros((rows, 64), np.float32)
    for j in range(n // 512):
        for e in range(8):
            acc = (acc.astype(np.float64) + p[:, j, :, e]).astype(np.float32)
    for s in (32, 16, 8, 4, 2, 1):
        acc = acc + acc[:, np.arange(64) ^ s]
    return acc[:, 0]


@pytest.mark.parametrize("d_in,d_out", [(8, 8), (72, 40), (520, 1000), (2048, 2056), (8200, 520), (32768, 136)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_the_row_dot_kernel_runs_where_it_is_asked_for(d_in, d_out, dt):
    """Bit for bit the sums of row dots in bf16 (in fp16 the hardware's two-element dot products sum in an order of their own),
    also on layers of 2^22 weights and more and with the matrix cores switched off."""
    L = synth.random_layer(d_in, d_out, 0, dt, seed=d_in + d_out)
    X16, _ = gu.tokens_for(L, 1)
    layer = gu.prepare(L, 0.5, max_batch=1, out_dtype=rs.F32, dense_rowmajor=1)
    for tuning in (dict(dense_kernel=2), dict(dense_kernel=2, mfma_min_batch=33), dict(dense_kernel=2, nontemporal=2)):
        rs.rsparse_set_tuning(layer, **tuning)
        got = gu.run_dense(layer, X16)
        gu.check_outputs(got, oracle.dense_linear(L.W16, X16, dt, dt, nthreads=8), rs.F32)
        if dt == synth.BF16:
            want = _row_dots(synth.decode16(L.W16, dt), synth.decode16(X16, dt)[0])
            assert np.array_equal(got[0].astype(np.float32).view(np.uint32), want.view(np.uint32)), tuning
    layer.destroy()


@pytest.mark.parametrize("B", [1, 2, 3, 4, 7, 8, 9, 32])
def test_row_dots_of_a_group_at_every_batch_tile(B):
    """Layers of different heights share the launch; every batch tile with the matrix cores off; NaN and infinities stay in
    their token."""
    dt = synth.F16
    Ls = [synth.random_layer(424, o, 0, dt, seed=70 + o) for o in (8, 264, 24)]
    X16, _ = gu.tokens_for(Ls[0], B, linear=B)
    x = synth.decode16(X16, dt)
    x[0, 423] = np.inf
    if B > 2:
        x[2, 0] = np.nan
    X16 = synth.encode16(x, dt)
    layers = [gu.prepare(L, 0.5, max_batch=32, out_dtype=rs.F32, dense_rowmajor=1) for L in Ls]
    for l in layers:
        rs.rsparse_set_tuning(l, dense_kernel=2, mfma_min_batch=33)
    Xd = gu.to_dev16(X16)
    Ys = [gu._alloc_out(l, B) for l in layers]
    rs.rsparse_dense_ref_group(layers, Xd.data_ptr(), B, [y.data_ptr() for y in Ys], gu.stream_ptr())
    for l, L, y in zip(layers, Ls, Ys):
        gu.check_outputs(gu._read_out(l, y), oracle.dense_linear(L.W16, X16, dt, dt, nthreads=8), rs.F32)
        l.destroy()


def test_row_dots_are_refused_without_the_copy_and_beyond_lds():
    dt = synth.BF16
    L = synth.random_layer(8200, 16, 0, dt, seed=1)
    X16, _ = gu.tokens_for(L, 8)
    for kw, B in ((dict(), 1), (dict(dense_rowmajor=1), 8)):
        layer = gu.prepare(L, 0.5, max_batch=8, **kw)
        rs.rsparse_set_tuning(layer, dense_kernel=2, mfma_min_batch=33)
        with pytest.raises(rs.RSparseError):
            gu.run_dense(layer, X16[:B])
        layer.destroy()
