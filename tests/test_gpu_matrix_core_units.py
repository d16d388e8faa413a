"""GPU tests of the matrix-core path where its units end: rows and ranks that leave part of a 16-row block, contractions
that leave part of a step or batch, token tiles, K slices of t, groups of layers, both launch forms, the dense product at
every batch, and the bounded wait for t.  Same oracle and tolerances as the other parity tests (gpu_util)."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth

pytestmark = pytest.mark.gpu


def _parity(layer, L, X16, tau, **kw):
    got = gu.run_linear(layer, X16)
    want = gu.oracle_linear(L, X16, tau, **kw)
    gu.check_lists(got, want)
    gu.check_outputs(got["Y"], want["Y"], rs.F32)


@pytest.mark.parametrize("d_in,d_out,rank", [(8, 8, 8), (24, 40, 0), (136, 24, 24), (520, 1000, 40), (1032, 264, 136), (4104, 520, 72)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_ragged_units(d_in, d_out, rank, dt):
    L = synth.random_layer(d_in, d_out, rank, dt, seed=41 + d_in + rank)
    for B, mode in ((5, 0), (16, 1), (17, 0), (32, 1)):
        X16, src = gu.tokens_for(L, B, linear=B)
        tau = gu.calibrated_tau(L, src, 0.5)
        layer = gu.prepare(L, tau, max_batch=32, out_dtype=rs.F32, dense_rowmajor=1, batch_mask_mode=mode)
        for launches in (1, 2, 1):
            rs.rsparse_set_tuning(layer, launches=launches)
            _parity(layer, L, X16, tau, batch_mask_mode=mode)
        # the same handle at the other number of token tiles: nothing of the last call shows
        other = X16[:7] if B > 16 else np.concatenate([X16, X16, X16, X16])[:20]
        _parity(layer, L, other, tau, batch_mask_mode=mode)
        layer.destroy()


@pytest.mark.parametrize("cmp_mode", [1, 2])
def test_strict_and_signed_thresholds_on_patterns(cmp_mode):
    """Thresholds on, between and beyond representable values, zeros of both signs, subnormals, infinities and NaN: the
    pattern comparison keeps exactly what the definition keeps."""
    for dt in (synth.F16, synth.BF16):
        L = synth.random_layer(136, 64, 16, dt, seed=7)
        rng = np.random.default_rng(3)
        X16 = synth.encode16(rng.standard_normal((6, 136)), dt)
        inf = 0x7C00 if dt == synth.F16 else 0x7F80
        X16[:, :12] = np.array([0, 0x8000, 1, 0x8001, inf, inf | 0x8000, inf + 1, (inf + 1) | 0x8000, inf - 1, (inf - 1) | 0x8000, 2, 0x8002],
                               dtype=np.uint16)
        vals = synth.decode16(np.abs(X16.view(np.int16)[0, 20:24]).view(np.uint16), dt)
        taus = [0.0, float(np.float32(vals[0])), float(np.nextafter(np.float32(vals[1]), np.float32(9))),
                float(np.nextafter(np.float32(vals[2]), np.float32(0))), 1e-30, 1e30, np.inf, -np.inf] + ([-0.25, -1e30] if cmp_mode == 2 else [])
        layer = gu.prepare(L, 0.0, max_batch=8, out_dtype=rs.F32, dense_rowmajor=1, cmp_mode=cmp_mode)
        for tau in taus:
            rs.rsparse_set_tau(layer, tau)
            got = gu.run_linear(layer, X16)
            want = gu.oracle_linear(L, X16, tau, cmp_mode=cmp_mode)
            gu.check_lists(got, want)
        layer.destroy()


def test_grouped_layers_share_one_launch_and_a_bias():
    """Four layers of different sizes and ranks (one without a low-rank part) on one input, several calls in a row."""
    shapes = [(528, 200), (528, 8), (528, 1032), (528, 16)]
    ranks = [40, 8, 0, 16]
    Ls = [synth.random_layer(a, b, r, synth.BF16, seed=90 + i) for i, ((a, b), r) in enumerate(zip(shapes, ranks))]
    X16, src = gu.tokens_for(Ls[0], 9, linear=3)
    tau = gu.calibrated_tau(Ls[0], src, 0.5)
    layers = [gu.prepare(L, tau, max_batch=16, out_dtype=rs.F32, dense_rowmajor=1) for L in Ls]
    bias = np.linspace(-1, 1, 1032).astype(np.float32)
    rs.rsparse_set_bias(layers[2], bias)
    Xd = gu.to_dev16(X16)
    for _ in range(3):
        Ys = [gu._alloc_out(l, 9) for l in layers]
        rs.rsparse_linear_group(layers, Xd.data_ptr(), 9, [y.data_ptr() for y in Ys], gu.stream_ptr())
        for i, (l, L, y) in enumerate(zip(layers, Ls, Ys)):
            want = gu.oracle_linear(L, X16, tau)["Y"] + (bias if i == 2 else 0)
            gu.check_outputs(gu._read_out(l, y), want, rs.F32)
            rs.rsparse_synchronize(l)


@pytest.mark.parametrize("B", [1, 2, 3, 5, 16, 17, 32])
def test_dense_product_at_every_batch(B):
    for d_in, d_out in ((8, 24), (1032, 1096), (2056, 2056)):        # below and above the row-dot limit
        L = synth.random_layer(d_in, d_out, 8, synth.F16, seed=d_in)
        X16, _ = gu.tokens_for(L, B, linear=B)
        layer = gu.prepare(L, 0.5, max_batch=32, out_dtype=rs.F32, dense_rowmajor=1)
        want = oracle.dense_linear(L.W16, X16, L.dtype, L.dtype, nthreads=8)
        for kernel in (0, 1, 2):
            rs.rsparse_set_tuning(layer, dense_kernel=kernel)
            gu.check_outputs(gu.run_dense(layer, X16), want, rs.F32)
        layer.destroy()


def test_bounded_wait_for_t_runs_out_and_the_handle_recovers():
    """Stage 1 sets no flag (test hook) and the wait is bounded to a few polls: the kernel ends, the call is reported
    as failed once, and the next calls are right again."""
    L = synth.random_layer(520, 328, 40, synth.BF16, seed=5)
    X16, src = gu.tokens_for(L, 12, linear=1)
    tau = gu.calibrated_tau(L, src, 0.5)
    layer = gu.prepare(L, tau, max_batch=16, out_dtype=rs.F32, dense_rowmajor=1)
    _parity(layer, L, X16, tau)
    rs.rsparse_set_tuning(layer, debug_skip_stage1=1, debug_wait_polls=4)
    with pytest.raises(rs.RSparseError):
        gu.run_linear(layer, X16)
    rs.rsparse_set_tuning(layer)
    for _ in range(2):
        _parity(layer, L, X16, tau)


@pytest.mark.parametrize("d_in,d_out,rank,group", [(32, 8, 0, 32), (96, 136, 8, 32), (1024, 264, 40, 1024), (1152, 1160, 72, 128), (4160, 520, 24, 64)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_q4_units(d_in, d_out, rank, group, dt):
    """4-bit weights: outputs that leave part of a 256-output unit or of its second half, contractions shorter than the waves
    of a workgroup, groups cut by wave shares, both token tiles, own and union masks, batches in any order on one handle, and
    the same results as the vector kernels."""
    L = synth.random_layer(d_in, d_out, rank, dt, seed=11 + d_in + d_out)
    Q, S16, Z = synth.quantize_q4(synth.decode16(L.W16, dt), dt, group)
    X16, src = gu.tokens_for(L, 32, linear=5)
    tau = gu.calibrated_tau(L, src, 0.5)
    U16, SV16 = (L.U16, L.SV16) if rank else (None, None)
    for mode in (0, 1):
        cfg = rs.make_config(d_in, d_out, rank, tau, dt, max_batch=32, out_dtype=rs.F32, batch_mask_mode=mode)
        layer = rs.rsparse_prepare_q4(cfg, Q, S16, Z, group, U16, SV16)
        for B in (16, 5, 32, 2, 17):
            want = oracle.rsparse_linear_q4(Q, S16, Z, U16, SV16, X16[:B], dt, tau, group=group, batch_mask_mode=mode)
            rs.rsparse_set_tuning(layer, mfma_min_batch=1)             # (left alone: from three tokens on)
            got = gu.run_linear(layer, X16[:B])
            gu.check_lists(got, want)
            gu.check_outputs(got["Y"], want["Y"], rs.F32)
            rs.rsparse_set_tuning(layer, mfma_min_batch=33)
            vec = gu.run_linear(layer, X16[:B])
            gu.check_lists(got, vec)
            gu.check_outputs(got["Y"], vec["Y"], rs.F32)
        layer.destroy()


@pytest.mark.parametrize("d_in,d_out,rank", [(8, 8, 8), (40, 136, 0), (136, 120, 24), (1032, 264, 136), (4104, 1032, 72)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_column_major_units(d_in, d_out, rank, dt):
    """Column-major W on the matrix cores: outputs that leave part of a 128-output unit, a last step partly past d_in, both
    token tiles, both mask modes, batches in any order on one handle, the dense product, and the vector kernels' results."""
    L = synth.random_layer(d_in, d_out, rank, dt, seed=17 + d_in + d_out)
    X16, src = gu.tokens_for(L, 32, linear=6)
    tau = gu.calibrated_tau(L, src, 0.5)
    for mode in (0, 1):
        layer = gu.prepare(L, tau, max_batch=32, out_dtype=rs.F32, batch_mask_mode=mode)
        for B in (16, 5, 32, 3, 17):
            _parity(layer, L, X16[:B], tau, batch_mask_mode=mode)
            got = gu.run_linear(layer, X16[:B])
            rs.rsparse_set_tuning(layer, mfma_min_batch=33)
            vec = gu.run_linear(layer, X16[:B])
            rs.rsparse_set_tuning(layer)
            gu.check_lists(got, vec)
            gu.check_outputs(got["Y"], vec["Y"], rs.F32)
            gu.check_outputs(gu.run_dense(layer, X16[:B]), oracle.dense_linear(L.W16, X16[:B], L.dtype, L.dtype, nthreads=8), rs.F32)
        layer.destroy()


def test_column_major_group_and_gate_up_pair():
    """A group of layers and the gate / up pair share the two launches at 9 tokens; signed threshold with a bias on one."""
    Ls = [synth.random_layer(520, o, r, synth.BF16, seed=60 + o) for o, r in ((264, 40), (264, 8), (72, 0))]
    X16, src = gu.tokens_for(Ls[0], 9, linear=2)
    tau = gu.calibrated_tau(Ls[0], src, 0.5)
    layers = [gu.prepare(L, tau, max_batch=9) for L in Ls]
    Xd = gu.to_dev16(X16)
    for _ in range(2):
        Ys = [gu._alloc_out(l, 9) for l in layers]
        rs.rsparse_linear_group(layers, Xd.data_ptr(), 9, [y.data_ptr() for y in Ys], gu.stream_ptr())
        outs = [gu._read_out(l, y) for l, y in zip(layers, Ys)]
        for l, L, y in zip(layers, Ls, outs):
            gu.check_outputs(y, gu.oracle_linear(L, X16, tau)["Y"], rs.BF16)
    H = gu._alloc_out(layers[0], 9)
    rs.rsparse_mlp_gate_up(layers[0], layers[1], Xd.data_ptr(), 9, H.data_ptr(), gu.stream_ptr())
    want = oracle.gated_input(synth.encode16(outs[0], synth.BF16), synth.encode16(outs[1], synth.BF16), synth.BF16)
    gu.check_outputs(gu._read_out(layers[0], H), synth.decode16(want, synth.BF16), rs.BF16)


def test_preparing_keeps_two_copies_of_w_at_a_time():
    """dense_rowmajor = 1 doubles the weight footprint, also while the layer is prepared (W goes up in slices): a second thread
    watches the free device memory.  Several slices give the layouts of one upload: the dense product by two kernels that read
    one layout each, and R-Sparse, on rows of the first, a middle and the last slice."""
    import threading

    torch = gu.torch_mod()
    dt, d_in, d_out = synth.F16, 8192, 16392
    L = synth.random_layer(d_in, d_out, 8, dt, seed=2)
    w = d_in * d_out * 2
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    least, stop = [free0], threading.Event()

    def watch():
        while not stop.is_set():
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])

    th = threading.Thread(target=watch)
    th.start()
    layer = gu.prepare(L, 0.5, max_batch=8, out_dtype=rs.F32, dense_rowmajor=1)
    stop.set()
    th.join()
    assert free0 - least[0] < 2 * w + (128 << 20), (free0 - least[0]) / w
    X16, src = gu.tokens_for(L, 5)
    rows = np.r_[0:64, 4000:4200, 8000:8300, d_out - 40:d_out]
    want = synth.decode16(X16, dt) @ synth.decode16(L.W16[rows], dt).T
    for tuning, B in ((dict(dense_kernel=1), 1), (dict(dense_kernel=2), 1), (dict(), 5)):
        rs.rsparse_set_tuning(layer, **tuning)
        gu.check_outputs(gu.run_dense(layer, X16[:B])[:, rows], want[:B], rs.F32)
    rs.rsparse_set_tau(layer, float("-inf"))                         # every channel kept: R-Sparse is the dense product too
    for B in (1, 5):
        gu.check_outputs(gu.run_linear(layer, X16[:B], lists=False)["Y"][:, rows], want[:B], rs.F32)
    layer.destroy()


@pytest.mark.parametrize("form,B", [("columns", 5), ("columns", 20), ("q4", 1), ("q4", 20)])
def test_replayed_graphs_of_the_two_launch_forms(form, B):
    """Column-major and 4-bit layers on the matrix cores inside a captured graph: every replay, with new tokens in the same
    buffer and an eager call at another batch size between replays, equals the oracle (the sums of the first
    launch are taken out by the second)."""
    torch = gu.torch_mod()
    dt = synth.BF16
    L = synth.random_layer(1056, 520, 40, dt, seed=77)
    X16, src = gu.tokens_for(L, 4 * B, linear=B)
    tau = gu.calibrated_tau(L, src, 0.5)
    if form == "q4":
        Q, S16, Z = synth.quantize_q4(synth.decode16(L.W16, dt), dt, 32)
        cfg = rs.make_config(L.d_in, L.d_out, L.rank, tau, dt, max_batch=32, out_dtype=rs.F32)
        layer = rs.rsparse_prepare_q4(cfg, Q, S16, Z, 32, L.U16, L.SV16)
        rs.rsparse_set_tuning(layer, mfma_min_batch=1)                 # (left alone: from three tokens on)
        oracle_of = lambda X: oracle.rsparse_linear_q4(Q, S16, Z, L.U16, L.SV16, X, dt, tau, group=32)["Y"]
    else:
        layer = gu.prepare(L, tau, max_batch=32, out_dtype=rs.F32)
        oracle_of = lambda X: gu.oracle_linear(L, X, tau)["Y"]
    Xd = gu.to_dev16(X16[:B])
    Y = gu._alloc_out(layer, B)
    rs.rsparse_linear(layer, Xd.data_ptr(), B, Y.data_ptr(), gu.stream_ptr())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rs.rsparse_linear(layer, Xd.data_ptr(), B, Y.data_ptr(), torch.cuda.current_stream().cuda_stream)
    for rep in range(4):
        xb = X16[rep * B:(rep + 1) * B]
        Xd.copy_(torch.from_numpy(np.ascontiguousarray(xb).view(np.int16)))
        Y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        gu.check_outputs(Y.cpu().numpy().astype(np.float64), oracle_of(xb), rs.F32)
        other = np.concatenate([xb, xb, xb, xb, xb])[:17 if B <= 16 else 5]
        gu.check_outputs(gu.run_linear(layer, other)["Y"], oracle_of(other), rs.F32)
    layer.destroy()
