"""The one-launch kernels after a bounded wait ran out, and which launches a layer gets.  A wait that runs out is forced from the
host (stage 1 publishes nothing, a few polls), so every kernel ends normally."""
import numpy as np
import pytest

import gpu_util as gu
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("strip_cols", [0, 64])
def test_the_static_entry_reports_the_wait_and_recovers(strip_cols):
    """On the library's own scratch as on the handle's: the documented message, and both entries are right afterwards."""
    L = synth.random_layer(520, 328, 40, synth.BF16, seed=6)
    X16, src = gu.tokens_for(L, 2, linear=2)
    tau = gu.calibrated_tau(L, src, 0.5)
    want = gu.oracle_linear(L, X16, tau)
    layer = gu.prepare(L, tau, max_batch=2, out_dtype=rs.F32, strip_cols=strip_cols)
    Xd = gu.to_dev16(X16)
    for entry in (rs.rsparse_linear_static, rs.rsparse_linear):
        Y = gu._alloc_out(layer, 2)
        rs.rsparse_set_tuning(layer, debug_skip_stage1=1, debug_wait_polls=4)
        entry(layer, Xd.data_ptr(), 2, Y.data_ptr(), gu.stream_ptr())
        with pytest.raises(rs.RSparseError, match="wait of the one-launch kernel ran out"):
            rs.rsparse_synchronize(layer)
        rs.rsparse_set_tuning(layer)
        for again in (entry, rs.rsparse_linear, rs.rsparse_linear_static):
            Y = gu._alloc_out(layer, 2)
            again(layer, Xd.data_ptr(), 2, Y.data_ptr(), gu.stream_ptr())
            rs.rsparse_synchronize(layer)
            gu.check_outputs(gu._read_out(layer, Y), want["Y"], rs.F32)
    layer.destroy()


@pytest.mark.parametrize("strip_cols", [0, 128])
@pytest.mark.parametrize("B", [3, 4, 7, 8])
@pytest.mark.parametrize("d_in,rows", [(3080, 5), (3080, 9), (6152, 32), (264, 8)])
def test_tokens_staged_for_stage_1(d_in, rows, B, strip_cols):
    """Four tokens and rows enough, eight tokens: the masked tokens lie in LDS, 6144 and 3072 channels at a time.  Chunks that end inside
    the last one, several rows a wave, waves without rows, own and union masks, calls of other batch sizes between (the tags of all
    token slots agree), and a wait that runs out."""
    L = synth.random_layer(d_in, 136, 40, synth.F16, seed=d_in)
    X16, src = gu.tokens_for(L, 8, linear=3)
    tau = gu.calibrated_tau(L, src, 0.5)
    for mode in (0, 1):
        layer = gu.prepare(L, tau, max_batch=8, out_dtype=rs.F32, strip_cols=strip_cols, batch_mask_mode=mode)
        forms = dict(launches=1, mfma_min_batch=33, lowrank_rows=rows)
        for b in (B, 1, B, 2, B):
            rs.rsparse_set_tuning(layer, **forms)
            got = gu.run_linear(layer, X16[:b])
            want = gu.oracle_linear(L, X16[:b], tau, batch_mask_mode=mode)
            gu.check_lists(got, want)
            gu.check_outputs(got["Y"], want["Y"], rs.F32)
        rs.rsparse_set_tuning(layer, **forms, debug_skip_stage1=1, debug_wait_polls=4)
        with pytest.raises(rs.RSparseError, match="ran out"):
            gu.run_linear(layer, X16[:B])
        rs.rsparse_set_tuning(layer, **forms)
        for _ in range(2):
            gu.check_outputs(gu.run_linear(layer, X16[:B])["Y"], gu.oracle_linear(L, X16[:B], tau, batch_mask_mode=mode)["Y"], rs.F32)
        layer.destroy()


def test_a_layer_above_the_column_kernels_descriptor():
    """65536 -> 16384: 2 GiB of W.  On the matrix cores, which do not read the column-major copy, it stays one launch: a wait that is
    made to run out is reported.  At one and four tokens it takes two launches, which have no such wait.  W is zero but for the
    first and last 64 rows, whose outputs are checked."""
    d_in, d_out, rank, dt = 65536, 16384, 8, synth.BF16
    small = synth.random_layer(d_in, 128, rank, dt, seed=12)
    W = np.zeros((d_out, d_in), dtype=np.uint16)
    U = np.zeros((d_out, rank), dtype=np.uint16)
    rows = np.r_[0:64, d_out - 64:d_out]
    W[rows], U[rows] = small.W16, small.U16
    X16, src = gu.tokens_for(small, 8, linear=4)
    tau = gu.calibrated_tau(small, src, 0.5, n_calib=8)
    cfg = rs.make_config(d_in, d_out, rank, tau, dt, max_batch=8, out_dtype=rs.F32, dense_rowmajor=1)
    layer = rs.rsparse_prepare_factors(cfg, W, U, small.SV16)
    del W

    def check(B):
        got, want = gu.run_linear(layer, X16[:B]), gu.oracle_linear(small, X16[:B], tau)
        rs.rsparse_synchronize(layer)
        gu.check_lists(got, want)
        gu.check_outputs(got["Y"][:, rows], want["Y"], rs.F32)

    for B in (8, 1, 4):
        check(B)
    Xd, Y = gu.to_dev16(X16), gu._alloc_out(layer, 8)
    rs.rsparse_set_tuning(layer, debug_skip_stage1=1, debug_wait_polls=4)
    rs.rsparse_linear(layer, Xd.data_ptr(), 8, Y.data_ptr(), gu.stream_ptr())
    with pytest.raises(rs.RSparseError, match="ran out"):
        rs.rsparse_synchronize(layer)
    rs.rsparse_linear(layer, Xd.data_ptr(), 1, Y.data_ptr(), gu.stream_ptr())
    rs.rsparse_synchronize(layer)
    rs.rsparse_set_tuning(layer)
    for B in (8, 1):
        check(B)
    layer.destroy()


def test_more_splits_than_the_kernels_division_covers():
    """2^20 outputs are 2048 column tiles: from 1024 splits on the workgroup numbers times the tiles pass 2^32."""
    L = synth.random_layer(8, 1 << 20, 8, synth.F16, seed=13)
    X16, src = gu.tokens_for(L, 1, linear=5)
    layer = gu.prepare(L, 0.0, out_dtype=rs.F32)
    for tuning in (dict(), dict(splits=1100, waves=1), dict(splits=2, waves=1, tile_map=2)):
        rs.rsparse_set_tuning(layer, **tuning)
        got, want = gu.run_linear(layer, X16), gu.oracle_linear(L, X16, 0.0)
        gu.check_lists(got, want)
        gu.check_outputs(got["Y"], want["Y"], rs.F32)
    layer.destroy()


@pytest.mark.parametrize("channel_major", [0, 1])
def test_one_handle_through_all_forms_in_turn(channel_major):
    """Tags and generations agree whatever a handle is called for in turn: the gate / up pair, either layer by itself, the group,
    one to three batch tiles, both forms of stage 1, two launches, the dense product, the static entry, and a wait that runs out in
    between.  512-wide tiles: 1096 outputs are three, the last ragged."""
    dt, tokens = synth.BF16, 20
    Ls = [synth.random_layer(1032, 1096, r, dt, seed=50 + r) for r in (40, 264)]
    X16, src = gu.tokens_for(Ls[0], tokens, linear=6)
    tau = gu.calibrated_tau(Ls[0], src, 0.5)
    layers = [gu.prepare(L, tau, max_batch=tokens, lowrank_channel_major=channel_major) for L in Ls]
    want = [gu.oracle_linear(L, X16, tau)["Y"] for L in Ls]
    Xd, s = gu.to_dev16(X16), gu.stream_ptr()
    forms = dict(mfma_min_batch=33, lowrank_wgs=7 * channel_major)

    def one(i, B, fn=rs.rsparse_linear):
        Y = gu._alloc_out(layers[i], B)
        fn(layers[i], Xd.data_ptr(), B, Y.data_ptr(), s)
        rs.rsparse_synchronize(layers[i])
        gu.check_outputs(gu._read_out(layers[i], Y), want[i][:B], dt)

    def group(B):
        Ys = [gu._alloc_out(l, B) for l in layers]
        rs.rsparse_linear_group(layers, Xd.data_ptr(), B, [y.data_ptr() for y in Ys], s)
        for l, y, w in zip(layers, Ys, want):
            rs.rsparse_synchronize(l)
            gu.check_outputs(gu._read_out(l, y), w[:B], dt)

    def pair(B):
        H = gu._alloc_out(layers[0], B)
        rs.rsparse_mlp_gate_up(layers[0], layers[1], Xd.data_ptr(), B, H.data_ptr(), s)
        for l in layers:
            rs.rsparse_synchronize(l)
        g, u = (synth.decode16(synth.encode16(w[:B], dt), dt) for w in want)
        h = g / (1.0 + np.exp(-g)) * u
        got = gu._read_out(layers[0], H)
        # one rounding each of g, u and h to bf16, 2^-9 at most; a sum in another order can move each by one step
        assert np.linalg.norm(got - h) <= 1.5e-2 * np.linalg.norm(h)

    for turn in range(2):
        for l in layers:
            rs.rsparse_set_tuning(l, **forms)
        for step in (lambda: pair(1), lambda: one(0, 1), lambda: group(3), lambda: one(1, 17), lambda: pair(8), lambda: one(1, 1), lambda: one(0, 20),
                     lambda: group(12), lambda: pair(2), lambda: one(0, 4, rs.rsparse_linear_static), lambda: one(1, 2), lambda: pair(4)):
            step()
        for l in layers:
            rs.rsparse_set_tuning(l, **dict(forms, lowrank_wgs=-1))
        pair(1), group(9), one(1, 3)
        rs.rsparse_set_tuning(layers[1], launches=2, mfma_min_batch=33)
        one(1, 5), one(1, 1)
        rs.rsparse_set_tuning(layers[1], **forms, debug_skip_stage1=1, debug_wait_polls=4)
        Y = gu._alloc_out(layers[1], 17)
        rs.rsparse_linear(layers[1], Xd.data_ptr(), 17, Y.data_ptr(), s)
        with pytest.raises(rs.RSparseError, match="ran out"):
            rs.rsparse_synchronize(layers[1])
    for l in layers:
        l.destroy()
