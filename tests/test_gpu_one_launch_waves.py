"""The one-launch column kernel where its waves' shares can go wrong: fewer chunks of 8 channels than waves, shares that end inside
a batch of loads or a group of 64 list entries, ranks that give a wave more rows of U_r^T than one group, t over several
rounds of rows, and 4-bit layers that share the vector kernels' launches.  Against the fp64 oracle, fp32 outputs: rel-L2 2e-5
(gpu_util.check_outputs: sums of up to 3e4 terms in 32 bits), lists equal."""
import pytest

import gpu_util as gu
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu
INF = float("inf")


@pytest.mark.parametrize("shape", [(8, 8, 8), (72, 520, 16), (520, 8, 8), (1032, 1096, 0), (2056, 520, 136), (4104, 1032, 8)])
@pytest.mark.parametrize("B", [1, 2, 4, 8])
@pytest.mark.parametrize("tuning", [dict(), dict(splits=1, waves=1), dict(splits=5, waves=2, lowrank_rows=3), dict(lowrank_rows=32)])
def test_shares_of_the_waves(shape, B, tuning):
    d_in, d_out, rank = shape
    L = synth.random_layer(d_in, d_out, rank, synth.BF16 if B % 2 else synth.F16, seed=95 + d_in)
    X16, src = gu.tokens_for(L, B, config=95)
    tau = gu.calibrated_tau(L, src, 0.5)
    for channel_major in (0, 1) if rank else (0,):
        layer = gu.prepare(L, tau, max_batch=B, out_dtype=rs.F32, lowrank_channel_major=channel_major)
        rs.rsparse_set_tuning(layer, launches=1, mfma_min_batch=33, lowrank_wgs=3 * channel_major, **tuning)
        for t in (tau, -INF, INF, tau):                       # half, all and none of the channels; the handle is reused
            rs.rsparse_set_tau(layer, t)
            got = gu.run_linear(layer, X16)
            want = gu.oracle_linear(L, X16, t)
            gu.check_lists(got, want)
            gu.check_outputs(got["Y"], want["Y"], rs.F32)
        layer.destroy()


@pytest.mark.parametrize("waves", [8, 2])
@pytest.mark.parametrize("rank", [0, 8, 40])
@pytest.mark.parametrize("B", [1, 4])
def test_batches_that_waves_claim(waves, rank, B):
    """Lists that end around the batches a wave starts with (four entries, two to a wave) and the first ones that are claimed, with
    and without rows of U_r^T behind them, which then start inside a batch: a fixed count gives the exact length at one token."""
    L = synth.random_layer(264, 1032, rank, synth.F16, seed=97)
    X16, _ = gu.tokens_for(L, B, config=97)
    first = 2 * waves * 4
    for k in sorted({1, 3, 4, 5, 4 * waves - 1, 4 * waves, 4 * waves + 1, first - rank % first, first - 1, first, first + 1, first + 6, 264}):
        for channel_major in (0, 1) if rank else (0,):
            layer = gu.prepare(L, 0.0, max_batch=B, out_dtype=rs.F32, topk=k, lowrank_channel_major=channel_major)
            rs.rsparse_set_tuning(layer, launches=1, mfma_min_batch=33, splits=1, waves=waves, lowrank_wgs=channel_major)
            got = gu.run_linear(layer, X16)
            want = gu.oracle_linear(L, X16, 0.0, topk=k)
            gu.check_lists(got, want)
            gu.check_outputs(got["Y"], want["Y"], rs.F32)
            layer.destroy()


@pytest.mark.parametrize("B,launches", [(1, 0), (3, 0), (9, 0), (1, 2), (3, 2), (9, 2), (20, 0)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_4_bit_layers_share_the_vector_launches(dt, B, launches):
    """Three 4-bit layers of different widths and ranks on one input, in one launch and in two (which batches above 16 tokens take
    by themselves): every layer's outputs and lists against the oracle's."""
    qs = [Q4Layer(synth.make_layer(1152, d_out, rank, dt, config=96, linear=i), 128) for i, (d_out, rank) in enumerate(((2120, 40), (72, 8), (1024, 0)))]
    X16, src = gu.tokens_for(qs[0].L, B, config=96)
    tau = gu.calibrated_tau(qs[0].L, src, 0.5)
    layers = [q.prepare(tau, max_batch=B, out_dtype=rs.F32) for q in qs]
    for l in layers:
        rs.rsparse_set_tuning(l, mfma_min_batch=33, launches=launches)
    Xd = gu.to_dev16(X16)
    for _ in range(2):
        Ys = [gu._alloc_out(l, B) for l in layers]
        rs.rsparse_linear_group(layers, Xd.data_ptr(), B, [y.data_ptr() for y in Ys], gu.stream_ptr())
        for q, l, y in zip(qs, layers, Ys):
            want = q.oracle(X16, tau)
            got = {"act": [rs.rsparse_last_active(l, b) for b in range(B)], "union": rs.rsparse_last_active(l, -1)}
            gu.check_lists(got, want)
            gu.check_outputs(gu._read_out(l, y), want["Y"], rs.F32)
    for l in layers:
        l.destroy()


# splits of the plain rule -> with slots left to stage 1: 32 -> 26, 28 -> 26, 22 -> 15
@pytest.mark.parametrize("shape", [(2048, (2048, 2048, 2048), 256), (2240, (3328, 3328), 280), (5120, (5120, 2048, 2048), 640)])
def test_groups_that_leave_slots_to_stage_1(shape):
    """Layers of a group with large ranks at one token, whose launch has fewer splits than its tiles alone would get: outputs and lists
    of every layer, each call twice on the same handles, and with a launch shape of the caller's in between."""
    d_in, d_outs, rank = shape
    Ls = [synth.random_layer(d_in, d_out, rank, synth.BF16, seed=98 + i) for i, d_out in enumerate(d_outs)]
    X16, src = gu.tokens_for(Ls[0], 1, config=98)
    tau = gu.calibrated_tau(Ls[0], src, 0.5)
    layers = [gu.prepare(L, tau, out_dtype=rs.F32) for L in Ls]
    want = [gu.oracle_linear(L, X16, tau) for L in Ls]
    Xd = gu.to_dev16(X16)
    for tuning in ({}, dict(splits=7), {}):
        for l in layers:
            rs.rsparse_set_tuning(l, **tuning)
        Ys = [gu._alloc_out(l, 1) for l in layers]
        rs.rsparse_linear_group(layers, Xd.data_ptr(), 1, [y.data_ptr() for y in Ys], gu.stream_ptr())
        for l, y, w in zip(layers, Ys, want):
            gu.check_lists({"act": [rs.rsparse_last_active(l, 0)], "union": rs.rsparse_last_active(l, -1)}, w)
            gu.check_outputs(gu._read_out(l, y), w["Y"], rs.F32)
    for l in layers:
        l.destroy()
