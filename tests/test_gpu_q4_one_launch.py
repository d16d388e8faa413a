"""The one-launch kernel of 4-bit weights where it can go wrong: groups shorter and longer than a wave's run of channels, runs of 8, 16 and
32 channels that end inside and at the ends of groups, more waves than runs, several tiles of 1024 columns with a ragged last one,
several batch tiles, coefficients too large to carry the codes' power of two, the gate / up pair, and a layer too large for it.  Against
the fp64 oracle, fp32 outputs: rel-L2 2e-5 (gpu_util.check_outputs), lists equal; the two-launch form of the same calls besides."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu
INF = float("inf")


def _check(layer, X16, t, want, **tuning):
    rs.rsparse_set_tuning(layer, mfma_min_batch=33, **tuning)
    rs.rsparse_set_tau(layer, t)
    got = gu.run_linear(layer, X16)
    gu.check_lists(got, want)
    gu.check_outputs(got["Y"], want["Y"], rs.F32)


# tiles * d_in / 32: 1 to 24 (runs of 8 channels), 640 (16), 1024 (32: one tile, two and sixteen)
SHAPES = [(32, 8, 8, 32), (96, 1032, 0, 32), (1152, 2120, 40, 128), (1024, 72, 16, 1024), (5120, 3080, 8, 64), (32768, 8, 8, 256), (16384, 1032, 24, 64)]


@pytest.mark.parametrize("shape,B", [(s, B) for s in SHAPES for B in (1, 2, 3, 9)] + [((2048, 16264, 24, 256), 1)])
def test_runs_groups_and_batch_tiles(shape, B):
    d_in, d_out, rank, group = shape
    q = Q4Layer(synth.random_layer(d_in, d_out, rank, synth.BF16 if B % 2 else synth.F16, seed=98 + d_in), group)
    X16, src = gu.tokens_for(q.L, B, config=98)
    tau = gu.calibrated_tau(q.L, src, 0.5)
    layer = q.prepare(tau, max_batch=B, out_dtype=rs.F32)
    wants = [(t, q.oracle(X16, t)) for t in (tau, -INF, INF)]          # half, all and none of the channels; the handle is reused
    for tuning in (dict(), dict(splits=1, waves=2, lowrank_rows=3), dict(splits=7, lowrank_rows=8), dict(launches=2)):
        for t, want in wants:
            _check(layer, X16, t, want, **tuning)
    layer.destroy()


@pytest.mark.parametrize("B", [1, 2])
def test_coefficients_beyond_the_carried_range(B):
    """bf16 tokens with entries from 1e27 on in some groups, in the middle of others and in none of the rest: those groups keep the
    codes' 2^24 in their scale."""
    q = Q4Layer(synth.random_layer(1024, 1032, 8, synth.BF16, seed=99), 128)
    X16, src = gu.tokens_for(q.L, B, config=99)
    tau = gu.calibrated_tau(q.L, src, 0.5)
    x = synth.decode16(X16, synth.BF16)
    x[:, [3, 200, 255]] = [[1e30, -3e28, 2e27]]
    layer = q.prepare(tau, max_batch=B, out_dtype=rs.F32)
    for splits in (1, 4):
        large = synth.encode16(x, synth.BF16)
        _check(layer, large, tau, q.oracle(large, tau), splits=splits)
    x[:, :] = 0.0                                              # the large ones alone: nothing of the small ones is lost beside them
    x[0, [300, 301]] = [1e30, 5e29]
    alone = synth.encode16(x, synth.BF16)
    _check(layer, alone, 1.0, q.oracle(alone, 1.0))
    layer.destroy()


@pytest.mark.parametrize("B,kw", [(1, {}), (2, {}), (4, {}), (1, dict(cmp_mode=2)), (2, dict(cmp_mode=2)), (4, dict(batch_mask_mode=1)), (3, dict(cmp_mode=2, batch_mask_mode=1))])
@pytest.mark.parametrize("ranks", [(40, 40), (40, 8), (0, 40)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_gate_and_up_in_one_launch(dt, ranks, B, kw):
    """H = round(silu(round(g)) round(u)) in the kernel's finish, ranks alike, different and zero on one side, with and without a bias
    on each (with a signed threshold too the form of the kernel that knows rules and biases).  Element by element: g and u are sums in
    32 bits, here up to 2e-5 of the token's largest from 64 bits (gpu_util.REL_L2_F32), so that each rounds to one of two or three neighbours; H is
    what the oracle's activation gives for some of them."""
    qs = [Q4Layer(synth.make_layer(1152, 2120, r, dt, config=97, linear=i), 128) for i, r in enumerate(ranks)]
    X16, src = gu.tokens_for(qs[0].L, B, config=97)
    tau = gu.calibrated_tau(qs[0].L, src, 0.5)
    layers = [q.prepare(tau, max_batch=B, **kw) for q in qs]
    for l in layers:
        rs.rsparse_set_tuning(l, mfma_min_batch=33)
    want = [q.oracle(X16, tau, **kw) for q in qs]
    sums = [w["Y"] for w in want]
    bias = [np.random.default_rng(97 + i).standard_normal(2120).astype(np.float32) for i in range(2)]
    Xd = gu.to_dev16(X16)
    for with_bias in (False, True):
        if with_bias:
            for l, b in zip(layers, bias):
                rs.rsparse_set_bias(l, b)
            sums = [y + b for y, b in zip(sums, bias)]
        near = [[synth.encode16(y + k * gu.REL_L2_F32 * np.abs(y).max(axis=1, keepdims=True), dt) for k in (-1, 0, 1)] for y in sums]
        H = np.stack([synth.decode16(oracle.gated_input(g, u, dt), dt) for g in near[0] for u in near[1]])
        for _ in range(2):
            Hd = gu._alloc_out(layers[0], B)
            rs.rsparse_mlp_gate_up(layers[0], layers[1], Xd.data_ptr(), B, Hd.data_ptr(), gu.stream_ptr())
            got = gu._read_out(layers[0], Hd)
            assert np.all((H.min(axis=0) <= got) & (got <= H.max(axis=0)))
            assert np.mean(got == H[4]) > 0.9                          # (the middle one: nearly all sums round alike)
            for i in range(2):
                for b in range(B):
                    assert np.array_equal(rs.rsparse_last_active(layers[i], b), want[i]["act"][b])
    for l in layers:
        l.destroy()


def test_a_layer_beyond_the_reach_of_one_launch():
    """U_r^T above 2 GiB less 16 MiB (1024 -> 2^20, rank 1024): two launches, vector kernel at one token and matrix cores at two, asked for or not.  The outputs
    of rows from the first, the last and other column tiles against the oracle's on these rows."""
    d_in, d_out, dt = 1024, 1 << 20, synth.F16
    rng = np.random.default_rng(96)
    Q = rng.integers(0, 16, (d_out, d_in), dtype=np.uint8)
    Z = rng.integers(5, 11, (d_out, 1), dtype=np.uint8)
    S16 = synth.encode16((0.75 + 0.5 * rng.random((d_out, 1))) * 1e-3, dt)
    U16 = rng.integers(0, 1 << 16, (d_out, d_in), dtype=np.uint16)
    U16 &= 0x87ff
    U16 |= 0x1000                                                      # (2^-11 to 2^-9, both signs)
    SV16 = synth.encode16(rng.standard_normal((d_in, d_in)) * 0.05, dt)
    X16 = synth.encode16(rng.standard_normal((2, d_in)), dt)
    rows = np.r_[0:40, 1000:1050, 524280:524300, d_out - 1030:d_out - 1010, d_out - 40:d_out]
    layer = rs.rsparse_prepare_q4(rs.make_config(d_in, d_out, d_in, 0.7, dt, max_batch=2, out_dtype=rs.F32), Q, S16, Z, d_in, U16, SV16)
    for B in (1, 2):
        want = oracle.rsparse_linear_q4(Q[rows], S16[rows], Z[rows], U16[rows], SV16, X16[:B], dt, 0.7, group=d_in)
        for tuning in ({}, dict(mfma_min_batch=33), dict(launches=1)):
            rs.rsparse_set_tuning(layer, **tuning)
            got = gu.run_linear(layer, X16[:B])
            gu.check_lists(got, want)
            gu.check_outputs(got["Y"][:, rows], want["Y"], rs.F32)
    layer.destroy()
