"""GPU parity for the variants of the activation rule and the output bias: fixed-count (top-k) activation with exact
ties, the signed threshold of Sec. 3.2 with a static bias, and the library-chosen mask mode (own masks up to 3
tokens, the union from 4).  Everything goes through the C ABI and is compared with the fp64 oracle: kept lists
bit-exact, outputs within the stated tolerances."""
import numpy as np
import pytest

import oracle
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _layer(d_in, d_out, rank, dt, seed=0):
    return synth.make_layer(d_in, d_out, rank, dt, config=70 + seed, linear=seed)


def _check(L, layer, X16, want):
    got = gu.run_linear(layer, X16)
    gu.check_lists(got, want)
    gu.check_outputs(got["Y"], want["Y"], layer.cfg.out_dtype)
    return got


@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
@pytest.mark.parametrize("strip_cols", [0, 64])
@pytest.mark.parametrize("launches", [1, 2])
def test_topk_keeps_exactly_k_with_lowest_channel_ties(dt, strip_cols, launches):
    L = _layer(1032, 1096, 64, dt)
    X16, _ = gu.tokens_for(L, 3)
    # plant runs of equal magnitudes (both signs) across the selection boundary
    X16[0, 100:140] = X16[0, 7]
    X16[0, 500:520] = X16[0, 7] ^ 0x8000
    X16[1, :] = X16[1, 3]                                   # one token made of a single magnitude
    for k in (1, 8, 300, 516, 1031, 1032):
        for B in (1, 3):
            layer = gu.prepare(L, 0.0, max_batch=4, out_dtype=rs.F32, strip_cols=strip_cols, topk=k)
            rs.rsparse_set_tuning(layer, launches=launches)
            want = gu.oracle_linear(L, X16[:B], 0.0, topk=k)
            got = _check(L, layer, X16[:B], want)
            for b in range(B):
                assert len(got["act"][b]) == k
            layer.destroy()


@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_topk_special_values(dt):
    L = _layer(256, 264, 16, dt, seed=1)
    x = np.zeros((4, 256))
    x[0, 5], x[0, 9], x[0, 200] = np.inf, -np.inf, 3.0     # infinities count as the largest
    x[1, :] = 0.0
    x[1, 17] = -0.0                                          # all zero: ties at magnitude 0, lowest channels win
    x[2, :] = np.linspace(-1, 1, 256)
    x[2, 40] = np.nan                                        # a NaN is never kept (and poisons the low-rank part)
    x[3, :] = 1e-7 if dt == synth.F16 else 1e-30            # tiny magnitudes (fp16: subnormal)
    x[3, ::3] *= 2
    X16 = synth.encode16(x, dt)
    for k in (2, 3, 100, 255, 256):
        layer = gu.prepare(L, 0.0, max_batch=4, out_dtype=rs.F32, topk=k)
        want = gu.oracle_linear(L, X16, 0.0, topk=k)
        _check(L, layer, X16, want)
        layer.destroy()


def test_topk_at_full_size_on_both_layouts_and_eight_tokens():
    dt = synth.BF16
    L = synth.random_layer(4096, 11008, 512, dt, seed=5)
    X16, _ = gu.tokens_for(L, 8)
    for strip_cols in (0, 128):
        for B, k in ((1, 2048), (8, 1229), (5, 4095)):
            layer = gu.prepare(L, 0.0, max_batch=8, strip_cols=strip_cols, topk=k)
            want = gu.oracle_linear(L, X16[:B], 0.0, topk=k)
            _check(L, layer, X16[:B], want)
            layer.destroy()


def test_topk_above_eight_tokens_runs_in_tiles_and_with_the_union_mask():
    dt = synth.F16
    L = _layer(1032, 520, 32, dt, seed=2)
    X16, _ = gu.tokens_for(L, 20)
    for mode in (0, 1):
        layer = gu.prepare(L, 0.0, max_batch=32, out_dtype=rs.F32, topk=200, batch_mask_mode=mode, dense_rowmajor=1)
        want = gu.oracle_linear(L, X16, 0.0, topk=200, batch_mask_mode=mode)
        got = gu.run_linear(layer, X16, lists=False)
        gu.check_outputs(got["Y"], want["Y"], rs.F32)
        layer.destroy()


def test_topk_grouped_call_with_different_k_per_layer():
    dt = synth.BF16
    La, Lb = _layer(1024, 512, 32, dt, seed=3), _layer(1024, 768, 32, dt, seed=4)
    X16, _ = gu.tokens_for(La, 2)
    a = gu.prepare(La, 0.0, max_batch=2, topk=100)
    b = gu.prepare(Lb, 0.0, max_batch=2, topk=700)
    torch = gu.torch_mod()
    Xd = gu.to_dev16(X16)
    Ya = torch.zeros((2, 512), dtype=torch.int16, device="cuda")
    Yb = torch.zeros((2, 768), dtype=torch.int16, device="cuda")
    rs.rsparse_linear_group([a, b], Xd.data_ptr(), 2, [Ya.data_ptr(), Yb.data_ptr()], gu.stream_ptr())
    torch.cuda.synchronize()
    for layer, L, Y, k in ((a, La, Ya, 100), (b, Lb, Yb, 700)):
        want = gu.oracle_linear(L, X16, 0.0, topk=k)
        gu.check_outputs(synth.decode16(Y.cpu().numpy().view(np.uint16), dt), want["Y"], dt)
        for t in range(2):
            assert np.array_equal(rs.rsparse_last_active(layer, t), want["act"][t])
    a.destroy()
    b.destroy()


@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
@pytest.mark.parametrize("strip_cols", [0, 64])
def test_signed_threshold_and_static_bias_of_the_multiphase_form(dt, strip_cols):
    """Sec. 3.2 end to end: sparse components x >= T_0 through the layer (rank 0 and rank > 0), residual as the static
    bias computed by the library's host routine from calibration tokens."""
    g = np.random.Generator(np.random.PCG64(12))
    for rank in (0, 32):
        L = _layer(1032, 520, rank, dt, seed=5)
        src = synth.DownInput(1032, config=75, linear=0)
        H_cal = synth.encode16(src.tokens(32, stream=synth.STREAM_CALIB), dt)
        X16 = synth.encode16(src.tokens(4), dt)
        X16[0, 11] = synth.encode16(np.array([0.25]), dt)[0]            # a tie at T_0
        T = [0.25, -0.1, -1.0]
        bias = rs.rsparse_multiphase_bias(L.W16, dt, H_cal, T)
        want_bias = oracle.static_bias(L.W16, dt, H_cal, dt, np.array(T))
        assert np.allclose(bias, want_bias, rtol=2e-6, atol=1e-7)
        for launches in (1, 2):
            layer = gu.prepare(L, T[0], max_batch=4, out_dtype=rs.F32, cmp_mode=2, strip_cols=strip_cols)
            rs.rsparse_set_tuning(layer, launches=launches)
            rs.rsparse_set_bias(layer, bias)
            want = gu.oracle_linear(L, X16, T[0], cmp_mode=2, bias=bias.astype(np.float64))
            _check(L, layer, X16, want)
            # the dense reference carries no bias
            dense = gu.run_dense(layer, X16)
            gu.check_outputs(dense, oracle.dense_linear(L.W16, X16, dt, dt, nthreads=4), rs.F32)
            rs.rsparse_set_bias(layer, None)
            _check(L, layer, X16, gu.oracle_linear(L, X16, T[0], cmp_mode=2))
            layer.destroy()


def test_bias_on_the_matrix_core_path_and_in_the_gated_pair():
    dt = synth.BF16
    L = _layer(1024, 520, 64, dt, seed=6)
    X16, src = gu.tokens_for(L, 16)
    tau = gu.calibrated_tau(L, src, 0.5)
    bias = np.random.Generator(np.random.PCG64(4)).standard_normal(520).astype(np.float32)
    layer = gu.prepare(L, tau, max_batch=16, out_dtype=rs.F32, dense_rowmajor=1)
    rs.rsparse_set_bias(layer, bias)
    want = gu.oracle_linear(L, X16, tau, bias=bias.astype(np.float64))
    _check(L, layer, X16, want)
    layer.destroy()
    # gate / up with the activation in the kernel's finish: each projection gets its own bias before silu(g) * u
    Lg, Lu = _layer(1024, 512, 32, dt, seed=7), _layer(1024, 512, 32, dt, seed=8)
    g = gu.prepare(Lg, tau, max_batch=1)
    u = gu.prepare(Lu, tau, max_batch=1)
    bg = np.linspace(-1, 1, 512).astype(np.float32)
    bu = np.linspace(2, -2, 512).astype(np.float32)
    rs.rsparse_set_bias(g, bg)
    rs.rsparse_set_bias(u, bu)
    torch = gu.torch_mod()
    Xd = gu.to_dev16(X16[:1])
    H = torch.zeros((1, 512), dtype=torch.int16, device="cuda")
    rs.rsparse_mlp_gate_up(g, u, Xd.data_ptr(), 1, H.data_ptr(), gu.stream_ptr())
    torch.cuda.synchronize()
    yg = oracle.rsparse_linear(Lg.W16, Lg.U16, Lg.SV16, X16[:1], dt, dt, tau, bias=bg.astype(np.float64))["Y"]
    yu = oracle.rsparse_linear(Lu.W16, Lu.U16, Lu.SV16, X16[:1], dt, dt, tau, bias=bu.astype(np.float64))["Y"]
    want_h = yg / (1.0 + np.exp(-yg)) * yu
    got_h = synth.decode16(H.cpu().numpy().view(np.uint16), dt)
    # three 16-bit roundings (g, u, h) on top of the layer's tolerance
    assert np.linalg.norm(got_h - want_h) <= 1.5e-2 * np.linalg.norm(want_h)
    g.destroy()
    u.destroy()


@pytest.mark.parametrize("strip_cols", [0, 64])
def test_mask_mode_left_to_the_library_switches_to_the_union_at_four_tokens(strip_cols):
    dt = synth.F16
    L = _layer(1032, 520, 32, dt, seed=9)
    X16, src = gu.tokens_for(L, 8)
    tau = gu.calibrated_tau(L, src, 0.5)
    layer = gu.prepare(L, tau, max_batch=8, out_dtype=rs.F32, batch_mask_mode=2, strip_cols=strip_cols)
    for B in (1, 2, 3, 4, 5, 8):
        want = gu.oracle_linear(L, X16[:B], tau, batch_mask_mode=1 if B >= 4 else 0)
        _check(L, layer, X16[:B], want)
    layer.destroy()


def test_topk_through_the_entry_point_that_allocates_nothing():
    dt = synth.BF16
    L = _layer(1032, 520, 32, dt, seed=10)
    X16, _ = gu.tokens_for(L, 4)
    layer = gu.prepare(L, 0.0, max_batch=4, topk=333)
    torch = gu.torch_mod()
    Xd = gu.to_dev16(X16)
    Y = torch.zeros((4, 520), dtype=torch.int16, device="cuda")
    rs.rsparse_linear_static(layer, Xd.data_ptr(), 4, Y.data_ptr(), gu.stream_ptr())
    torch.cuda.synchronize()
    want = gu.oracle_linear(L, X16, 0.0, topk=333)
    gu.check_outputs(synth.decode16(Y.cpu().numpy().view(np.uint16), dt), want["Y"], dt)
    for b in range(4):
        assert np.array_equal(rs.rsparse_last_active(layer, b), want["act"][b])
    layer.destroy()


def test_planned_call_runs_dense_where_the_byte_model_says_so():
    """rsparse_linear_group_planned: a small attention projection and any layer at 8 tokens run the dense kernel (exact
    dense product), a large MLP layer at one token runs R-Sparse; results match the corresponding oracle either way."""
    dt = synth.BF16
    torch = gu.torch_mod()
    small = synth.random_layer(4096, 4096, 256, dt, seed=21)
    big = synth.random_layer(4096, 14336, 256, dt, seed=22)
    for L, B, expect in ((small, 1, False), (big, 1, True), (big, 8, False)):
        X16, src = gu.tokens_for(L, B)
        tau = gu.calibrated_tau(L, src, 0.5)
        layer = gu.prepare(L, tau, max_batch=8, dense_rowmajor=1)
        Xd = gu.to_dev16(X16)
        Y = torch.zeros((B, L.d_out), dtype=torch.int16, device="cuda")
        used = rs.rsparse_linear_group_planned([layer], Xd.data_ptr(), B, [Y.data_ptr()], 0.5, gu.stream_ptr())
        torch.cuda.synchronize()
        assert used == expect == rs.rsparse_plan_layer(L.d_in, L.d_out, L.rank, 0.5, 1, B)[2]
        got = synth.decode16(Y.cpu().numpy().view(np.uint16), dt)
        want = gu.oracle_linear(L, X16, tau)["Y"] if used else oracle.dense_linear(L.W16, X16, dt, dt, nthreads=8)
        gu.check_outputs(got, want, dt)
        layer.destroy()


def test_planned_call_knows_which_dense_kernel_a_layer_has():
    """Three tokens, 4096 -> 14336: the dense product of a layer that keeps the operand layout beats R-Sparse (22 against 30 us),
    the one over column-major W alone does not (34 us)."""
    dt = synth.BF16
    torch = gu.torch_mod()
    L = synth.random_layer(4096, 14336, 256, dt, seed=22)
    X16, src = gu.tokens_for(L, 3)
    tau = gu.calibrated_tau(L, src, 0.5)
    for rowmajor in (0, 1):
        layer = gu.prepare(L, tau, max_batch=3, dense_rowmajor=rowmajor)
        Xd = gu.to_dev16(X16)
        Y = torch.zeros((3, L.d_out), dtype=torch.int16, device="cuda")
        used = rs.rsparse_linear_group_planned([layer], Xd.data_ptr(), 3, [Y.data_ptr()], 0.5, gu.stream_ptr())
        torch.cuda.synchronize()
        assert used == (not rowmajor)
        want = gu.oracle_linear(L, X16, tau)["Y"] if used else oracle.dense_linear(L.W16, X16, dt, dt, nthreads=8)
        gu.check_outputs(synth.decode16(Y.cpu().numpy().view(np.uint16), dt), want, dt)
        with pytest.raises(rs.RSparseError):
            rs.rsparse_linear_group_planned([layer], Xd.data_ptr(), 3, [Y.data_ptr()], 1.5, gu.stream_ptr())
        layer.destroy()


@pytest.mark.parametrize("strip_cols", [0, 64])
def test_topk_with_bias_in_a_replayed_graph(strip_cols):
    """The rule-writing kernel of the fixed-count activation is part of the captured call: every replay, with new token
    values in the same buffer and an eager call between replays, selects afresh and matches the oracle."""
    torch = gu.torch_mod()
    dt = synth.BF16
    L = _layer(1032, 520, 32, dt, seed=9)
    X16, _ = gu.tokens_for(L, 8)
    bias = np.random.Generator(np.random.PCG64(6)).standard_normal(520).astype(np.float32)
    B, k = 2, 300
    layer = gu.prepare(L, 0.0, max_batch=B, out_dtype=rs.F32, strip_cols=strip_cols, topk=k)
    rs.rsparse_set_bias(layer, bias)
    Xd = gu.to_dev16(X16[:B])
    Y = gu._alloc_out(layer, B)
    Ye = gu._alloc_out(layer, B)
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
        got = Y.cpu().numpy().astype(np.float64)
        rs.rsparse_linear(layer, Xd.data_ptr(), B, Ye.data_ptr(), gu.stream_ptr())
        torch.cuda.synchronize()
        want = gu.oracle_linear(L, xb, 0.0, topk=k, bias=bias.astype(np.float64))
        gu.check_outputs(got, want["Y"], rs.F32)
        eager = Ye.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - eager) <= 1e-5 * np.linalg.norm(eager)
        for b in range(B):
            assert np.array_equal(rs.rsparse_last_active(layer, b), want["act"][b])
    layer.destroy()


@pytest.mark.parametrize("d_in", [8, 8192, 8200, 16384, 16392, 65536])
def test_topk_rules_of_a_group_at_the_edges_of_a_threads_share(d_in):
    """1024 threads with one, two or up to eight chunks of 8 channels each; three layers' rules come from one launch.  Kept
    lists bit-exact with ties across threads, at the first channels and at the last."""
    dt = synth.F16
    Ls = [synth.random_layer(d_in, 16, 8, dt, seed=90 + i) for i in range(3)]
    X16, _ = gu.tokens_for(Ls[0], 2)
    X16[0, ::3] = X16[0, 7]                                  # ties over all threads
    X16[1, -8:] = X16[1, 0] ^ 0x8000                         # ties in the first and the last chunk
    ks = (1, max(1, d_in // 3), d_in - 1)
    layers = [gu.prepare(L, 0.0, max_batch=2, topk=k) for L, k in zip(Ls, ks)]
    torch = gu.torch_mod()
    Xd = gu.to_dev16(X16)
    Ys = [torch.zeros((2, 16), dtype=torch.int16, device="cuda") for _ in Ls]
    rs.rsparse_linear_group(layers, Xd.data_ptr(), 2, [Y.data_ptr() for Y in Ys], gu.stream_ptr())
    torch.cuda.synchronize()
    for layer, L, Y, k in zip(layers, Ls, Ys, ks):
        want = gu.oracle_linear(L, X16, 0.0, topk=k)
        gu.check_outputs(synth.decode16(Y.cpu().numpy().view(np.uint16), dt), want["Y"], dt)
        for t in range(2):
            assert np.array_equal(rs.rsparse_last_active(layer, t), want["act"][t])
        layer.destroy()
