"""GPU tests of t = (S_r V_r^T) x on the matrix cores at the ends of its range: |t| beyond fp16's largest number, infinite t,
and t far below fp16's normal numbers, in all three weight forms (column-major, operand layout, 4-bit: below three tokens with launches = 2),
next to the oracle and next to the vector kernels, which hold t in fp32."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth

pytestmark = pytest.mark.gpu

FORMS = [("columns", 5), ("columns", 20), ("operand", 5), ("operand", 20), ("q4", 1), ("q4", 2), ("q4", 5), ("q4", 20)]


class _Form:
    """One layer in one weight form: prepare, and the oracle's result."""

    def __init__(self, form, d_in, d_out, rank, dt, seed):
        self.form, self.L = form, synth.random_layer(d_in, d_out, rank, dt, seed=seed)
        if form == "q4":
            self.q4 = synth.quantize_q4(synth.decode16(self.L.W16, dt), dt, 32)

    def prepare(self, tau, B, **kw):
        L = self.L
        if self.form != "q4":
            return gu.prepare(L, tau, max_batch=max(B, 5), out_dtype=rs.F32, dense_rowmajor=int(self.form == "operand"), **kw)
        cfg = rs.make_config(L.d_in, L.d_out, L.rank, tau, L.dtype, max_batch=B, out_dtype=rs.F32, **kw)
        return rs.rsparse_prepare_q4(cfg, *self.q4, 32, L.U16, L.SV16)

    def oracle(self, X16, tau, **kw):
        L = self.L
        if self.form != "q4":
            return gu.oracle_linear(L, X16, tau, **kw)
        return oracle.rsparse_linear_q4(*self.q4, L.U16, L.SV16, X16, L.dtype, tau, group=32, **kw)


@pytest.mark.parametrize("form,B", FORMS)
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_t_beyond_the_largest_fp16_number(form, B, dt):
    """A signed threshold drops large negative activations: |t| up to several 1e5 with finite results, in some rank indices and
    tokens only."""
    F = _Form(form, 320, 264, 72, dt, seed=3 + B)
    L = F.L
    sv = synth.decode16(L.SV16, dt)
    sv[5::16] *= 3000.0 / np.abs(sv[5::16]).max()
    L.SV16 = synth.encode16(sv, dt)
    X16, _ = gu.tokens_for(L, B, linear=B)
    x = synth.decode16(X16, dt)
    x[::2, 7] = -200.0
    X16 = synth.encode16(x, dt)
    t = synth.decode16(L.SV16, dt) @ np.where(x >= 0.5, 0.0, x).T
    assert np.abs(t).max() > 1e5 and (B == 1 or np.abs(t[:, 1]).max() < 65504)
    layer = F.prepare(0.5, B, cmp_mode=2)
    want = F.oracle(X16, 0.5, cmp_mode=2)
    assert np.all(np.isfinite(want["Y"]))
    for tuning in ({}, dict(launches=2), dict(mfma_min_batch=33), {}):
        rs.rsparse_set_tuning(layer, **tuning)
        got = gu.run_linear(layer, X16)
        gu.check_lists(got, want)
        gu.check_outputs(got["Y"], want["Y"], rs.F32)
    layer.destroy()


@pytest.mark.parametrize("form,B", FORMS)
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_infinite_t_gives_infinite_outputs(form, B, dt):
    """A dropped -Inf with factors of one sign: the definition gives -Inf in every output of that token, not NaN; a dropped NaN
    gives NaN; the other tokens are not touched."""
    F = _Form(form, 96, 40, 24, dt, seed=11 + B)
    L = F.L
    for a in ("U16", "SV16"):
        setattr(L, a, synth.encode16(np.abs(synth.decode16(getattr(L, a), dt)) + 0.01, dt))
    X16, _ = gu.tokens_for(L, B, linear=B)
    x = synth.decode16(X16, dt)
    x[0, 9] = -np.inf
    if B > 2:
        x[2, 9] = np.nan
    X16 = synth.encode16(x, dt)
    layer = F.prepare(0.5, B, cmp_mode=2)
    want = F.oracle(X16, 0.5, cmp_mode=2)["Y"]
    assert np.all(np.isneginf(want[0])) and (B <= 2 or np.all(np.isnan(want[2])))
    for tuning in ({}, dict(launches=2), dict(mfma_min_batch=33), {}):
        rs.rsparse_set_tuning(layer, **tuning)
        got = gu.run_linear(layer, X16)["Y"]
        assert np.array_equal(np.isneginf(got), np.isneginf(want)) and np.array_equal(np.isnan(got), np.isnan(want))
        gu.check_outputs(got, want, rs.F32)
    layer.destroy()


@pytest.mark.parametrize("form,B", [f for f in FORMS if f[0] != "operand"])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_small_t_keeps_its_32_bits(form, B, dt):
    """Every channel dropped, so that y = U_r t alone, with t around 1e-6, where two fp16 parts would hold 2^-36 at best (1e-5 of
    it).  Two chains of fp32 sums over 320 and 72 terms in any order: at most (320 + 72) 2^-24 = 2.3e-5 of the terms' sum of
    magnitudes, and with independent roundings sqrt(320 + 72) 2^-24 = 1.2e-6 of the result."""
    F = _Form(form, 320, 264, 72, dt, seed=23 + B)
    L = F.L
    L.SV16 = synth.encode16(synth.decode16(L.SV16, dt) * (1e-2 / np.abs(synth.decode16(L.SV16, dt)).max()), dt)
    rng = np.random.default_rng(B)
    X16 = synth.encode16(rng.standard_normal((B, 320)) * 1e-4, dt)
    layer = F.prepare(1.0, B)
    want = F.oracle(X16, 1.0)["Y"]
    for tuning in ({}, dict(launches=2), dict(mfma_min_batch=33)):
        rs.rsparse_set_tuning(layer, **tuning)
        got = gu.run_linear(layer, X16)["Y"]
        err = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
        assert np.all(err <= 1.2e-6), err
    layer.destroy()
