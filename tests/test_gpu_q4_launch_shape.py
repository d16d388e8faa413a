"""How the matrix-core launch of 4-bit weights divides its work: one workgroup per compute unit, two (long runs; a ragged last tile), more
units than slots (one split each), with and without a t part, at both counts of token tiles.  Against the fp64 oracle,
fp32 outputs: rel-L2 2e-5 (gpu_util.check_outputs), lists equal; each call twice on one handle (the sums are left zero)."""
import pytest

import gpu_util as gu
import paper_2504_19449_amd as rs
from paper_2504_19449_amd import synth
from test_gpu_q4 import Q4Layer

pytestmark = pytest.mark.gpu


# units x token tiles (of 512 slots): 178 (two per compute unit, six steps a wave; with and without t), 516 (more than slots), few (cut to the steps),
# 138 (three splits, short runs), 68 (the nearest to one per unit: runs of two steps)
@pytest.mark.parametrize("shape", [(1536, 22536, 40, 128, 17), (1536, 22536, 0, 128, 32), (64, 65800, 8, 32, 17), (96, 648, 72, 32, 3),
                                   (1024, 17416, 16, 128, 20), (1024, 17408, 24, 128, 9)])
@pytest.mark.parametrize("dt", [synth.F16, synth.BF16])
def test_division(shape, dt):
    d_in, d_out, rank, group, B = shape
    q = Q4Layer(synth.random_layer(d_in, d_out, rank, dt, seed=101 + d_in), group)
    X16, src = gu.tokens_for(q.L, B, config=101)
    tau = gu.calibrated_tau(q.L, src, 0.5)
    layer = q.prepare(tau, max_batch=B, out_dtype=rs.F32)
    want = q.oracle(X16, tau)
    for _ in range(2):
        got = gu.run_linear(layer, X16)
        gu.check_lists(got, want)
        gu.check_outputs(got["Y"], want["Y"], rs.F32)
    layer.destroy()
