"""The one-launch kernels after a bounded wait ran out, and which launches a layer gets.  A wait that runs out is forced from the
host (stage 1 publishes nothing, a few polls), so every kernel ends normally."""
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
