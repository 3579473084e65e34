"""GPU tests of row sums and maxima around the row length that one block covers (8192 fp32, 16384 16-bit elements): equal to the
oracle on either side of it, with nothing written past the last row, and with the output laid over the input."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from oracle import tbik_oracle as orc
from paper_2511_17826_amd import binding as tb

pytestmark = pytest.mark.gpu


def _call(x, x_dtype, out, op, M, V):
    nbytes = tb.lib().tbik_row_reduce_workspace_bytes(M, V, op)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    assert tb.lib().tbik_row_reduce(x.data_ptr(), x_dtype, out.data_ptr(), op, M, V, ws.data_ptr(), nbytes, None) == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("over_input", [False, True])
@pytest.mark.parametrize("M", [1, 5, 300])
@pytest.mark.parametrize("dtype,V", [(torch.float32, 4), (torch.float32, 8188), (torch.float32, 8192), (torch.float32, 8196),
                                     (torch.bfloat16, 8), (torch.bfloat16, 16384), (torch.bfloat16, 16392),
                                     (torch.float16, 16376), (torch.float16, 16384)])
def test_sum_and_max(dtype, V, M, over_input):
    rng = np.random.default_rng(V + M)
    x = torch.from_numpy(rng.standard_normal((M, V)).astype(np.float32)).to(dtype)
    x[M // 2, V // 2] = -0.0
    x[0] = -0.0                                             # a row of zeros of one sign
    x[-1, V - 1] = float("inf") if M > 1 else 3.0
    wide = x.float().numpy()
    leaf = orc.LEAF_F32 if dtype == torch.float32 else orc.LEAF_BF16
    want = {tb.TBIK_SUM: orc.row_sum(wide, leaf), tb.TBIK_MAX: wide.max(axis=1)}
    for op in (tb.TBIK_SUM, tb.TBIK_MAX):
        # the rows, and room behind them so that an output of M floats fits over the shortest of them
        buf = torch.full((M * V + 4 * M + 8,), -7.0, dtype=dtype, device="cuda")
        buf[:M * V] = x.reshape(-1).cuda()
        frame = torch.full((M + 2,), -7.0, device="cuda")
        out = buf.view(torch.float32)[:M] if over_input else frame[1:M + 1]
        _call(buf, tb._DTYPES[dtype], out, op, M, V)
        got = gu.host_f32(out)
        if op == tb.TBIK_SUM:
            assert np.array_equal(gu.u32(got), gu.u32(want[op])), (op, V, M)
        else:
            assert np.array_equal(got, want[op]), (op, V, M)
        assert float(frame[0]) == -7.0 and float(frame[-1]) == -7.0
