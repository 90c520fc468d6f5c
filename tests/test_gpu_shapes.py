"""Launch shapes of matrices with 1024 to 8256 input channels and 4097 to 8192 columns: against the CPU oracle, and
the calls that stand for one another bit for bit."""
import numpy as np
import pytest

import teal_inputs as ti
from oracle import teal_oracle as orc
from test_gpu_parity import T, TIGHT, dev, rel_l2, run_bf16, survivors, workspace  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,tile,splits", [(1024, 4352, 192, 8), (1536, 5120, 192, 8), (1600, 5120, 192, 7),
                                             (2048, 8192, 256, 8), (2112, 8192, 256, 7), (2560, 5120, 192, 8),
                                             (4096, 4352, 192, 11), (4096, 6144, 192, 8), (8192, 5120, 192, 8),
                                             (8256, 5120, 192, 8)])
def test_planned_shapes_of_4097_to_8192_columns(T, m, n, tile, splits):   # noqa: F811
    status, plan = T.teal_gemv_plan(16, m, n)
    assert status == 0 and (plan["tile_cols"], plan["splits"]) == (tile, splits)
    w = ti.weights_bf16(n, m, seed=m + n)
    wt, ws = dev(ti.to_input_channel_major(w)), workspace(T, m, n)
    x = ti.make_x(m, m + 3 * n, "laplace")
    xd, t = dev(x), ti.quantile_threshold(x, 0.5)
    y = run_bf16(T, wt, xd, t, m, n, ws)
    rows = np.arange(0, n, 37, dtype=np.int32)
    assert rel_l2(y[rows], orc.sparse_gemv_bf16_rows(w, x, t, rows)) <= TIGHT
    assert survivors(T, ws) == [orc.sparsify(x, t)[3]]
    again = torch.empty(n, device="cuda")
    T.check(T.teal_sparse_gemv_bf16_static(wt, xd, t, again, m, n))
    assert np.array_equal(again.cpu().numpy(), y)
    stack_ws = torch.zeros(T.teal_workspace_bytes_stack([1], [n], [m]), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_gemv_bf16_stack([1], [wt], [t], [again], [n], [xd], [m], stack_ws))
    assert np.array_equal(again.cpu().numpy(), y)
