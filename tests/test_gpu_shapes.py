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


@pytest.mark.parametrize("m,n", [(1536, 5120), (2048, 8192), (2560, 5120), (4096, 4352), (4096, 6144)])
def test_formed_inputs_in_the_planned_shapes(T, m, n):   # noqa: F811
    """The calls that form their input, at the same sizes: bit for bit the producer kernel and the plain call; and
    the MLP whose W_down has this shape bit for bit the calls that it stands for."""
    g = torch.Generator(device="cuda").manual_seed(m + n)
    wt = (0.02 * torch.randn(m, n, generator=g, device="cuda")).to(torch.bfloat16)
    gate, up = torch.randn(m, generator=g, device="cuda"), torch.randn(m, generator=g, device="cuda")
    x, ws = torch.empty(m, dtype=torch.float16, device="cuda"), workspace(T, m, n)
    ys = [torch.empty(n, device="cuda") for _ in range(2)]
    T.check(T.teal_swiglu_f16(gate, up, x, m))
    T.check(T.teal_sparse_gemv_bf16(wt, x, 0.25, ys[0], m, n, ws))
    T.check(T.teal_sparse_gemv_bf16_swiglu(wt, gate, up, 0.25, ys[1], m, n, ws))
    assert torch.equal(ys[0], ys[1])
    gamma = 0.5 + 0.1 * up
    T.check(T.teal_rmsnorm_f16(gate, gamma, 2.0 ** -17, x, m))
    T.check(T.teal_sparse_gemv_bf16(wt, x, 0.3, ys[0], m, n, ws))
    T.check(T.teal_sparse_gemv_bf16_rmsnorm_multi([wt], [0.3], ys[1:], [n], gate, gamma, 2.0 ** -17, m, ws))
    assert torch.equal(ys[0], ys[1])
    d, f = 1024, m                                             # the MLP d -> f -> n
    w_gu = [(0.02 * torch.randn(d, f, generator=g, device="cuda")).to(torch.bfloat16) for _ in range(2)]
    xd = torch.randn(d, generator=g, device="cuda").half()
    gu, one = [torch.empty(f, device="cuda") for _ in range(2)], [torch.empty(f, device="cuda") for _ in range(2)]
    status, shape = T.teal_mlp_plan(16, d, f, n)
    assert status == 0
    wm = torch.zeros(T.teal_workspace_bytes_mlp(d, f, n), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_mlp_bf16(*w_gu, wt, xd, 0.5, 0.5, 0.05, *one, ys[0], d, f, n, wm, shape=shape))
    wg = workspace(T, d, f)
    for w, o in zip(w_gu, gu):
        T.check(T.teal_sparse_gemv_bf16_ex(w, xd, 0.5, o, d, f, wg, lanes_per_row=shape.gu_lanes_per_row,
                                           tile_cols=shape.gu_tile_cols, splits=shape.gu_splits, waves=8, unroll=4))
    T.check(T.teal_sparse_gemv_bf16_swiglu(wt, *gu, 0.05, ys[1], f, n, ws))
    assert all(torch.equal(a, b) for a, b in zip(one + ys[:1], gu + ys[1:]))
