"""The split-K combine at the edges of its own rules, against the CPU oracle through the C ABI:
arrival counters with a line each or packed (by the number of output tiles), and the calls
that follow on the same workspace."""
import numpy as np
import pytest

import teal_inputs as ti
from oracle import teal_oracle as orc
from test_gpu_parity import T, TIGHT, dev, rel_l2, run_bf16, survivors  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def bf16_case(n, m, seed, p=0.5):
    w = ti.weights_bf16(n, m, seed)
    x = ti.make_x(m, seed + 1, "laplace")
    t = ti.quantile_threshold(x, p)
    return dev(ti.to_input_channel_major(w)), dev(x), t, orc.sparse_gemv_bf16(w, x, t), orc.sparsify(x, t)[3]


@pytest.mark.parametrize("tiles", [8191, 8192, 8193])
def test_counters_with_a_line_each_and_packed(T, tiles):   # noqa: F811
    """8 columns per tile: up to 8192 tiles each counter has a 128-byte line, beyond that the
    counters are packed.  A second, ordinary call on the same workspace must find it ready."""
    m, n = 130, 8 * tiles
    wt, x, t, want, kept = bf16_case(n, m, 9700 + tiles)
    ws = torch.zeros(T.teal_workspace_bytes(2048, n), dtype=torch.uint8, device="cuda")
    wt2, x2, t2, want2, kept2 = bf16_case(1032, 2048, 9800)
    for _ in range(2):
        y = run_bf16(T, wt, x, t, m, n, ws, lanes_per_row=8, tile_cols=8, splits=2)
        assert rel_l2(y, want) <= TIGHT and survivors(T, ws) == [kept]
        y = run_bf16(T, wt2, x2, t2, 2048, 1032, ws)
        assert rel_l2(y, want2) <= TIGHT and survivors(T, ws) == [kept2]
