"""The compaction of a slice at the edges of its forms, against the CPU oracle through the C ABI: short
slices (2, 4 or 8 segments of 64 channels, every wavefront for itself), longer ones (2, 4, 8 or 16 segments
per wavefront) and pieces of 4096, on any address.  Survivor counts are exact; a channel that is missing, doubled or
misplaced moves y by far more than the tolerance."""
import numpy as np
import pytest

import teal_inputs as ti
from oracle import teal_oracle as orc
from test_gpu_parity import T, TIGHT, dev, rel_l2, run_bf16, survivors, workspace  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def shifted(x, by):
    """x on the device, `by` elements behind a 256-byte boundary."""
    buf = torch.zeros(x.size + by, dtype=torch.int16, device="cuda")
    buf[by:] = dev(x)
    return buf[by:]


@pytest.mark.parametrize("waves", [4, 8, 16])
@pytest.mark.parametrize("m", [1, 63, 128, 130, 256, 257, 504, 512, 513, 520, 1016, 1024, 1032, 2047, 2048,
                               2056, 4088, 4096, 4104, 8191, 8192])
def test_slice_lengths_and_addresses(T, m, waves):   # noqa: F811
    """One split, so that the slice is the whole state (pieces of 4096 beyond that); x on an address that
    is a multiple of 4 bytes and on one that is not."""
    n = 72
    w = ti.weights_bf16(n, m, seed=3 * m + waves)
    wt, ws = dev(ti.to_input_channel_major(w)), workspace(T, m, n)
    x = ti.make_x(m, 5 * m + 1, "laplace")
    for p in (0.0, 0.5, 0.97):
        t = ti.quantile_threshold(x, p)
        want, kept = orc.sparse_gemv_bf16(w, x, t), orc.sparsify(x, t)[3]
        got = [run_bf16(T, wt, shifted(x, by), t, m, n, ws, lanes_per_row=16, splits=1, waves=waves, unroll=4)
               for by in (0, 1, 2)]
        assert rel_l2(got[0], want) <= TIGHT and survivors(T, ws) == [kept], (m, p)
        assert all(np.array_equal(g, got[0]) for g in got), (m, p)


@pytest.mark.parametrize("m", [100, 200, 500, 1000, 1001])
def test_thresholds_between_and_beyond_fp16_values(T, m):   # noqa: F811
    """Short slices compare in fp16: every threshold splits the magnitudes as the fp32 compare does,
    between two values, at one, among the subnormals, and beyond the largest."""
    n = 16
    wt, ws = dev(np.ones((m, n), np.uint16)), workspace(T, m, n)      # weights of about 1e-40
    bits = np.random.default_rng(m).integers(0, 1 << 16, m).astype(np.uint16)
    bits[:12] = [0, 0x8000, 1, 0x8001, 2, 0x3FF, 0x400, 0x7BFF, 0xFBFF, 0x7C00, 0xFC00, 0x7E00]
    x = bits.view(np.float16)
    for t in (0.0, 2.0 ** -30, 2.0 ** -24, 1.5 * 2.0 ** -24, 2.0 ** -14, 1.0, 1.00048828125, float(np.float32(1.0004)),
              65504.0, 65519.0, 65536.0, 2.0 ** 100):
        run_bf16(T, wt, dev(x), t, m, n, ws, splits=1)
        assert survivors(T, ws) == [orc.sparsify(x, t)[3]], t


@pytest.mark.parametrize("m", [1000, 1001, 1024, 1032, 2048, 2056, 4096])
def test_formed_inputs(T, m):   # noqa: F811
    """SiLU(gate) * up: bitwise the producer kernel and the plain call, in one slice (a
    matrix wide enough to go without split-K) and in short ones."""
    for n in (264, 33000):
        g = torch.Generator(device="cuda").manual_seed(m + n)
        wt = (0.02 * torch.randn(m, n, generator=g, device="cuda")).to(torch.bfloat16)
        gate, up = torch.randn(m, generator=g, device="cuda"), torch.randn(m, generator=g, device="cuda")
        h = torch.empty(m, dtype=torch.float16, device="cuda")
        T.check(T.teal_swiglu_f16(gate, up, h, m))
        t = ti.quantile_threshold(h.cpu().numpy(), 0.5)
        ws, ys = workspace(T, m, n), [torch.empty(n, device="cuda") for _ in range(2)]
        T.check(T.teal_sparse_gemv_bf16(wt, h, t, ys[0], m, n, ws))
        T.check(T.teal_sparse_gemv_bf16_swiglu(wt, gate, up, t, ys[1], m, n, ws))
        assert torch.equal(ys[0], ys[1]), n


@pytest.mark.parametrize("m", [2048, 2304, 4096, 4352, 8192])
def test_w4_groups_of_long_slices(T, m):   # noqa: F811
    """128 tiles of 1024 columns leave two splits: slices of 1024 to 4096 channels, whose groups of 128 the
    int4 kernel walks by the positions that the compaction leaves."""
    n = 131072
    g = torch.Generator(device="cuda").manual_seed(m)
    q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
    scale = (0.01 + 0.01 * torch.rand(m // 128, n, generator=g, device="cuda")).half()
    x = torch.randn(m, generator=g, device="cuda").half()
    t = ti.quantile_threshold(x.cpu().numpy(), 0.5)
    ws, y = workspace(T, m, n), torch.empty(n, device="cuda")
    T.check(T.teal_sparse_gemv_w4(q, scale, 128, x, t, y, m, n, ws))
    cols = torch.arange(0, n, 509, device="cuda")
    b = q[:, cols // 2].view(torch.int8)
    w = torch.where(cols % 2 == 0, (b << 4) >> 4, b >> 4).double() * scale[:, cols].double().repeat_interleave(128, 0)
    kept = x.float().abs() > t
    want = (torch.where(kept, x.double(), 0.0)[:, None] * w).sum(0).cpu().numpy()
    assert rel_l2(y[cols].cpu().numpy(), want) <= TIGHT and survivors(T, ws) == [int(kept.sum())]


@pytest.mark.parametrize("m", [2048, 4096, 8192])
def test_w4_one_large_or_infinite_survivor_of_a_long_slice(T, m):   # noqa: F811
    """Two splits of 1024 to 4096 channels: how large the survivors are comes from the strips of 8 wavefronts,
    and one survivor beyond 127, or one infinity, in any of them is enough."""
    n = 131072
    assert T.teal_gemv_plan(4, m, n)[1]["splits"] == 2
    g = torch.Generator(device="cuda").manual_seed(m + 1)
    q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
    scale = (0.01 + 0.01 * torch.rand(m // 128, n, generator=g, device="cuda")).half()
    x = torch.randn(m, generator=g, device="cuda").half()
    ws, y = workspace(T, m, n), torch.empty(n, device="cuda")
    cols = torch.arange(0, n, 509, device="cuda")
    b = q[:, cols // 2].view(torch.int8)
    w = torch.where(cols % 2 == 0, (b << 4) >> 4, b >> 4).double() * scale[:, cols].double().repeat_interleave(128, 0)
    strip = m // 16
    for place in (0, 3 * strip + 77, 7 * strip, m // 2 - 1, m // 2, m // 2 + 4 * strip + 1, m - 1):
        xl = x.clone()
        xl[place] = 2000.0
        T.check(T.teal_sparse_gemv_w4(q, scale, 128, xl, 0.5, y, m, n, ws))
        want = (torch.where(xl.abs() > 0.5, xl.double(), 0.0)[:, None] * w).sum(0).cpu().numpy()
        assert rel_l2(y[cols].cpu().numpy(), want) <= TIGHT, place
        for inf in (float("inf"), -float("inf")):
            xl[place] = inf
            T.check(T.teal_sparse_gemv_w4(q, scale, 128, xl, 0.5, y, m, n, ws))
            assert bool(y.isnan().all()), (place, inf)


@pytest.mark.parametrize("m,n", [(1024, 512), (4096, 4096), (4096, 131072)])
def test_w4_formed_input_that_overflows(T, m, n):   # noqa: F811
    """SiLU(gate) * up beyond 65504 is an infinity of the state that W_down reads, as in the separate calls."""
    g = torch.Generator(device="cuda").manual_seed(m + n)
    q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
    scale = (0.01 + 0.01 * torch.rand(m // 128, n, generator=g, device="cuda")).half()
    gate, up = torch.randn(m, generator=g, device="cuda"), torch.randn(m, generator=g, device="cuda")
    ws, y, h = workspace(T, m, n), torch.empty(n, device="cuda"), torch.empty(m, dtype=torch.float16, device="cuda")
    for place in (0, m // 2 - 1, m - 1):
        for high, nan in ((250.0, False), (300.0, True)):      # 62500 and 90000
            gl, ul = gate.clone(), up.clone()
            gl[place], ul[place] = high, high
            T.check(T.teal_swiglu_f16(gl, ul, h, m))
            assert bool(h[place].isinf()) == nan
            T.check(T.teal_sparse_gemv_w4_swiglu(q, scale, 128, gl, ul, 0.25, y, m, n, ws))
            assert bool(y.isnan().all()) == nan and bool(y.isnan().any()) == nan, (place, high)
            if not nan:
                plain = torch.empty(n, device="cuda")
                T.check(T.teal_sparse_gemv_w4(q, scale, 128, h, 0.25, plain, m, n, ws))
                assert torch.equal(y, plain), place


@pytest.mark.parametrize("m", [8, 4096, 5000, 16384])
@pytest.mark.parametrize("scale", [1e-38, 1e-30, 1e-12, 1.0, 1e12, 1e30])
def test_scale_of_the_normalisation_over_its_range(T, m, scale):   # noqa: F811
    """The iteration for 1 / sqrt and, where its result is out of the ordinary range, the operations it stands
    for: bit for bit the oracle's state."""
    h, gamma = ti.norm_inputs(m, 7 * m)
    h = (h * np.float32(scale)).astype(np.float32)
    x = torch.empty(m, dtype=torch.int16, device="cuda")
    for eps in (0.0, 2.0 ** -20):
        T.check(T.teal_rmsnorm_f16(dev(h), dev(gamma), eps, x, m))
        got, want = x.cpu().numpy().view(np.float16), orc.rmsnorm_f16(h, gamma, eps)
        assert np.array_equal(np.isnan(got), np.isnan(want)), eps
        keep = ~np.isnan(want)
        assert np.array_equal(got.view(np.uint16)[keep], want.view(np.uint16)[keep]), eps
