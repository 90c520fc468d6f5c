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


def w4_case(n, m, seed):
    q, scale = ti.quantize_w4(ti.weights_bf16(n, m, seed))
    b = q.view(np.int8)
    lo, hi = (b << 4).astype(np.int8) >> 4, b >> 4
    w = np.stack([lo, hi], axis=2).reshape(m, n).astype(np.float64)
    w *= np.repeat(scale.astype(np.float64), 128, axis=0)
    return dev(q), dev(scale), w


def w4_bound(m, xk, w):
    """Exact integer sums per run (a wavefront's rows of a group), put together from three pairs of
    digits with at most 8 roundings of a term each (the pairs' magnitudes add up to at most 3.02 of
    the value's: 3.02 for the conversions, 3.02 and 1 for the two sums), then fp32 sums over at most
    m / 128 runs, 8 wavefronts and 16 splits."""
    return (8 + m / 128 + 8 + 16) * 2.0 ** -24 * (np.abs(xk)[:, None] * np.abs(w)).sum(0)


@pytest.mark.parametrize("kind", ["mixed range", "subnormal", "one", "equal", "large", "ends"])
@pytest.mark.parametrize("m,n", [(128, 32), (512, 544), (1152, 1056), (4096, 1024), (2048, 28672)])
def test_w4_integer_activations(T, kind, m, n):   # noqa: F811
    """The int4 kernel's activations are integers in units of 2^-24: values over all of fp16's range,
    subnormals alone, a single survivor, equal values, and survivors only at the ends of the
    128-channel groups; slices of one and of several passes, both tile widths."""
    rng = np.random.default_rng(m + n)
    q, scale, w = w4_case(n, m, 9900 + m + n)
    x = rng.standard_normal(m)
    t = 0.5
    if kind == "mixed range":
        x, t = np.sign(x) * 2.0 ** rng.uniform(-24, 15.9, m), 0.0
    elif kind == "subnormal":
        x, t = x * 2.0 ** -18, 2.0 ** -18
    elif kind == "one":
        x = np.zeros(m)
        x[m - 1] = -3.0
    elif kind == "equal":
        x = np.full(m, 0.50048828125)
    elif kind == "large":
        x, t = x * 20000, 9000.0
        x = np.clip(x, -65504, 65504)
    else:
        x = np.zeros(m)
        x[0::128], x[127::128] = 1.5, -2.5
    x = x.astype(np.float16)
    kept = np.abs(x.astype(np.float32)) > np.float32(t)
    xk = np.where(kept, x, 0).astype(np.float64)
    y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_gemv_w4(q, scale, 128, dev(x), t, y, m, n, ws))
    torch.cuda.synchronize()
    assert survivors(T, ws) == [int(kept.sum())]
    assert np.all(np.abs(y.cpu().numpy() - xk @ w) <= w4_bound(m, xk, w))


def test_w4_infinite_activation_gives_nan(T):   # noqa: F811
    m, n = 1024, 512
    q, scale, _ = w4_case(n, m, 9950)
    x = np.ones(m, np.float16)
    x[700] = -np.inf
    y = torch.zeros(n, dtype=torch.float32, device="cuda")
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_gemv_w4(q, scale, 128, dev(x), 0.5, y, m, n, ws))
    torch.cuda.synchronize()
    assert torch.isnan(y).all()


@pytest.mark.parametrize("m,n", [(1024, 544), (4096, 1056), (2048, 28672)])
def test_w4_infinite_scale_gives_the_sign_of_its_sum(T, m, n):   # noqa: F811
    """A group whose scale is infinite in some columns: products of one sign give an infinity of that
    sign there, whatever digits the activations have, and leave the other columns alone."""
    rng = np.random.default_rng(m)
    q = rng.integers(1, 8, (m, n)) * np.where(np.arange(n) % 2, -1, 1)
    packed = ((q[:, 0::2] & 15) | ((q[:, 1::2] & 15) << 4)).astype(np.uint8)
    scale = np.full((m // 128, n), 0.01, np.float16)
    scale[3, ::3] = np.inf
    x = (2.0 ** rng.integers(-6, 7, m)).astype(np.float16)
    x[::5] *= np.float16(1.2001953125)
    y = torch.zeros(n, dtype=torch.float32, device="cuda")
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_gemv_w4(dev(packed), dev(scale), 128, dev(x), 0.0, y, m, n, ws))
    torch.cuda.synchronize()
    got, hit = y.cpu().numpy(), np.arange(n) % 3 == 0
    assert np.array_equal(got[hit], np.where(np.arange(n) % 2, -np.inf, np.inf)[hit].astype(np.float32))
    want = x.astype(np.float64) @ (q * np.repeat(scale.astype(np.float64), 128, 0))[:, ~hit]
    assert rel_l2(got[~hit], want) <= TIGHT


@pytest.mark.parametrize("large", [127.0, -127.0625, 128.0, -2000.0, 65504.0])
@pytest.mark.parametrize("m,n", [(128, 32), (640, 544), (4096, 1056), (2048, 28672)])
def test_w4_small_activations_beside_a_large_one(T, large, m, n):   # noqa: F811
    """Four digits up to 127, six beyond: one large activation whose weights are zero in some columns,
    or whose group's scale is, must leave the other activations' products in those columns as
    exact as they are without it (a bound per column, from that column's own terms)."""
    rng = np.random.default_rng(n + int(abs(large)))
    q, scale = ti.quantize_w4(ti.weights_bf16(n, m, 9960 + m))
    q, scale = q.copy(), scale.copy()
    at = m - 77
    q[at, : n // 4] = 0                                 # columns 0 .. n / 2
    scale[at // 128, n // 2 + 5:: 3] = 0
    b = q.view(np.int8)
    w = np.stack([(b << 4).astype(np.int8) >> 4, b >> 4], axis=2).reshape(m, n).astype(np.float64)
    w *= np.repeat(scale.astype(np.float64), 128, axis=0)
    for spread in (0.01, 2.0 ** -22):
        x = (rng.standard_normal(m) * spread).astype(np.float16)
        x[at] = large
        y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
        T.check(T.teal_sparse_gemv_w4(dev(q), dev(scale), 128, dev(x), 0.0, y, m, n, ws))
        torch.cuda.synchronize()
        assert survivors(T, ws) == [int(np.count_nonzero(x))]
        xd = x.astype(np.float64)
        assert np.all(np.abs(y.cpu().numpy() - xd @ w) <= w4_bound(m, xd, w)), spread


@pytest.mark.parametrize("m", [512, 4096])
def test_w4_fused_calls_with_large_activations_are_the_plain_calls(T, m):   # noqa: F811
    """Six digits where the input is formed in the kernel: bitwise the producer kernel followed by
    the plain call, with a few activations far beyond 127."""
    rng = np.random.default_rng(m)
    ns = [1056, 544]
    mats = [ti.quantize_w4(ti.weights_bf16(n, m, 9970 + n), 128) for n in ns]
    qd, sd = [dev(q) for q, _ in mats], [dev(s) for _, s in mats]
    h = rng.standard_normal(m).astype(np.float32)
    h[::97] *= 40
    gamma = np.full(m, 60.0, np.float32)
    up = (rng.standard_normal(m) * 30).astype(np.float32)
    gate = (rng.standard_normal(m) * 4).astype(np.float32)
    up[::101] = 900.0
    gate[::101] = 9.0
    hd, gd, ud, ad = dev(h), dev(gamma), dev(up), dev(gate)
    ws = torch.zeros(T.teal_workspace_bytes(m, sum(ns)), dtype=torch.uint8, device="cuda")
    xd = torch.empty(m, dtype=torch.int16, device="cuda")
    ys = [[torch.empty(n, dtype=torch.float32, device="cuda") for n in ns] for _ in range(2)]
    T.check(T.teal_rmsnorm_f16(hd, gd, 1e-5, xd, m))
    T.check(T.teal_sparse_gemv_w4_multi(qd, sd, 128, [5.0, 0.0], ys[0], ns, xd, m, ws))
    T.check(T.teal_sparse_gemv_w4_rmsnorm_multi(qd, sd, 128, [5.0, 0.0], ys[1], ns, hd, gd, 1e-5, m, ws))
    torch.cuda.synchronize()
    x = xd.cpu().numpy().view(np.float16)
    assert np.abs(x).max() > 200
    for k, n in enumerate(ns):
        assert torch.equal(ys[0][k], ys[1][k])
        want = orc.sparse_gemv_w4(mats[k][0], mats[k][1], 128, x, [5.0, 0.0][k])
        assert rel_l2(ys[0][k].cpu().numpy(), want) <= TIGHT
    T.check(T.teal_swiglu_f16(ad, ud, xd, m))
    T.check(T.teal_sparse_gemv_w4(qd[0], sd[0], 128, xd, 1.0, ys[0][0], m, ns[0], ws))
    T.check(T.teal_sparse_gemv_w4_swiglu(qd[0], sd[0], 128, ad, ud, 1.0, ys[1][0], m, ns[0], ws))
    torch.cuda.synchronize()
    assert xd.view(torch.float16).abs().max().item() > 2000
    assert torch.equal(ys[0][0], ys[1][0])


@pytest.mark.parametrize("m,n,slices", [(2048, 2048, 16), (2176, 2048, 17), (4096, 1024, 32), (3584, 3072, 28), (4096, 4096, 32),
                                        (8192, 5120, 22), (8192, 5664, 16), (128, 32, 1)])
def test_w4_slices_cut_finer_for_one_matrix(T, m, n, slices):   # noqa: F811
    """Up to 160 blocks of 16 slices a single int4 matrix runs in finer ones (22 of 384 channels where 25 would
    take 328), a group of one does not, and the plans of either say so: both within the bound, the same survivors, reproducible."""
    rng = np.random.default_rng(m + n)
    q, scale, w = w4_case(n, m, 9950 + m + n)
    x = rng.standard_normal(m).astype(np.float16)
    t = 0.4
    kept = np.abs(x.astype(np.float32)) > np.float32(t)
    xk = np.where(kept, x.astype(np.float64), 0.0)
    bound = w4_bound(m, xk, w) + 32 * 2.0 ** -24 * (np.abs(xk)[:, None] * np.abs(w)).sum(0)
    want = xk @ w
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    got = []
    for one in (True, True, False):
        y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
        if one:
            T.check(T.teal_sparse_gemv_w4(q, scale, 128, dev(x), t, y, m, n, ws))
        else:
            T.check(T.teal_sparse_gemv_w4_multi([q], [scale], 128, [t], [y], [n], dev(x), m, ws))
        torch.cuda.synchronize()
        assert survivors(T, ws) == [int(kept.sum())]
        got.append(y.cpu().numpy())
        assert np.all(np.abs(got[-1] - want) <= bound)
    assert np.array_equal(got[0], got[1])
    st, plan = T.teal_gemv_plan(4, m, n)
    st, of_one = T.teal_gemv_plan_multi(4, m, [n])
    assert plan["splits"] == slices and plan["tile_cols"] == of_one["tile_cols"]
    if slices == of_one["splits"]:
        assert np.array_equal(got[0], got[2])


@pytest.mark.parametrize("m,f,d", [(256, 4096, 2048), (512, 2176, 1024)])
@pytest.mark.parametrize("down_splits", [1, 4, 16, None])
def test_w4_mlp_runs_in_the_shape_it_is_given(T, m, f, d, down_splits):   # noqa: F811
    """W_down of the one-launch int4 MLP in the caller's splits, also fewer than planned; without a shape in
    the planned ones, which are those of the call by itself."""
    mats = [ti.quantize_w4(ti.weights_bf16(b, a, 9990 + a + b), 128) for a, b in ((m, f), (m, f), (f, d))]
    q, sc = [dev(a) for a, _ in mats], [dev(b) for _, b in mats]
    x = dev(ti.make_x(m, 17, "laplace"))
    st, shape = T.teal_mlp_plan(4, m, f, d)
    planned = T.teal_gemv_plan(4, f, d)[1]
    assert (shape.down_tile_cols, shape.down_splits) == (planned["tile_cols"], planned["splits"])
    if down_splits:
        shape.down_splits = down_splits
    blocks = T.teal_mlp_block_info(4, m, f, d, shape, -1)[1][0]
    last = T.teal_mlp_block_info(4, m, f, d, shape, blocks - 1)[1]
    ks = -(-(-(-f // shape.down_splits)) // 128) * 128
    assert last[1] == 2 and last[3] + 1 == -(-f // ks)
    ys = [[torch.full((k,), float("nan"), dtype=torch.float32, device="cuda") for k in (f, f, d)] for _ in range(2)]
    ws = torch.zeros(T.teal_workspace_bytes_mlp(m, f, d), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_mlp_w4(*q, *sc, 128, x, 0.1, 0.1, 1e-4, *ys[0], m, f, d, ws, shape=shape))
    T.check(T.teal_sparse_mlp_w4(*q, *sc, 128, x, 0.1, 0.1, 1e-4, *ys[1], m, f, d, ws))
    wd = torch.zeros(T.teal_workspace_bytes(f, d), dtype=torch.uint8, device="cuda")
    yd = torch.full((d,), float("nan"), dtype=torch.float32, device="cuda")
    T.check(T.teal_sparse_gemv_w4_swiglu(q[2], sc[2], 128, ys[0][0], ys[0][1], 1e-4, yd, f, d, wd))
    torch.cuda.synchronize()
    assert torch.equal(ys[1][2], yd) and (down_splits or torch.equal(ys[0][2], yd))
    assert rel_l2(ys[0][2].cpu().numpy(), yd.cpu().numpy()) <= TIGHT
