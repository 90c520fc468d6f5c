"""Where the K-slices of a tile meet: column words (whole numbers added by atomics) or arrival counters and
partial rows, over column magnitudes from 1e-36 to 1e30, sums that the grid of whole numbers holds or does
not, infinities and NaN."""
import numpy as np
import pytest

from test_gpu_parity import T, survivors  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# magnitudes of the columns of a matrix, repeated over its columns
SCALES = [1.0, 1e-2, 3e-5, 1e-6, 1e-9, 1e-20, 1e-36, 300.0, 1e4, 1e6, 1e10, 1e20, 1e30]


def matrix(m, n, seed):
    """[m][n] bf16 weights, column j of magnitude SCALES[j % 13] * 0.02, exact in binary64."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    scale = torch.tensor(SCALES, device="cuda").repeat(-(-n // len(SCALES)))[:n]
    return (torch.randn((m, n), generator=g, device="cuda") * 0.02 * scale).to(torch.bfloat16)


def state(m, seed, kept=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(m, generator=g, device="cuda")
    if kept is not None:
        x = torch.where(torch.arange(m, device="cuda") % max(1, m // kept) == 0, x + 2 * x.sign(), 0.0)
    return x.half()


def run(T, wt, x, t, ws, **shape):
    m, n = wt.shape
    y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    T.check(T.teal_sparse_gemv_bf16_ex(wt, x, t, y, m, n, ws, **shape))
    torch.cuda.synchronize()
    return y


def check(y, wt, x, t, splits):
    """32-bit sums of exact products in any order: (kept + wavefronts) * 2^-24 of the sum of magnitudes for
    every column.  And the columns of a magnitude together: a lane adds at most a chain of `chain` products of random
    sign, whose roundings add up to 2^-24 * sqrt(chain / 6) of the norm, the sums of the lanes and of eight
    wavefronts to less than 2 units more, and the meeting adds half a unit; bounded by twice that."""
    kept = x.float().abs() > t
    xk = torch.where(kept, x.double(), 0.0)
    w = wt.double()
    want = xk @ w
    fin = torch.isfinite(want)
    mag = xk.abs() @ torch.nan_to_num(w.abs(), 0.0, 0.0)
    assert torch.equal(torch.isnan(y), torch.isnan(want))
    inf = torch.isinf(want)
    assert torch.equal(y[inf].double(), want[inf])
    err = (y.double() - want).abs()[fin]
    bound = (2 * int(kept.sum()) + 16 + 4 * splits) * 2.0 ** -24 * mag[fin] + 2.0 ** -149
    assert bool((err <= bound).all()), float((err / (bound + 1e-300)).max())
    chain = -(-int(kept.sum()) // (8 * splits)) + 1
    for k in range(len(SCALES)):
        cols = torch.arange(len(y), device=y.device) % len(SCALES) == k
        cols &= fin & (want.abs() > 2.0 ** -120)                # (below, sums have fewer bits)
        if int(cols.sum()) >= 8:
            rel = float((y.double() - want)[cols].norm() / want[cols].norm())
            assert rel <= 2 * 2.0 ** -24 * (2.5 + (chain / 6) ** 0.5), (SCALES[k], rel)
    return int(kept.sum())


@pytest.mark.parametrize("m,n,splits,p", [(128, 8, 2, 0.5), (130, 520, 2, 0.0), (1000, 264, 7, 0.5), (2048, 1048, 16, 0.5),
                                          (2048, 2048, 16, 0.99), (2176, 1048, 17, 0.5), (4096, 4096, 8, 0.5),
                                          (4096, 520, 32, 0.5), (2112, 520, 33, 0.5)])
def test_columns_of_all_magnitudes(T, m, n, splits, p):   # noqa: F811
    """Counts of 4 bits up to 16 splits and of 5 bits up to 32, which are the most that column words take; 33 use
    the counters.  Two calls, the second on a
    workspace whose rows hold the first one's: same bits, and the counters' area is zero again."""
    wt, x = matrix(m, n, m + n), state(m, 3 * m + n)
    t = float(torch.quantile(x.float().abs(), p)) if p else 0.0
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    head = T.teal_survivors_offset()
    ws[head:].fill_(0x5A)
    first = run(T, wt, x, t, ws, splits=splits)
    kept = check(first, wt, x, t, splits)
    assert survivors(T, ws) == [kept]
    assert not bool(ws[:head].any())
    assert torch.equal(run(T, wt, x, t, ws, splits=splits), first)
    assert not bool(ws[:head].any())


# Exponents of the columns' unit below, from far below the grid's step to beyond its end.
EXPONENTS = list(range(-75, 6))


def whole_sums(m, n, splits, seed):
    """[m][n] weights and an input whose products are whole multiples of 2^EXPONENTS[column] with less than 2^24
    units in all, so that 32-bit sums in any order are exact.  In the second half of the columns the first and the
    last channel of a slice (its first and last wavefront's) add 2^23 units and take them off again."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    units = torch.randint(-(1 << 22) // m, (1 << 22) // m + 1, (m, n), generator=g, device="cuda").double()
    units = units.clamp(-256, 256)
    units[:, n // 2:] = units[:, n // 2:].abs() * (torch.rand((m, n - n // 2), generator=g, device="cuda") < 0.05)
    ks = (-(-m // splits) + 63) // 64 * 64
    first = m // ks // 2 * ks
    last = min(m, first + ks) - 1
    units[first, n // 2:], units[last, n // 2:] = 2.0 ** 23, -(2.0 ** 23)
    unit = torch.tensor([2.0 ** e for e in EXPONENTS], device="cuda", dtype=torch.float64).repeat(-(-n // len(EXPONENTS)))[:n]
    wt = (units * unit).to(torch.bfloat16)
    assert torch.equal(wt.double(), units * unit)
    x = torch.randint(0, 2, (m,), generator=g, device="cuda").half()
    x[first] = x[last] = 1.0
    return wt, x, (x.double() @ units) * unit


@pytest.mark.parametrize("m,n,splits", [(1000, 1304, 2), (2048, 1304, 4), (2048, 1304, 5), (4096, 2048, 16), (4096, 1304, 32),
                                        (700, 682 * 128, 5), (700, 682 * 128 + 8, 5)])
def test_no_bit_of_a_slice_is_lost(T, m, n, splits):   # noqa: F811
    """Sums that are exact in every slice come out exactly, also those that cancel to less than the grid's
    step: words with and without flag words, and counters (the last)."""
    wt, x, want = whole_sums(m, n, splits, m + splits)
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    shape = dict(lanes_per_row=16, tile_cols=128, splits=splits)
    for _ in range(2):
        y = run(T, wt, x, 0.5, ws, **shape)
        bad = (y.double() != want).nonzero()[:, 0]
        assert bad.numel() == 0, (sorted({EXPONENTS[int(c) % len(EXPONENTS)] for c in bad}), len(bad))
        assert not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("batch", [1, 2, 3])
@pytest.mark.parametrize("splits", [4, 16])
def test_no_bit_of_a_batch_is_lost(T, batch, splits):   # noqa: F811
    m, n = 2048, 1304
    wt, x, want = whole_sums(m, n, splits, 5 * splits)
    X = torch.stack([x * (1 if b % 2 == 0 else -1) for b in range(batch)])
    ws = torch.zeros(T.teal_workspace_bytes_batch(m, n, batch), dtype=torch.uint8, device="cuda")
    Y = torch.full((batch, n), float("nan"), dtype=torch.float32, device="cuda")
    T.check(T.teal_sparse_gemv_bf16_batch_ex(wt, X, batch, 0.5, Y, m, n, ws, splits=splits))
    torch.cuda.synchronize()
    for b in range(batch):
        assert torch.equal(Y[b].double(), want if b % 2 == 0 else -want), b


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("e", [-24, -12, 0, 15])
@pytest.mark.parametrize("fmt,m,n", [("w8", 2048, 2048), ("w8", 4096, 16384), ("w4", 2048, 2048), ("w4", 4096, 1024)])
def test_no_bit_of_a_quantised_slice_is_lost(T, fmt, m, n, e, dense):   # noqa: F811
    """Sums of less than 2^24 units of 2^e, or of 2^e times the group's scale: exact in every slice and in all, in
    words (16, 4 and 32 slices) and, in the dense calls on large inputs, kept apart."""
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n + e)
    x = (torch.randint(-1, 2, (m,), generator=g, device="cuda").float() * 2.0 ** e).half()
    t = 0.0 if dense else 0.75 * 2.0 ** e
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    if fmt == "w8":
        q = torch.randint(-127, 128, (m, n), generator=g, device="cuda", dtype=torch.int8)
        sc = (2.0 ** -torch.arange(n, device="cuda").remainder(8).float()).half()
        want = (x.double() @ q.double()) * sc.double()
    else:
        q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
        sc = (2.0 ** -torch.arange(n, device="cuda").remainder(8).float()).half().expand(m // 128, n).contiguous()
        b = q.view(torch.int8)
        want = (x.double() @ torch.stack([(b << 4) >> 4, b >> 4], 2).reshape(m, n).double()) * sc[0].double()
    call = (lambda: T.teal_sparse_gemv_w8(q, sc, x, t, y, m, n, ws)) if fmt == "w8" else \
        (lambda: T.teal_sparse_gemv_w4(q, sc, 128, x, t, y, m, n, ws))
    for _ in range(2):
        y.fill_(float("nan"))
        T.check(call())
        torch.cuda.synchronize()
        assert torch.equal(y.double(), want)
        assert not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("e", [-13, -8, 0, 6, 11])
@pytest.mark.parametrize("fmt", ["bf16", "w8", "w4", "batch"])
def test_ordinary_sums_take_the_short_way_whatever_the_size_of_the_inputs(T, fmt, e):   # noqa: F811
    """Inputs of size 2^e at 50 %: the step follows the threshold, so next to none of the slices' sums is kept
    apart (int8 and int4: none, they are whole multiples of it).  A sum kept apart is written to its slice's row.
    The step gets no finer than 2^-44 (int4: 2^-43), and an fp32 sum below 2^-21 (2^-20) may have a bit below it: of sums about
    0.2 * 2^e (0.1 * 2^e) a share of 4 * 2^(-21 - e) (8 * 2^(-20 - e), at e = -13 alone: above, all products are multiples)."""
    m = n = 2048
    g = torch.Generator(device="cuda")
    g.manual_seed(e + 100)
    x = (torch.randn(m, generator=g, device="cuda") * 2.0 ** e).half()
    t = 0.6744898 * 2.0 ** e
    size = T.teal_workspace_bytes(m, n)
    ws = torch.zeros(max(size, T.teal_workspace_bytes_batch(m, n, 2)), dtype=torch.uint8, device="cuda")
    rows = ws[size - 4 * 128 * n:].view(torch.int32)      # 128 rows behind the head and the report
    rows.fill_(0x5A5A5A5A)
    y = torch.full((2, n), float("nan"), dtype=torch.float32, device="cuda")
    if fmt in ("bf16", "batch"):
        w = (torch.randn((m, n), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
        if fmt == "bf16":
            T.check(T.teal_sparse_gemv_bf16(w, x, t, y[0], m, n, ws))
        else:
            T.check(T.teal_sparse_gemv_bf16_batch(w, torch.stack([x, -x]), 2, t, y, m, n, ws))
    elif fmt == "w8":
        q = torch.randint(-127, 128, (m, n), generator=g, device="cuda", dtype=torch.int8)
        T.check(T.teal_sparse_gemv_w8(q, torch.full((n,), 2e-4, device="cuda").half(), x, t, y[0], m, n, ws))
    else:
        q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
        sc = (torch.rand((m // 128, n), generator=g, device="cuda") * 0.005).half()
        T.check(T.teal_sparse_gemv_w4(q, sc, 128, x, t, y[0], m, n, ws))
    torch.cuda.synchronize()
    apart = int((rows != 0x5A5A5A5A).sum())
    share = 0.0 if fmt == "w8" else 0.001 + 2 * 4 * 2.0 ** (-21 - e)
    if fmt == "w4":
        share = 8 * 2.0 ** (-20 - e) if e == -13 else 0.0
    assert apart <= 16 * n * share, apart
    assert bool(torch.isfinite(y[0]).all()) and not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("t", [1e-6, 1e-4, 1e-3])
@pytest.mark.parametrize("size", [1.0, 8.0])
@pytest.mark.parametrize("fmt", ["bf16", "w4", "batch"])
def test_low_thresholds_take_the_short_way_too(T, fmt, size, t):   # noqa: F811
    """A threshold that drops next to nothing says as little of the inputs' size as none: sums of ordinary inputs
    stay within the grid (int4 here in 32 slices, whose end is nearer).  Off it are bf16 sums near zero: below 2^-21 of
    about 0.2, and int4's of scales with bits below 2^-18."""
    m = n = 4096 if fmt == "w4" else 2048
    g = torch.Generator(device="cuda")
    g.manual_seed(int(size))
    x = (torch.randn(m, generator=g, device="cuda") * size).half()
    bytes_ = T.teal_workspace_bytes(m, n)
    ws = torch.zeros(max(bytes_, T.teal_workspace_bytes_batch(m, n, 2)), dtype=torch.uint8, device="cuda")
    rows = ws[bytes_ - 4 * 128 * n:].view(torch.int32)
    rows.fill_(0x5A5A5A5A)
    y = torch.full((2, n), float("nan"), dtype=torch.float32, device="cuda")
    if fmt == "w4":
        q = torch.randint(0, 256, (m, n // 2), generator=g, device="cuda", dtype=torch.uint8)
        sc = (torch.rand((m // 128, n), generator=g, device="cuda") * 0.005).half()
        T.check(T.teal_sparse_gemv_w4(q, sc, 128, x, t, y[0], m, n, ws))
    else:
        w = (torch.randn((m, n), generator=g, device="cuda") * 0.02).to(torch.bfloat16)
        if fmt == "bf16":
            T.check(T.teal_sparse_gemv_bf16(w, x, t, y[0], m, n, ws))
        else:
            T.check(T.teal_sparse_gemv_bf16_batch(w, torch.stack([x, -x]), 2, t, y, m, n, ws))
    torch.cuda.synchronize()
    apart = int((rows != 0x5A5A5A5A).sum())
    assert apart <= 32 * n // 1000, apart
    assert bool(torch.isfinite(y[0]).all()) and not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("kept", [1, 3, 40])
def test_few_survivors(T, kept):   # noqa: F811
    """Slices without a survivor and slices whose sum is one product: exact where the column has one."""
    m, n = 2048, 1040
    wt, x = matrix(m, n, 71), state(m, 72, kept)
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    y = run(T, wt, x, 0.5, ws, splits=16)
    assert check(y, wt, x, 0.5, 16) >= kept
    if kept == 1:
        i = int(x.float().abs().argmax())
        assert torch.equal(y, x[i].float() * wt[i].float())


def test_infinities_and_nans_stay_in_their_columns(T):   # noqa: F811
    m, n = 2048, 1040
    wt, x = matrix(m, n, 81), state(m, 82)
    x[5], x[1999] = 3.0, -2.0
    inf = float("inf")
    wt[5, 3], wt[1999, 4], wt[5, 130], wt[5, 17], wt[1999, 17] = inf, inf, float("nan"), inf, inf   # (17: NaN)
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        y = run(T, wt, x, 0.5, ws, splits=16)
        check(y, wt, x, 0.5, 16)
        assert y[3] == inf and y[4] == -inf and bool(y[[17, 130]].isnan().all())
        assert not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("m,splits,tiles", [(300, 2, 1023), (700, 5, 682), (2048, 16, 682), (2048, 32, 682)])
def test_words_and_counters_give_the_same_bits(T, m, splits, tiles):   # noqa: F811
    """The most tiles of 128 columns that have words (fewer with more than four slices, which need flag
    words), and one tile more, which uses the counters: the same columns, the same bits."""
    n = tiles * 128
    wide = matrix(m, n + 8, 91)
    narrow, x = wide[:, :n].contiguous(), state(m, 92)
    t = 0.5
    ws = torch.zeros(T.teal_workspace_bytes(m, n + 8), dtype=torch.uint8, device="cuda")
    shape = dict(lanes_per_row=16, tile_cols=128, splits=splits)
    a, b = run(T, wide, x, t, ws, **shape), run(T, narrow, x, t, ws, **shape)
    kept = check(b, narrow, x, t, splits)
    assert survivors(T, ws) == [kept]
    assert torch.equal(a[:n].view(torch.int32), b.view(torch.int32))
    again = run(T, wide, x, t, ws, **shape)
    assert torch.equal(again, a) and survivors(T, ws) == [kept]
    assert not bool(ws[:T.teal_survivors_offset()].any())


@pytest.mark.parametrize("batch", [1, 2, 3])
@pytest.mark.parametrize("m,n,splits", [(2048, 1040, 4), (2050, 520, 16)])
def test_batches(T, batch, m, n, splits):   # noqa: F811
    """One and two rows meet in words, three by counters."""
    wt = matrix(m, n, 11 + m)
    X = torch.stack([state(m, 20 + b) for b in range(batch)])
    ws = torch.zeros(T.teal_workspace_bytes_batch(m, n, batch), dtype=torch.uint8, device="cuda")
    got = []
    for _ in range(2):
        Y = torch.full((batch, n), float("nan"), dtype=torch.float32, device="cuda")
        T.check(T.teal_sparse_gemv_bf16_batch_ex(wt, X, batch, 0.5, Y, m, n, ws, splits=splits))
        torch.cuda.synchronize()
        assert not bool(ws[:T.teal_survivors_offset()].any())
        got.append(Y)
    assert torch.equal(got[0], got[1])
    kept = X.double().abs().sum(0) > batch * 0.5
    assert survivors(T, ws) == [int(kept.sum())]
    xk = torch.where(kept, X.double(), 0.0)
    want, mag = xk @ wt.double(), xk.abs() @ wt.double().abs()
    # as for one vector, twice: high and low parts of the activations are summed on their own
    bound = 2 * (2 * int(kept.sum()) + 16 + 4 * splits) * 2.0 ** -24 * mag + 2.0 ** -148
    err = (Y.double() - want).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("scale", [1e-7, 1.0, 1e5])
@pytest.mark.parametrize("fmt", ["bf16", "w8", "w4"])
def test_one_launch_mlp_waits_for_every_column(T, fmt, scale):   # noqa: F811
    """gate and up in several slices, whose columns may be written by different blocks: as the calls one
    by one, and the same bits every time, also where sums are kept apart."""
    m, f = 1024, 2816
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(m, generator=g, device="cuda").half()
    dims = [(m, f), (m, f), (f, m)]
    if fmt == "bf16":
        W = [(torch.randn(d, generator=g, device="cuda") * 0.02 * s).to(torch.bfloat16)
             for d, s in zip(dims, (scale, 1 / scale, 1.0))]
        sc = []
    else:
        rows = {"w8": lambda a: 1, "w4": lambda a: a // 128}[fmt]
        width = {"w8": lambda b: b, "w4": lambda b: b // 2}[fmt]
        W = [torch.randint(-127, 128, (a, width(b)), generator=g, device="cuda", dtype=torch.int8) for a, b in dims]
        sc = [(torch.rand((rows(a), b), generator=g, device="cuda") * 1e-3 * min(max(s, 1e-3), 10.0)).half()
              for (a, b), s in zip(dims, (scale, 1 / scale, 1.0))]
    st, shape = T.teal_mlp_plan({"bf16": 16, "w8": 8, "w4": 4}[fmt], m, f, m)
    assert st == T.TEAL_OK and shape.gu_splits > 1
    ws = torch.zeros(T.teal_workspace_bytes_mlp(m, f, m), dtype=torch.uint8, device="cuda")
    ws1 = torch.zeros(T.teal_workspace_bytes(f, 2 * f), dtype=torch.uint8, device="cuda")

    def outs():
        return [torch.full((k,), float("nan"), dtype=torch.float32, device="cuda") for k in (f, f, m)]
    ts = (0.5, 0.25, 1e-3)
    mlp = {"bf16": T.teal_sparse_mlp_bf16, "w8": T.teal_sparse_mlp_w8, "w4": T.teal_sparse_mlp_w4}[fmt]
    group = [128] if fmt == "w4" else []
    first = None
    for _ in range(8):
        o = outs()
        T.check(mlp(*W, *sc, *group, x, *ts, *o, m, f, m, ws, shape=shape))
        torch.cuda.synchronize()
        assert first is None or all(torch.equal(a, b) for a, b in zip(o, first))
        first = o
    assert not any(bool(a.isnan().any()) for a in first)
    r = outs()
    multi = {"bf16": T.teal_sparse_gemv_bf16_multi, "w8": T.teal_sparse_gemv_w8_multi,
             "w4": T.teal_sparse_gemv_w4_multi}[fmt]
    down = {"bf16": T.teal_sparse_gemv_bf16_swiglu, "w8": T.teal_sparse_gemv_w8_swiglu,
            "w4": T.teal_sparse_gemv_w4_swiglu}[fmt]
    T.check(multi(W[:2], *([sc[:2]] if sc else []), *group, ts[:2], r[:2], [f, f], x, m, ws1))
    T.check(down(W[2], *sc[2:], *group, first[0], first[1], ts[2], r[2], f, m, ws1))
    torch.cuda.synchronize()
    for a, b in zip(first, r):
        tol = 3e-7 * float(b.norm())          # (the calls one by one may have other launch shapes)
        assert float((a - b).norm()) <= tol


@pytest.mark.parametrize("scale", [1e-6, 1.0, 1000.0])
def test_int8_sums_before_their_scale(T, scale):   # noqa: F811
    """int8 sums meet before the channel's scale, on a coarser grid."""
    m, n = 2048, 2064
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    q = torch.randint(-127, 128, (m, n), generator=g, device="cuda", dtype=torch.int8)
    sc = (torch.rand(n, generator=g, device="cuda") * 0.01).half()
    x = (torch.randn(m, generator=g, device="cuda") * scale).clamp(-60000, 60000).half()
    t = 0.5 * scale
    y = torch.full((n,), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.zeros(T.teal_workspace_bytes(m, n), dtype=torch.uint8, device="cuda")
    T.check(T.teal_sparse_gemv_w8(q, sc, x, t, y, m, n, ws))
    torch.cuda.synchronize()
    kept = x.float().abs() > t
    xk = torch.where(kept, x.double(), 0.0)
    want = (xk @ q.double()) * sc.double()
    mag = (xk.abs() @ q.double().abs()) * sc.double()
    err = (y.double() - want).abs()
    bound = (2 * int(kept.sum()) + 64) * 2.0 ** -24 * mag
    assert bool((err <= bound).all()), float((err / (bound + 1e-300)).max())
    assert survivors(T, ws) == [int(kept.sum())] and not bool(ws[:T.teal_survivors_offset()].any())
