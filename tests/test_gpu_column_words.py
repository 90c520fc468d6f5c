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
    """32-bit sums of exact products in any order: (kept + wavefronts) * 2^-24 of the sum of magnitudes;
    the grid's rounding is below 2^-22 of the largest of a slice's eight terms."""
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
    return int(kept.sum())


@pytest.mark.parametrize("m,n,splits,p", [(128, 8, 2, 0.5), (130, 520, 2, 0.0), (1000, 264, 7, 0.5), (2048, 1048, 16, 0.5),
                                          (2048, 2048, 16, 0.99), (2176, 1048, 17, 0.5), (4096, 4096, 8, 0.5)])
def test_columns_of_all_magnitudes(T, m, n, splits, p):   # noqa: F811
    """16 splits are the most that column words take; 17 use the counters.  Two calls, the second on a
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


@pytest.mark.parametrize("m,splits", [(300, 2), (2048, 16)])
def test_words_and_counters_give_the_same_bits(T, m, splits):   # noqa: F811
    """682 tiles of 128 columns have words, 683 use the counters: the same columns, the same bits."""
    n = 682 * 128
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
