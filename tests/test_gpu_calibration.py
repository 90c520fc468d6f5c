"""GPU parity for threshold calibration (Section 4.2): histogram of fp16
magnitudes and the thresholds read off it, bit-exact against the oracle
(which sorts)."""
import numpy as np
import pytest

import teal_inputs as ti
from oracle import teal_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LEVELS = [0.0, 0.1, 0.25, 0.3, 0.4, 0.5, 0.65, 0.8, 0.9, 0.999, 1.0]


@pytest.fixture(scope="module")
def T():
    import paper_2408_14690_amd as T
    assert torch.cuda.is_available()
    T.load_library()
    return T


def dev16(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda()


def gpu_hist(T, batches):
    hist = torch.zeros(T.TEAL_HIST_BINS, dtype=torch.int64, device="cuda")
    for x in batches:
        xd = dev16(x) if x.size else torch.empty(1, dtype=torch.int16, device="cuda")
        T.check(T.teal_abs_histogram(xd, x.size, hist))
    torch.cuda.synchronize()
    return hist


def gpu_thresholds(T, hist, levels):
    t = torch.full((len(levels),), -1.0, dtype=torch.float32, device="cuda")
    T.check(T.teal_histogram_thresholds(hist, levels, t))
    torch.cuda.synchronize()
    return t.cpu().numpy()


@pytest.mark.parametrize("count", [0, 1, 7, 8, 9, 1000, 4096, 14336, 100_003, 4096 * 512])
@pytest.mark.parametrize("dist", ["gaussian", "laplace"])
def test_histogram_and_thresholds_bit_exact(T, count, dist):
    x = ti.make_x(count, 40 + count, dist) if count else np.zeros(0, np.float16)
    hist = gpu_hist(T, [x])
    want = orc.abs_histogram(x)
    assert np.array_equal(hist.cpu().numpy().astype(np.uint64), want)
    got = gpu_thresholds(T, hist, LEVELS)
    for p, t in zip(LEVELS, got):
        assert float(t) == orc.quantile_threshold(x, p), (count, p)


def test_batches_accumulate_and_misaligned_starts(T):
    x = np.concatenate([ti.gaussian_x(30_000, 1), ti.laplace_x(20_001, 2)])
    whole = gpu_hist(T, [x])
    parts = gpu_hist(T, [x[:12_345], x[12_345:40_000], x[40_000:]])
    assert torch.equal(whole, parts)
    # a view that starts 2, 6 or 14 bytes past a 16-byte boundary
    base = dev16(x)
    for off in (1, 3, 7):
        hist = torch.zeros(T.TEAL_HIST_BINS, dtype=torch.int64, device="cuda")
        T.check(T.teal_abs_histogram(base.data_ptr() + 2 * off, x.size - off, hist))
        torch.cuda.synchronize()
        assert np.array_equal(hist.cpu().numpy().astype(np.uint64), orc.abs_histogram(x[off:]))


def test_special_values_and_heavy_ties(T):
    x = np.array([np.nan, -np.inf, 0.0, -0.0, 6e-8, -65504.0, np.nan, 2.0, -2.0, 1.9990234375],
                 np.float16)
    hist = gpu_hist(T, [x])
    assert np.array_equal(hist.cpu().numpy().astype(np.uint64), orc.abs_histogram(x))
    got = gpu_thresholds(T, hist, LEVELS)
    for p, t in zip(LEVELS, got):
        assert float(t) == orc.quantile_threshold(x, p)
    # every sample in one bin (all zeros) and in one high bin
    for v in (0.0, 3.5):
        z = np.full(300_000, v, np.float16)
        h = gpu_hist(T, [z])
        assert int(h[np.array([v], np.float16).view(np.uint16)[0]].item()) == z.size
        assert float(gpu_thresholds(T, h, [0.5])[0]) == v
    # only NaNs: nothing counted, t = 0
    h = gpu_hist(T, [np.full(100, np.nan, np.float16)])
    assert int(h.sum().item()) == 0 and float(gpu_thresholds(T, h, [0.5])[0]) == 0.0


def test_calibrated_threshold_gives_the_requested_sparsity(T):
    """End to end: calibrate on a sample, threshold fresh states with the result."""
    sample = np.concatenate([ti.gaussian_x(4096, 100 + k) for k in range(64)])
    hist = gpu_hist(T, [sample])
    t50 = float(gpu_thresholds(T, hist, [0.5])[0])
    assert t50 == orc.quantile_threshold(sample, 0.5)
    x = ti.gaussian_x(4096, 999)
    xd = dev16(x)
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    T.check(T.teal_sparsify(xd, 4096, t50, None, None, count))
    torch.cuda.synchronize()
    kept = int(count.item())
    assert kept == orc.sparsify(x, t50)[3]
    assert abs(1 - kept / 4096 - 0.5) < 0.03       # a fresh draw: binomial spread ~0.008


@pytest.mark.parametrize("count,off", [(1, 0), (7, 1), (8191, 3), (8192 * 256, 0), (8192 * 256 + 9, 5),
                                       (8192 * 700 + 4095, 0)])
def test_histogram_shares_zeros_and_nans(T, count, off):
    """Contiguous shares of the blocks (one value, less than a unit, a unit per block, ragged),
    many zeros (counted lane by lane), NaNs (left out) and every sign."""
    rng = np.random.default_rng(count)
    x = rng.standard_normal(count).astype(np.float16)
    x[rng.random(count) < 0.4] = np.float16(0.0)
    x[rng.random(count) < 0.1] = np.float16(-0.0)
    x[rng.random(count) < 0.01] = np.float16(np.nan)
    x[rng.random(count) < 0.01] = np.float16(-np.inf)
    buf = torch.zeros(count + 8, dtype=torch.int16, device="cuda")
    buf[off:off + count] = torch.from_numpy(x.view(np.int16)).cuda()
    hist = torch.zeros(T.TEAL_HIST_BINS, dtype=torch.int64, device="cuda")
    for _ in range(2):
        T.check(T.teal_abs_histogram(buf[off:off + count], count, hist))
    torch.cuda.synchronize()
    mag = x.view(np.uint16).astype(np.int64) & 0x7FFF
    want = 2 * np.bincount(mag[mag <= 0x7C00], minlength=T.TEAL_HIST_BINS)
    assert np.array_equal(hist.cpu().numpy(), want)


def test_thresholds_at_every_row_and_wavefront_edge(T):
    """Ranks whose bin is the first or last of a lane's pair, of a row of 128 bins and of a
    wavefront's 2048 bins, counts beyond 32 bits, and levels 0 and 1."""
    bins = [0, 1, 2, 127, 128, 2047, 2048, 2175, 2176, 4095, 4096, 20000, 30719, 30720, 31743, 31744]
    hist = np.zeros(T.TEAL_HIST_BINS, np.int64)
    hist[bins] = [3, 1, 5, 2, 2, 7, 1, 1, 4, 9, (1 << 33) + 1, 2, 6, 1, 1, 2]
    total = int(hist.sum())
    cum = np.cumsum(hist)
    ranks = sorted({int(r) for b in bins for r in (cum[b], cum[b] - hist[b] + 1)})
    hd = torch.from_numpy(hist).cuda()
    levels = [0.0, 1.0] + [r / total for r in ranks]
    for i in range(0, len(levels), 16):
        part = levels[i:i + 16]
        t = torch.full((len(part),), -1.0, dtype=torch.float32, device="cuda")
        T.check(T.teal_histogram_thresholds(hd, part, t))
        torch.cuda.synchronize()
        for p, got in zip(part, t.cpu().numpy()):
            k = min(total, max(0, int(np.ceil(p * float(total) - 1e-9))))
            want = 0.0 if k == 0 else float(np.uint16(np.searchsorted(cum, k)).view(np.float16))
            assert got == want, (p, k)
