"""The arithmetic in which the K-slices of a column meet (csrc/grid_sum.h), compiled for the host: the slices'
fp32 sums, in column words in any order of arrival and by rows, against exact rational sums."""
import ctypes
import os
import random
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "grid_sum.h"
#include <cstring>
using namespace teal;
// One column: slice order[i] arrives i-th at a word that was left at zero.  Returns what the one that finds the
// others complete writes; -1 arrivals if none or several did.
extern "C" int meet_words(int unit, const float *sums, const int *order, int splits, float *y)
{
    const Grid grid{unit, splits};
    unsigned long long word = 0;
    unsigned flags = 0;
    int wrote = 0;
    for (int i = 0; i < splits; ++i) {
        const int s = order[i];
        const GridSum g = grid_sum(sums[s], grid);
        const unsigned long long mine = g.apart ? word_addend_apart(s, splits) : word_addend_on(g, splits);
        if (g.apart) flags |= 1u << s;
        const unsigned long long found = word;
        word += mine;
        if (!word_complete(found, splits)) continue;
        ++wrote;
        const unsigned told = word_told(mine, found, splits);
        const unsigned from = !told ? 0 : splits <= kWordFlagged ? told : flags;
        double apart = 0.0;
        if (told)
            for (int j = 0; j < splits; ++j) apart += from >> j & 1u ? (double)sums[j] : 0.0;
        *y = grid_value(word_whole(mine, found, splits), apart, grid);
    }
    return wrote;
}
extern "C" float meet_rows(int unit, const float *sums, int splits)
{
    const Grid grid{unit, splits};
    GridTotal total;
    for (int j = 0; j < splits; j += kGridRows) {
        float v[kGridRows] = {};
        const int n = splits - j < kGridRows ? splits - j : kGridRows;
        std::memcpy(v, sums + j, n * sizeof(float));
        grid_add_rows(total, v, n, grid);
    }
    return grid_value(total.whole, total.apart, grid);
}
extern "C" int off_grid(int unit, int splits, float sum) { return grid_sum(sum, Grid{unit, splits}).apart; }
extern "C" int unit_of(int bits, float t)
{
    return bits == 16 ? grid_unit_bf16(t) : bits == 8 ? grid_unit_w8(t) : grid_unit_w4(t);
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("grid_sum")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Wextra", "-Wno-unknown-pragmas", "-Werror", "-fPIC", "-shared",
                    "-I", os.path.join(ROOT, "paper_2408_14690_amd", "csrc"), str(d / "driver.cpp"),
                    "-o", str(d / "driver.so")], check=True)
    lib = ctypes.CDLL(str(d / "driver.so"))
    lib.meet_rows.restype = ctypes.c_float
    lib.unit_of.argtypes = [ctypes.c_int, ctypes.c_float]
    lib.off_grid.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_float]
    return lib


def meet(host, sums, unit, rng):
    """The column's output, the same bits in three orders of arrival and by rows."""
    v = np.asarray(sums, np.float32)
    ptr = v.ctypes.data_as(ctypes.c_void_p)
    got = [np.float32(host.meet_rows(unit, ptr, len(v)))]
    for order in (list(range(len(v))), list(range(len(v)))[::-1], rng.sample(range(len(v)), len(v))):
        y = ctypes.c_float(float("nan"))
        o = (ctypes.c_int * len(v))(*order)
        assert host.meet_words(unit, ptr, o, len(v), ctypes.byref(y)) == 1
        got.append(np.float32(y.value))
    assert len({np.float32(g).tobytes() if g == g else "nan" for g in got}) == 1, (sums, got)
    return got[0]


SPLITS = [2, 3, 4, 5, 8, 15, 16, 17, 22, 31, 32]


@pytest.mark.parametrize("unit", [49, 40, 24, -5])
@pytest.mark.parametrize("splits", SPLITS)
def test_no_bit_of_a_slice_is_lost(host, unit, splits):
    """Sums that are small whole multiples of one power of two, from far below the grid's step to far above its
    end, so that their total is an fp32 number: it has to come out exactly.  Among them a slice of 2^(22 - unit) and
    a last bit below the step, one that cancels to less than the step, and both ends of the grid."""
    rng = random.Random(splits)
    u = 2.0 ** -unit
    for e in range(max(-149, -unit - 70), -unit + 60):
        for _ in range(3):
            k = [rng.randint(-(2 ** 18), 2 ** 18) for _ in range(splits)]
            if rng.random() < 0.5:
                k = [q if rng.random() < 0.3 else 0 for q in k]
            sums = [q * 2.0 ** e for q in k]
            assert meet(host, sums, unit, rng) == np.float32(sum(k) * 2.0 ** e), (e, k)
    zeros = [0.0] * (splits - 1)
    for one in (2.0 ** 22 * u * (1 + 2.0 ** -23), -(2.0 ** 23) * u * (1 - 2.0 ** -24), u / 2, -u / 2 ** 5, 2.0 ** -149, -0.0):
        assert meet(host, [one] + zeros, unit, rng) == np.float32(one)
    top = 2.0 ** (51 if splits <= 16 else 48) * u
    for one in (top, -top, top * (1 - 2.0 ** -24), top * (1 + 2.0 ** -23), 2.0 ** 127):
        assert meet(host, [one] + zeros, unit, rng) == np.float32(one)
        assert meet(host, zeros + [one], unit, rng) == np.float32(one)
    assert meet(host, [top * (1 - 2.0 ** -24)] * splits, unit, rng) == np.float32(splits * top * (1 - 2.0 ** -24))
    assert meet(host, [-top * (1 - 2.0 ** -24)] * splits, unit, rng) == np.float32(-splits * top * (1 - 2.0 ** -24))


@pytest.mark.parametrize("unit", [49, 40, 24, -5])
@pytest.mark.parametrize("splits", SPLITS)
def test_sums_of_any_size(host, unit, splits):
    """Random fp32 sums with a spread of 2^40 and more: within the rounding to fp32 once, and of fp64 sums of
    at most `splits` terms."""
    rng = random.Random(100 + splits)
    for _ in range(400):
        centre, spread = rng.uniform(-60, 40), rng.choice([1, 10, 40])
        sums = [np.float32(rng.choice([-1, 1]) * 2.0 ** (centre + rng.uniform(-spread, spread))) for _ in range(splits)]
        exact = sum((Fraction(float(v)) for v in sums), Fraction(0))
        mag = sum(abs(Fraction(float(v))) for v in sums)
        got = Fraction(float(meet(host, sums, unit, rng)))
        assert abs(got - exact) <= abs(exact) / 2 ** 24 + mag * (splits + 2) / 2 ** 52 + Fraction(1, 2 ** 149)


@pytest.mark.parametrize("splits", SPLITS)
def test_infinities_and_nans(host, splits):
    rng = random.Random(200 + splits)
    rest = [rng.gauss(0, 1) for _ in range(splits - 1)]
    inf = float("inf")
    assert meet(host, [inf] + rest, 40, rng) == inf and meet(host, rest + [-inf], 40, rng) == -inf
    assert np.isnan(meet(host, [float("nan")] + rest, 40, rng))
    assert np.isnan(meet(host, [inf] + rest[1:] + [-inf], 40, rng))


THRESHOLDS = [0.0, 1e-30, 2.0 ** -24, 3e-7, 1e-5, 2.0 ** -15, 1e-4, 1e-3, 0.02, 0.03125, 0.3, 0.6744898, 1.0, 1.999, 2.0, 5.0, 100.0, 1000.0,
              32768.0, 65503.0]


@pytest.mark.parametrize("t", THRESHOLDS)
def test_sums_of_quantised_weights_are_on_the_grid(host, t):
    """Whatever the surviving inputs: int8 products, and int4 products with their group's scale (for thresholds that
    are not far below the inputs), are whole multiples of the step; long sums stay below the limit."""
    rng = np.random.default_rng(int(t) + 7)
    u8, u4 = host.unit_of(8, t), host.unit_of(4, t)
    x = np.abs(rng.integers(0, 0x7C00, 4000, dtype=np.uint16).view(np.float16).astype(np.float64))
    x = np.append(x, float(np.float16(min(t * (1 + 2.0 ** -8), 65504))))
    x = x[x > t]
    assert np.all(np.ldexp(x, u8) % 1 == 0)
    scale = rng.integers(0, 0x7C00, len(x), dtype=np.uint16).view(np.float16).astype(np.float64)
    if t == 0 or t >= 2.0 ** -14:
        # inputs above t are multiples of 2^(e - 10), which with scales of 2^-24 gives the step down to its finest,
        # 2^-43; below that, and dense, scales of that much more
        low = max(2.0 ** -24, 2.0 ** (-33 - np.floor(np.log2(t)))) if t else 2.0 ** -16
        assert np.all(np.ldexp(x * np.maximum(np.round(scale / low) * low, low), u4) % 1 == 0)
    ordinary = max(t, 2.0 ** -9)
    for bits, gain in ((8, 127 * 64), (4, 0.05 * 7 * 64), (16, 0.05 * 64)):
        for splits in (16, 32):
            assert not host.off_grid(host.unit_of(bits, t), splits, gain * ordinary), (bits, splits)


@pytest.mark.parametrize("e", range(-14, 12))
def test_unit_follows_the_inputs(host, e):
    """Inputs of size 2^e with half of them dropped: sums of bf16 weights of 0.02 over 64 to 2048 channels, whose
    sizes are some 0.05 to 1 times the inputs', are on the grid from 2^-7 of that on to 16 times it (for the smallest
    inputs from 2^-21 on: an odd last bit of less is below the finest step of 2^-44)."""
    unit = host.unit_of(16, 0.67 * 2.0 ** e)
    for s in (0.05 * 2.0 ** -6, 0.05, 1.0, 16.0):
        v = np.float32(max(s * 2.0 ** e, 2.0 ** -21))
        assert not host.off_grid(unit, 16, np.nextafter(v, np.float32(np.inf))), s
    assert host.unit_of(16, 0.0) == 40 and host.unit_of(4, 0.0) == 40 and host.unit_of(8, 0.0) == 24


@pytest.mark.parametrize("t", [1e-9, 2.0 ** -24, 1e-6, 1e-5, 1e-4, 4e-4, 1e-3])
def test_low_thresholds_on_ordinary_inputs(host, t):
    """Thresholds that drop next to nothing of inputs about 1 to 8: the sums of 1024 such inputs with weights of 0.02
    (0.64 to 5.1) are on the grid up to six times that."""
    for bits in (16, 4):
        for splits in (2, 16, 32):
            if (bits, splits) == (16, 32):          # (by a caller's own shape only: they end at 16)
                continue
            for v in (0.64, 5.1, 6 * 5.1):
                for v32 in (np.float32(v), -np.nextafter(np.float32(v), np.float32(0))):
                    assert not host.off_grid(host.unit_of(bits, t), splits, v32), (bits, splits, v)
