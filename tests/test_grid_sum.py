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
template <int UNIT> static int words(const float *sums, const int *order, int splits, float *y)
{
    unsigned long long word = 0;
    unsigned flags = 0;
    int wrote = 0;
    for (int i = 0; i < splits; ++i) {
        const int s = order[i];
        const GridSum g = grid_sum<UNIT>(sums[s], grid_limit<UNIT>(splits));
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
        *y = grid_value<UNIT>(word_whole(mine, found, splits), apart);
    }
    return wrote;
}
template <int UNIT> static float rows(const float *sums, int splits)
{
    GridTotal total;
    for (int j = 0; j < splits; j += kGridRows) {
        float v[kGridRows] = {};
        const int n = splits - j < kGridRows ? splits - j : kGridRows;
        std::memcpy(v, sums + j, n * sizeof(float));
        grid_add_rows<UNIT>(total, v, n, splits);
    }
    return grid_value<UNIT>(total.whole, total.apart);
}
extern "C" int meet_words(int unit, const float *sums, const int *order, int splits, float *y)
{
    return unit == 40 ? words<40>(sums, order, splits, y) : words<28>(sums, order, splits, y);
}
extern "C" float meet_rows(int unit, const float *sums, int splits)
{
    return unit == 40 ? rows<40>(sums, splits) : rows<28>(sums, splits);
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


@pytest.mark.parametrize("unit", [40, 28])
@pytest.mark.parametrize("splits", SPLITS)
def test_no_bit_of_a_slice_is_lost(host, unit, splits):
    """Sums that are small whole multiples of one power of two, from far below the grid's step to far above its
    end, so that their total is an fp32 number: it has to come out exactly.  Among them a slice of 2^(22 - unit) and
    a last bit below the step, one that cancels to less than the step, and both ends of the grid."""
    rng = random.Random(splits)
    u = 2.0 ** -unit
    for e in list(range(-unit - 70, -unit + 60)):
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


@pytest.mark.parametrize("unit", [40, 28])
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
