// How the fp32 sums of the K-slices of a column are added (Section 4.4's split-K combine) so that the order
// of their arrival does not matter: as whole multiples of 2^-unit, which add up to the same in any order.
// Plain arithmetic shared by the kernels and the host (the host side is what the CPU tests add up slices
// with), so the two cannot drift apart.
//
// A slice's sum is on the grid if it is a whole multiple of 2^-unit below 2^51 (more than 16 slices: 2^48) of
// them.  An fp32 number of 2^(23 - unit) or more is such a multiple whatever its last bit, and so is what two
// or more of that size cancel to, so that in ordinary data hardly a sum is off the grid.  Nothing is rounded to
// the grid: a sum off it (smaller with bits below the step, larger, an infinity, a NaN) is kept apart whole, and
// what is kept apart is added in fp64, in the order of the slices.  The total is rounded to fp32 at the end.  So
// the unit changes no result but what fp64 rounds; it only says which sums take the short way.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define TEAL_HD_INLINE __host__ __device__ __forceinline__
#else
#define TEAL_HD_INLINE inline
#endif

namespace teal {

// Column words: the lowest bits, 4 for up to 16 slices and 5 for up to 32, count the arrivals; as many above
// them tell which of up to four slices kept their sum apart, of more slices how many (a flag word
// then tells which); the other bits are the sum.  All arrivals but the last find counts that fit.
constexpr int kWordSplits = 32, kWordFlagged = 4;
TEAL_HD_INLINE int word_count_bits(int splits) { return splits <= 16 ? 4 : 5; }

// 16 sums below 2^51 steps fit the 56 bits of such a word, 32 below 2^48 the 54 of the other.
constexpr double kGridMagic = 0x1.8p52;         // x + kGridMagic rounds |x| < 2^51 to a whole number, in the low bits of the sum
struct Grid {
    int unit, splits;
};

// The unit of a call, from its threshold: the one thing every block knows of the size of the inputs that survive.  A
// sum kept apart costs the call two to four trips to memory more.  With a unit of 40 (int8: 28) for all, every
// column took them where the outputs were below 2^-13 or above 2^11; us per call at 50 % for inputs about 1 / 2^-14 / 2^12, and
// by partial rows: bf16 2048 x 2048 4.15 / 5.26 / 5.33, 4.65, with the unit from the threshold 4.14 / 4.22 / 4.22; int8 4096 x
// 4096 at 2^12 6.69, 6.53, now 5.86; int4 4096 x 4096 5.58 / 5.66 / 7.77, 6.75, now 5.57 / 5.58 / 5.57.  What is
// left are weights of an unusual size (bf16 2048 x 2048 of 2^-10 or 2^14 times 0.02: 4.85 and 5.37) and inputs of one in
// dense calls (t = 0; about 2^-12 or 2^12: 5.69 and 5.78, by rows 5.18).
// A low threshold belongs to small inputs or to ordinary ones of which hardly any are dropped.  So the step stops
// getting finer (`finest`) where both still take the short way.  With 48, whose sums end at 8 (more than 16 slices: at 1),
// the latter went the long way.  us, by rows / 48 / as below: int4 4096 x 4096, inputs about 1, t = 1e-4 6.61 / 7.47 / 5.88;
// bf16 2048 x 2048, t = 1e-4, inputs about 64 4.95 / 5.73 / 4.58, about 1 with some of 300 4.99 / 5.51 / 4.60; the other end,
// inputs about 2^-15 at 50 %: bf16 4.50 / 4.19 / 4.56, int4 4096 x 4096 with scales about 2^-8 6.72 / 5.50 / 5.50.  Left on the
// long way: int4 in more than 16 slices for inputs about 64 with t below 2^-8 (by rows 7.10, 7.93), or about 2^-12 and less with scales
// about 2^-9 (6.77, 7.18).
// floor(log2 t); kNoExponent and less for a t that keeps every input but zeros.
constexpr int kNoExponent = -25;
TEAL_HD_INLINE int threshold_exponent(float t) { return (int)(__builtin_bit_cast(unsigned, t) >> 23 & 255u) - 127; }
TEAL_HD_INLINE int grid_unit(float t, int at_one, int finest, int dense)
{
    const int e = threshold_exponent(t), unit = at_one - e;
    return e <= kNoExponent ? dense : unit < finest ? unit : finest;
}
// int8, whose sums meet before the channel's scale: an fp16 number above 2^e is a whole multiple of 2^(e - 10), and
// every one is of 2^-24, so all sums are multiples of the step.  The 8192 products a slice may have stay below the
// limit for inputs up to 2^21 times the threshold (t = 0: up to 2^7).
TEAL_HD_INLINE int grid_unit_w8(float t) { return grid_unit(t, 10, 24, 24); }
// int4: fp16 scales are multiples of 2^-24, so the sums are of 2^(e - 34); and of 2^-43, whatever the inputs, where the scales are
// 2^-9 or more.
TEAL_HD_INLINE int grid_unit_w4(float t) { return grid_unit(t, 34, 43, 40); }
// bf16 weights have any exponent: the sums of a slice of ordinary weights (about 0.02) are some 2^-2 of the inputs'
// size, in the middle of the 28 powers of two between 2^(23 - unit) and the limit.
TEAL_HD_INLINE int grid_unit_bf16(float t) { return grid_unit(t, 38, 44, 40); }

struct GridSum {
    unsigned long long shifted;     // the bits of sum * 2^unit + kGridMagic
    bool apart;                     // off the grid
};
TEAL_HD_INLINE GridSum grid_sum(float sum, const Grid &grid)
{
    const double x = __builtin_ldexp((double)sum, grid.unit);
    const double shifted = x + kGridMagic;
    return GridSum{__builtin_bit_cast(unsigned long long, shifted),
                   !((__builtin_fabs(x) < (grid.splits <= 16 ? 0x1p51 : 0x1p48)) & (shifted - kGridMagic == x))};
}
TEAL_HD_INLINE unsigned long long grid_magic_bits() { return __builtin_bit_cast(unsigned long long, kGridMagic); }

TEAL_HD_INLINE float grid_value(long long whole, double apart, const Grid &grid)
{
    return (float)(__builtin_ldexp((double)whole, -grid.unit) + apart);
}

// What a slice adds to a column's word: its sum and one arrival, or one arrival and the note that it keeps its
// sum apart (word_told() of what the last one finds says whether any did).
TEAL_HD_INLINE unsigned long long word_addend_on(const GridSum &g, int splits)
{
    const int bits = word_count_bits(splits);
    return (g.shifted << 2 * bits) + (1u - (grid_magic_bits() << 2 * bits));
}
TEAL_HD_INLINE unsigned long long word_addend_apart(int s, int splits)
{
    return 1u + (1u << word_count_bits(splits) << (splits > kWordFlagged ? 0 : s));
}
TEAL_HD_INLINE bool word_complete(unsigned long long found, int splits)
{
    return ((unsigned)found & ((1u << word_count_bits(splits)) - 1u)) == (unsigned)splits - 1u;
}
TEAL_HD_INLINE unsigned word_told(unsigned long long mine, unsigned long long found, int splits)
{
    const int bits = word_count_bits(splits);
    return (unsigned)(found | mine) >> bits & ((1u << bits) - 1u);
}
TEAL_HD_INLINE long long word_whole(unsigned long long mine, unsigned long long found, int splits)
{
    const int bits = word_count_bits(splits);
    return ((long long)found >> 2 * bits) + ((long long)mine >> 2 * bits);
}

// The same by partial rows (a slice's row holds its sum as it is), up to kGridRows at a time in the order of
// the slices (v[u]: row u; rows past the last are zeros).
constexpr int kGridRows = 8;          // (16 cost the stack kernel a block per unit)
struct GridTotal {
    long long whole = 0;
    double apart = 0.0;
};
TEAL_HD_INLINE void grid_add_rows(GridTotal &total, const float (&v)[kGridRows], int rows, const Grid &grid)
{
    long long whole = 0;
    bool apart = false;
#pragma unroll
    for (int q = 0; q < kGridRows; q += 4) {
        if (q >= rows) break;                             // block-uniform
#pragma unroll
        for (int u = q; u < q + 4; ++u) {
            const GridSum g = grid_sum(v[u], grid);
            whole += (long long)(g.shifted - grid_magic_bits());
            apart |= g.apart;
        }
    }
    if (__builtin_expect(apart, 0)) {
        whole = 0;
#pragma unroll
        for (int u = 0; u < kGridRows; ++u) {
            const GridSum g = grid_sum(v[u], grid);
            whole += g.apart ? 0 : (long long)(g.shifted - grid_magic_bits());
            total.apart += g.apart ? (double)v[u] : 0.0;
        }
    }
    total.whole += whole;
}

}  // namespace teal
