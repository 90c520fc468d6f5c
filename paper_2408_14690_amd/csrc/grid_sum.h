// How the fp32 sums of the K-slices of a column are added (Section 4.4's split-K combine) so that the order
// of their arrival does not matter: as whole multiples of 2^-UNIT, which add up to the same in any order.
// Plain arithmetic shared by the kernels and the host (the host side is what the CPU tests add up slices
// with), so the two cannot drift apart.
//
// A slice's sum is on the grid if it is a whole multiple of 2^-UNIT and |sum| < grid_limit().  An fp32 number
// of 2^(23 - UNIT) or more is such a multiple whatever its last bit, and so is what two or more of that size
// cancel to, so that in ordinary data hardly a sum is off the grid.  Nothing is rounded to the grid: a
// sum off it (smaller with bits below the step, larger, an infinity, a NaN) is kept apart whole, and what is
// kept apart is added in fp64, in the order of the slices.  The total is rounded to fp32 at the end.
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
template <int UNIT>
TEAL_HD_INLINE float grid_limit(int splits)
{
    constexpr float kScale = (float)(1ull << UNIT);
    return splits <= 16 ? (float)(1ull << 51) / kScale : (float)(1ull << 48) / kScale;
}

struct GridSum {
    unsigned long long shifted;     // the bits of sum * 2^UNIT + kGridMagic
    bool apart;                     // off the grid
};
template <int UNIT>
TEAL_HD_INLINE GridSum grid_sum(float sum, float limit)
{
    const double x = (double)sum * (double)(1ull << UNIT);       // exact, so fusing it with the next line changes nothing
    const double shifted = x + kGridMagic;
    return GridSum{__builtin_bit_cast(unsigned long long, shifted),
                   !((__builtin_fabsf(sum) < limit) & (shifted - kGridMagic == x))};
}
TEAL_HD_INLINE unsigned long long grid_magic_bits() { return __builtin_bit_cast(unsigned long long, kGridMagic); }

template <int UNIT>
TEAL_HD_INLINE float grid_value(long long whole, double apart)
{
    return (float)((double)whole * (1.0 / (double)(1ull << UNIT)) + apart);
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
template <int UNIT>
TEAL_HD_INLINE void grid_add_rows(GridTotal &total, const float (&v)[kGridRows], int rows, int splits)
{
    const float limit = grid_limit<UNIT>(splits);
    long long whole = 0;
    bool apart = false;
#pragma unroll
    for (int q = 0; q < kGridRows; q += 4) {
        if (q >= rows) break;                             // block-uniform
#pragma unroll
        for (int u = q; u < q + 4; ++u) {
            const GridSum g = grid_sum<UNIT>(v[u], limit);
            whole += (long long)(g.shifted - grid_magic_bits());
            apart |= g.apart;
        }
    }
    if (__builtin_expect(apart, 0)) {
        whole = 0;
#pragma unroll
        for (int u = 0; u < kGridRows; ++u) {
            const GridSum g = grid_sum<UNIT>(v[u], limit);
            whole += g.apart ? 0 : (long long)(g.shifted - grid_magic_bits());
            total.apart += g.apart ? (double)v[u] : 0.0;
        }
    }
    total.whole += whole;
}

}  // namespace teal
