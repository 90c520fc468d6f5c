// y = s_t(x) W^T for weight-quantised W (Section 5.3 names the formats; a kernel
// that is both sparse and quantised is what that section leaves open).
//   int8: W[j][i] = q[i][j] * scale[j]            (channel-wise)
//   int4: W[j][i] = nibble(i, j) * scale[i/128][j] (groups of 128 input channels)
// Dequantisation happens in registers; only surviving rows are read.
#include <type_traits>

#include "gemv_common.h"
#include "gemv_dispatch.h"
#include "gemv_mlp.h"

namespace teal {

struct FmtW8 {
    static constexpr int kElemsPerLane = 16;   // 16 bytes = 16 int8
    static constexpr int kBitsPerElem = 8;
    static __device__ __forceinline__ int grid_unit(float t) { return grid_unit_w8(t); }
    struct Args {
        const void *W;
        const __half *scale;
        int ld = 0;             // elements from one row of W to the next; 0 = n
    };
    static __device__ __forceinline__ void read_now(const Args (&a)[4])
    {
        asm volatile("" ::"s"(a[0].ld), "s"(a[1].ld), "s"(a[2].ld), "s"(a[3].ld), "s"(a[0].scale),
                     "s"(a[1].scale), "s"(a[2].scale), "s"(a[3].scale));
    }
    static __device__ __forceinline__ void select(Args &a, const Args &b, bool take)
    {
        a.W = take ? b.W : a.W;
        a.scale = take ? b.scale : a.scale;
        a.ld = take ? b.ld : a.ld;
    }
    static __device__ __forceinline__ void fma(float (&acc)[16], u32x4 v, float xv)
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const int wq = (int)(v[q] << (24 - 8 * b)) >> 24;   // sign-extend byte b
                acc[4 * q + b] = fmaf(xv, (float)wq, acc[4 * q + b]);
            }
        }
    }
    // The per-output-channel scale factors out of the sum over input channels.
    typedef __half ColumnScale;
    static __device__ __forceinline__ ColumnScale column_scale(const Args &a, int col)
    {
        return a.scale[col];
    }
    static __device__ __forceinline__ float finish(float sum, ColumnScale sc)
    {
        return sum * __half2float(sc);
    }
};

struct FmtW4 {
    static constexpr int kElemsPerLane = 32;   // 16 bytes = 32 nibbles
    static constexpr int kBitsPerElem = 4;
    static __device__ __forceinline__ int grid_unit(float t) { return grid_unit_w4(t); }
    struct Args {
        const void *W;
        const __half *scale;
    };
    static __device__ __forceinline__ void select(Args &a, const Args &b, bool take)
    {
        a.W = take ? b.W : a.W;
        a.scale = take ? b.scale : a.scale;
    }
    struct ColumnScale {};
    static __device__ __forceinline__ ColumnScale column_scale(const Args &, int) { return {}; }
    static __device__ __forceinline__ float finish(float sum, ColumnScale) { return sum; }
};

constexpr int kGroup = 128;
constexpr int kW4Waves = 8;
constexpr int kW4Unroll = 4;

// The int4 products run on the matrix cores, in integers.  With fp32 FMAs every weight costs its FMA
// and 0.75 instructions to extract it, 71 vector instructions per 16-byte load with the
// addressing: the row stream was bound by instruction issue (two wavefronts per SIMD), not by HBM
// (dense 28672 x 8192: 21 us of rows for 14.7 us of bytes at the peak).
//
// v_mfma_i32_16x16x64_i8: a lane's 16 bytes are 16 of the 64 values of K, its lane % 16 the row of A,
// lane / 16 the quarter of K, so with 16 lanes to a weight row the weights go in as they were
// loaded, 8 bytes of one row and 8 of the same columns of another.  B separates the bytes again: it
// is zero except where the byte's place in its row equals the column's, B[16 g + 8 i + j][j] =
// the activation of the i-th of lane group g's rows, so the product of half a chunk (a chunk: 16
// bytes, 32 output columns) with column j is the sum over the rows of activation times byte j, and
// the eight rows of two loads are added by the instruction.  A byte is two nibbles: each, masked into
// the upper half of a byte of its own, is 16 times its signed value, so extraction is an AND and
// a shift-and-AND per 4 bytes, 12 instructions per 16-byte load.
//
// Activations enter as integers too: an fp16 value is a whole multiple of 2^-24, X = x 2^24, below
// 2^40, in signed base-256 digits; columns j and j + 8 of B take two digits, so two
// instructions take four digits (|x| <= 127) and three take six (all of fp16).  How many is
// decided per slice by its survivors.  The products of a wavefront's rows of a 128-channel
// group and their sums are exact; a group's sum is rounded when it is put together from its digits,
// and its scale is applied in fp32.  An infinite activation makes every column NaN.
// (us at 50 %, FMAs / four digits / six: 4096 -> 4096 8.1 / 7.2 / 7.8, 14336 -> 4096 11.4 / 10.1 / 10.8,
// 8192 -> 2 x 28672 29.8 / 26.6 / 27.3.  Activations scaled by the slice's largest to 30 bits
// took four digits everywhere, but with 2000 beside values around 0.001 a column whose weight
// of the 2000 is zero was 2e-4 off; with six digits it is 8e-8.)
struct FixedDigits {
    static constexpr bool kMagnitude = true;
    static constexpr float kUnit = 5.9604644775390625e-8f;       // 2^-24
    // Four digits reach to 127 (2^24 + 2^16 + 2^8 + 1).
    static_assert(kModestLimit <= 127.f, "slices of modest survivors need four digits");
    // Digits 0 to 3 in the second word, 4 and 5 in the lower half of the first, below the channel
    // counted from the slice's first.  Digit d of X is byte d: adding 128 to each digit that a higher
    // one follows makes the bytes of X unsigned digits without a borrow, and the flip of their
    // top bits takes it off again.  X is put together from the nearest whole number and what is left.
    static_assert(kMaxSlice <= 1 << 15, "a channel of a slice fits the upper half of a word");
    static __device__ __forceinline__ int2 entry(int, int offset, float x)
    {
        const float whole = rintf(x);
        const unsigned rest = (unsigned)(int)((x - whole) * 16777216.f) + 0x00808080u;   // below 2^25
        const unsigned upper = (unsigned)(int)whole + 0x8080u + (rest >> 24);            // digits 3, 4, 5
        const unsigned low = __builtin_amdgcn_perm(upper, rest, 0x04020100u) ^ 0x80808080u;
        const unsigned high = __builtin_amdgcn_perm((unsigned)offset, upper ^ 0x8000u, 0x05040201u);
        return make_int2((int)high, (int)low);
    }
};

typedef int i32x4 __attribute__((ext_vector_type(4)));


// One batch of row loads of the int4 kernel: U wavefront loads of 4 rows, all from one 128-channel
// group, and the group's scales for the columns this lane holds sums of.
template <int U, int P>
struct W4Batch {
    u32x4 v[U];
    int x[U][P - 1];  // digits of the activations: 0..3, and 4, 5
    unsigned sc[4];   // fp16 pairs: chunk 4 * (lane / 16) + r, byte lane % 16, at [r]
    int rows;         // live rows in this batch (wavefront-uniform); 0 = the share is exhausted
    bool ends_run;    // wavefront-uniform
};

// Integer sums over the rows of one run (a wavefront's rows of one group), P pairs of digits: lane
// (n = lane % 16, g = lane / 16) holds, in register r, chunk 4 g + r, byte n % 8 of half h, digit
// n / 8 + 2 p.  At most 128 rows of |digit| <= 128 and |16 nibble| <= 128: 2^21, a pair 2^29.
template <int P>
struct W4Sums {
    i32x4 v[2][2][P];      // [nibble][h][p] sum of digit * 16 * nibble
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int p = 0; p < P; ++p) v[k][h][p] = i32x4{0, 0, 0, 0};
    }
};

// Work of one block for int4 weights with group scales: output tile `tile`
// (tile_cols columns) x K-slice `s` (ks channels, a multiple of 128).
//
// A wavefront covers 512 columns (16 lanes of 32, four rows per load).  With LPR = 32 (tiles of up to
// 1024 columns) the even wavefronts take the left half of the tile and the odd ones the right, and a
// pair shares its rows.  The wavefronts take equal contiguous shares of the compacted list, as for
// the other formats.  The list is ascending, so each 128-channel group is a
// run of it, delimited by the segment prefixes (two 64-channel segments per
// group), and a wavefront's share crosses few group boundaries: the scales are applied once per
// (wavefront, group it touches).  Batches never straddle a group, and two batches are in flight
// per wavefront across group boundaries.
// Returns how many of the tile's outputs this thread wrote.
template <int LPR, int WAVES, int U, class XS>
__device__ __forceinline__ int w4_block(const FmtW4::Args &a, const XS &x,
                                         float t, float *partial, const Meeting &meet, int gtile, float *y, int m,
                                         int n, int ks, int tile, int s, int tile_cols, int splits,
                                         const SurvivorReport &report)
{
    using F = FmtW4;
    constexpr int EPL = F::kElemsPerLane;
    constexpr int R = 4;                          // rows per wavefront load
    constexpr int PARTS = LPR / 16;               // wavefronts side by side over the tile's columns
    constexpr int SHARES = WAVES / PARTS;
    constexpr int PART_COLS = 16 * EPL;
    static_assert(LPR == 16 || LPR == 32, "tiles of up to 512 or 1024 columns");
    extern __shared__ __align__(16) unsigned char smem[];
    int2 *list = reinterpret_cast<int2 *>(smem);
    float *red = reinterpret_cast<float *>(smem + (size_t)ks * sizeof(int2));
    __shared__ int counts[kCompactInts];

    asm volatile("" ::"s"(a.W), "s"(a.scale), "s"(partial), "s"(meet.counters), "s"(y));   // as in gemv_block
    const int k0 = s * ks;                       // multiple of 128
    const int k1 = min(m, k0 + ks);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = w % PARTS, share = w / PARTS;
    int group_excl;                    // lane j: where group j of the slice begins in the list
    int cnt = 0;
    int magnitude = kModest;
    bool compacted = false;
    if constexpr (XS::kPlainHalf) {
        if (k1 - k0 <= kPrivateSlice) {         // block-uniform: short slices need no barrier
            cnt = compact_slice_private<FixedDigits>(x.x, t, k0, k1, share, SHARES, list, group_excl,
                                                     &magnitude);
            compacted = true;
        }
    }
    if (!compacted)
        cnt = compact_slice<WAVES, XS, FixedDigits>(x, t, k0, k1, list, counts, group_excl, nullptr, false,
                                                    &magnitude);

    trace_mark(2);
    if (tile == 0 && !meet.word_step && threadIdx.x == (WAVES - 1) * 64) report_slice(report, s, splits, cnt);
    const int lane = threadIdx.x & 63;
    const int l = lane & 15, g = lane >> 4;
    const int col0 = tile * tile_cols;
    const int part0 = col0 + part * PART_COLS;
    const int part_cols = tile_cols - part * PART_COLS;
    const unsigned row_bytes = (unsigned)(n / 2);
    const unsigned char *lane_base =
        static_cast<const unsigned char *>(a.W) + (size_t)k0 * row_bytes +
        lane_column<EPL>(part0, part_cols, n, l) / 2;
    // columns this lane adds up: chunk 4 g + r, byte l
    const __half *scale_base = a.scale + (size_t)(k0 / kGroup) * n + 2 * l;
    int scale_col[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) scale_col[r] = lane_column<EPL>(part0, part_cols, n, 4 * g + r);
    // B: this lane's column takes byte l % 8 of a lane, from digit l / 8 + 2 p of the row (of digits
    // 4 and 5, digit l / 8 of the channel's word)
    unsigned pick[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const unsigned at = 8 * (l & 3), digit = 2 * p + (l >> 3);
            pick[p][q] = ((l >> 2) & 1) == q ? (0x0C0C0C0Cu & ~(0xFFu << at)) | (digit << at)
                                             : 0x0C0C0C0Cu;
        }

    float acc[2][4];                              // [nibble][r]: chunk 4 g + r, byte l
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[q][r] = 0.f;
    // where a digit's sum lies when the two lanes that hold a pair of digits join them
    const int own_shift = l < 8 ? 0 : 8, other_shift = 8 - own_shift;
    int start, mine;
    // Told to be uniform: without this the walk over the groups is compiled with masks and vector compares, 30
    // registers and a loop of its own more per batch.
    cnt = __builtin_amdgcn_readfirstlane(cnt);
    magnitude = __builtin_amdgcn_readfirstlane(magnitude);
    wave_share(cnt, share, SHARES, start, mine);
    // Walk state (all wavefront-uniform): next list position, end of the share, current
    // group of the slice and the end of this wavefront's rows in it.
    // list offset at which group j of the slice begins (past the last group: the total)
    auto group_begin = [&](int j) { return __builtin_amdgcn_readlane(group_excl, j); };
    int cur = start;
    const int end = start + mine;
    int gi = 0, gend = min(end, group_begin(1));

    auto stream = [&](auto pairs) {
        constexpr int P = pairs.value;
        W4Sums<P> sums;
        sums.clear();
        // Every call issues exactly U row loads and the four scale loads of the batch's group,
        // whether or not rows are left: the compiler then knows how many loads are outstanding at
        // every wait and waits for a batch's own loads only.  (With a conditional scale load and an
        // early return for an exhausted share it waited for older loads between the loads of a
        // batch, and little more than one batch was ever in flight.)  A batch past the end of the
        // share re-reads the share's last row with zero multipliers.
        auto issue = [&](W4Batch<U, P> &b) {
            const bool live = cur < end;                  // wavefront-uniform
            if (live) {
                while (cur >= gend) {                     // next group with rows in this share
                    ++gi;
                    gend = min(end, group_begin(gi + 1));
                }
            }
            const int nb = live ? min(U * R, gend - cur) : 0;
            const int last = live ? cur + nb - 1 : end - 1;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = cur + u * R + g;
                const int2 ent = list[min(e, last)];
                const bool ours = live && e <= last;
                b.x[u][0] = ours ? ent.y : 0;
                if constexpr (P == 3) b.x[u][1] = ours ? ent.x : 0;
                b.v[u] = load_stream16(lane_base + (size_t)((unsigned)ent.x >> 16) * row_bytes);
            }
            b.rows = nb;
            b.ends_run = live && cur + nb == gend;
            const __half *sp = scale_base + (size_t)gi * n;
#pragma unroll
            for (int r = 0; r < 4; ++r) b.sc[r] = *reinterpret_cast<const unsigned *>(sp + scale_col[r]);
            cur += nb;
        };
        auto consume = [&](const W4Batch<U, P> &b) {
#pragma unroll
            for (int u = 0; u < U; u += 2) {          // slots past the end of a run multiply by zero
                i32x4 half[2][2], B[P];               // [nibble][h] of two rows
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const unsigned v = b.v[u + i][q];
                        half[0][q / 2][2 * i + q % 2] = (int)((v << 4) & 0xF0F0F0F0u);
                        half[1][q / 2][2 * i + q % 2] = (int)(v & 0xF0F0F0F0u);
                    }
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int q = 0; q < 2; ++q) {
                            const unsigned digits = (unsigned)b.x[u + i][p / 2];
                            B[p][2 * i + q] = (int)__builtin_amdgcn_perm(digits, digits, pick[p % 2][q]);
                        }
#pragma unroll
                for (int k = 0; k < 4 * P; ++k) {
                    const int q = k / (2 * P), h = k / P % 2, p = k % P;
                    sums.v[q][h][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(half[q][h], B[p],
                                                                            sums.v[q][h][p], 0, 0, 0);
                }
            }
            if (!b.ends_run) return;
            // The lanes l < 8 take the first half of a chunk and give the second to the lane 8 further,
            // which holds the other digit of a pair.  A column's sum is complete before the group's
            // scale multiplies it: an infinite scale then gives what it gives the whole sum.
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    int pair[P];
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        const int first = sums.v[q][0][p][r], second = sums.v[q][1][p][r];
                        const int own = l < 8 ? first : second, give = l < 8 ? second : first;
                        const int got = __builtin_amdgcn_update_dpp(0, give, 0x128 /* row_ror:8 */, 0xF,
                                                                    0xF, false);
                        pair[p] = (int)(((unsigned)own << own_shift) + ((unsigned)got << other_shift));
                    }
                    float sum = (float)pair[P - 1];       // each pair weighs 2^16 more than the one before
#pragma unroll
                    for (int p = P - 2; p >= 0; --p) sum = fmaf(sum, 65536.f, (float)pair[p]);
                    const __half2 sc = __builtin_bit_cast(__half2, b.sc[r]);
                    acc[q][r] = fmaf(q ? __high2float(sc) : __low2float(sc), sum, acc[q][r]);
                }
            sums.clear();
        };

        // Two batches in flight.  The fences keep the compiler from sinking a batch's loads into
        // the consumption of the batch before it.  (A third batch in flight was measured 2 to 6 %
        // slower.)
        if (mine > 0) {                               // wavefront-uniform
            W4Batch<U, P> b0, b1;
            issue(b0);
            while (b0.rows > 0) {
                issue(b1);
                __builtin_amdgcn_sched_barrier(0);
                consume(b0);
                __builtin_amdgcn_sched_barrier(0);
                if (b1.rows <= 0) break;
                issue(b0);
                __builtin_amdgcn_sched_barrier(0);
                consume(b1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (magnitude != kModest) stream(std::integral_constant<int, 3>{});
    else stream(std::integral_constant<int, 2>{});
    trace_mark(3);
    trace_mark_thread(1, (WAVES - 1) * 64);
    const float unit = magnitude == kInfinite ? __uint_as_float(0x7FC00000u) : 0.0625f * FixedDigits::kUnit;
    float *row = red + share * combine_row<EPL, LPR> + part * PART_COLS + 2 * l;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        *reinterpret_cast<float2 *>(row + EPL * (4 * g + r)) =
            make_float2(acc[0][r] * unit, acc[1][r] * unit);
    return block_finish<F, LPR, WAVES, SHARES>(red, partial, meet, gtile, y, tile, col0, tile_cols, s,
                                               splits, n, a, report, cnt, t);
}

template <int LPR, int WAVES, int U>
__global__ __launch_bounds__(WAVES * 64) void sparse_gemv_w4_kernel(
    FmtW4::Args a, const __half *__restrict__ x, float t, float *partial, Meeting meet, float *y,
    int m, int n, int ks, int tile_cols, int splits)
{
    trace_mark(0);
    const int tile = blockIdx.x;
    w4_block<LPR, WAVES, U>(a, HalfSource{x}, t, partial, meet, tile, y, m, n, ks, tile, blockIdx.y, tile_cols, splits,
                            survivor_report(meet.counters, 0, splits));
    trace_mark(6);
}

// The int4 product with its input formed in the kernel from the two products that precede
// W_down (Appendix A.3), as sparse_gemv_swiglu_kernel does for the other formats.
template <int LPR, int WAVES, int U>
__global__ __launch_bounds__(WAVES * 64) void sparse_gemv_w4_swiglu_kernel(
    FmtW4::Args a, const float *__restrict__ gate, const float *__restrict__ up, float t,
    float *partial, Meeting meet, float *y, int m, int n, int ks, int tile_cols,
    int splits)
{
    trace_mark(0);
    const int tile = blockIdx.x;
    w4_block<LPR, WAVES, U>(a, SwigluSource{gate, up}, t, partial, meet, tile, y, m, n, ks, tile, blockIdx.y, tile_cols,
                            splits, survivor_report(meet.counters, 0, splits));
}

// Several int4 matrices that read the same hidden state in one launch; the block finds its
// matrix from its tile index as in sparse_gemv_multi_kernel.
template <int LPR, int WAVES, int U, class XS>
__device__ __forceinline__ void w4_multi_block(const MultiArgs<FmtW4> &ma, const XS &x,
                                               float *partial, Meeting meet, int m, int ks,
                                               int tile_cols, int splits, int gtile, int s)
{
    trace_mark(0);
    int k = 0, first = 0, n = ma.n[0];      // as in multi_block
    size_t partial_off = 0;
    FmtW4::Args a = ma.a[0];
    float *y = ma.y[0];
    float t = ma.t[0];
    asm volatile("" ::"s"(ma.y[0]), "s"(ma.y[1]), "s"(ma.y[2]), "s"(ma.y[3]), "s"(ma.n[0]), "s"(ma.n[1]),
                 "s"(ma.n[2]), "s"(ma.n[3]), "s"(ma.t[0]), "s"(ma.t[1]), "s"(ma.t[2]), "s"(ma.t[3]),
                 "s"(ma.a[0].W), "s"(ma.a[1].W), "s"(ma.a[2].W), "s"(ma.a[3].W), "s"(ma.tile_begin[4]),
                 "s"(partial), "s"(meet.counters), "s"(splits), "s"(ma.a[0].scale), "s"(ma.a[1].scale), "s"(ma.a[2].scale),
                 "s"(ma.a[3].scale));
#pragma unroll
    for (int j = 1; j < kMaxMulti; ++j) {
        const bool here = j < ma.count && gtile >= ma.tile_begin[j];
        partial_off += here ? (size_t)splits * ma.n[j - 1] : 0;
        k = here ? j : k;
        first = here ? ma.tile_begin[j] : first;
        n = here ? ma.n[j] : n;
        y = here ? ma.y[j] : y;
        t = here ? ma.t[j] : t;
        FmtW4::select(a, ma.a[j], here);
    }
    w4_block<LPR, WAVES, U>(a, x, t, partial + partial_off, meet, gtile, y, m, n, ks, gtile - first, s, tile_cols, splits,
                            survivor_report(meet.counters, k, splits));
    trace_mark(6);
}

template <int LPR, int WAVES, int U>
__global__ __launch_bounds__(WAVES * 64) void sparse_gemv_w4_multi_kernel(
    MultiArgs<FmtW4> ma, const __half *__restrict__ x, float *partial, Meeting meet, int m,
    int ks, int tile_cols, int splits)
{
    asm volatile("" ::"s"(x));                 // as in multi_block
    w4_multi_block<LPR, WAVES, U>(ma, HalfSource{x}, partial, meet, m, ks, tile_cols, splits,
                                  (int)blockIdx.x, (int)blockIdx.y);
}

// The grouped int4 launch with its shared input formed from the hidden state before the
// normalisation layer, as sparse_gemv_rmsnorm_multi_kernel does for the other formats.
template <int LPR, int U>
__global__ __launch_bounds__(kNormWaves * 64) void sparse_gemv_w4_rmsnorm_multi_kernel(
    MultiArgs<FmtW4> ma, const float *__restrict__ h, const float *__restrict__ gamma, float eps,
    double inv_m, float *partial, Meeting meet, int m, int ks, int tile_cols, int splits)
{
    __shared__ double wave_sums[kMaxNormChunks * kNormWaves];
    asm volatile("" ::"s"(h), "s"(gamma), "s"(eps), "s"(inv_m));      // as in multi_block
    w4_multi_block<LPR, kNormWaves, U>(ma, RmsnormSource{h, gamma, m, inv_m, eps, wave_sums}, partial,
                                       meet, m, ks, tile_cols, splits, (int)blockIdx.x, (int)blockIdx.y);
}

// Independent int4 groups in one launch (see sparse_gemv_stack_kernel).
template <int WAVES, int U>
__global__ __launch_bounds__(WAVES * 64) void sparse_gemv_w4_stack_kernel(StackArgs<FmtW4> sa)
{
    int block;
    const StackGroup<FmtW4> &sg = sa.g[stack_group_of_block(sa, block)];
    const int tiles = sg.ma.tile_begin[sg.ma.count], gtile = block % tiles, s = block / tiles;
    if (sg.lanes_per_row == 32)
        w4_multi_block<32, WAVES, U>(sg.ma, HalfSource{sg.x}, sg.partial, sg.meet, sg.m, sg.ks,
                                     sg.tile_cols, sg.splits, gtile, s);
    else
        w4_multi_block<16, WAVES, U>(sg.ma, HalfSource{sg.x}, sg.partial, sg.meet, sg.m, sg.ks,
                                     sg.tile_cols, sg.splits, gtile, s);
}

hipError_t launch_gemv_w8_stack(int groups, const StackGroupDesc *d, hipStream_t stream)
{
    StackArgs<FmtW8> sa{};
    size_t lds;
    const hipError_t e = fill_stack_args<FmtW8>(
        sa, lds, groups, d, 64, 8, 64, [](FmtW8::Args &a, const StackGroupDesc &g, int k) {
            a.W = g.Wt[k];
            a.scale = static_cast<const __half *>(g.scale[k]);
        });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sparse_gemv_stack_kernel<FmtW8, 8, 4, true>), dim3(sa.block_begin[groups]),
                       dim3(8 * 64), lds, stream, sa);
    return hipGetLastError();
}

hipError_t launch_gemv_w4_stack(int groups, const StackGroupDesc *d, hipStream_t stream)
{
    StackArgs<FmtW4> sa{};
    size_t lds;
    const hipError_t e = fill_stack_args<FmtW4>(
        sa, lds, groups, d, kGroup, 16, 32, [](FmtW4::Args &a, const StackGroupDesc &g, int k) {
            a.W = g.Wt[k];
            a.scale = static_cast<const __half *>(g.scale[k]);
        });
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sparse_gemv_w4_stack_kernel<kW4Waves, kW4Unroll>),
                       dim3(sa.block_begin[groups]), dim3(kW4Waves * 64), lds, stream, sa);
    return hipGetLastError();
}

hipError_t launch_gemv_w8(const int8_t *Wq, const void *scale_f16, const void *x_f16, float t,
                          float *y, int m, int n, float *partial, int *counters,
                          const GemvShape &sh, hipStream_t stream)
{
    const GemvGeometry g = gemv_geometry(m, n, sh, FmtW8::kElemsPerLane, 64);
    const Meeting meet = meeting_of(counters, g.tiles, g.tile_cols, g.splits);
    FmtW8::Args a{Wq, static_cast<const __half *>(scale_f16)};
    const __half *x = static_cast<const __half *>(x_f16);
#define TEAL_LAUNCH(F, LPR, WAVES, U)                                                          \
    hipLaunchKernelGGL((sparse_gemv_kernel<F, LPR, WAVES, U>), dim3(g.tiles, g.splits), \
                       dim3(WAVES * 64), g.lds, stream, a, x, t, partial, meet, y, m, n,   \
                       g.ks, g.tile_cols, g.splits)
    TEAL_DISPATCH(TEAL_LAUNCH, FmtW8, sh);
#undef TEAL_LAUNCH
    return hipGetLastError();
}

hipError_t launch_gemv_w8_multi(int count, const int8_t *const *Wq, const int *row_pitch,
                                const void *const *scale_f16, const float *t, float *const *y,
                                const int *n, const void *x_f16, int m, float *partial,
                                int *counters, const GemvShape &sh, hipStream_t stream)
{
    int n_max = 0;
    for (int k = 0; k < count; ++k) n_max = n[k] > n_max ? n[k] : n_max;
    // slice length, split count and LDS size do not depend on n
    const GemvGeometry g = gemv_geometry(m, n_max, sh, FmtW8::kElemsPerLane, 64, kMaxLongSlice);
    MultiArgs<FmtW8> ma{};
    ma.count = count;
    ma.tile_begin[0] = 0;
    for (int k = 0; k < count; ++k) {
        ma.a[k].W = Wq[k];
        ma.a[k].ld = row_pitch ? row_pitch[k] : 0;
        ma.a[k].scale = static_cast<const __half *>(scale_f16[k]);
        ma.y[k] = y[k];
        ma.t[k] = t[k];
        ma.n[k] = n[k];
        ma.tile_begin[k + 1] = ma.tile_begin[k] + (n[k] + g.tile_cols - 1) / g.tile_cols;
    }
    const int tiles = ma.tile_begin[count];
    const Meeting meet = meeting_of(counters, tiles, g.tile_cols, g.splits);
    const __half *x = static_cast<const __half *>(x_f16);
#define TEAL_LAUNCH(F, LPR, WAVES, U)                                                          \
    do {                                                                                       \
        if (!allow_large_lds(sparse_gemv_multi_kernel<F, LPR, WAVES, U>, g.lds))               \
            return hipErrorInvalidValue;                                                       \
        hipLaunchKernelGGL((sparse_gemv_multi_kernel<F, LPR, WAVES, U>),                       \
                           dim3(tiles, g.splits), dim3(WAVES * 64), g.lds, stream, ma, x,     \
                           partial, meet, m, g.ks, g.tile_cols, g.splits);                 \
    } while (0)
    TEAL_DISPATCH(TEAL_LAUNCH, FmtW8, sh);
#undef TEAL_LAUNCH
    return hipGetLastError();
}

static bool w8_lanes_supported(const GemvShape &s)
{
    const int l = s.lanes_per_row;
    return (l == 8 || l == 16 || l == 32 || l == 64) && s.splits >= 1 && s.tile_cols >= 0 &&
           s.tile_cols % FmtW8::kElemsPerLane == 0 && s.tile_cols <= l * FmtW8::kElemsPerLane;
}

// The int8 kernels with their input formed in the kernel (the activation sources of the bf16
// kernels: Appendix A.3's MLP intermediate, the normalised hidden state).  Shapes with 8
// wavefronts and 4 loads per batch, which is what the launch-shape rule produces.
hipError_t launch_gemv_w8_swiglu(const int8_t *Wq, const void *scale_f16, const float *gate,
                                 const float *up, float t, float *y, int m, int n, float *partial,
                                 int *counters, const GemvShape &sh, hipStream_t stream)
{
    if (sh.waves != 8 || sh.unroll != 4 || !w8_lanes_supported(sh)) return hipErrorInvalidValue;
    const GemvGeometry g = gemv_geometry(m, n, sh, FmtW8::kElemsPerLane, 64);
    const Meeting meet = meeting_of(counters, g.tiles, g.tile_cols, g.splits);
    FmtW8::Args a{Wq, static_cast<const __half *>(scale_f16)};
#define TEAL_LAUNCH_S(LPR)                                                                     \
    hipLaunchKernelGGL((sparse_gemv_swiglu_kernel<FmtW8, LPR, 8, 4>), dim3(g.tiles, g.splits), \
                       dim3(8 * 64), g.lds, stream, a, gate, up, t, partial, meet, y, m, n, \
                       g.ks, g.tile_cols, g.splits)
    if (sh.lanes_per_row == 64) TEAL_LAUNCH_S(64);
    else if (sh.lanes_per_row == 32) TEAL_LAUNCH_S(32);
    else if (sh.lanes_per_row == 16) TEAL_LAUNCH_S(16);
    else TEAL_LAUNCH_S(8);
#undef TEAL_LAUNCH_S
    return hipGetLastError();
}

hipError_t launch_gemv_w8_rmsnorm_multi(int count, const int8_t *const *Wq, const int *row_pitch,
                                        const void *const *scale_f16, const float *t,
                                        float *const *y, const int *n, const float *h,
                                        const float *gamma, float eps, int m, float *partial,
                                        int *counters, const GemvShape &sh, hipStream_t stream)
{
    if (m < 8 || m > kMaxNormDim || m % 8 != 0 || sh.waves != kNormWaves || sh.unroll != 4 ||
        !w8_lanes_supported(sh))
        return hipErrorInvalidValue;
    int n_max = 0;
    for (int k = 0; k < count; ++k) n_max = n[k] > n_max ? n[k] : n_max;
    const GemvGeometry g = gemv_geometry(m, n_max, sh, FmtW8::kElemsPerLane, 64);
    MultiArgs<FmtW8> ma{};
    ma.count = count;
    ma.tile_begin[0] = 0;
    for (int k = 0; k < count; ++k) {
        ma.a[k].W = Wq[k];
        ma.a[k].ld = row_pitch ? row_pitch[k] : 0;
        ma.a[k].scale = static_cast<const __half *>(scale_f16[k]);
        ma.y[k] = y[k];
        ma.t[k] = t[k];
        ma.n[k] = n[k];
        ma.tile_begin[k + 1] = ma.tile_begin[k] + (n[k] + g.tile_cols - 1) / g.tile_cols;
    }
    const int tiles = ma.tile_begin[count];
    const Meeting meet = meeting_of(counters, tiles, g.tile_cols, g.splits);
#define TEAL_LAUNCH_N(LPR)                                                                     \
    hipLaunchKernelGGL((sparse_gemv_rmsnorm_multi_kernel<FmtW8, LPR, 4>),                      \
                       dim3(tiles, g.splits), dim3(kNormWaves * 64), g.lds, stream, ma, h,    \
                       gamma, eps, 1.0 / m, partial, meet, m, g.ks, g.tile_cols, g.splits)
    if (sh.lanes_per_row == 64) TEAL_LAUNCH_N(64);
    else if (sh.lanes_per_row == 32) TEAL_LAUNCH_N(32);
    else if (sh.lanes_per_row == 16) TEAL_LAUNCH_N(16);
    else TEAL_LAUNCH_N(8);
#undef TEAL_LAUNCH_N
    return hipGetLastError();
}

hipError_t launch_gemv_w4(const uint8_t *Wq, const void *scale_f16, const void *x_f16, float t,
                          float *y, int m, int n, float *partial, int *counters,
                          const GemvShape &sh, hipStream_t stream)
{
    GemvShape w4 = sh;
    w4.waves = kW4Waves;                          // the int4 kernel is built for 8 wavefronts
    const GemvGeometry g = gemv_geometry(m, n, w4, FmtW4::kElemsPerLane, kGroup);
    const Meeting meet = meeting_of(counters, g.tiles, g.tile_cols, g.splits);
    FmtW4::Args a{Wq, static_cast<const __half *>(scale_f16)};
    const __half *x = static_cast<const __half *>(x_f16);
#define TEAL_LAUNCH_W4(LPR)                                                                    \
    hipLaunchKernelGGL((sparse_gemv_w4_kernel<LPR, kW4Waves, kW4Unroll>),                      \
                       dim3(g.tiles, g.splits), dim3(kW4Waves * 64), g.lds, stream, a, x, t,  \
                       partial, meet, y, m, n, g.ks, g.tile_cols, g.splits)
    // A lane covers 32 columns: 16 lanes per row (tiles up to 512 columns) or 32 lanes
    // per row (up to 1024 columns).
    if (sh.lanes_per_row == 32) TEAL_LAUNCH_W4(32);
    else TEAL_LAUNCH_W4(16);
#undef TEAL_LAUNCH_W4
    return hipGetLastError();
}

hipError_t launch_gemv_w4_swiglu(const uint8_t *Wq, const void *scale_f16, const float *gate,
                                 const float *up, float t, float *y, int m, int n, float *partial,
                                 int *counters, const GemvShape &sh, hipStream_t stream)
{
    GemvShape w4 = sh;
    w4.waves = kW4Waves;
    const GemvGeometry g = gemv_geometry(m, n, w4, FmtW4::kElemsPerLane, kGroup);
    const Meeting meet = meeting_of(counters, g.tiles, g.tile_cols, g.splits);
    FmtW4::Args a{Wq, static_cast<const __half *>(scale_f16)};
#define TEAL_LAUNCH_W4S(LPR)                                                                   \
    hipLaunchKernelGGL((sparse_gemv_w4_swiglu_kernel<LPR, kW4Waves, kW4Unroll>),               \
                       dim3(g.tiles, g.splits), dim3(kW4Waves * 64), g.lds, stream, a, gate,  \
                       up, t, partial, meet, y, m, n, g.ks, g.tile_cols, g.splits)
    if (sh.lanes_per_row == 32) TEAL_LAUNCH_W4S(32);
    else TEAL_LAUNCH_W4S(16);
#undef TEAL_LAUNCH_W4S
    return hipGetLastError();
}

hipError_t launch_gemv_w4_rmsnorm_multi(int count, const uint8_t *const *Wq,
                                        const void *const *scale_f16, const float *t,
                                        float *const *y, const int *n, const float *h,
                                        const float *gamma, float eps, int m, float *partial,
                                        int *counters, const GemvShape &sh, hipStream_t stream)
{
    if (m < 8 || m > kMaxNormDim || m % kGroup != 0 || kW4Waves != kNormWaves)
        return hipErrorInvalidValue;
    int n_max = 0;
    for (int k = 0; k < count; ++k) n_max = n[k] > n_max ? n[k] : n_max;
    GemvShape w4 = sh;
    w4.waves = kW4Waves;
    const GemvGeometry g = gemv_geometry(m, n_max, w4, FmtW4::kElemsPerLane, kGroup);
    MultiArgs<FmtW4> ma{};
    ma.count = count;
    ma.tile_begin[0] = 0;
    for (int k = 0; k < count; ++k) {
        ma.a[k].W = Wq[k];
        ma.a[k].scale = static_cast<const __half *>(scale_f16[k]);
        ma.y[k] = y[k];
        ma.t[k] = t[k];
        ma.n[k] = n[k];
        ma.tile_begin[k + 1] = ma.tile_begin[k] + (n[k] + g.tile_cols - 1) / g.tile_cols;
    }
    const int tiles = ma.tile_begin[count];
    const Meeting meet = meeting_of(counters, tiles, g.tile_cols, g.splits);
#define TEAL_LAUNCH_W4N(LPR)                                                                   \
    hipLaunchKernelGGL((sparse_gemv_w4_rmsnorm_multi_kernel<LPR, kW4Unroll>),                  \
                       dim3(tiles, g.splits), dim3(kNormWaves * 64), g.lds, stream, ma, h,    \
                       gamma, eps, 1.0 / m, partial, meet, m, g.ks, g.tile_cols, g.splits)
    if (sh.lanes_per_row == 32) TEAL_LAUNCH_W4N(32);
    else TEAL_LAUNCH_W4N(16);
#undef TEAL_LAUNCH_W4N
    return hipGetLastError();
}

hipError_t launch_gemv_w4_multi(int count, const uint8_t *const *Wq, const void *const *scale_f16,
                                const float *t, float *const *y, const int *n, const void *x_f16,
                                int m, float *partial, int *counters, const GemvShape &sh,
                                hipStream_t stream)
{
    int n_max = 0;
    for (int k = 0; k < count; ++k) n_max = n[k] > n_max ? n[k] : n_max;
    GemvShape w4 = sh;
    w4.waves = kW4Waves;
    const GemvGeometry g = gemv_geometry(m, n_max, w4, FmtW4::kElemsPerLane, kGroup);
    MultiArgs<FmtW4> ma{};
    ma.count = count;
    ma.tile_begin[0] = 0;
    for (int k = 0; k < count; ++k) {
        ma.a[k].W = Wq[k];
        ma.a[k].scale = static_cast<const __half *>(scale_f16[k]);
        ma.y[k] = y[k];
        ma.t[k] = t[k];
        ma.n[k] = n[k];
        ma.tile_begin[k + 1] = ma.tile_begin[k] + (n[k] + g.tile_cols - 1) / g.tile_cols;
    }
    const int tiles = ma.tile_begin[count];
    const Meeting meet = meeting_of(counters, tiles, g.tile_cols, g.splits);
    const __half *x = static_cast<const __half *>(x_f16);
#define TEAL_LAUNCH_W4M(LPR)                                                                   \
    hipLaunchKernelGGL((sparse_gemv_w4_multi_kernel<LPR, kW4Waves, kW4Unroll>),                \
                       dim3(tiles, g.splits), dim3(kW4Waves * 64), g.lds, stream, ma, x,      \
                       partial, meet, m, g.ks, g.tile_cols, g.splits)
    if (sh.lanes_per_row == 32) TEAL_LAUNCH_W4M(32);
    else TEAL_LAUNCH_W4M(16);
#undef TEAL_LAUNCH_W4M
    return hipGetLastError();
}

// The int4 block body for the one-launch MLP.
struct W4Body {
    typedef FmtW4 Format;
    template <int LPR, class XS>
    static __device__ __forceinline__ int run(const FmtW4::Args &a, const XS &x, float t,
                                               float *partial, const Meeting &meet, int gtile, float *y, int m,
                                               int n, int ks, int tile, int s, int tile_cols,
                                               int splits, const SurvivorReport &report)
    {
        static_assert(LPR == 16 || LPR == 32, "a lane covers 32 int4 columns");
        return w4_block<LPR, kW4Waves, kW4Unroll>(a, x, t, partial, meet, gtile, y, m, n, ks, tile,
                                                  s, tile_cols, splits, report);
    }
};

static void set_wq_args(const void *&W, const __half *&scale, const void *w, const void *sc)
{
    W = w;
    scale = static_cast<const __half *>(sc);
}

hipError_t launch_mlp_w8(const MlpHostArgs &h, const MlpLaunch &L, hipStream_t stream)
{
    if (!mlp_shape_ok(L.gu, 16) || !mlp_shape_ok(L.down, 16)) return hipErrorInvalidValue;
    MlpArgs<FmtW8> A{};
    size_t lds;
    if (!fill_mlp_args<FmtW8>(A, lds, h, L, 64, [](FmtW8::Args &a, const void *W, const void *sc, int pitch) {
            set_wq_args(a.W, a.scale, W, sc);
            a.ld = pitch;
        }))
        return hipErrorInvalidValue;
    return launch_mlp_kernel<GemvBody<FmtW8>, true>(A, L.gu.lanes_per_row, L.down.lanes_per_row,
                                                    lds, stream);
}

hipError_t launch_mlp_w4(const MlpHostArgs &h, const MlpLaunch &L, hipStream_t stream)
{
    if (!mlp_shape_ok(L.gu, 32) || !mlp_shape_ok(L.down, 32)) return hipErrorInvalidValue;
    if (h.m % kGroup != 0 || h.f % kGroup != 0) return hipErrorInvalidValue;
    if (h.gu_pitch != 0 || h.down_pitch != 0) return hipErrorInvalidValue;   // rows are packed
    const auto lanes_ok = [](int l) { return l == 16 || l == 32; };
    if (!lanes_ok(L.gu.lanes_per_row) || !lanes_ok(L.down.lanes_per_row))
        return hipErrorInvalidValue;
    MlpArgs<FmtW4> A{};
    size_t lds;
    if (!fill_mlp_args<FmtW4>(A, lds, h, L, kGroup,
                              [](FmtW4::Args &a, const void *W, const void *sc, int) {
                                  set_wq_args(a.W, a.scale, W, sc);
                              }))
        return hipErrorInvalidValue;
    const dim3 grid(mlp_blocks(A.grid)), block(kW4Waves * 64);
#define TEAL_MLP_W4(LG, LD)                                                                    \
    hipLaunchKernelGGL((sparse_mlp_kernel<W4Body, LG, LD>), grid, block, lds, stream, A)
    if (L.gu.lanes_per_row == 32) {
        if (L.down.lanes_per_row == 32) TEAL_MLP_W4(32, 32);
        else TEAL_MLP_W4(32, 16);
    } else {
        if (L.down.lanes_per_row == 32) TEAL_MLP_W4(16, 32);
        else TEAL_MLP_W4(16, 16);
    }
#undef TEAL_MLP_W4
    return hipGetLastError();
}

}  // namespace teal

#ifdef TEAL_TRACE_BLOCKS
extern "C" int teal_trace_read_wq(unsigned long long *host, size_t count) { return teal::read_trace(host, count); }
#endif
