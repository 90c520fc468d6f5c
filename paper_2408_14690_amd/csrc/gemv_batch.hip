// Small-batch variant of the thresholded product (Section 5.4.4): one set of
// channels is dropped for the whole batch, chosen by the magnitude averaged
// over the batch dimension, and every row of the batch is multiplied with the
// surviving rows of the input-channel-major weights.  The weight stream is the
// same as for one vector (each surviving row is read once).
//
// The products run on the matrix cores.  With fp32 FMAs a 16-byte load costs 64 FMAs and 8
// conversions per lane at 8 batch rows, which is more issue than the stream leaves (8 rows
// took 1.5 times the time of one vector).  v_mfma_f32_16x16x32_bf16 takes 16 columns x 32
// input channels of weights and 32 channels x 16 columns of activations: bf16 weights go in
// as they are, and an fp16 activation is the exact sum of two bf16 numbers (8 + 3
// significand bits), so 8 batch rows x (high, low) fill its 16 columns and the products
// are exact.  What a 16-byte load costs then is 4 byte permutes (a lane's 8 weights of 8
// rows become 8 rows of 8 columns) and one matrix instruction, whatever the batch size.
// Llama-3-8B-shaped block at 50 %, 8 rows: 81.0 us with FMAs, 58.9 us this way (220 MB: 3.7 TB/s;
// one vector 52 us).  The row stream is bound by HBM; what remains above it is the compaction of 8
// activation vectors by every block (1.4 us at 512 channels, 3.4 us at 4096) and the combine.
//
// At one and two rows up to 4 wavefronts lie side by side over a tile of up to 512 columns (PARTS):
// with the narrow tile alone 2 rows of large matrices were slower than with FMAs in wide tiles
// (us per block, FMAs / narrow / now: 70B shape 156 / 167 / 153, 13B 76 / 82 / 72, ragged 4664-wide
// 71 / 81 / 67; 4096 -> 50264 40.1 / 55.0 / 41.7, whose unaligned rows cost more in pieces of 256
// bytes).  From three rows on the narrow tile is ahead of the FMAs at every size.
#include "gemv_common.h"

namespace teal {

namespace {

// Channel i survives iff (1 / batch) * sum_b |X[b][i]| > t.  Evaluated as
// sum > batch * t in fp64: fp16 -> fp32 -> fp64 and |.| are exact, a sum of
// up to kMaxBatch fp16 magnitudes is exact in fp64 and so is batch * t, so the
// decision involves no rounding and does not depend on the order of the batch.
// A NaN makes the sum NaN, which compares false (the channel is dropped).
// The activations of a channel are kept as fp16 pairs (batch rows 2k and 2k + 1); `batch` of the
// NB values count.
template <int NB>
__device__ __forceinline__ bool survives_batch(const unsigned (&pair)[NB / 2], int batch, double bound)
{
    double s = 0.0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const unsigned short h = (unsigned short)(pair[b / 2] >> (16 * (b & 1)));
        s += b < batch ? (double)fabsf(__half2float(__ushort_as_half(h))) : 0.0;
    }
    return s > bound;
}

// The same decision for a wavefront's 64 channels, as a ballot, from an fp32 sum (weight[b] = 1
// for batch rows that count, else 0).  The sum is within 2^-21 of the exact one, and bound
// rounded to fp32 within 2^-24, so where the two lie further apart than 2^-20 of each the fp32
// comparison is the exact one; only if that leaves a lane open (a sum next to the bound, an
// infinity, a NaN, zeros against t = 0) the wavefront evaluates the fp64 form.
template <int NB>
__device__ __forceinline__ unsigned long long ballot_batch(const unsigned (&pair)[NB / 2],
                                                           const float (&weight)[NB], int batch,
                                                           double bound)
{
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NB / 2; ++k) {
        const __half2 h = __builtin_bit_cast(__half2, pair[k]);
        s = fmaf(fabsf(__low2float(h)), weight[2 * k], s);
        s = fmaf(fabsf(__high2float(h)), weight[2 * k + 1], s);
    }
    const float bf = (float)bound;
    const float margin = 9.5367431640625e-7f * (s + bf);      // 2^-20
    const float d = s - bf;
    const bool keep = d > margin;
    if (__ballot(!keep && !(d < -margin)) == 0) return __ballot(keep);
    return __ballot(survives_batch<NB>(pair, batch, bound));
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Rows one matrix instruction takes (K), and the output columns of a wavefront: 16 lanes share a
// weight row, 8 columns each; the four groups of 16 lanes hold different rows.
constexpr int kChunkRows = 32;
constexpr int kBatchTile = 128;
// Activations of one surviving channel in LDS: 8 fp16 values (batch rows past NB are never written
// and feed matrix columns that are never read).  They are split into their high and low parts
// when a chunk is multiplied, where vector instructions are to be had under the row stream, and
// not in the compaction, where every block waits for them (4.4 -> 3.4 us at 4096 channels
// and 8 rows).
constexpr int kActBytes = 16;

// Rows of one wavefront: equal contiguous shares, in multiples of the 4 rows that one
// wavefront load covers.
template <int SHARES>
__device__ __forceinline__ int batch_share_rows(int cnt)
{
    return 4 * ((cnt + 4 * SHARES - 1) / (4 * SHARES));
}

// compact_slice for a batch: list_idx[] receives the surviving channels of [k0, k1) in
// ascending order and act[] their activations.  Same scheme: ballots and popcounts, counts
// through LDS, every wavefront scans them.  A lane looks at VEC (1, 2, 4) consecutive channels with
// one load per batch row (2 * VEC bytes aligned), PASSES times: the slice has at most
// 64 * VEC * PASSES * WAVES channels, a multiple of VEC.  What this takes is vector instructions (8
// cycles each with two wavefronts to a SIMD), so a channel's values stay packed.
template <int NB, int WAVES, int VEC, int PASSES>
__device__ __forceinline__ int compact_slice_batch(const __half *__restrict__ X, int batch, int m,
                                                   double bound, int k0, int k1, int *list_idx,
                                                   unsigned char *act, int *seg_cnt)
{
    constexpr int WORDS = (VEC + 1) / 2;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nseg = (k1 - k0 + 64 * VEC - 1) / (64 * VEC);

    // All loads are in flight together, from one position per pass (clamped to the slice; what lies past it is
    // left out below) and a scalar offset per batch row.  Batch rows past the last repeat it and have no
    // weight in the sums.  Single channels are loaded by address: 64 two-byte loads through a descriptor took longer
    // (8 rows, 2050 -> 28672 15.0 us a call instead of 14.3, 11006 -> 4096 13.2 instead of 12.8).
    const Buffer states = buffer_of(X, 2u * (unsigned)batch * (unsigned)m);
    unsigned raw[PASSES][NB][WORDS];
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int channel = min(k0 + ((w + j * WAVES) * 64 + lane) * VEC, k1 - VEC);
        const int at = 2 * channel;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            [[maybe_unused]] const int row = 2 * min(b, batch - 1) * m;
            if constexpr (VEC == 1) {
                raw[j][b][0] = *reinterpret_cast<const unsigned short *>(X + (size_t)min(b, batch - 1) * m + channel);
            } else if constexpr (VEC == 2) {
                raw[j][b][0] = __builtin_amdgcn_raw_buffer_load_b32(states, at, row, 0);
            } else {
                const auto u = __builtin_amdgcn_raw_buffer_load_b64(states, at, row, 0);
                raw[j][b][0] = u[0];
                raw[j][b][WORDS - 1] = u[1];
            }
        }
    }
    float weight[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) weight[b] = b < batch ? 1.f : 0.f;
    unsigned pair[PASSES][VEC][NB / 2];
    unsigned long long bal[PASSES][VEC];
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int seg = w + j * WAVES;
        const unsigned long long inside = __ballot(k0 + (seg * 64 + lane) * VEC < k1);
        int kept = 0;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
#pragma unroll
            for (int k = 0; k < NB / 2; ++k)
                pair[j][e][k] = __builtin_amdgcn_perm(raw[j][2 * k + 1][e / 2], raw[j][2 * k][e / 2],
                                                      (e & 1) ? 0x07060302u : 0x05040100u);
            bal[j][e] = ballot_batch<NB>(pair[j][e], weight, batch, bound) & inside;
            kept += __popcll(bal[j][e]);
        }
        if (lane == 0 && seg < nseg) seg_cnt[seg] = kept;
    }
    __syncthreads();
    const int c = lane < nseg ? seg_cnt[lane] : 0;
    const int incl = wave_inclusive_scan(c);
    const int seg_excl = incl - c;
    const int total = __builtin_amdgcn_readlane(incl, 63);
#pragma unroll
    for (int j = 0; j < PASSES; ++j) {
        const int seg = w + j * WAVES;
        if (seg >= nseg) continue;                     // wavefront-uniform
        int rank = __builtin_amdgcn_readlane(seg_excl, seg);
#pragma unroll
        for (int e = 0; e < VEC; ++e) rank += lanes_below(bal[j][e]);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if ((bal[j][e] >> lane) & 1ull) {
                list_idx[rank] = k0 + (seg * 64 + lane) * VEC + e;
                unsigned *dst = reinterpret_cast<unsigned *>(act + rank * kActBytes);
#pragma unroll
                for (int k = 0; k < NB / 2; ++k) dst[k] = pair[j][e][k];
                ++rank;
            }
        }
    }
    __syncthreads();
    return total;
}

// The accumulators of one lane: v[c][r] belongs to activation column lane % 16 and to output
// column 8 * (4 * (lane / 16) + r) + c of the tile.
struct BatchAcc {
    f32x4 v[8];
};

// Multiplies a chunk in: rows[u] holds this lane's 8 weights of row 4 u + lane / 16, `x` the
// activations.  Two rows' weights of one column are joined by one byte permute.
__device__ __forceinline__ void multiply_chunk(BatchAcc &acc, const u32x4 (&rows)[8], bf16x8 x)
{
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        u32x4 a;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            a[k] = __builtin_amdgcn_perm(rows[2 * k + 1][c / 2], rows[2 * k][c / 2],
                                         (c & 1) ? 0x07060302u : 0x05040100u);
        acc.v[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), x,
                                                           acc.v[c], 0, 0, 0);
    }
}

// The activations of one chunk for this lane: rows 4 u + lane / 16, u = 0..7, of batch row
// lane % 8, the high part in lanes with lane % 16 < 8, else the low part.  A transposing LDS read
// gives each of 16 lanes one column of a 4 x 16 block of 16-bit values, of which every lane
// addresses four neighbouring columns of one row (columns 8..15 are 0..7 again): `act` is what
// this lane addresses in the first block, the second lies 16 rows further.  High part: the upper
// 16 bits of the value in fp32; the rest has at most 3 significant bits (an infinity leaves a
// NaN, see the sums in block_finish_batch).  Rows from `rows_left` on belong to another wavefront
// (or to nobody) and count as zeros.
__device__ __forceinline__ bf16x8 chunk_activations(const unsigned char *act, int rows_left,
                                                     int lane)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)act);
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(act + 16 * kActBytes));
    const uint2 wa = __builtin_bit_cast(uint2, a), wb = __builtin_bit_cast(uint2, b);
    u32x4 x = {wa.x, wa.y, wb.x, wb.y};
    if (rows_left < kChunkRows) {                     // wavefront-uniform
        const int live = rows_left - (lane >> 4);     // rows 4 u < live are ours
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x[k] &= (8 * k < live ? 0x0000FFFFu : 0u) | (8 * k + 4 < live ? 0xFFFF0000u : 0u);
    }
    const unsigned take = (lane & 8) ? 0xFFFF0000u : 0u;         // what the low part leaves out
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const __half2 h = __builtin_bit_cast(__half2, (unsigned)x[k]);
        const float f0 = __low2float(h), f1 = __high2float(h);
        const float v0 = f0 - __uint_as_float(__float_as_uint(f0) & take);
        const float v1 = f1 - __uint_as_float(__float_as_uint(f1) & take);
        x[k] = __builtin_amdgcn_perm(__float_as_uint(v1), __float_as_uint(v0), 0x07060302u);
    }
    return __builtin_bit_cast(bf16x8, x);
}

// stream_rows for a batch: the `mine` rows of a wavefront's share in chunks of 32, 8 loads of 16
// bytes per lane each, two chunks in flight.  Slots behind the end of the share load its last
// row again (no new traffic) and count as zeros.
__device__ __forceinline__ void stream_rows_batch(BatchAcc &acc, const int *list_idx, int start,
                                                  int mine, const unsigned char *act,
                                                  const unsigned char *__restrict__ lane_base,
                                                  unsigned row_bytes)
{
    if (mine <= 0) return;
    // the lane from its own instruction: one register across the loop (128 are all there are)
    const int lane = lanes_below(~0ull);
    const int last = mine - 1;
    const int chunks = (mine + kChunkRows - 1) / kChunkRows;
    const int *share = list_idx + start;
    const unsigned char *act_lane =
        act + (start + 4 * ((lane & 15) >> 2) + (lane >> 4)) * kActBytes + (lane & 1) * 8;

    auto issue = [&](u32x4 (&rows)[8], int chunk) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int row = share[min(chunk * kChunkRows + 4 * u + (lane >> 4), last)];
            rows[u] = load_stream16(lane_base + (size_t)(unsigned)row * row_bytes);
        }
    };
    auto consume = [&](const u32x4 (&rows)[8], int chunk) {
        multiply_chunk(acc, rows, chunk_activations(act_lane + chunk * kChunkRows * kActBytes,
                                                    kChunkRows, lane));
    };
    auto consume_last = [&](u32x4 (&rows)[8]) {
        const int rows_left = mine - (chunks - 1) * kChunkRows;
        // 0 times an infinite weight is a NaN: the weights of the slots behind the share go, too
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (4 * u + (lane >> 4) >= rows_left) rows[u] = u32x4{0u, 0u, 0u, 0u};
        multiply_chunk(acc, rows,
                       chunk_activations(act_lane + (chunks - 1) * kChunkRows * kActBytes, rows_left,
                                         lane));
    };

    // Scheduling fences keep the two chunks apart: without them the compiler issues both
    // back to back and drains the queue before the next pair.
    u32x4 b0[8], b1[8];
    issue(b0, 0);
    int it = 0;
    for (; it + 2 < chunks; it += 2) {
        issue(b1, it + 1);
        __builtin_amdgcn_sched_barrier(0);
        consume(b0, it);
        __builtin_amdgcn_sched_barrier(0);
        issue(b0, it + 2);
        __builtin_amdgcn_sched_barrier(0);
        consume(b1, it + 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (it + 1 < chunks) {
        issue(b1, it + 1);
        __builtin_amdgcn_sched_barrier(0);
        consume(b0, it);
        __builtin_amdgcn_sched_barrier(0);
        consume_last(b1);
    } else {
        consume_last(b0);
    }
}

constexpr int kBatchWordRows = 2;                      // most rows of a batch that meet in column words

// One activation column of the combine buffer, padded so that the 16 columns a row of lanes
// holds are written to different LDS banks.
constexpr int kBatchRedRow = kBatchTile + 8;
constexpr int kBatchRedWave = 16 * kBatchRedRow;       // floats per wavefront

// Leaves this wavefront's accumulators in red[], laid out [wavefront][activation column][tile
// column]: high part of batch row b in activation column b, low part in column b + 8.
__device__ __forceinline__ void batch_sums_to_lds(const BatchAcc &acc, float *red, int w)
{
    const int lane = lanes_below(~0ull);
    float *dst = red + w * kBatchRedWave + (lane & 15) * kBatchRedRow +
                 32 * (lane >> 4);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < 2; ++q)
            *reinterpret_cast<float4 *>(dst + 8 * r + 4 * q) =
                make_float4(acc.v[4 * q][r], acc.v[4 * q + 1][r], acc.v[4 * q + 2][r],
                            acc.v[4 * q + 3][r]);
}

__device__ __forceinline__ void store_coherent2(float *p, float2 v)      // 8-byte aligned
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(p),
                       __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_coherent2(const float *p)        // 8-byte aligned
{
    return __builtin_bit_cast(
        float2, __hip_atomic_load(reinterpret_cast<const unsigned long long *>(p),
                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// block_finish for a batch, with a word (or a place in the partial rows, [split][batch row][n]) per batch row
// and column.  red[] (WAVES x kBatchRedWave floats) lies over the list, which is dead once every
// wavefront has left the row stream.  Wavefront w holds sums of part w % PARTS of the tile's columns.  A
// thread owns two neighbouring columns of one batch row.
template <int NB, int WAVES, int PARTS>
__device__ __forceinline__ void block_finish_batch(const BatchAcc &acc, float *red,
                                                   float *partial, const Meeting &meet, int gtile, float *Y,
                                                   int tile, int col0, int tile_cols, int s, int splits,
                                                   int n, int batch, int w,
                                                   const SurvivorReport &report, int cnt, double bound)
{
    constexpr int PAIRS = PARTS * kBatchTile / 2;
    static_assert(NB * PAIRS <= WAVES * 64, "one pair of columns per thread");
    __shared__ int last_flag;
    const int thread = w * 64 + lanes_below(~0ull);
    const int cols = min(tile_cols, n - col0);
    __syncthreads();                   // every wavefront is done with the list
    batch_sums_to_lds(acc, red, w);
    __syncthreads();
    trace_mark(7);
    const int bb = thread / PAIRS;
    const int c = 2 * (thread % PAIRS);
    const bool owner = bb < batch && c < cols;          // cols is a multiple of 8
    float2 sum = make_float2(0.f, 0.f);
    if (owner) {
        // The high parts of all wavefronts, then the low ones.  Where the high sum is not
        // finite it is the result: an infinite weight or activation makes it infinite or a NaN,
        // as the product is, and the low part a NaN.
        const float *hi = red + c / kBatchTile * kBatchRedWave + bb * kBatchRedRow + c % kBatchTile;
        const float *lo = hi + 8 * kBatchRedRow;
        float2 h = make_float2(0.f, 0.f), l = h;
#pragma unroll
        for (int q = 0; q < WAVES; q += PARTS) {
            const float2 a = *reinterpret_cast<const float2 *>(hi + q * kBatchRedWave);
            const float2 b = *reinterpret_cast<const float2 *>(lo + q * kBatchRedWave);
            h.x += a.x; h.y += a.y;
            l.x += b.x; l.y += b.y;
        }
        sum.x = fabsf(h.x) < INFINITY ? h.x + l.x : h.x;
        sum.y = fabsf(h.y) < INFINITY ? h.y + l.y : h.y;
    }
    float *y = Y + (size_t)bb * n + col0 + c;
    if (splits == 1) {
        if (owner) {
            store_coherent(y, sum.x);
            store_coherent(y + 1, sum.y);
        }
        return;
    }
    float *p = partial + (size_t)bb * n + col0 + c;
    const size_t split_stride = (size_t)batch * n;
    // Words for one or two rows.  With more, the atomics themselves take longer than the trips they save (8 rows,
    // Llama-3-8B block: 56.4 us by partial rows, 59.8 by words; 4 rows 52.1 and 52.3; 2 rows 53.2 and 52.0).
    constexpr bool kWords = NB <= kBatchWordRows;
    const Grid grid{grid_unit_bf16((float)bound), splits};
    if constexpr (kWords) {
        if (meet.word_step) {
            const ColumnWords words = column_words(meet, gtile, partial + col0, (unsigned)batch * n,
                                                   ((unsigned)splits * batch - 1u) * n + cols);
            const int at = bb * tile_cols + c, place = bb * n + c;
            unsigned long long mine_x = 0, mine_y = 0, found_x = 0, found_y = 0;
            if (owner) {
                mine_x = word_addend(words, grid, sum.x, at, place, s, splits);
                mine_y = word_addend(words, grid, sum.y, at + 1, place + 1, s, splits);
                found_x = word_add(words.word + at, mine_x);
                found_y = word_add(words.word + at + 1, mine_y);
            }
            unsigned long long *const counts = count_word(meet, report.matrix);
            const bool reports = tile == 0 && thread == (WAVES - 1) * 64;
            unsigned long long counted = 0;
            if (reports) counted = count_slice(counts, cnt);
            trace_mark(4);
            if (owner && word_complete(found_x, splits))
                store_coherent(y, word_value(words, grid, mine_x, found_x, at, place, splits));
            if (owner && word_complete(found_y, splits))
                store_coherent(y + 1, word_value(words, grid, mine_y, found_y, at + 1, place + 1, splits));
            if (reports) count_total(report, counts, cnt, splits, counted);
            trace_mark(5);
            return;
        }
    }
    const bool on_grid = kWords && splits <= kWordSplits;
    if (owner) store_coherent2(p + s * split_stride, sum);
    wait_vector_memory();
    __syncthreads();
    trace_mark(4);
    // the ticket wraps to zero with the last arrival: ready for the next call
    if (thread == 0)
        last_flag = atomicInc(reinterpret_cast<unsigned *>(meet.counters + (size_t)gtile * meet.counter_step),
                              (unsigned)splits - 1u) ==
                    (unsigned)splits - 1u;
    __syncthreads();
    trace_mark(5);
    if (!last_flag) return;
    if (tile == 0 && w == WAVES - 1) report_total(report, splits);

    // Second pass, up to 16 loads in flight; every output is summed in split order, so the
    // result does not depend on which block is last.
    if (!owner) return;
    constexpr int MAXLD = kWords ? kGridRows : 16;
    sum = make_float2(0.f, 0.f);
    GridTotal total_x, total_y;
    for (int j = 0; j < splits; j += MAXLD) {
        float2 v[MAXLD];
#pragma unroll
        for (int u = 0; u < MAXLD; ++u)
            v[u] = j + u < splits ? load_coherent2(p + (size_t)(j + u) * split_stride)
                                  : make_float2(0.f, 0.f);
#pragma unroll
        for (int u = 0; u < MAXLD; ++u) {
            sum.x += v[u].x;
            sum.y += v[u].y;
        }
        if constexpr (kWords) {
            if (on_grid) {
                float vx[MAXLD], vy[MAXLD];
#pragma unroll
                for (int u = 0; u < MAXLD; ++u) vx[u] = v[u].x, vy[u] = v[u].y;
                grid_add_rows(total_x, vx, splits - j, grid);
                grid_add_rows(total_y, vy, splits - j, grid);
            }
        }
    }
    if (on_grid)
        sum = make_float2(grid_value(total_x.whole, total_x.apart, grid),
                          grid_value(total_y.whole, total_y.apart, grid));
    store_coherent(y, sum.x);
    store_coherent(y + 1, sum.y);
}

// Work of one block: output tile `tile` x K-slice `s` of one matrix, all batch rows.  The tile has
// up to PARTS x kBatchTile columns; PARTS wavefronts side by side share their rows.
template <int NB, int WAVES, int PARTS>
__device__ __forceinline__ void batch_block(const void *__restrict__ W,
                                            const __half *__restrict__ X, int batch, double bound,
                                            float *partial, const Meeting &meet, int gtile, float *Y, int m, int n,
                                            int ks, int tile, int s, int tile_cols, int splits,
                                            const SurvivorReport &report)
{
    extern __shared__ __align__(16) unsigned char smem[];
    // [activations: ks rows, and a chunk that may be read past the last][list_idx: ks ints];
    // red[] reuses the front.
    int *list_idx = reinterpret_cast<int *>(smem + (size_t)(ks + kChunkRows) * kActBytes);
    float *red = reinterpret_cast<float *>(smem);
    __shared__ int seg_cnt[kMaxSegs];

    trace_mark(0);
    asm volatile("" ::"s"(W), "s"(partial), "s"(meet.counters), "s"(Y));      // as in gemv_block
    const int k0 = s * ks;
    const int k1 = min(m, k0 + ks);
    // Channels per lane by the length of the slice, so that short slices occupy every wavefront;
    // one by one where the rows of X do not lie on 8-byte boundaries, in as many passes as the
    // slice needs (8 rows 4097 -> 4096: 14.6 us with always 8 passes, 12.4 us).
    constexpr int kLanes = 64 * WAVES;
    const int len = k1 - k0;                           // block-uniform
    const bool vec = (m & 3) == 0 && (reinterpret_cast<uintptr_t>(X) & 7) == 0;
#define TEAL_COMPACT(VEC, PASSES)                                                                \
    compact_slice_batch<NB, WAVES, VEC, PASSES>(X, batch, m, bound, k0, k1, list_idx, smem, seg_cnt)
    int cnt;
    if (len <= kLanes) cnt = TEAL_COMPACT(1, 1);
    else if (vec)
        cnt = len <= 2 * kLanes   ? TEAL_COMPACT(2, 1)
              : len <= 4 * kLanes ? TEAL_COMPACT(4, 1)
                                  : TEAL_COMPACT(4, kMaxLongSliceBatch / (4 * kLanes));
    else
        cnt = len <= 2 * kLanes   ? TEAL_COMPACT(1, 2)
              : len <= 4 * kLanes ? TEAL_COMPACT(1, 4)
                                  : TEAL_COMPACT(1, kMaxLongSliceBatch / kLanes);
#undef TEAL_COMPACT

    trace_mark(2);
    if (tile == 0 && !meet.word_step && threadIdx.x == (WAVES - 1) * 64) report_slice(report, s, splits, cnt);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int share = batch_share_rows<WAVES / PARTS>(cnt);
    const int start = w / PARTS * share;
    const int mine = min(max(cnt - start, 0), share);

    const int col0 = tile * tile_cols;
    const int part0 = w % PARTS * kBatchTile;      // lanes past the tile's edge re-read its last columns
    const int col = lane_column<8>(col0 + part0, min(tile_cols - part0, kBatchTile), n, threadIdx.x & 15);
    const unsigned row_bytes = (unsigned)n * 2u;
    const unsigned char *lane_base = static_cast<const unsigned char *>(W) + (size_t)col * 2;

    BatchAcc acc;
#pragma unroll
    for (int c = 0; c < 8; ++c) acc.v[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    stream_rows_batch(acc, list_idx, start, mine, smem, lane_base, row_bytes);
    trace_mark(3);
    trace_mark_thread(1, (WAVES - 1) * 64);
    block_finish_batch<NB, WAVES, PARTS>(acc, red, partial, meet, gtile, Y, tile, col0, tile_cols, s, splits,
                                  n, batch, w, report, cnt, bound);
    trace_mark(6);
}

// 4 wavefronts per SIMD (at most 128 registers): two blocks share a unit, so that one's compaction
// and combine lie under the other's row stream where there are more blocks than units.
template <int NB, int WAVES, int PARTS>
__global__ __launch_bounds__(WAVES * 64, 4) void sparse_gemv_batch_kernel(
    const void *__restrict__ W, const __half *__restrict__ X, int batch, double bound,
    float *partial, Meeting meet, float *Y, int m, int n, int ks, int tile_cols, int splits)
{
    const int tile = blockIdx.x;
    batch_block<NB, WAVES, PARTS>(W, X, batch, bound, partial, meet, tile, Y, m, n, ks, tile, blockIdx.y,
                                  tile_cols, splits, survivor_report(meet.counters, 0, splits));
}

// Several matrices that read the same batch of hidden states (q/k/v, gate/up:
// Appendix A.3), each with its own threshold, in one launch; the block finds its
// matrix from its tile index as in sparse_gemv_multi_kernel.
struct BatchMultiArgs {
    const void *W[kMaxMulti];
    float *Y[kMaxMulti];
    double bound[kMaxMulti];          // batch * t_k
    int n[kMaxMulti];
    int tile_begin[kMaxMulti + 1];
    int count;
};

template <int NB, int WAVES, int PARTS>
__global__ __launch_bounds__(WAVES * 64, 4) void sparse_gemv_batch_multi_kernel(
    BatchMultiArgs ma, const __half *__restrict__ X, int batch, float *partial, Meeting meet,
    int m, int ks, int tile_cols, int splits)
{
    const int gtile = blockIdx.x, s = blockIdx.y;
    // all matrices' arguments at once, as in multi_block
    int k = 0, first = 0, n = ma.n[0];
    size_t partial_off = 0;            // each matrix owns splits * batch * n floats of partial rows
    const void *W = ma.W[0];
    float *Y = ma.Y[0];
    double bound = ma.bound[0];
    asm volatile("" ::"s"(ma.W[0]), "s"(ma.W[1]), "s"(ma.W[2]), "s"(ma.W[3]), "s"(ma.Y[0]), "s"(ma.Y[1]),
                 "s"(ma.Y[2]), "s"(ma.Y[3]), "s"(ma.bound[0]), "s"(ma.bound[1]), "s"(ma.bound[2]),
                 "s"(ma.bound[3]), "s"(ma.n[0]), "s"(ma.n[1]), "s"(ma.n[2]), "s"(ma.n[3]),
                 "s"(ma.tile_begin[4]), "s"(partial), "s"(meet.counters), "s"(X), "s"(batch), "s"(m), "s"(splits));
#pragma unroll
    for (int j = 1; j < kMaxMulti; ++j) {
        const bool here = j < ma.count && gtile >= ma.tile_begin[j];
        partial_off += here ? (size_t)splits * batch * ma.n[j - 1] : 0;
        k = here ? j : k;
        first = here ? ma.tile_begin[j] : first;
        n = here ? ma.n[j] : n;
        W = here ? ma.W[j] : W;
        Y = here ? ma.Y[j] : Y;
        bound = here ? ma.bound[j] : bound;
    }
    batch_block<NB, WAVES, PARTS>(W, X, batch, bound, partial + partial_off, meet, gtile, Y, m, n, ks,
                                  gtile - first, s, tile_cols, splits, survivor_report(meet.counters, k, splits));
}

constexpr int kBatchWaves = 8;

// One block thresholds the batch like sparsify_kernel does one vector: groups of 4 chunks
// of 1024 channels, the loads of a group (all batch rows) in flight together.
constexpr int kSparsifyWaves = 16;
constexpr int kSparsifyChunk = kSparsifyWaves * 64;
constexpr int kSparsifyGroup = 4;
__global__ __launch_bounds__(kSparsifyChunk) void sparsify_batch_kernel(
    const __half *__restrict__ X, int batch, int m, double bound, uint8_t *__restrict__ mask,
    int32_t *__restrict__ idx, int32_t *__restrict__ count)
{
    __shared__ int wave_cnt[2][kSparsifyGroup][kSparsifyWaves];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    int base = 0;
    int buf = 0;
    for (int c0 = 0; c0 < m; c0 += kSparsifyGroup * kSparsifyChunk, buf ^= 1) {
        __half raw[kSparsifyGroup][kMaxBatch];
#pragma unroll
        for (int j = 0; j < kSparsifyGroup; ++j) {
            const int i = min(c0 + j * kSparsifyChunk + (int)threadIdx.x, m - 1);
#pragma unroll
            for (int b = 0; b < kMaxBatch; ++b)       // rows past the batch repeat the last row
                raw[j][b] = X[(size_t)min(b, batch - 1) * m + i];
        }
        unsigned long long bal[kSparsifyGroup];
#pragma unroll
        for (int j = 0; j < kSparsifyGroup; ++j) {
            const int i = c0 + j * kSparsifyChunk + (int)threadIdx.x;
            double s = 0.0;
#pragma unroll
            for (int b = 0; b < kMaxBatch; ++b)
                s += b < batch ? (double)fabsf(__half2float(raw[j][b])) : 0.0;
            const bool keep = i < m && s > bound;
            if (i < m && mask) mask[i] = keep ? 1 : 0;
            bal[j] = __ballot(keep);
            if (lane == 0) wave_cnt[buf][j][w] = __popcll(bal[j]);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kSparsifyGroup; ++j) {
            if (c0 + j * kSparsifyChunk < m) {        // block-uniform
                int below = 0, total = 0;
#pragma unroll
                for (int ww = 0; ww < kSparsifyWaves; ++ww) {
                    const int c = wave_cnt[buf][j][ww];
                    below += ww < w ? c : 0;
                    total += c;
                }
                if (idx && ((bal[j] >> lane) & 1ull))
                    idx[base + below + lanes_below(bal[j])] =
                        c0 + j * kSparsifyChunk + (int)threadIdx.x;
                base += total;
            }
        }
        // wave_cnt is double-buffered: the next group writes the other half, and that
        // group's barrier orders it against this group's reads.
    }
    if (threadIdx.x == 0 && count) *count = base;
}

// The same result with eight channels per thread (one 16-byte load per batch row), for X on
// a 16-byte boundary and m a multiple of 8 (so that every row is): the block-wide prefix and
// the stores are shared by eight channels, as in the single-vector kernel of this shape.
constexpr int kVecChannels = 8;
constexpr int kVecPass = kSparsifyChunk * kVecChannels;

template <int P>
__global__ __launch_bounds__(kSparsifyChunk) void sparsify_batch_vec_kernel(
    const __half *__restrict__ X, int batch, int m, double bound, uint8_t *__restrict__ mask,
    bool mask_aligned, int32_t *__restrict__ idx, int32_t *__restrict__ count)
{
    __shared__ int wave_tot[2][P][kSparsifyWaves];
    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    int base = 0;
    int buf = 0;
    for (int c0 = 0; c0 < m; c0 += P * kVecPass, buf ^= 1) {
        unsigned bits[P];
        int cnt[P], incl[P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            const int i0 = c0 + (p * kSparsifyChunk + (int)threadIdx.x) * kVecChannels;
            const int ic = min(i0, m - kVecChannels);     // m >= 8 and m % 8 == 0
            uint4 raw[kMaxBatch];
#pragma unroll
            for (int b = 0; b < kMaxBatch; ++b)           // rows past the batch repeat the last row
                raw[b] = *reinterpret_cast<const uint4 *>(X + (size_t)min(b, batch - 1) * m + ic);
            double sum[kVecChannels];
#pragma unroll
            for (int e = 0; e < kVecChannels; ++e) sum[e] = 0.0;
#pragma unroll
            for (int b = 0; b < kMaxBatch; ++b) {
                if (b < batch) {                          // block-uniform
                    const unsigned wd[4] = {raw[b].x, raw[b].y, raw[b].z, raw[b].w};
#pragma unroll
                    for (int e = 0; e < kVecChannels; ++e) {
                        const unsigned short h = (unsigned short)(wd[e >> 1] >> (16 * (e & 1)));
                        sum[e] += (double)fabsf(__half2float(__ushort_as_half(h)));
                    }
                }
            }
            unsigned bb = 0;
#pragma unroll
            for (int e = 0; e < kVecChannels; ++e) bb |= (sum[e] > bound ? 1u : 0u) << e;
            if (i0 >= m) bb = 0;
            bits[p] = bb;
            cnt[p] = __popc(bb);
            incl[p] = wave_inclusive_scan(cnt[p]);
            if (lane == 63) wave_tot[buf][p][w] = incl[p];
            if (mask && i0 < m) {
                if (mask_aligned) {
                    const unsigned lo = bb & 0xFu, hi = (bb >> 4) & 0xFu;
                    uint2 mv;
                    mv.x = (lo & 1u) | ((lo & 2u) << 7) | ((lo & 4u) << 14) | ((lo & 8u) << 21);
                    mv.y = (hi & 1u) | ((hi & 2u) << 7) | ((hi & 4u) << 14) | ((hi & 8u) << 21);
                    *reinterpret_cast<uint2 *>(mask + i0) = mv;
                } else {
#pragma unroll
                    for (int e = 0; e < kVecChannels; ++e) mask[i0 + e] = (uint8_t)((bb >> e) & 1u);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (c0 + p * kVecPass < m) {                  // block-uniform
                int below = 0, total = 0;
#pragma unroll
                for (int ww = 0; ww < kSparsifyWaves; ++ww) {
                    const int c = wave_tot[buf][p][ww];
                    below += ww < w ? c : 0;
                    total += c;
                }
                if (idx) {
                    const int i0 = c0 + (p * kSparsifyChunk + (int)threadIdx.x) * kVecChannels;
                    int o = base + below + incl[p] - cnt[p];
#pragma unroll
                    for (int e = 0; e < kVecChannels; ++e)
                        if ((bits[p] >> e) & 1u) idx[o++] = i0 + e;
                }
                base += total;
            }
        }
    }
    if (threadIdx.x == 0 && count) *count = base;
}

}  // namespace

bool gemv_batch_shape_supported(int batch, const GemvShape &s)
{
    if (batch < 1 || batch > kMaxBatch) return false;
    const int nb = batch <= 2 ? 2 : batch <= 4 ? 4 : 8;
    const bool lpr = s.lanes_per_row == 64 || s.lanes_per_row == 32 || s.lanes_per_row == 16;
    const bool tc = s.tile_cols >= 0 && s.tile_cols % 8 == 0 && s.tile_cols <= s.lanes_per_row * 8;
    // (the limit of the documented interface; see batch_tile for the width a launch runs in)
    const bool fits = nb * s.lanes_per_row <= 256;
    return lpr && tc && fits && s.waves == kBatchWaves && s.splits >= 1;
}

// At one or two rows a block takes tiles of up to 512 columns, else of at most kBatchTile; a wider
// request runs in tiles of that width.
static GemvShape batch_tile(int batch, GemvShape sh)
{
    if (sh.tile_cols <= 0) sh.tile_cols = sh.lanes_per_row * 8;
    if (batch <= 2) return sh;
    sh.lanes_per_row = 16;
    if (sh.tile_cols > kBatchTile) sh.tile_cols = kBatchTile;
    return sh;
}

// Dynamic LDS of a block: the activations of a slice that survives whole and its index list;
// the combine buffer reuses it.
static size_t batch_lds(int ks)
{
    const size_t list = (size_t)(ks + kChunkRows) * kActBytes + (size_t)ks * sizeof(int);
    const size_t red = (size_t)kBatchWaves * kBatchRedWave * sizeof(float);
    return list > red ? list : red;
}

static Meeting batch_meeting(int *counters, int tiles, int batch, const GemvGeometry &g)
{
    Meeting m = meeting_of(counters, tiles, batch * g.tile_cols, g.splits);
    if (batch > kBatchWordRows) m.word_step = 0;
    return m;
}

hipError_t launch_gemv_bf16_batch(const void *Wt, const void *X_f16, int batch, float t, float *Y,
                                  int m, int n, float *partial, int *counters,
                                  const GemvShape &sh, hipStream_t stream)
{
    if (!gemv_batch_shape_supported(batch, sh)) return hipErrorInvalidValue;
    const GemvGeometry g = gemv_geometry(m, n, batch_tile(batch, sh), 8, 64);
    if (g.ks > kMaxLongSliceBatch) return hipErrorInvalidValue;
    const int lanes = batch_tile(batch, sh).lanes_per_row;
    const size_t lds = batch_lds(g.ks);
    const double bound = (double)batch * (double)t;
    const Meeting meet = batch_meeting(counters, g.tiles, batch, g);
    const __half *X = static_cast<const __half *>(X_f16);
#define TEAL_LAUNCH_B(NB, PARTS)                                                                        \
    do {                                                                                         \
        if (!allow_large_lds(sparse_gemv_batch_kernel<NB, kBatchWaves, PARTS>, lds))                    \
            return hipErrorInvalidValue;                                                         \
        hipLaunchKernelGGL((sparse_gemv_batch_kernel<NB, kBatchWaves, PARTS>), dim3(g.tiles, g.splits), \
                           dim3(kBatchWaves * 64), lds, stream, Wt, X, batch, bound, partial,    \
                           meet, Y, m, n, g.ks, g.tile_cols, g.splits);                          \
    } while (0)
    if (batch > 4) TEAL_LAUNCH_B(8, 1);
    else if (batch > 2) TEAL_LAUNCH_B(4, 1);
    else if (lanes == 64) TEAL_LAUNCH_B(2, 4);
    else if (lanes == 32) TEAL_LAUNCH_B(2, 2);
    else TEAL_LAUNCH_B(2, 1);
#undef TEAL_LAUNCH_B
    return hipGetLastError();
}

hipError_t launch_gemv_bf16_batch_multi(int count, const void *const *Wt, const float *t,
                                        float *const *Y, const int *n, const void *X_f16,
                                        int batch, int m, float *partial, int *counters,
                                        const GemvShape &sh, hipStream_t stream)
{
    int n_max = 0;
    for (int k = 0; k < count; ++k) n_max = n[k] > n_max ? n[k] : n_max;
    if (!gemv_batch_shape_supported(batch, sh)) return hipErrorInvalidValue;
    const GemvGeometry g = gemv_geometry(m, n_max, batch_tile(batch, sh), 8, 64);
    if (g.ks > kMaxLongSliceBatch) return hipErrorInvalidValue;
    const int lanes = batch_tile(batch, sh).lanes_per_row;
    const size_t lds = batch_lds(g.ks);
    BatchMultiArgs ma{};
    ma.count = count;
    ma.tile_begin[0] = 0;
    for (int k = 0; k < count; ++k) {
        ma.W[k] = Wt[k];
        ma.Y[k] = Y[k];
        ma.bound[k] = (double)batch * (double)t[k];
        ma.n[k] = n[k];
        ma.tile_begin[k + 1] = ma.tile_begin[k] + (n[k] + g.tile_cols - 1) / g.tile_cols;
    }
    const int tiles = ma.tile_begin[count];
    const Meeting meet = batch_meeting(counters, tiles, batch, g);
    const __half *X = static_cast<const __half *>(X_f16);
#define TEAL_LAUNCH_BM(NB, PARTS)                                                                       \
    do {                                                                                         \
        if (!allow_large_lds(sparse_gemv_batch_multi_kernel<NB, kBatchWaves, PARTS>, lds))              \
            return hipErrorInvalidValue;                                                         \
        hipLaunchKernelGGL((sparse_gemv_batch_multi_kernel<NB, kBatchWaves, PARTS>),                    \
                           dim3(tiles, g.splits), dim3(kBatchWaves * 64), lds, stream, ma, X,   \
                           batch, partial, meet, m, g.ks, g.tile_cols, g.splits);                \
    } while (0)
    if (batch > 4) TEAL_LAUNCH_BM(8, 1);
    else if (batch > 2) TEAL_LAUNCH_BM(4, 1);
    else if (lanes == 64) TEAL_LAUNCH_BM(2, 4);
    else if (lanes == 32) TEAL_LAUNCH_BM(2, 2);
    else TEAL_LAUNCH_BM(2, 1);
#undef TEAL_LAUNCH_BM
    return hipGetLastError();
}

hipError_t launch_sparsify_batch(const void *X_f16, int batch, int m, float t, uint8_t *mask,
                                 int32_t *idx, int32_t *count, hipStream_t stream)
{
    const __half *X = static_cast<const __half *>(X_f16);
    const double bound = (double)batch * (double)t;
    if (m >= kVecChannels && m % kVecChannels == 0 && (reinterpret_cast<uintptr_t>(X_f16) & 15) == 0) {
        const bool mask_aligned = (reinterpret_cast<uintptr_t>(mask) & 7) == 0;
        if (m <= kVecPass)
            hipLaunchKernelGGL(sparsify_batch_vec_kernel<1>, dim3(1), dim3(kSparsifyChunk), 0, stream,
                               X, batch, m, bound, mask, mask_aligned, idx, count);
        else
            hipLaunchKernelGGL(sparsify_batch_vec_kernel<2>, dim3(1), dim3(kSparsifyChunk), 0, stream,
                               X, batch, m, bound, mask, mask_aligned, idx, count);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sparsify_batch_kernel, dim3(1), dim3(kSparsifyWaves * 64), 0, stream, X,
                       batch, m, bound, mask, idx, count);
    return hipGetLastError();
}

}  // namespace teal

#ifdef TEAL_TRACE_BLOCKS
extern "C" int teal_trace_read_batch(unsigned long long *host, size_t count) { return teal::read_trace(host, count); }
#endif
