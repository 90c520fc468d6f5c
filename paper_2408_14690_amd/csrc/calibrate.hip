// Threshold calibration (Section 4.2): t_p is read off an empirical
// distribution of |x| built from activations collected offline.  fp16
// magnitudes have only 32768 bit patterns and non-negative fp16 values order
// like their bit patterns, so an exact histogram over the patterns yields the
// exact order statistic: no sorting, any number of batches.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include "teal_internal.h"

namespace teal {

namespace {

constexpr int kBins = 32768;              // fp16 magnitude bit patterns
constexpr int kHistThreads = 1024;
constexpr int kHistBlocks = 256;          // one per compute unit: the 128 KB of counters fill most of its LDS
constexpr int kHistLoads = 4;             // 16-byte loads per batch; a thread keeps two batches in flight
constexpr int kFlushBins = 0x7C00;       // 31 * 1024: bins 1 .. 0x7C00
constexpr unsigned kDumpBin = 0x7C01u;    // every NaN is counted here, and this counter is never flushed
constexpr unsigned kZeroBins = 0x7C40u;   // zeros, one counter per lane (patterns of NaNs, otherwise unused)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct HistBatch {
    u32x4 d[kHistLoads];
    __device__ __forceinline__ void load(const u32x4 *p)
    {
#pragma unroll
        for (int u = 0; u < kHistLoads; ++u) d[u] = __builtin_nontemporal_load(p + u * kHistThreads);
    }
};

// Inclusive prefix sums over the lanes of a wavefront, with data-parallel primitives (the steps
// of wave_inclusive_scan in gemv_common.h, on both halves of a 64-bit value).
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long lanes_from(unsigned long long v)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROWS, 0xF, true);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xF, true);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long wave_scan_u64(unsigned long long v)
{
    v += lanes_from<0x111, 0xF>(v);       // row_shr:1, 2, 4, 8
    v += lanes_from<0x112, 0xF>(v);
    v += lanes_from<0x114, 0xF>(v);
    v += lanes_from<0x118, 0xF>(v);
    v += lanes_from<0x142, 0xA>(v);       // row_bcast:15 -> rows 1, 3
    v += lanes_from<0x143, 0xC>(v);       // row_bcast:31 -> rows 2, 3
    return v;
}
__device__ __forceinline__ unsigned long long last_lane(unsigned long long v)
{
    return ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 63) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 63);
}

// Every block counts its share of x in a private histogram of all 32768
// patterns in LDS (32-bit counters: a block never sees 2^32 values, the
// entry point bounds count), then adds the non-empty counters to the global
// 64-bit histogram.  NaNs are left out.  The next batch of loads is issued
// before the current one is counted, so the stream never drains.
// Bound by HBM (2 bytes per value) and then by the flush, 3-5 M atomics at about 250 G/s (one per
// clock and memory channel).  134 MB of normal values: 45.6 us with every block walking the bins
// from the same end, 43.8 us this way (34 MB 30.1 -> 26.7 us, 8 MB 20.9 -> 19.6 us); the same with
// half of the values zero 137 -> 40 us.  (Shares that grow from block to block, so that the flushes
// follow each other under the reading, take another 7 us off the 134 MB but make samples of
// few distinct values, which the LDS atomics bound, up to 1.5 times as slow: not done.)
__global__ __launch_bounds__(kHistThreads) void abs_histogram_kernel(
    const uint16_t *__restrict__ x, size_t count, unsigned long long *__restrict__ hist)
{
    extern __shared__ __align__(16) unsigned int lds_hist[];   // kBins counters
    const int tid = threadIdx.x;
#pragma unroll
    for (int b = 0; b < kBins / (4 * kHistThreads); ++b)
        reinterpret_cast<u32x4 *>(lds_hist)[b * kHistThreads + tid] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();

    // branch-free: patterns above +Inf (NaNs) collapse onto the dump counter, and a zero goes to
    // the lane's own counter (a sample with many zeros would otherwise count lane by lane)
    const unsigned zero_bin = kZeroBins + (tid & 63);
    auto add = [&](unsigned mag) {
        atomicAdd(&lds_hist[mag == 0u ? zero_bin : min(mag, kDumpBin)], 1u);
    };
    auto add8 = [&](const u32x4 d) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            add(d[q] & 0x7FFFu);
            add((d[q] >> 16) & 0x7FFFu);
        }
    };
    // 16-byte loads over the aligned body, scalar loads over the ragged head and tail
    const size_t head = (size_t)((16 - ((uintptr_t)x & 15)) & 15) / 2;
    const size_t lead = head < count ? head : count;
    const size_t vecs = (count - lead) / 8;
    const u32x4 *xv = reinterpret_cast<const u32x4 *>(x + lead);
    const size_t units = (vecs + kHistThreads - 1) / kHistThreads;   // a contiguous range per block
    const size_t begin = units * blockIdx.x / gridDim.x * kHistThreads;
    size_t end = units * (blockIdx.x + 1) / gridDim.x * kHistThreads;
    if (end > vecs) end = vecs;
    const u32x4 *p = xv + begin + tid;
    const size_t mine = end > begin ? end - begin : 0;                   // block-uniform
    const size_t batches = mine / ((size_t)kHistLoads * kHistThreads);   // whole batches
    if (batches) {
        HistBatch cur, nxt;
        cur.load(p);
        for (size_t b = 1; b < batches; ++b) {
            p += kHistLoads * kHistThreads;
            nxt.load(p);
#pragma unroll
            for (int u = 0; u < kHistLoads; ++u) add8(cur.d[u]);
            cur = nxt;
        }
        p += kHistLoads * kHistThreads;
#pragma unroll
        for (int u = 0; u < kHistLoads; ++u) add8(cur.d[u]);
    }
    for (; p < xv + end; p += kHistThreads) add8(__builtin_nontemporal_load(p));
    const size_t tail0 = lead + vecs * 8;
    const size_t gtid = (size_t)blockIdx.x * kHistThreads + tid;
    if (gtid < lead) add(x[gtid] & 0x7FFFu);                             // at most 7 values each
    if (gtid < count - tail0) add(x[tail0 + gtid] & 0x7FFFu);
    __syncthreads();
    if (tid < 64) {
        const unsigned long long zeros = last_lane(wave_scan_u64(lds_hist[zero_bin]));
        if (tid == 0 && zeros) atomicAdd(&hist[0], zeros);
    }
    // Bins 1 .. 0x7C00 (+Inf), every block from a place of its own: with all blocks walking the
    // bins from the same end, 256 of them wanted the same lines at the same time.
    const int from = (int)(blockIdx.x % kHistBlocks) * (kFlushBins / kHistBlocks) + tid;
    for (int b0 = from; b0 < from - tid + kFlushBins; b0 += kHistThreads) {
        const int b = 1 + (b0 < kFlushBins ? b0 : b0 - kFlushBins);
        const unsigned c = lds_hist[b];
        if (c) atomicAdd(&hist[b], (unsigned long long)c);
    }
}

constexpr int kMaxLevels = 16;
struct Levels {
    double p[kMaxLevels];
    int count;
};

constexpr int kLevelWaves = 16;
constexpr int kWaveBins = kBins / kLevelWaves;          // bins of a wavefront
constexpr int kLevelRows = kWaveBins / 128;             // rows of 128 bins, two per lane
static_assert(kLevelRows * 128 * kLevelWaves == kBins, "the wavefronts' rows cover the bins");

// One block.  Wavefront w owns bins [2048 w, 2048 w + 2048), read in rows of 128 with 16-byte loads
// (one thread per 32 consecutive bins made every load touch 64 lines, each fetched 8 times: 12.2 us;
// 6.1 us now, most of it one compute unit reading 256 KB).  The 16 wavefront totals go
// through LDS; for each level the wavefront whose range contains rank k walks its rows.
__global__ __launch_bounds__(kLevelWaves * 64) void histogram_thresholds_kernel(
    const unsigned long long *__restrict__ hist, Levels lv, float *__restrict__ t_out)
{
    __shared__ unsigned long long totals[kLevelWaves];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    ulonglong2 own[kLevelRows];
    unsigned long long sum = 0;
#pragma unroll
    for (int j = 0; j < kLevelRows; ++j) {
        const unsigned long long *p = hist + w * kWaveBins + j * 128 + 2 * lane;
        own[j] = make_ulonglong2(p[0], p[1]);
    }
#pragma unroll
    for (int j = 0; j < kLevelRows; ++j) sum += own[j].x + own[j].y;
    sum = last_lane(wave_scan_u64(sum));
    if (lane == 0) totals[w] = sum;
    __syncthreads();
    unsigned long long below = 0, total = 0;
#pragma unroll
    for (int k = 0; k < kLevelWaves; ++k) {
        below += k < w ? totals[k] : 0ull;
        total += totals[k];
    }
    for (int l = 0; l < lv.count; ++l) {
        // rank k = ceil(p N - 1e-9), each operation rounded once (no fused multiply-add), so
        // that the integer decision is the one plain IEEE double arithmetic makes anywhere
        double k_real = ceil(__dadd_rn(__dmul_rn(lv.p[l], (double)total), -1e-9));
        if (k_real < 0.0) k_real = 0.0;
        if (k_real > (double)total) k_real = (double)total;
        const unsigned long long k = (unsigned long long)k_real;
        if (k == 0) {
            if (threadIdx.x == 0) t_out[l] = 0.f;
            continue;
        }
        if (k <= below || k > below + sum) continue;             // wavefront-uniform
        unsigned long long c = below;                            // samples below the row
        bool found = false;
#pragma unroll
        for (int j = 0; j < kLevelRows; ++j) {
            if (found) continue;                                 // wavefront-uniform
            const unsigned long long incl = wave_scan_u64(own[j].x + own[j].y);
            const unsigned long long row = last_lane(incl);
            if (k <= c + row) {
                const unsigned long long first = c + incl - own[j].y, second = c + incl;
                const unsigned long long before = first - own[j].x;
                if (k > before && k <= second) {                 // exactly one lane
                    const int bin = w * kWaveBins + j * 128 + 2 * lane + (k > first ? 1 : 0);
                    t_out[l] = __half2float(__ushort_as_half((unsigned short)bin));
                }
                found = true;
            }
            c += row;
        }
    }
}

}  // namespace

hipError_t launch_abs_histogram(const void *x_f16, size_t count, unsigned long long *hist,
                                hipStream_t stream)
{
    if (count == 0) return hipSuccess;
    size_t want = (count / 8 + kHistThreads - 1) / kHistThreads;
    int blocks = want < 1 ? 1 : want > (size_t)kHistBlocks ? kHistBlocks : (int)want;
    hipLaunchKernelGGL(abs_histogram_kernel, dim3(blocks), dim3(kHistThreads),
                       kBins * sizeof(unsigned int), stream,
                       static_cast<const uint16_t *>(x_f16), count, hist);
    return hipGetLastError();
}

hipError_t launch_histogram_thresholds(const unsigned long long *hist, const double *p, int np,
                                       float *t_out, hipStream_t stream)
{
    Levels lv{};
    lv.count = np;
    for (int l = 0; l < np; ++l) lv.p[l] = p[l];
    hipLaunchKernelGGL(histogram_thresholds_kernel, dim3(1), dim3(kLevelWaves * 64), 0, stream, hist,
                       lv, t_out);
    return hipGetLastError();
}

}  // namespace teal
