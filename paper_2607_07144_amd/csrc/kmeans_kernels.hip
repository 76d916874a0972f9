// kmeans_kernels.hip -- one Lloyd update of a residual stage of per-head
// codebooks (Sec. 3 "Setup": codebooks are trained by k-means), for gfx950.
//
// The assignment step is fkv_rvq_assign.  Accumulate: one block per book and
// 64-dimension slice sorts the member tokens by cluster; one lane per 8
// dimensions of a member token forms the stage input r = x - (codewords of the
// earlier stages) exactly in fp64, sums it in registers over a run of one
// cluster, and adds the run, as integers in units of 2^-24 (every binary16 value
// is a multiple of 2^-24), to the cluster's sum with 64-bit LDS atomics -- exact
// at every step, so the sums do not depend on any order (few tokens, and narrow
// rows, are added one by one without the sort).  Finalize: mean = sum /
// count * 2^-24 in fp64, rounded once to binary16; an empty cluster keeps its
// centroid.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include <algorithm>
#include <mutex>

#include "fkv.h"
#include "fkv_hip_common.h"

#pragma clang fp contract(off)

namespace fkv {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
constexpr int kThreads = 256;
constexpr int kAccThreads = 1024;
constexpr int kAccBatch = 4;     // tokens per thread whose loads are in flight together
constexpr int kChunk = 8192;     // tokens sorted by cluster at a time
constexpr int kSlice = 64;

// One element of a stage input in units of 2^-24.  A NaN adds nothing, and an
// infinity the largest or smallest multiple of 2^32 that an int64 holds.
__device__ __forceinline__ unsigned long long fixed24(double r)
{
    if (__builtin_isnan(r)) return 0;
    if (__builtin_isinf(r)) return r > 0.0 ? 0x7FFFFFFF00000000ull : 0x8000000000000000ull;
    return (unsigned long long)(long long)ldexp(r, 24);
}

// One block per (book, 64-dimension slice): the block owns that slice of the
// book's cluster sums in LDS, and at the end adds it to the global sums with
// plain read-modify-writes (no other block touches it in this launch).  The
// member tokens are taken 8192 at a time and sorted by cluster (a counting sort
// of 16-bit positions in LDS); each group of dc/8 lanes then walks a run of the
// sorted list with its eight dimensions per lane summed in registers, and adds
// them to LDS only where the cluster changes.  Adding every token to LDS with
// 64-bit atomics was what bounded this kernel (17 LDS cycles per wave
// instruction, eight per 8 tokens): 512 books of 256 x 128, 32,732 tokens each,
// stage 0 1.28 -> 0.98 ms, stage 1 1.49 -> 1.19, stage 2 1.75 -> 1.47 (3.4 -> 4.4
// TB/s of vectors at stage 0; they take 0.7 ms at 6 TB/s, the sort about a
// quarter of a chunk's time, since one block fills a compute unit's LDS).
// A register sum of n terms r = x - (earlier codewords), each a multiple of 2^-24
// below 2^16 (stage + 1), is exact in fp64 while n (stage + 1) 2^40 < 2^53; a
// group's run has at most kChunk / groups <= 64 tokens (8192 / 1024 per lane of a
// row), so 64 * 8 * 2^40 = 2^49.
// A run that holds a NaN or an infinity (its register sum is not finite) is
// walked again token by token instead, so that every finite element still counts
// exactly and the sums still do not depend on any order.
// A cluster's row in LDS is dc + 1 words long: with an odd number of 8-byte
// words per row, the same dimension of different clusters falls in different
// banks.
//
// ST >= 0: the stage is fixed at compile time, so the loops over the earlier
// stages unroll and all their codeword reads of a task batch are issued
// together.  ST = -1 takes the stage at run time (stages 5..7, where the
// unrolled form would spill).  B, the tokens whose loads are in flight together,
// is what the registers hold (128 for 16 waves): with four, stages 3, 4 and 5.. keep
// 16, 92 and 76 bytes of scratch.  512 books of 8192 tokens of 128, four, three and
// two (us): stage 3 523, 536, 537; stage 4 649, 627, 638; stage 5 1358, 1373, 1152.
template <int ST>
__global__ __launch_bounds__(kAccThreads) void kmeans_accumulate_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ books, const int32_t* __restrict__ stream_book,
    const uint8_t* __restrict__ symbols, unsigned long long* __restrict__ sums, uint32_t* __restrict__ counts,
    int64_t n_streams, int64_t T, int64_t t_begin, int64_t Ta, int d, int S, int K, int stage_rt)
{
    const int stage = ST >= 0 ? ST : stage_rt;
    constexpr int B = ST == 4 ? 3 : ST < 0 ? 2 : kAccBatch;
    extern __shared__ __align__(16) uint8_t lds[];
    const int n_slices = (d + kSlice - 1) / kSlice;
    const int b = blockIdx.x / n_slices, slice = blockIdx.x - b * n_slices;
    const int e0 = slice * kSlice, dc = min(kSlice, d - e0);   // this block's dimensions [e0, e0 + dc)
    const int nch = dc / 8;
    const int pitch = dc + 1;                                    // words per cluster row
    const int tid = threadIdx.x;
    unsigned long long* ls = (unsigned long long*)lds;           // [K][pitch]
    uint32_t* lc = (uint32_t*)(ls + (size_t)K * pitch);          // [K] members so far
    uint32_t* cnt = lc + K;                                      // [256] members in the chunk, then their places
    uint32_t* wsum = cnt + 256;                                  // [4] wave totals of the scan
    int* match = (int*)(wsum + 4);                               // [kAccThreads]: streams of a window using book b
    int* n_match = match + kAccThreads;
    uint16_t* order = (uint16_t*)(n_match + 1);                  // [kChunk] the chunk's positions by cluster
    for (int i = tid; i < K * pitch; i += kAccThreads) ls[i] = 0;
    for (int i = tid; i < K; i += kAccThreads) lc[i] = 0;
    const int n_groups = kAccThreads / nch, group = tid / nch, ch = tid - group * nch;
    const float inv_Ta = 1.0f / (float)Ta;
    // The streams are scanned kAccThreads at a time, one per thread, and those
    // of book b listed in LDS (their order does not matter: integer sums).
    for (int64_t s0 = 0; s0 < n_streams; s0 += kAccThreads) {
        if (tid == 0) *n_match = 0;
        __syncthreads();
        if (s0 + tid < n_streams && stream_book[s0 + tid] == b) match[atomicAdd(n_match, 1)] = tid;
        __syncthreads();
        const int64_t total = (int64_t)*n_match * Ta;   // the window's member tokens, stream by stream
        for (int64_t c0 = 0; c0 < total; c0 += kChunk) {
            const int n = (int)min((int64_t)kChunk, total - c0);
            const int m0 = (int)(c0 / Ta), r0 = (int)(c0 - (int64_t)m0 * Ta);
            // position `rel` of the chunk: its stream and token (u + 1/2 is at
            // least 1/(2 Ta) off every quotient's edge, far over the rounding)
            auto locate = [&](int rel, int64_t& s, int64_t& t) {
                const uint32_t u = (uint32_t)r0 + (uint32_t)rel;   // Ta < 2^31
                const uint32_t q = Ta >= kChunk ? (u >= (uint32_t)Ta) : (uint32_t)(((float)u + 0.5f) * inv_Ta);
                s = s0 + match[m0 + (int)q];
                t = u - q * (uint32_t)Ta;
            };
            if (tid < 256) cnt[tid] = 0;
            __syncthreads();
            int place[kChunk / kAccThreads];   // cluster and rank within it; -1: past the end, or skipped
#pragma unroll
            for (int i = 0; i < kChunk / kAccThreads; ++i) {
                const int rel = i * kAccThreads + tid;
                place[i] = -1;
                if (rel < n) {
                    int64_t s, t;
                    locate(rel, s, t);
                    const uint8_t* sym = symbols + (s * Ta + t) * S;
                    bool bad = false;
                    int cl = 0;
                    for (int st = 0; st <= stage; ++st) {
                        cl = sym[st];
                        bad = bad || cl >= K;   // outside the book: skipped
                    }
                    if (!bad) place[i] = cl << 16 | (int)atomicAdd(cnt + cl, 1u);
                }
            }
            __syncthreads();
            // exclusive prefix sums of the cluster sizes
            uint32_t own = 0, inc = 0;
            if (tid < 256) {
                own = inc = cnt[tid];
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t v = __shfl_up(inc, o);
                    if ((tid & 63) >= o) inc += v;
                }
                if ((tid & 63) == 63) wsum[tid >> 6] = inc;
                if (tid < K) lc[tid] += own;
            }
            __syncthreads();
            if (tid < 256) {
                for (int w = 0; w < (tid >> 6); ++w) inc += wsum[w];
                cnt[tid] = inc - own;
            }
            const int nv = (int)(wsum[0] + wsum[1] + wsum[2] + wsum[3]);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < kChunk / kAccThreads; ++i)
                if (place[i] >= 0) order[cnt[place[i] >> 16] + (place[i] & 0xffff)] = (uint16_t)(i * kAccThreads + tid);
            __syncthreads();

            const int per = (nv + n_groups - 1) / n_groups;
            const int p0 = min(nv, group * per), p1 = group < n_groups ? min(nv, p0 + per) : 0;
            int cur = -1;
            bool again = false;   // a run was left out because its sum is not finite
            double acc[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = 0.0;
            auto flush = [&] {
                if (cur < 0) return;
                unsigned long long* dst = ls + (size_t)cur * pitch + ch * 8;
                // to units of 2^-24: |acc| 2^24 < 2^51, so adding 3 * 2^51 leaves the
                // integer in the low mantissa bits, exactly, under the exponent of 2^52
                // (all ones if acc is not finite)
                long long m[8];
                uint32_t top = 0;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    m[e] = __double_as_longlong(__builtin_fma(acc[e], 0x1p24, 0x1.8p52));
                    top = max(top, (uint32_t)(m[e] >> 32));
                }
                if (top >= 0x7FF00000u) {
                    again = true;
                    return;
                }
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    atomicAdd(dst + e, (unsigned long long)(m[e] - __double_as_longlong(0x1.8p52)));
            };
            for (int p = p0; p < p1; p += B) {
                int64_t row[B];     // token row of x
                const uint8_t* sym[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    int64_t s, t;
                    locate(order[min(p + u, p1 - 1)], s, t);
                    row[u] = s * T + t_begin + t;
                    sym[u] = symbols + (s * Ta + t) * S;
                }
                half8 xv[B];
#pragma unroll
                for (int u = 0; u < B; ++u) xv[u] = *(const half8*)(x + row[u] * d + e0 + ch * 8);
                uint64_t sy[B];     // the token's symbols of stages 0..stage, one byte each
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    sy[u] = 0;
                    for (int st = 0; st <= stage; ++st) sy[u] |= (uint64_t)sym[u][st] << (8 * st);
                }
                double r[B][8];
#pragma unroll
                for (int u = 0; u < B; ++u)
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[u][e] = (double)xv[u][e];
#pragma unroll
                for (int st = 0; st < stage; ++st) {
                    half8 c[B];
#pragma unroll
                    for (int u = 0; u < B; ++u)
                        c[u] = *(const half8*)(books + (((int64_t)b * S + st) * K + (int)((sy[u] >> (8 * st)) & 255u)) * d +
                                               e0 + ch * 8);
#pragma unroll
                    for (int u = 0; u < B; ++u)
#pragma unroll
                        for (int e = 0; e < 8; ++e) r[u][e] = r[u][e] - (double)c[u][e];
                }
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (p + u >= p1) continue;
                    const int cl = (int)((sy[u] >> (8 * stage)) & 255u);
                    if (cl != cur) {
                        flush();
                        cur = cl;
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] = r[u][e];
                    } else {
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] = acc[e] + r[u][e];
                    }
                }
            }
            flush();
            if (again) {
                // the runs that hold a NaN or an infinity, token by token
                auto cluster = [&](int q) {
                    int64_t s, t;
                    locate(order[q], s, t);
                    return (int)symbols[(s * Ta + t) * S + stage];
                };
                auto element = [&](int q, int e) {
                    int64_t s, t;
                    locate(order[q], s, t);
                    const uint8_t* sym = symbols + (s * Ta + t) * S;
                    double r = (double)x[(s * T + t_begin + t) * d + e0 + ch * 8 + e];
#pragma unroll 1
                    for (int st = 0; st < stage; ++st)
                        r = r - (double)books[(((int64_t)b * S + st) * K + sym[st]) * d + e0 + ch * 8 + e];
                    return r;
                };
                int end;
#pragma unroll 1
                for (int p = p0; p < p1; p = end) {
                    const int cl = cluster(p);
                    bool finite = true;
#pragma unroll 1
                    for (end = p; end < p1 && cluster(end) == cl; ++end)
#pragma unroll 1
                        for (int e = 0; e < 8; ++e) finite = finite && __builtin_isfinite(element(end, e));
                    if (finite) continue;   // counted already
#pragma unroll 1
                    for (int i = 0; i < 8 * (end - p); ++i)
                        atomicAdd(ls + (size_t)cl * pitch + ch * 8 + (i & 7), fixed24(element(p + (i >> 3), i & 7)));
                }
            }
            __syncthreads();   // the chunk's order and counts are consumed
        }
        __syncthreads();   // the list is rewritten for the next window
    }
    for (int i = tid; i < K * dc; i += kAccThreads) {
        const int j = i / dc, e = i - j * dc;
        const unsigned long long v = ls[j * pitch + e];
        if (v) sums[((int64_t)b * K + j) * d + e0 + e] += v;
    }
    if (slice == 0)
        for (int j = tid; j < K; j += kAccThreads)
            if (lc[j]) counts[(int64_t)b * K + j] += lc[j];
}

// The same without the sort: stream by stream, each lane adds its eight elements
// of every member token to LDS with 64-bit atomics.
template <int ST>
__global__ __launch_bounds__(kAccThreads) void kmeans_direct_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ books, const int32_t* __restrict__ stream_book,
    const uint8_t* __restrict__ symbols, unsigned long long* __restrict__ sums, uint32_t* __restrict__ counts,
    int64_t n_streams, int64_t T, int64_t t_begin, int64_t Ta, int d, int S, int K, int stage_rt)
{
    const int stage = ST >= 0 ? ST : stage_rt;
    extern __shared__ __align__(16) uint8_t lds[];
    const int n_slices = (d + kSlice - 1) / kSlice;
    const int b = blockIdx.x / n_slices, slice = blockIdx.x - b * n_slices;
    const int e0 = slice * kSlice, dc = min(kSlice, d - e0);   // this block's dimensions [e0, e0 + dc)
    const int nch = dc / 8;
    const int pitch = dc + 1;                                    // words per cluster row
    unsigned long long* ls = (unsigned long long*)lds;           // [K][pitch]
    uint32_t* lc = (uint32_t*)(ls + (size_t)K * pitch);          // [K]
    int* match = (int*)(lc + K);                                 // [kAccThreads]: streams of a chunk using book b
    int* n_match = match + kAccThreads;
    for (int i = threadIdx.x; i < K * pitch; i += kAccThreads) ls[i] = 0;
    for (int i = threadIdx.x; i < K; i += kAccThreads) lc[i] = 0;
    // The streams are scanned kAccThreads at a time, one per thread, and those
    // of book b listed in LDS (their order does not matter: integer sums).
    for (int64_t s0 = 0; s0 < n_streams; s0 += kAccThreads) {
        if (threadIdx.x == 0) *n_match = 0;
        __syncthreads();
        if (s0 + threadIdx.x < n_streams && stream_book[s0 + threadIdx.x] == b)
            match[atomicAdd(n_match, 1)] = (int)threadIdx.x;
        __syncthreads();
        const int nm = *n_match;
        for (int m = 0; m < nm; ++m) {
            const int64_t s = s0 + match[m];
            // 32-bit task walk (the host checks that Ta * nch fits).  Each thread
            // takes kAccBatch tasks at a time and issues all their loads before
            // any sum, so the latencies of the batch overlap.
            const int n_task = (int)(Ta * nch);
            for (int task0 = threadIdx.x; task0 < n_task; task0 += kAccThreads * kAccBatch) {
                int cl[kAccBatch];          // cluster of each task, -1: none (past the end, or skipped)
                int64_t row[kAccBatch];     // token row of x
                const uint8_t* sym[kAccBatch];
                int chn[kAccBatch];
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u) {
                    const int task = task0 + u * kAccThreads;
                    const int t = task / nch;
                    chn[u] = task - t * nch;
                    sym[u] = symbols + (s * Ta + (task < n_task ? t : 0)) * S;
                    row[u] = s * T + t_begin + (task < n_task ? t : 0);
                    cl[u] = task < n_task ? 0 : -1;
                }
                uint64_t sy[kAccBatch];     // the task's symbols of stages 0..stage, one byte each
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u) {
                    sy[u] = 0;
                    for (int st = 0; st <= stage; ++st) sy[u] |= (uint64_t)sym[u][st] << (8 * st);
                }
                half8 xv[kAccBatch];
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u) xv[u] = *(const half8*)(x + row[u] * d + e0 + chn[u] * 8);
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u) {
                    bool bad = cl[u] < 0;
                    for (int st = 0; st <= stage; ++st) bad = bad || (int)((sy[u] >> (8 * st)) & 255u) >= K;
                    cl[u] = bad ? -1 : (int)((sy[u] >> (8 * stage)) & 255u);   // outside the book: skipped
                }
                double r[kAccBatch][8];
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u)
#pragma unroll
                    for (int e = 0; e < 8; ++e) r[u][e] = (double)xv[u][e];
#pragma unroll
                for (int st = 0; st < stage; ++st) {
                    half8 c[kAccBatch];
#pragma unroll
                    for (int u = 0; u < kAccBatch; ++u)
                        c[u] = *(const half8*)(books +
                                               (((int64_t)b * S + st) * K + (cl[u] < 0 ? 0 : (int)((sy[u] >> (8 * st)) & 255u))) * d +
                                               e0 + chn[u] * 8);
#pragma unroll
                    for (int u = 0; u < kAccBatch; ++u)
#pragma unroll
                        for (int e = 0; e < 8; ++e) r[u][e] = r[u][e] - (double)c[u][e];
                }
#pragma unroll
                for (int u = 0; u < kAccBatch; ++u) {
                    if (cl[u] < 0) continue;
                    unsigned long long* dst = ls + (size_t)cl[u] * pitch + chn[u] * 8;
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        atomicAdd(dst + e, (unsigned long long)(long long)ldexp(r[u][e], 24));   // NaN and infinities as fixed24
                    if (chn[u] == 0 && slice == 0) atomicAdd(lc + cl[u], 1u);
                }
            }
        }
        __syncthreads();   // the list is rewritten for the next chunk
    }
    for (int i = threadIdx.x; i < K * dc; i += kAccThreads) {
        const int j = i / dc, e = i - j * dc;
        const unsigned long long v = ls[j * pitch + e];
        if (v) sums[((int64_t)b * K + j) * d + e0 + e] += v;
    }
    if (slice == 0)
        for (int j = threadIdx.x; j < K; j += kAccThreads)
            if (lc[j]) counts[(int64_t)b * K + j] += lc[j];
}

__global__ __launch_bounds__(kThreads) void kmeans_finalize_kernel(
    const unsigned long long* __restrict__ sums, const uint32_t* __restrict__ counts, _Float16* __restrict__ books,
    int d, int S, int K, int stage, int64_t n_elems)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n_elems; i += (int64_t)gridDim.x * kThreads) {
        const int64_t bj = i / d;   // book * K + j
        const int e = (int)(i - bj * d);
        const uint32_t c = counts[bj];
        if (c == 0) continue;
        const int64_t b = bj / K, j = bj - b * K;
        const double m = ldexp((double)(long long)sums[i] / (double)c, -24);
        books[((b * S + stage) * K + j) * d + e] = f64_to_f16(m);
    }
}

int64_t grid_for(int64_t n)
{
    const int64_t b = (n + kThreads - 1) / kThreads;
    return b < 1 ? 1 : (b > 4096 ? 4096 : b);
}

// Zero fill of n 8-byte words (the scratch sums and counts before an update;
// a kernel rather than a memset so that the call can be captured in a graph).
__global__ __launch_bounds__(kThreads) void zero_words_kernel(unsigned long long* __restrict__ p, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) p[i] = 0;
}

// Device scratch of the allocation-free k-means update: the cluster sums
// (int64, [n_books][K][d]) followed by the counts (u32, [n_books][K]).  Each
// device the library runs on holds its own copy until the process ends.  In
// host code this name is not a device address: kernels get the per-device
// address taken once with hipGetSymbolAddress.
static __device__ __align__(256) unsigned long long scratch[FKV_NOALLOC_SCRATCH_BYTES / 8];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];

// Address of the current device's scratch array (taken once per device);
// nullptr when the device is unknown or the runtime refuses.
void* scratch_address()
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        g_scratch_ptr[dev] = p;
    }
    return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace fkv

using namespace fkv;

extern "C" int fkv_kmeans_accumulate(const fkv_rvq_desc* desc, const uint16_t* x_f16, const uint16_t* books_f16,
                                     const int32_t* stream_book, const uint8_t* symbols, int32_t stage,
                                     int64_t* sums, uint32_t* counts, void* stream)
{
    if (!desc) return FKV_ERR_INVALID_ARG;
    const fkv_rvq_desc& D = *desc;
    if (D.n_streams < 0 || D.T < 0 || D.t_begin < 0 || D.t_end < D.t_begin || D.t_end > D.T) return FKV_ERR_INVALID_ARG;
    if (D.d < 8 || D.d > 256 || D.d % 8 != 0 || D.S < 1 || D.S > 8 || D.K < 1 || D.K > 256 || D.n_books < 1)
        return FKV_ERR_INVALID_ARG;
    if (stage < 0 || stage >= D.S) return FKV_ERR_INVALID_ARG;
    const int64_t Ta = D.t_end - D.t_begin;
    if (D.n_streams == 0 || Ta == 0) return FKV_OK;
    if (!x_f16 || !books_f16 || !stream_book || !symbols || !sums || !counts) return FKV_ERR_INVALID_ARG;
    if (!aligned(x_f16, 16) || !aligned(books_f16, 16) || !aligned(sums, 8) || !aligned(counts, 4) ||
        !aligned(stream_book, 4))
        return FKV_ERR_INVALID_ARG;
    const int n_slices = (D.d + kSlice - 1) / kSlice;
    if (Ta * (std::min(kSlice, (int)D.d) / 8) > 0x7fffffff - kAccThreads * kAccBatch) return FKV_ERR_UNSUPPORTED;
    auto lds_bytes = [](int K, int dc, bool sort) {
        return (size_t)K * (dc + 1) * 8 + (size_t)K * 4 + (kAccThreads + 1) * 4 + (sort ? (256 + 4) * 4 + kChunk * 2 : 0);
    };
    const int dc = std::min(kSlice, (int)D.d);
    // The sort costs a chunk about 5 us of barriers, which few tokens do not repay,
    // and the direct form pays 1.3 us per stream of a book.  A narrow row takes few
    // lanes, so the atomics it saves are few, and two direct blocks fit a compute
    // unit; at stage 0, whose registers allow it too, so they do for up to 150
    // codewords.  Measured, direct and sorted (us): one stream per book, K = 256: d = 64,
    // 16 tokens 12.2 and 17.1, 300 tokens 25.5 and 30.0, 2500 tokens 68.1 and 58.3;
    // d = 8, 4000 tokens 19.4 and 31.0; d = 48, 20,000 tokens in two streams 273 and
    // 321.  200 books of 64 x 256: 4 streams of 64 tokens 18.7 and 19.0, 32 streams
    // of 64 tokens 71.8 and 55.5.  Stage 0, 288 books of 64 x 128: 950 tokens 26.5 and 31.0,
    // 2500 52.3 and 46.5; of 256 x 100 (1152 blocks): 2500 122 and 142, 4000 183 and 195.
    const bool few = D.n_streams < 4 * (int64_t)D.n_books, narrow = D.d <= 24 || (D.d < 56 && D.n_books > 256);
    const int64_t blocks = (int64_t)D.n_books * n_slices;
    const bool pairs = stage == 0 && blocks > 256 && 2 * lds_bytes(D.K, dc, false) <= 160 * 1024;
    const int paired = (1000 + 10 * (int)D.K) * (blocks > 1024 || dc < kSlice ? 2 : 1);
    const int64_t repays = std::max(pairs ? paired : 900, 8 * (int)D.K);
    const bool sort = narrow ? !few && Ta < 1024 : !few || D.n_streams * Ta >= D.n_books * repays;
    const size_t shm = lds_bytes(D.K, dc, sort);
    static std::once_flag once[12];   // one per kernel instance below
    auto go = [&](int slot, auto kern) {
        std::call_once(once[slot], [&] {
            (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds_bytes(256, kSlice, slot < 6));
        });
        (void)hipGetLastError();
        hipLaunchKernelGGL(kern, dim3((unsigned)(D.n_books * n_slices)), dim3(kAccThreads), shm, (hipStream_t)stream,
                           (const _Float16*)x_f16, (const _Float16*)books_f16, stream_book, symbols,
                           (unsigned long long*)sums, counts, D.n_streams, D.T, D.t_begin, Ta, D.d, D.S, D.K, stage);
        return launch_status();
    };
    auto pick = [&](int slot, auto st) {
        constexpr int ST = decltype(st)::value;
        return sort ? go(slot, kmeans_accumulate_kernel<ST>) : go(6 + slot, kmeans_direct_kernel<ST>);
    };
    switch (stage) {
    case 0: return pick(0, std::integral_constant<int, 0>{});
    case 1: return pick(1, std::integral_constant<int, 1>{});
    case 2: return pick(2, std::integral_constant<int, 2>{});
    case 3: return pick(3, std::integral_constant<int, 3>{});
    case 4: return pick(4, std::integral_constant<int, 4>{});
    default: return pick(5, std::integral_constant<int, -1>{});
    }
}

extern "C" int fkv_kmeans_finalize(int32_t n_books, int32_t S, int32_t K, int32_t d, int32_t stage,
                                   const int64_t* sums, const uint32_t* counts, uint16_t* books_f16, void* stream)
{
    if (n_books < 1 || S < 1 || S > 8 || K < 1 || K > 256 || d < 8 || d > 256 || d % 8 != 0) return FKV_ERR_INVALID_ARG;
    if (stage < 0 || stage >= S || !sums || !counts || !books_f16) return FKV_ERR_INVALID_ARG;
    if (!aligned(sums, 8) || !aligned(counts, 4) || !aligned(books_f16, 2)) return FKV_ERR_INVALID_ARG;
    const int64_t n_elems = (int64_t)n_books * K * d;
    hipLaunchKernelGGL(kmeans_finalize_kernel, dim3((unsigned)grid_for(n_elems)), dim3(kThreads), 0,
                       (hipStream_t)stream, (const unsigned long long*)sums, counts, (_Float16*)books_f16, d, S, K,
                       stage, n_elems);
    return launch_status();
}

extern "C" size_t fkv_kmeans_update_noalloc_bytes(int32_t n_books, int32_t K, int32_t d)
{
    if (n_books < 1 || K < 1 || d < 1) return 0;
    return (size_t)n_books * K * d * 8 + (size_t)n_books * K * 4;
}

extern "C" int fkv_kmeans_update_noalloc(const fkv_rvq_desc* desc, const uint16_t* x_f16, uint16_t* books_f16,
                                         const int32_t* stream_book, const uint8_t* symbols, int32_t stage,
                                         uint32_t* counts_out, void* stream)
{
    if (!desc) return FKV_ERR_INVALID_ARG;
    const fkv_rvq_desc& D = *desc;
    if (D.n_streams < 0 || D.T < 0 || D.t_begin < 0 || D.t_end < D.t_begin || D.t_end > D.T) return FKV_ERR_INVALID_ARG;
    if (D.d < 8 || D.d > 256 || D.d % 8 != 0 || D.S < 1 || D.S > 8 || D.K < 1 || D.K > 256 || D.n_books < 1)
        return FKV_ERR_INVALID_ARG;
    if (stage < 0 || stage >= D.S) return FKV_ERR_INVALID_ARG;
    if (!x_f16 || !books_f16 || !stream_book || !symbols) return FKV_ERR_INVALID_ARG;
    if (!aligned(x_f16, 16) || !aligned(books_f16, 16) || !aligned(stream_book, 4) ||
        (counts_out && !aligned(counts_out, 4)))
        return FKV_ERR_INVALID_ARG;
    const size_t need = fkv_kmeans_update_noalloc_bytes(D.n_books, D.K, D.d);
    if (need > (size_t)FKV_NOALLOC_SCRATCH_BYTES) return FKV_ERR_SCRATCH_TOO_SMALL;
    const int64_t Ta = D.t_end - D.t_begin;
    if (Ta * (std::min(kSlice, (int)D.d) / 8) > 0x7fffffff - kAccThreads * kAccBatch) return FKV_ERR_UNSUPPORTED;
    void* base = scratch_address();
    if (!base) return FKV_ERR_NO_DEVICE;
    const hipStream_t st = (hipStream_t)stream;
    unsigned long long* sums = (unsigned long long*)base;
    const int64_t n_sum = (int64_t)D.n_books * D.K * D.d;
    uint32_t* counts = (uint32_t*)(sums + n_sum);
    // the previous call's contents are cleared first: sums and counts start at zero
    const int64_t n_words = (int64_t)((need + 7) / 8);
    hipLaunchKernelGGL(zero_words_kernel, dim3((unsigned)grid_for(n_words)), dim3(kThreads), 0, st, sums, n_words);
    int rc = launch_status();
    if (rc != FKV_OK) return rc;
    if (D.n_streams > 0 && Ta > 0) {
        rc = fkv_kmeans_accumulate(desc, x_f16, books_f16, stream_book, symbols, stage, (int64_t*)sums, counts,
                                   stream);
        if (rc != FKV_OK) return rc;
    }
    rc = fkv_kmeans_finalize(D.n_books, D.S, D.K, D.d, stage, (const int64_t*)sums, counts, books_f16, stream);
    if (rc != FKV_OK) return rc;
    if (counts_out) {
        if (hipMemcpyAsync(counts_out, counts, (size_t)D.n_books * D.K * 4, hipMemcpyDeviceToDevice, st) != hipSuccess) {
            (void)hipGetLastError();
            return FKV_ERR_LAUNCH;
        }
    }
    return FKV_OK;
}
