// rvq_kernels.hip -- per-head residual vector quantization (assignment) on
// gfx950 matrix cores.
//
// Method (Sec. 3 "Setup" of the paper): an archived K or V head vector x is
// stored as S codebook indices whose centroids sum to its reconstruction.
// Greedy residual VQ: r_0 = x; for stage s, i_s = argmin_j ||r_s - C_s[j]||^2
// (lowest j on exact ties), then r_{s+1} = r_s - C_s[i_s].
//
// Formulation.  For a token with residual r and stage codebook C:
//     u_j = r.c_j - ||c_j||^2/2 - b  =  -||r - c_j||^2/2 - (b - ||r||^2/2),
// with a per-token bias b >= ||r||^2/2, so every u_j is a negative float whose
// magnitude orders like the squared distance.  All of u_j comes out of the
// matrix cores (v_mfma_f32_32x32x16_f16, codebook = A operand from LDS,
// 32 tokens = B operand in registers):
//   * one "bias step" per 32x32 tile: A row i = (-||c_i||^2/2 split exactly
//     into three fp16 parts, 1, 2^14), B column j = (1, 1, 1, b_j parts), so
//     the tile starts at -||c_i||^2/2 - b_j.  b only has to be an upper bound
//     of ||r||^2/2 (it shifts every score of a token equally), so it is
//     rounded up into fp16 freely;
//   * the d/16 data steps add r.c_i.
// In the 32x32 accumulator layout lane l owns token l%32 and 16 of the tile's
// 32 codewords, so the argmin is in-lane: a negative float's bits, read as an
// unsigned integer, grow with its magnitude; with the low 5 bits replaced by
// the codeword's position among the 32 that the lane holds in a pair of
// consecutive tiles, they form a key whose minimum (v_min3_u32) is the
// nearest codeword and carries its index.  Dropping 5 mantissa bits coarsens
// the comparison to 2^-18 relative, inside the 1e-5 near-tie band.  Tile pairs
// merge on the value bits (earlier pair wins ties), then lane l with lane
// l^32.  Stage s's bias is the winning |u| of stage s-1 (||r_s||^2/2 plus the
// previous margin), grown by 2^-10.
//
// Exact operands.  Stage 0 multiplies fp16 x by fp16 codewords (every product
// exact in fp32).  Stage 1 uses r_1 = x - c_0 as two fp16 passes, x.c and
// (-c_0).c, both exact.  From stage 2 on the residual is carried as an fp16
// pair hi + lo (about 22 bits, rebuilt in fp32 and split again after every
// stage) and both halves go through the matrix cores.
//
// Codebooks.  Each stage's codebook is copied global -> LDS with the
// asynchronous global_load_lds_dwordx4 into two alternating buffers, so the
// next stage's book streams in while the current one is in use (one buffer
// where two or three blocks share a compute unit and cover each other's copies).  An LDS row
// holds a codeword's 16-byte chunks followed by its bias-step chunk; the odd
// chunk count per row spreads the 32 rows of an A fragment over distinct banks.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <mutex>

#include "fkv.h"
#include "fkv_hip_common.h"
#include "fkv_internal.h"

namespace fkv {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kLdsBudget = 160 * 1024;
constexpr float kBiasHiScale = 16384.0f;   // weight of the bias's second fp16 slot
constexpr int kItemTokens = 256;           // tokens per block of the staged kernels
constexpr int kMaxGroup = 256;             // streams per group in the grouped form (<= threads per block)

// One LDS book buffer: Kp rows of row_p bytes, then a 16-byte zero pad.
__host__ __device__ constexpr size_t buf_bytes_of(int row_p, int Kp)
{
    return (size_t)Kp * row_p + 16;
}

template <int D>
struct Shape {
    static constexpr int KS = D / 16;                    // 16-deep matrix steps along d
    static constexpr int NCH = D / 8;                    // 16-byte chunks of a codeword
    // LDS row: the codeword's NCH chunks, then its bias-step A chunk.  The odd
    // number of 16-byte chunks per row puts any 16 consecutive rows on 16
    // distinct bank groups, so fragment reads are conflict-free without a
    // swizzle and a lane's fragments sit at fixed offsets from one base.
    static constexpr int ROW_P = (NCH + 1) * 16;
    static constexpr int TILE_P = 32 * ROW_P;            // one 32-codeword tile
};

// Block shapes.  The narrow one (four waves of two token tiles, two blocks per
// compute unit, three at d <= 64) serves large launches: a fragment read from
// LDS feeds two token tiles, and while one block waits for its rows or the next
// book the other has the matrix cores.  The wide one (eight waves of one token
// tile, one block per compute unit, two book buffers) serves d > 128, where two
// token tiles do not fit the registers, and launches of at most one block per
// compute unit, where twice the waves share a block's 256 tokens.
// Measured, wide and narrow, 256-token items (us): d = 128, S = 3, K = 256:
// 2^18 items 22.0-22.9 and 20.0-20.4 ms (602 -> 650 TFLOP/s); 2048 items 182
// and 160, 384 items 44.9 and 40.8, 256 items 26.4 and 27.5, 64 items 19.6 and
// 22.4.  d = 80, S = 3, K = 100: 512 items 21.9 and 19.0, 256 items 9.9 and 11.7.
// One 8-wave block of two token tiles per compute unit (512 tokens a book pass)
// instead of two 4-wave blocks: 22.2 ms, its waves wait at the same barriers.
template <int D, bool WIDE>
struct Cfg : Shape<D> {
    using Shape<D>::ROW_P;
    static constexpr int TT = WIDE ? 1 : 2;              // 32-token tiles per wave
    static constexpr int WAVES = WIDE ? 8 : 4;
    static constexpr int THREADS = 64 * WAVES;
    static_assert(WAVES * TT * 32 == kItemTokens, "a block takes one item");
    static constexpr int BLOCKS = WIDE ? 1 : D <= 64 ? 3 : 2;   // resident blocks per compute unit
    // two book buffers when two full (K = 256) books fit, else one
    static constexpr int NBUF = BLOCKS * 2 * buf_bytes_of(ROW_P, 256) <= kLdsBudget ? 2 : 1;
};

template <int D, bool WIDE>
size_t lds_bytes(int Kp)
{
    return (size_t)Cfg<D, WIDE>::NBUF * buf_bytes_of(Cfg<D, WIDE>::ROW_P, Kp);
}

// Asynchronously copies stage codebook C ([K][D] fp16) into an LDS buffer of
// Kp rows.  Each 64-lane copy fills 64 consecutive 16-byte LDS chunks; a
// row's bias-step slot gets a placeholder (its last data chunk) that
// book_bias_rows overwrites, and rows >= K are copies of row K-1, so they tie
// with it and lose to its lower index.
template <int D, int WAVES>
__device__ __forceinline__ void book_to_lds_async(const _Float16* __restrict__ C, int K, int Kp,
                                                  uint8_t* buf, int wave, int lane)
{
    constexpr int NCH = Shape<D>::NCH, CH = NCH + 1, STEP = WAVES * 64;
    const int chunks = Kp * CH;   // a multiple of 64 (Kp is)
    for (int q0 = __builtin_amdgcn_readfirstlane(wave) * 64; q0 < chunks; q0 += STEP) {
        const uint32_t q = (uint32_t)(q0 + lane);
        const uint32_t row = q / CH, slot = q - row * CH;
        const uint32_t off = min(row, (uint32_t)K - 1) * D + min(slot, (uint32_t)NCH - 1) * 8;
        const _Float16* src = C + off;
        __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                         (void __attribute__((address_space(3)))*)(buf + (size_t)q0 * 16),
                                         16, 0, 0);
    }
}

// Bias-step A chunk of a codeword with squared norm `acc`: (-||c||^2/2 as hi +
// mid + lo fp16 parts, 1, 2^14, 0, 0, 0).
__device__ __forceinline__ half8 bias_row(float acc)
{
    const float n = -0.5f * acc;
    const _Float16 hi = (_Float16)n;
    const float rem = n - (float)hi;
    const _Float16 mid = (_Float16)rem;
    const _Float16 lo = (_Float16)(rem - (float)mid);
    half8 a = (half8)(_Float16)0;
    a[0] = hi;
    a[1] = mid;
    a[2] = lo;
    a[3] = (_Float16)1.0f;
    a[4] = (_Float16)kBiasHiScale;
    return a;
}

// The bias-step A chunk of every row of NB buffers, written into the row's last slot.  All rows'
// LDS reads are issued before any norm is formed, so their latencies overlap.
template <int D, int THREADS, int NB>
__device__ __forceinline__ void book_bias_rows(uint8_t* buf0, uint8_t* buf1, int Kp)
{
    constexpr int NCH = Shape<D>::NCH;
    for (int r = threadIdx.x; r < Kp; r += THREADS) {
        uint8_t* row[2] = {buf0 + (size_t)r * Shape<D>::ROW_P, buf1 + (size_t)r * Shape<D>::ROW_P};
        half8 v[NB][NCH];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int p = 0; p < NCH; ++p) v[b][p] = *(const half8*)(row[b] + p * 16);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            float acc = 0.0f;
#pragma unroll
            for (int p = 0; p < NCH; ++p) {
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2 h = {v[b][p][e], v[b][p][e + 1]};
                    acc = __builtin_amdgcn_fdot2(h, h, acc, false);
                }
            }
            *(half8*)(row[b] + NCH * 16) = bias_row(acc);
        }
    }
}

// The value lane l ^ 32 holds (hh: this lane's half-wave).
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v, int hh)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return hh ? r[0] : r[1];
}

// Bias-step B column of a token: slots 0-2 multiply the norm parts (1, 1, 1),
// slots 3-4 hold -b rounded up in magnitude, b <= 32768 in slot 3 directly,
// larger b in slot 4 in units of 2^14.  Lanes holding k = 8..15 give zeros.
__device__ __forceinline__ half8 bias_column(float b, int hh)
{
    half8 v = (half8)(_Float16)0;
    if (hh == 0) {
        const float bu = fmaxf(b * (1.0f + 0x1p-9f), 0x1p-24f);
        v[0] = v[1] = v[2] = (_Float16)1.0f;
        if (bu <= 32768.0f)
            v[3] = (_Float16)(-bu);
        else
            v[4] = (_Float16)(-fminf(bu * (1.0f / kBiasHiScale), 65504.0f));
    }
    return v;
}

__device__ __forceinline__ void wait_all_and_sync()
{
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}

// A-operand fragments of one 32-codeword tile: its d/16 data steps and the
// bias step.
template <int D>
struct Frag {
    half8 a[Shape<D>::KS];
    half8 bias;
};

// A lane's fragments of tile ct start at buf + base + ct * TILE_P, with
// base = col * ROW_P + 16 hh: data step ks at +32 ks, the bias chunk at
// +16 NCH.  For the upper half-wave (k = 8..15 of the bias step) that chunk is
// the next row's first chunk or the buffer's zero pad: finite values that
// meet the zero half of the token's bias column.
template <int D>
__device__ __forceinline__ void load_frag(Frag<D>& f, const uint8_t* buf, uint32_t base, int ct)
{
    const uint8_t* tile = buf + base + (size_t)ct * Shape<D>::TILE_P;
#pragma unroll
    for (int ks = 0; ks < Shape<D>::KS; ++ks) f.a[ks] = *(const half8*)(tile + ks * 32);
    f.bias = *(const half8*)(tile + Shape<D>::NCH * 16);
}

// acc = bias step + A(tile) x B over all k-steps; with TWO a second B operand
// accumulates into the same tile.
template <int D, bool TWO>
__device__ __forceinline__ void issue_tile(const Frag<D>& f, const half8& bz, const half8 (&bA)[Shape<D>::KS],
                                           const half8 (&bB)[Shape<D>::KS], floatx16& acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.bias, bz, (floatx16)0.0f, 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < Shape<D>::KS; ++ks) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[ks], bA[ks], acc, 0, 0, 0);
        if (TWO) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[ks], bB[ks], acc, 0, 0, 0);
    }
}

// Minimum over a lane's 16 scores of (float bits with the low 5 bits replaced
// by base + register index), as a tree of three-input minima.
template <uint32_t BASE>
__device__ __forceinline__ uint32_t tile_min_key(const floatx16& a)
{
    uint32_t k[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) k[v] = (__float_as_uint(a[v]) & ~31u) | (BASE + (uint32_t)v);
    const uint32_t m0 = min(min(k[0], k[1]), k[2]);
    const uint32_t m1 = min(min(k[3], k[4]), k[5]);
    const uint32_t m2 = min(min(k[6], k[7]), k[8]);
    const uint32_t m3 = min(min(k[9], k[10]), k[11]);
    const uint32_t m4 = min(min(k[12], k[13]), k[14]);
    const uint32_t m5 = min(min(m0, m1), m2);
    const uint32_t m6 = min(min(m3, m4), k[15]);
    return min(m5, m6);
}

// Adds the scores of the second tile of pair `pair` (positions 16..31) to the key
// minimum pk of its first tile (positions 0..15) and folds the pair into the
// running best; an earlier pair wins ties on the value bits.
__device__ __forceinline__ void pair_second(const floatx16& acc, uint32_t pk, int pair, uint32_t& bkey, int& bpair)
{
    const uint32_t k = min(pk, tile_min_key<16>(acc));
    if ((k & ~31u) < (bkey & ~31u)) {
        bkey = k;
        bpair = pair;
    }
}

// Instruction-interleaving hints for one pipelined step: every MFMA of the tile
// being issued is followed by a few VALU ops of the previous tile's argmin and,
// early on, the LDS reads of the next tile's fragments, so one wave keeps its
// matrix core busy while its vector ALU and LDS work proceed.
template <int NMFMA, int NVALU, int NDS, int GAP>
__device__ __forceinline__ void interleave_hint()
{
    constexpr int per = (NVALU + NMFMA - 1) / NMFMA;
#pragma unroll
    for (int i = 0; i < NMFMA; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);      // one MFMA
        if (i % GAP == 0 && i / GAP < NDS) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
        __builtin_amdgcn_sched_group_barrier(0x002, per, 0);    // a few VALU
    }
}

// One stage's scores over all nct (even) codeword tiles, software-pipelined:
// the fragments of tile ct+2 load and the MFMAs of tile ct+1 run while the
// argmin of tile ct executes on the VALU.  Tiles 2p and 2p+1 form pair p.
template <int D, bool TWO>
__device__ __forceinline__ void stage_scan(const uint8_t* buf, uint32_t fa, int nct, const half8& bz,
                                           const half8 (&bA)[Shape<D>::KS], const half8 (&bB)[Shape<D>::KS],
                                           uint32_t& bkey, int& bpair)
{
    constexpr int NM = 1 + Shape<D>::KS * (TWO ? 2 : 1);   // MFMAs per tile
    constexpr int NV = 26;                                 // VALU ops of one tile's argmin
    constexpr int ND = Shape<D>::KS + 1;                   // LDS reads of one tile's fragments
    Frag<D> f0, f1;
    floatx16 acc0, acc1;
    uint32_t pk;
    load_frag<D>(f0, buf, fa, 0);
    load_frag<D>(f1, buf, fa, 1);
    issue_tile<D, TWO>(f0, bz, bA, bB, acc0);
    int ct = 0;
    for (; ct + 2 < nct; ct += 2) {
        issue_tile<D, TWO>(f1, bz, bA, bB, acc1);
        load_frag<D>(f0, buf, fa, ct + 2);
        pk = tile_min_key<0>(acc0);
        interleave_hint<NM, NV, ND, 1>();
        issue_tile<D, TWO>(f0, bz, bA, bB, acc0);
        load_frag<D>(f1, buf, fa, min(ct + 3, nct - 1));
        pair_second(acc1, pk, ct >> 1, bkey, bpair);
        interleave_hint<NM, NV, ND, 1>();
    }
    issue_tile<D, TWO>(f1, bz, bA, bB, acc1);
    pk = tile_min_key<0>(acc0);
    pair_second(acc1, pk, ct >> 1, bkey, bpair);
}

// One stage's scores for two token tiles with one fragment buffer and one
// accumulator per token tile: while token tile 1 takes codeword tile ct, token
// tile 0's scores of it are reduced and each fragment, used for the last time,
// is replaced by the next codeword tile's; then token tile 0 takes that one
// while token tile 1 is reduced.  Half the LDS reads of two one-tile scans, and
// 196 registers at d = 128 beside the keys, so that two waves fit a SIMD.
template <int D, bool TWO>
__device__ __forceinline__ void stage_scan_two(const uint8_t* buf, uint32_t fa, int nct, const half8 (&bz)[2],
                                               const half8 (&bA)[2][Shape<D>::KS], const half8 (&bB)[2][Shape<D>::KS],
                                               uint32_t (&bkey)[2], int (&bpair)[2])
{
    constexpr int NM = 1 + Shape<D>::KS * (TWO ? 2 : 1);   // MFMAs per codeword tile and token tile
    constexpr int ND = Shape<D>::KS + 1;                   // LDS reads of one tile's fragments
    constexpr int GAP = TWO ? 2 : 1;                       // MFMAs per fragment
    Frag<D> f;
    floatx16 a0, a1;
    uint32_t pk[2];
    auto issue0 = [&] { issue_tile<D, TWO>(f, bz[0], bA[0], bB[0], a0); };
    auto issue1 = [&] { issue_tile<D, TWO>(f, bz[1], bA[1], bB[1], a1); };
    auto first = [&](int tt, const floatx16& a) { pk[tt] = tile_min_key<0>(a); };
    auto second = [&](int tt, const floatx16& a, int pair) {
        pair_second(a, pk[tt], pair, bkey[tt], bpair[tt]);
    };
    load_frag<D>(f, buf, fa, 0);
    issue0();
    int ct = 0;
    for (; ct + 2 < nct; ct += 2) {
        issue1();
        load_frag<D>(f, buf, fa, ct + 1);
        first(0, a0);
        interleave_hint<NM, 26, ND, GAP>();
        issue0();
        first(1, a1);
        interleave_hint<NM, 26, 0, 1>();
        issue1();
        load_frag<D>(f, buf, fa, ct + 2);
        second(0, a0, ct >> 1);
        interleave_hint<NM, 30, ND, GAP>();
        issue0();
        second(1, a1, ct >> 1);
        interleave_hint<NM, 30, 0, 1>();
    }
    issue1();
    load_frag<D>(f, buf, fa, ct + 1);
    first(0, a0);
    interleave_hint<NM, 26, ND, GAP>();
    issue0();
    first(1, a1);
    interleave_hint<NM, 26, 0, 1>();
    issue1();
    second(0, a0, ct >> 1);
    second(1, a1, ct >> 1);
}

// Re-split of a residual pair: for the two fp16 lanes q of the words a (hi),
// b (lo) and c (chosen codeword), rv = (a + b) - c in fp32 (each operation
// rounded once, as written), then hi' = fp16(rv) and lo' = fp16(rv - hi'),
// with the mixed-precision FMAs (fp16 operands read from either half of a
// word, fp32 arithmetic, an fp16 result written into one half).
__device__ __forceinline__ void resplit2(uint32_t a, uint32_t b, uint32_t c, uint32_t& na, uint32_t& nb)
{
    float t0, t1, r0, r1;
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,1]" : "=v"(t0) : "v"(a), "v"(b));
    asm("v_fma_mix_f32 %0, %1, 1.0, %2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(t1) : "v"(a), "v"(b));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=v"(r0) : "v"(c), "v"(t0));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r1) : "v"(c), "v"(t1));
    uint32_t h, l;
    asm("v_fma_mixlo_f16 %0, %1, 1.0, 0 op_sel_hi:[0,0,0]" : "=&v"(h) : "v"(r0));
    asm("v_fma_mixhi_f16 %0, %1, 1.0, 0 op_sel_hi:[0,0,0]" : "+v"(h) : "v"(r1));
    asm("v_fma_mixlo_f16 %0, %1, -1.0, %2 op_sel:[0,0,0] op_sel_hi:[1,0,0]" : "=&v"(l) : "v"(h), "v"(r0));
    asm("v_fma_mixhi_f16 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(l) : "v"(h), "v"(r1));
    na = h;
    nb = l;
}

// GRP: a work item is a group of G streams that share one book (groups[g * G
// + e] is member e of group g) and its tokens are the members' archived
// tokens, member by member, so that one block serves all of them with a single
// copy of the book (the per-token arithmetic is that of the per-stream form).
// PERS: a block takes ipb consecutive work items (token ranges, mostly of one
// stream) and loads the next item's token rows into registers during the current
// item's last stage, so a new item does not start by waiting on HBM.
template <int D, bool WIDE, bool ENC, bool GRP, bool PERS>
__global__ __launch_bounds__((Cfg<D, WIDE>::THREADS), (Cfg<D, WIDE>::BLOCKS)) void rvq_assign_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ books,
    const int32_t* __restrict__ stream_book, uint8_t* __restrict__ symbols,
    float* __restrict__ residual, uint32_t* __restrict__ n_bad, int64_t T, int64_t t_begin,
    int64_t Ta, int S, int NS, int K, int Kp, int n_books, int64_t blocks_per_stream, int64_t tpb,
    double2* __restrict__ points, const double2* __restrict__ vtab, double cr, int cN, int cL, int64_t n_spans,
    const int32_t* __restrict__ groups, int G, int64_t n_streams, int64_t ipb, int64_t n_items)
{
    static_assert(!(GRP && ENC), "the grouped form has no fused encode");
    using C = Cfg<D, WIDE>;
    constexpr int KS = C::KS, TT = C::TT, NBUF = C::NBUF;
    extern __shared__ __align__(16) uint8_t lds[];
    // LDS: NBUF buffers of Kp rows (codeword + bias-step chunk) and a zero
    // pad; addressed from `lds` so every access stays an LDS access.
    const size_t buf_bytes = buf_bytes_of(C::ROW_P, Kp);

    // XCD-aware order: blocks dispatched to one XCD (every 8th) take consecutive
    // work items, so the blocks of one stream share that XCD's L2 copy of its book.
    const uint32_t nblk = gridDim.x, q8 = nblk / 8, r8 = nblk % 8;
    const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int64_t bidx = (int64_t)xcd * q8 + min(xcd, r8) + slot;
    const int64_t it0 = PERS ? bidx * ipb : bidx;
    const int64_t it1 = PERS ? min(it0 + ipb, n_items) : it0 + 1;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, hh = lane >> 5;
    half8 bN[TT][KS];   // PERS: the next item's token rows
    bool have_next = false;
    for (int64_t item = it0; item < it1; ++item) {
        const int64_t s = item / blocks_per_stream;                // the stream (GRP: the group)
        const int64_t Tv = GRP ? (int64_t)G * Ta : Ta;             // the item's tokens
        const int64_t tb = (item - s * blocks_per_stream) * tpb;   // first token of the block
        const int64_t te = min(Tv, tb + tpb);                      // one past its last

        uint8_t* sym_s = symbols + s * Ta * S;
        int b = GRP ? -1 : stream_book[s];

        // this lane's tokens (independent of the book id, so their loads overlap its)
        int64_t tok[TT];
        bool valid[TT];
        int64_t srow[TT];               // GRP: the token's row in the [n_streams][Ta] outputs
        half8 bA[TT][KS], bB[TT][KS];   // B operands of the current stage's passes
        half8 bz[TT];                   // bias-step B operand
        const bool prefetched = PERS && have_next;
        have_next = false;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            tok[tt] = tb + (int64_t)(wave * TT + tt) * 32 + col;
            valid[tt] = tok[tt] < te;
            int64_t xr;
            if constexpr (GRP) {
                // member e's token t; a member id out of range rejects the group
                // below, and meanwhile reads stream 0
                const int64_t tv = valid[tt] ? tok[tt] : tb;
                const int64_t e = tv / Ta, t = tv - e * Ta;
                const int64_t m = groups[s * G + e];
                const int64_t mm = (m >= 0 && m < n_streams) ? m : 0;
                srow[tt] = mm * Ta + t;
                xr = mm * T + t_begin + t;
            } else {
                srow[tt] = 0;
                xr = s * T + t_begin + (valid[tt] ? tok[tt] : 0);
            }
            const _Float16* row = x + xr * D + 8 * hh;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (prefetched)
                    bA[tt][ks] = bN[tt][ks];
                else
                    bA[tt][ks] = valid[tt] ? *(const half8*)(row + 16 * ks) : (half8)(_Float16)0;
                bB[tt][ks] = (half8)(_Float16)0;
            }
        }
        if constexpr (GRP) {
            // the group's book: its first member's, which every member must share
            const int32_t m0 = groups[s * G];
            const int gb = (m0 >= 0 && m0 < n_streams) ? stream_book[m0] : -1;
            int bad = gb < 0 || gb >= n_books;
            if (tid < G) {
                const int32_t m = groups[s * G + tid];
                bad |= m < 0 || m >= n_streams || stream_book[m] != gb;
            }
            b = __syncthreads_or(bad) ? -1 : gb;
        }

        if (b < 0 || b >= n_books) {
            if constexpr (GRP) {
                // every in-range member's symbols (and residual) of the block's tokens
                for (int64_t i = tb * S + tid; i < te * S; i += C::THREADS) {
                    const int64_t j = i / S, e = j / Ta, m = groups[s * G + e];
                    if (m >= 0 && m < n_streams) symbols[(m * Ta + (j - e * Ta)) * S + (i - j * S)] = 0xFF;
                }
                if (residual)
                    for (int64_t i = tb * D + tid; i < te * D; i += C::THREADS) {
                        const int64_t j = i / D, e = j / Ta, m = groups[s * G + e];
                        if (m >= 0 && m < n_streams) residual[(m * Ta + (j - e * Ta)) * D + (i - j * D)] = NAN;
                    }
                if (tid == 0 && tb == 0 && n_bad) atomicAdd(n_bad, 1u);
                return;
            }
            for (int64_t i = tb * S + tid; i < te * S; i += C::THREADS) sym_s[i] = 0xFF;
            if (ENC)   // the block's spans encode 0xFF symbols: NaN points, as a separate encode gives
                for (int64_t j = tb * S / cL + tid; j < (te * S + cL - 1) / cL; j += C::THREADS)
                    points[s * n_spans + j] = make_double2(NAN, NAN);
            if (residual)
                for (int64_t i = tb * D + tid; i < te * D; i += C::THREADS) residual[s * Ta * D + i] = NAN;
            if (tid == 0 && tb == 0 && n_bad) atomicAdd(n_bad, 1u);
            continue;
        }
        const _Float16* bk = books + (int64_t)b * S * K * D;

        // Fused span encode: the vertex table (NaN beyond the alphabet) and the
        // block's symbols live after the book buffers.
        double2* V_l = (double2*)(lds + NBUF * buf_bytes);
        uint8_t* sym_l = (uint8_t*)(V_l + 256);
        if (ENC && tid < 256) V_l[tid] = tid < cN ? vtab[tid] : make_double2(NAN, NAN);

        // start the first books' copies; zero the buffers' end pads
        book_to_lds_async<D, C::WAVES>(bk, K, Kp, lds, wave, lane);
        if (NBUF > 1 && NS > 1) book_to_lds_async<D, C::WAVES>(bk + (size_t)K * D, K, Kp, lds + buf_bytes, wave, lane);
        if (tid < NBUF) *(half8*)(lds + tid * buf_bytes + (size_t)Kp * C::ROW_P) = (half8)(_Float16)0;

#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            float n2 = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2 h = {bA[tt][ks][e], bA[tt][ks][e + 1]};
                    n2 = __builtin_amdgcn_fdot2(h, h, n2, false);
                }
            }
            n2 += __uint_as_float(lane_xor32(__float_as_uint(n2), hh));
            bz[tt] = bias_column(0.5f * n2 * (1.0f + 0x1p-10f), hh);
        }
        const uint32_t fa = (uint32_t)(col * C::ROW_P + hh * 16);

        wait_all_and_sync();
        if (NBUF > 1 && NS > 1)
            book_bias_rows<D, C::THREADS, 2>(lds, lds + buf_bytes, Kp);
        else
            book_bias_rows<D, C::THREADS, 1>(lds, lds, Kp);
        __syncthreads();

        const int nct = Kp / 32;  // even
        // GRP: a wave without tokens (short items, such as one token per member)
        // skips the scans and only takes part in the book pipeline
        const bool wave_on = !GRP || __builtin_amdgcn_readfirstlane((int)(tb + (int64_t)wave * TT * 32 < te));
        // One stage: TWO (stages 1..) scans with two passes per tile.  Stage 0 is
        // issued on its own, ahead of the loop over the later stages: with one
        // loop body holding both scan forms the register allocator kept both
        // forms' values live across the loop and spilled (d = 128, three stages,
        // wide shape: 256 VGPRs and 32 bytes of scratch per lane, against 188 and
        // none; the narrow shape holds 256 and 16-24 bytes, outside its scan).
        auto stage = [&](const int st, auto two_c) {
            constexpr bool TWO = decltype(two_c)::value;
            if (PERS && st + 1 == NS && item + 1 < it1) {
                // the next item's token rows, in flight during this stage
                const int64_t sn = (item + 1) / blocks_per_stream;
                const int64_t tbn = (item + 1 - sn * blocks_per_stream) * tpb;
                const int64_t ten = min(Ta, tbn + tpb);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const int64_t tk = tbn + (int64_t)(wave * TT + tt) * 32 + col;
                    const bool v = tk < ten;
                    const _Float16* row = x + (sn * T + t_begin + (v ? tk : 0)) * D + 8 * hh;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
                        bN[tt][ks] = v ? *(const half8*)(row + 16 * ks) : (half8)(_Float16)0;
                }
                have_next = true;
            }
            const int cur = NBUF > 1 ? (st & 1) : 0;
            const uint8_t* buf = lds + cur * buf_bytes;
            uint32_t bkey[TT];
            int bpair[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                bkey[tt] = 0xFFFFFFFFu;
                bpair[tt] = 0;
            }
            if (wave_on) {
                if constexpr (TT == 2)
                    stage_scan_two<D, TWO>(buf, fa, nct, bz, bA, bB, bkey, bpair);
                else
                    stage_scan<D, TWO>(buf, fa, nct, bz[0], bA[0], bB[0], bkey[0], bpair[0]);
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const int li = (int)(bkey[tt] & 31u);
                    int cw = (2 * bpair[tt] + (li >> 4)) * 32 + 8 * ((li & 15) >> 2) + 4 * hh + (li & 3);
                    cw = min(cw, K - 1);  // only reachable with all-NaN scores; keeps reads in bounds
                    uint32_t val = bkey[tt] & ~31u;
                    const uint32_t oval = lane_xor32(val, hh);
                    const int ocw = (int)lane_xor32((uint32_t)cw, hh);
                    if (oval < val || (oval == val && ocw < cw)) {
                        val = oval;
                        cw = ocw;
                    }
                    if (hh == 0 && valid[tt]) {
                        if (GRP)
                            symbols[srow[tt] * S + st] = (uint8_t)cw;
                        else
                            sym_s[tok[tt] * S + st] = (uint8_t)cw;
                        if (ENC) sym_l[(tok[tt] - tb) * S + st] = (uint8_t)cw;
                    }
                    // next stage's bias: this stage's winning |u| grown by 2^-10
                    bz[tt] = bias_column(-__uint_as_float(val) * (1.0f + 0x1p-10f), hh);
                    // this lane's chunks of the chosen codeword
                    half8 cv[KS];
                    const uint8_t* crow = buf + (size_t)cw * C::ROW_P + hh * 16;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) cv[ks] = *(const half8*)(crow + ks * 32);
                    const bool last = st + 1 == NS;
                    if (TWO && !last) {
                        // r = (hi + lo) - c for st >= 2, (x - c_0) - c_1 for st == 1; split again
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                            const u32x4 a = __builtin_bit_cast(u32x4, bA[tt][ks]), b = __builtin_bit_cast(u32x4, bB[tt][ks]),
                                        c = __builtin_bit_cast(u32x4, cv[ks]);
                            u32x4 na, nb;
#pragma unroll
                            for (int w = 0; w < 4; ++w) {
                                uint32_t x, y;
                                resplit2(a[w], b[w], c[w], x, y);
                                na[w] = x;
                                nb[w] = y;
                            }
                            bA[tt][ks] = __builtin_bit_cast(half8, na);
                            bB[tt][ks] = __builtin_bit_cast(half8, nb);
                        }
                    }
                    if (last && residual && valid[tt]) {
                        float* out = residual + (GRP ? srow[tt] : s * Ta + tok[tt]) * D + 8 * hh;
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            floatx4 lo4, hi4;
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float rv = (float)bA[tt][ks][e] + (TWO ? (float)bB[tt][ks][e] : 0.0f) -
                                                 (float)cv[ks][e];
                                if (e < 4) lo4[e] = rv; else hi4[e - 4] = rv;
                            }
                            *(floatx4*)(out + 16 * ks) = lo4;
                            *(floatx4*)(out + 16 * ks + 4) = hi4;
                        }
                    }
                    if (!TWO && !last) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) bB[tt][ks] = -cv[ks];
                    }
                }
            }   // wave_on
            if (st + 1 < NS && (NBUF == 1 || st >= 1 || st + 2 < NS)) {
                // Book pipeline: buffer `cur` is free once every wave is past here.
                wait_all_and_sync();
                if (NBUF == 1) {
                    book_to_lds_async<D, C::WAVES>(bk + (size_t)(st + 1) * K * D, K, Kp, lds, wave, lane);
                    wait_all_and_sync();
                } else if (st + 2 < NS) {
                    book_to_lds_async<D, C::WAVES>(bk + (size_t)(st + 2) * K * D, K, Kp, lds + cur * buf_bytes, wave, lane);
                }
                if (NBUF == 1 || st >= 1) {
                    uint8_t* nb = lds + (NBUF > 1 ? ((st + 1) & 1) : 0) * buf_bytes;
                    book_bias_rows<D, C::THREADS, 1>(nb, nb, Kp);
                }
                __syncthreads();
            }
        };
        stage(0, std::false_type{});
        for (int st = 1; st < NS; ++st) stage(st, std::true_type{});
        if (ENC) {
            // Span encode of the block's symbols (Sec. 1 "The code"): the block's
            // token range holds whole spans, each walked from the anchor (0,0) with
            // p <- V + r (p - V), operation for operation as the encode kernel, and
            // stored with a streaming store (measured: faster on the four-stage
            // d = 64 shape, neutral elsewhere; slower in the small-book kernel).
            __syncthreads();
            const int64_t n_sym = Ta * S;
            for (int64_t j = tb * S / cL + tid; j < (te * S + cL - 1) / cL; j += C::THREADS) {
                const int64_t a = j * cL;
                const int len = (int)min((int64_t)cL, n_sym - a);
                const uint8_t* my = sym_l + (a - tb * S);
                double px = 0.0, py = 0.0;
                for (int k0 = 0; k0 < len; k0 += 8) {
                    // the vertices of up to 8 symbols first (they do not depend on p),
                    // then the dependent steps
                    double2 v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = k0 + u < len ? V_l[my[k0 + u]] : make_double2(0.0, 0.0);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        if (k0 + u < len) {
                            const double tx = px - v[u].x, ty = py - v[u].y;
                            const double ux = cr * tx, uy = cr * ty;
                            px = v[u].x + ux;
                            py = v[u].y + uy;
                        }
                    }
                }
                store_point_stream(points + s * n_spans + j, px, py);
            }
        }
        if (item + 1 < it1) __syncthreads();   // the next item's book copies overwrite the buffers
    }
}

// LDS after the book buffers for the fused span encode: 256 vertices and the
// block's symbols.
constexpr size_t enc_lds_bytes()
{
    return 256 * 16 + (size_t)kItemTokens * 8;
}

// ---- small books: at most 64 codewords and two stages (d <= 64) ----------
// Every stage's book then fits in LDS for the whole block, so one block walks
// several token items of one stream: the books are copied and their norms
// formed once, no barrier separates the stages or the items, and the next
// item's token rows load while the current item is assigned.  The block's
// symbols are staged in LDS and its spans encoded once, after its last item.
constexpr int kSmallK = 64;
constexpr int kSmallBlocks = 3;     // resident blocks per compute unit
constexpr int kSmallMaxItems = 8;   // token items per block (bounds the symbol staging)

// One stage over the two codeword tiles of a small book with a single
// fragment buffer.
template <int D, bool TWO>
__device__ __forceinline__ void stage_scan_small(const uint8_t* buf, uint32_t fa, const half8& bz,
                                                 const half8 (&bA)[Shape<D>::KS], const half8 (&bB)[Shape<D>::KS],
                                                 uint32_t& bkey, int& bpair)
{
    Frag<D> f;
    floatx16 acc0, acc1;
    load_frag<D>(f, buf, fa, 0);
    issue_tile<D, TWO>(f, bz, bA, bB, acc0);
    load_frag<D>(f, buf, fa, 1);
    issue_tile<D, TWO>(f, bz, bA, bB, acc1);
    const uint32_t pk = tile_min_key<0>(acc0);
    pair_second(acc1, pk, 0, bkey, bpair);
}

// A block barrier that orders LDS only: each wave's LDS operations complete
// before it, while its global loads (the next item's token rows) and stores
// stay in flight (__syncthreads also waits for those).
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int D>
__device__ __forceinline__ void load_rows(half8 (&dst)[Shape<D>::KS], const _Float16* __restrict__ x, int64_t row,
                                          bool valid, int hh)
{
    const _Float16* p = x + row * D + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < Shape<D>::KS; ++ks) dst[ks] = valid ? *(const half8*)(p + 16 * ks) : (half8)(_Float16)0;
}

template <int D, bool ENC>
__global__ __launch_bounds__((Cfg<D, false>::THREADS), kSmallBlocks) void rvq_small_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ books, const int32_t* __restrict__ stream_book,
    uint8_t* __restrict__ symbols, float* __restrict__ residual, uint32_t* __restrict__ n_bad, int64_t T,
    int64_t t_begin, int64_t Ta, int S, int NS, int K, int Kp, int n_books, int64_t blocks_per_stream, int64_t tpi,
    int64_t ipb, double2* __restrict__ points, const double2* __restrict__ vtab, double cr, int cN, int cL,
    int64_t n_spans)
{
    using C = Cfg<D, false>;
    constexpr int KS = C::KS, TOK = C::WAVES * 32;
    extern __shared__ __align__(16) uint8_t lds[];
    const size_t buf_bytes = buf_bytes_of(C::ROW_P, Kp);

    // XCD-aware order, as in rvq_assign_kernel
    const uint32_t nblk = gridDim.x, q8 = nblk / 8, r8 = nblk % 8;
    const uint32_t xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int64_t item = (int64_t)xcd * q8 + min(xcd, r8) + slot;
    const int64_t s = item / blocks_per_stream;
    const int64_t tb0 = (item - s * blocks_per_stream) * ipb * tpi;   // the block's first token
    const int64_t te0 = min(Ta, tb0 + ipb * tpi);                      // one past its last

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int col = lane & 31, hh = lane >> 5;
    uint8_t* sym_s = symbols + s * Ta * S;
    const int b = stream_book[s];
    const _Float16* xs = x + (s * T + t_begin) * D;

    half8 bA[1][KS];   // token rows of the block's first item
    load_rows<D>(bA[0], xs, tb0 + wave * 32 + col, tb0 + wave * 32 + col < min(te0, tb0 + tpi), hh);

    if (b < 0 || b >= n_books) {
        for (int64_t i = tb0 * S + tid; i < te0 * S; i += C::THREADS) sym_s[i] = 0xFF;
        if (ENC)
            for (int64_t j = tb0 * S / cL + tid; j < (te0 * S + cL - 1) / cL; j += C::THREADS)
                points[s * n_spans + j] = make_double2(NAN, NAN);
        if (residual)
            for (int64_t i = tb0 * D + tid; i < te0 * D; i += C::THREADS) residual[s * Ta * D + i] = NAN;
        if (tid == 0 && tb0 == 0 && n_bad) atomicAdd(n_bad, 1u);
        return;
    }
    const _Float16* bk = books + (int64_t)b * S * K * D;

    double2* V_l = (double2*)(lds + 2 * buf_bytes);
    uint8_t* sym_l = (uint8_t*)(V_l + 256);   // the block's symbols, token-major from tb0
    if (ENC && tid < 256) V_l[tid] = tid < cN ? vtab[tid] : make_double2(NAN, NAN);
    book_to_lds_async<D, C::WAVES>(bk, K, Kp, lds, wave, lane);
    if (NS > 1) book_to_lds_async<D, C::WAVES>(bk + (size_t)K * D, K, Kp, lds + buf_bytes, wave, lane);
    if (tid < 2) *(half8*)(lds + tid * buf_bytes + (size_t)Kp * C::ROW_P) = (half8)(_Float16)0;
    wait_all_and_sync();
    if (NS > 1)
        book_bias_rows<D, C::THREADS, 2>(lds, lds + buf_bytes, Kp);
    else
        book_bias_rows<D, C::THREADS, 1>(lds, lds, Kp);
    __syncthreads();

    const uint32_t fa = (uint32_t)(col * C::ROW_P + hh * 16);
    // One token item on rows `cur`; the next item's rows load into `nxt`
    // (the two register sets alternate, so the load is first waited for when
    // the next item starts).
    auto run_item = [&](int64_t tb, half8 (&cur)[1][KS], half8 (&nxt)[1][KS]) {
        const int64_t te = min(te0, tb + tpi);
        const int64_t tok = tb + wave * 32 + col;
        const bool valid = tok < te;
        const int64_t tbn = tb + tpi;
        if (tbn < te0) load_rows<D>(nxt[0], xs, tbn + wave * 32 + col, tbn + wave * 32 + col < min(te0, tbn + tpi), hh);

        half8 bz[1], bB[1][KS];
        float n2 = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bB[0][ks] = (half8)(_Float16)0;
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                const half2 h = {cur[0][ks][e], cur[0][ks][e + 1]};
                n2 = __builtin_amdgcn_fdot2(h, h, n2, false);
            }
        }
        n2 += __uint_as_float(lane_xor32(__float_as_uint(n2), hh));
        bz[0] = bias_column(0.5f * n2 * (1.0f + 0x1p-10f), hh);

        // stage 0, then stage 1 (as in rvq_assign_kernel: one body per scan form)
        auto stage = [&](const int st, auto two_c) {
            constexpr bool TWO = decltype(two_c)::value;
            const uint8_t* buf = lds + st * buf_bytes;
            uint32_t bkey[1] = {0xFFFFFFFFu};
            int bpair[1] = {0};
            stage_scan_small<D, TWO>(buf, fa, bz[0], cur[0], bB[0], bkey[0], bpair[0]);
            const int li = (int)(bkey[0] & 31u);
            int cw = (li >> 4) * 32 + 8 * ((li & 15) >> 2) + 4 * hh + (li & 3);
            cw = min(cw, K - 1);  // only reachable with all-NaN scores; keeps reads in bounds
            uint32_t val = bkey[0] & ~31u;
            const uint32_t oval = lane_xor32(val, hh);
            const int ocw = (int)lane_xor32((uint32_t)cw, hh);
            if (oval < val || (oval == val && ocw < cw)) {
                val = oval;
                cw = ocw;
            }
            if (hh == 0 && valid) {
                sym_s[tok * S + st] = (uint8_t)cw;
                if (ENC) sym_l[(tok - tb0) * S + st] = (uint8_t)cw;
            }
            bz[0] = bias_column(-__uint_as_float(val) * (1.0f + 0x1p-10f), hh);
            half8 cv[KS];
            const uint8_t* crow = buf + (size_t)cw * C::ROW_P + hh * 16;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) cv[ks] = *(const half8*)(crow + ks * 32);
            const bool last = st + 1 == NS;
            if (last && residual && valid) {
                float* out = residual + (s * Ta + tok) * D + 8 * hh;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    floatx4 lo4, hi4;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float rv = (float)cur[0][ks][e] + (TWO ? (float)bB[0][ks][e] : 0.0f) -
                                         (float)cv[ks][e];
                        if (e < 4) lo4[e] = rv; else hi4[e - 4] = rv;
                    }
                    *(floatx4*)(out + 16 * ks) = lo4;
                    *(floatx4*)(out + 16 * ks + 4) = hi4;
                }
            }
            if (!TWO && !last) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) bB[0][ks] = -cv[ks];
            }
        };
        stage(0, std::false_type{});
        if (NS > 1) stage(1, std::true_type{});
    };
    half8 rB[1][KS];
    for (int64_t tb = tb0; tb < te0; tb += 2 * tpi) {
        run_item(tb, bA, rB);
        if (tb + tpi < te0) run_item(tb + tpi, rB, bA);
    }
    if (ENC) {
        // the block's token range holds whole spans (tpi is a multiple of
        // L / gcd(L, S)), each walked from the anchor (0,0) with
        // p <- V + r (p - V), operation for operation as the encode kernel
        lds_barrier();
        const int64_t n_sym = Ta * S;
        for (int64_t j = tb0 * S / cL + tid; j < (te0 * S + cL - 1) / cL; j += C::THREADS) {
            const int64_t a = j * cL;
            const int len = (int)min((int64_t)cL, n_sym - a);
            const uint8_t* my = sym_l + (a - tb0 * S);
            double px = 0.0, py = 0.0;
            for (int k0 = 0; k0 < len; k0 += 8) {
                double2 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = k0 + u < len ? V_l[my[k0 + u]] : make_double2(0.0, 0.0);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    if (k0 + u < len) {
                        const double tx = px - v[u].x, ty = py - v[u].y;
                        const double ux = cr * tx, uy = cr * ty;
                        px = v[u].x + ux;
                        py = v[u].y + uy;
                    }
                }
            }
            points[s * n_spans + j] = make_double2(px, py);
        }
    }
}

// ---- few tokens per book: at most 32 per work item --------------------------
// A decoding step's eviction assigns one token per stream (per group of streams
// sharing a book: a few).  Its work is reading the books once (100 MB for 512
// books of 3 x 256 x 128), so nothing is staged: wave w owns codeword tile w of
// every stage, loads its A fragments straight from global memory into
// registers, forms the tile's norms there, and the block's waves meet only to
// compare their best codewords and to pass the chosen rows on.  The token rows
// and their residual parts live in LDS.  Two 8-wave blocks (three at d <= 64)
// fit a compute unit, so their loads and scans overlap; the staged form runs
// one block per compute unit, which waits on three 64 KB copies for the scan of
// a single wave.  512 books of 3 x 256 x 128, four tokens each: 36.0 -> 21.4 us
// (2.8 -> 4.7 TB/s of books); 576 of 4 x 256 x 64: 39.5 -> 23 us.  Counters of the
// first case: vector ALU 42% busy, matrix cores 13%, LDS 13%, the L1 0.6 tag
// lookups per busy cycle (32-byte pieces of 32 rows per load), a quarter of the
// waves' cycles waiting; a stage's loads are issued only after the compare of the
// stage before.  The grouped instances keep 12-40 bytes of scratch at d <= 64 and
// 24 at d = 128.  Slower: the next stage's fragments in registers too (more scratch,
// or one block per compute unit: 29-60 us), its lines touched ahead (34 us).
// Scores, keys, biases and residual splits are rvq_assign_kernel's, operation
// for operation, and the winner is the lowest (score key, codeword) there too.
constexpr int kFewTokens = 32;

template <int D>
struct FewLds {
    static constexpr int PITCH = (D / 8 + 1) * 16;   // bytes per token row: odd number of 16-byte chunks
    alignas(16) uint8_t hi[kFewTokens * PITCH];
    uint8_t lo[kFewTokens * PITCH], chosen[kFewTokens * PITCH];
    uint64_t best[8][kFewTokens];                    // each wave's best (score key, codeword) per token
};

template <int D, bool GRP>
__global__ __launch_bounds__(512, D <= 64 ? 6 : D <= 128 ? 4 : 2) void rvq_few_kernel(
    const _Float16* __restrict__ x, const _Float16* __restrict__ books, const int32_t* __restrict__ stream_book,
    uint8_t* __restrict__ symbols, float* __restrict__ residual, uint32_t* __restrict__ n_bad, int64_t T,
    int64_t t_begin, int64_t Ta, int S, int NS, int K, int n_books, const int32_t* __restrict__ groups, int G,
    int64_t n_streams, int64_t n_items)
{
    constexpr int KS = D / 16, NCH = D / 8, PITCH = FewLds<D>::PITCH;
    __shared__ FewLds<D> l;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, hh = lane >> 5, n_waves = blockDim.x >> 6;
    const int nt = (int)(GRP ? G * Ta : Ta);   // <= kFewTokens
    for (int64_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        // token i of the item: member stream and position, output row
        auto token = [&](int i, int64_t& xr, int64_t& orow) {
            const int e = GRP ? i / (int)Ta : 0, t = GRP ? i - e * (int)Ta : i;
            const int64_t m = GRP ? (int64_t)groups[item * G + e] : item;
            const bool in = m >= 0 && m < n_streams;
            xr = (in ? m : 0) * T + t_begin + t;
            orow = in ? m * Ta + t : -1;
        };
        int b;
        if constexpr (GRP) {
            const int32_t m0 = groups[item * G];
            const int gb = (m0 >= 0 && m0 < n_streams) ? stream_book[m0] : -1;
            int bad = gb < 0 || gb >= n_books;
            if (tid < G) {
                const int32_t m = groups[item * G + tid];
                bad |= m < 0 || m >= n_streams || stream_book[m] != gb;
            }
            b = __syncthreads_or(bad) ? -1 : gb;
        } else {
            b = stream_book[item];
            if (b < 0 || b >= n_books) b = -1;
            __syncthreads();   // the previous item's rows are consumed
        }
        if (b < 0) {
            for (int i = tid; i < nt * S; i += blockDim.x) {
                int64_t xr, orow;
                token(i / S, xr, orow);
                if (orow >= 0) symbols[orow * S + i % S] = 0xFF;
            }
            if (residual)
                for (int i = tid; i < nt * D; i += blockDim.x) {
                    int64_t xr, orow;
                    token(i / D, xr, orow);
                    if (orow >= 0) residual[orow * D + i % D] = NAN;
                }
            if (tid == 0 && n_bad) atomicAdd(n_bad, 1u);
            continue;
        }
        const _Float16* bk = books + (int64_t)b * S * K * D;

        // rows >= K read row K - 1: they tie with it and give its index
        const _Float16* my_row = bk + (int64_t)min(32 * wave + col, K - 1) * D + 8 * hh;
        half8 f[KS];
        auto load_frags = [&](int st) {
            const _Float16* p = my_row + (int64_t)st * K * D;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) f[ks] = *(const half8*)(p + 16 * ks);
        };
        load_frags(0);
        for (int i = tid; i < kFewTokens * NCH; i += blockDim.x) {
            const int t = i / NCH, c = i - t * NCH;
            half8 v = (half8)(_Float16)0;
            if (t < nt) {
                int64_t xr, orow;
                token(t, xr, orow);
                v = *(const half8*)(x + xr * D + 8 * c);
            }
            *(half8*)(l.hi + t * PITCH + 16 * c) = v;
            *(half8*)(l.lo + t * PITCH + 16 * c) = (half8)(_Float16)0;
        }
        // this lane's token: member stream and position
        const int my_e = GRP ? min(col, nt - 1) / (int)Ta : 0, my_t = min(col, nt - 1) - my_e * (int)Ta;
        const int64_t my_m = GRP ? (int64_t)groups[item * G + my_e] : item;
        __syncthreads();

        const uint8_t* hi_l = l.hi + col * PITCH + 16 * hh;
        const uint8_t* lo_l = l.lo + col * PITCH + 16 * hh;
        float bias;
        {
            float n2 = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const half8 v = *(const half8*)(hi_l + 32 * ks);
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2 h = {v[e], v[e + 1]};
                    n2 = __builtin_amdgcn_fdot2(h, h, n2, false);
                }
            }
            n2 += __uint_as_float(lane_xor32(__float_as_uint(n2), hh));
            bias = 0.5f * n2 * (1.0f + 0x1p-10f);
        }

        for (int st = 0; st < NS; ++st) {
            const bool last = st + 1 == NS;
            // bias-step fragment: the row's norm summed chunk by chunk in order
            // (each half-wave holds every second chunk; the swap gives both
            // halves the even and the odd one)
            half8 fb = (half8)(_Float16)0;
            {
                typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                float acc = 0.0f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const u32x4 own = __builtin_bit_cast(u32x4, f[ks]);
                    uint32_t odd[4];
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const auto r = __builtin_amdgcn_permlane32_swap(own[w], own[w], false, false);
                        const uint32_t even = r[0];
                        odd[w] = r[1];
                        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2, even), __builtin_bit_cast(half2, even),
                                                     acc, false);
                    }
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(half2, odd[w]), __builtin_bit_cast(half2, odd[w]),
                                                     acc, false);
                }
                const half8 a = bias_row(acc);
                if (hh == 0) fb = a;
            }
            const half8 bz = bias_column(bias, hh);
            floatx16 acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(fb, bz, (floatx16)0.0f, 0, 0, 0);
            if (st == 0) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[ks], *(const half8*)(hi_l + 32 * ks), acc, 0, 0, 0);
            } else {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[ks], *(const half8*)(hi_l + 32 * ks), acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(f[ks], *(const half8*)(lo_l + 32 * ks), acc, 0, 0, 0);
                }
            }
            const uint32_t key = tile_min_key<0>(acc);
            const int li = (int)(key & 31u);
            uint32_t cw = min((uint32_t)(32 * wave + 8 * (li >> 2) + 4 * hh + (li & 3)), (uint32_t)K - 1);
            uint32_t val = key & ~31u;
            {
                const uint32_t oval = lane_xor32(val, hh), ocw = lane_xor32(cw, hh);
                if (oval < val || (oval == val && ocw < cw)) {
                    val = oval;
                    cw = ocw;
                }
            }
            if (hh == 0) l.best[wave][col] = (uint64_t)val << 32 | cw;
            __syncthreads();
            uint64_t best = l.best[0][col];
            for (int w = 1; w < n_waves; ++w) best = min(best, l.best[w][col]);
            cw = (uint32_t)best;
            bias = -__uint_as_float((uint32_t)(best >> 32)) * (1.0f + 0x1p-10f);
            if (wave == 0 && hh == 0 && col < nt) symbols[(my_m * Ta + my_t) * S + st] = (uint8_t)cw;
            if (last && !residual) break;
            // the wave that owns a token's chosen row passes it on
            for (uint64_t mine = __ballot(lane < nt && (int)(cw >> 5) == wave); mine; mine &= mine - 1) {
                const int t = __builtin_ctzll(mine);
                if (col == (__builtin_amdgcn_readlane((int)cw, t) & 31)) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) *(half8*)(l.chosen + t * PITCH + 16 * hh + 32 * ks) = f[ks];
                }
            }
            if (!last) load_frags(st + 1);
            __syncthreads();
            for (int i = tid; i < nt * NCH; i += blockDim.x) {
                const int t = i / NCH, c = i - t * NCH;
                const half8 cv = *(const half8*)(l.chosen + t * PITCH + 16 * c);
                if (last) {
                    const half8 hv = *(const half8*)(l.hi + t * PITCH + 16 * c);
                    const half8 lv = *(const half8*)(l.lo + t * PITCH + 16 * c);
                    int64_t xr, ro;
                    token(t, xr, ro);
                    floatx4 lo4, hi4;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float rv = (float)hv[e] + (st > 0 ? (float)lv[e] : 0.0f) - (float)cv[e];
                        if (e < 4) lo4[e] = rv; else hi4[e - 4] = rv;
                    }
                    *(floatx4*)(residual + ro * D + 8 * c) = lo4;
                    *(floatx4*)(residual + ro * D + 8 * c + 4) = hi4;
                } else if (st == 0) {
                    *(half8*)(l.lo + t * PITCH + 16 * c) = -cv;
                } else {
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    const u32x4 a = *(const u32x4*)(l.hi + t * PITCH + 16 * c), bb = *(const u32x4*)(l.lo + t * PITCH + 16 * c),
                                cc = __builtin_bit_cast(u32x4, cv);
                    u32x4 na, nb;
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        uint32_t p, q;
                        resplit2(a[w], bb[w], cc[w], p, q);
                        na[w] = p;
                        nb[w] = q;
                    }
                    *(u32x4*)(l.hi + t * PITCH + 16 * c) = na;
                    *(u32x4*)(l.lo + t * PITCH + 16 * c) = nb;
                }
            }
            __syncthreads();
        }
    }
}

// Fused encode parameters (points == nullptr: assignment only).
struct EncArgs {
    double2* points;
    const double2* vtab;
    double r;
    int N, L;
};

// Stream groups of the grouped form (on = false: the per-stream form).
struct GroupArgs {
    bool on;
    const int32_t* groups;
    int64_t n_groups;
    int G;
};

template <int D, bool WIDE, bool ENC, bool GRP, bool PERS>
int launch_rvq_t(const fkv_rvq_desc* dsc, int ns, const uint16_t* x, const uint16_t* books,
                 const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad,
                 const EncArgs& enc, const GroupArgs& grp, hipStream_t stream)
{
    static std::once_flag once;
    const int Kp = (dsc->K + 63) / 64 * 64;  // whole pairs of 32-codeword tiles
    std::call_once(once, [] {
        (void)hipFuncSetAttribute((const void*)rvq_assign_kernel<D, WIDE, ENC, GRP, PERS>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)(lds_bytes<D, WIDE>(256) + (ENC ? enc_lds_bytes() : 0)));
    });
    (void)hipGetLastError();
    const int64_t Ta = dsc->t_end - dsc->t_begin;
    // Tokens per block: with the fused encode, a multiple of L / gcd(L, S) so
    // that every block holds whole spans.
    int64_t tpb = kItemTokens;
    if (ENC) {
        int a = enc.L, b = dsc->S;
        while (b) {
            const int t = a % b;
            a = b;
            b = t;
        }
        const int unit = enc.L / a;
        tpb = (int64_t)(kItemTokens / unit) * unit;
    }
    const int64_t items = GRP ? grp.n_groups : dsc->n_streams;
    const int64_t bps = ((GRP ? grp.G * Ta : Ta) + tpb - 1) / tpb;
    const int64_t n_items = bps * items;
    // 16 items per block once there are at least 64 blocks' worth per compute
    // unit
    const int64_t ipb = (PERS && ns > 2 && n_items >= 256 * 64) ? 16 : 1;
    const int64_t nblk = (n_items + ipb - 1) / ipb;
    if (nblk > 0x7fffffff) return FKV_ERR_UNSUPPORTED;
    const int64_t n_spans = ENC ? (Ta * dsc->S + enc.L - 1) / enc.L : 0;
    const size_t shm = lds_bytes<D, WIDE>(Kp) + (ENC ? enc_lds_bytes() : 0);
    hipLaunchKernelGGL((rvq_assign_kernel<D, WIDE, ENC, GRP, PERS>), dim3((unsigned)nblk), dim3(Cfg<D, WIDE>::THREADS), shm,
                       stream, (const _Float16*)x, (const _Float16*)books, stream_book, symbols, residual, n_bad,
                       dsc->T, dsc->t_begin, Ta, dsc->S, ns, dsc->K, Kp, dsc->n_books, bps, tpb, enc.points, enc.vtab,
                       enc.r, enc.N, enc.L, n_spans, grp.groups, grp.G, dsc->n_streams, ipb, n_items);
    return launch_status();
}

// Small books: token items of 128 (whole spans with the fused encode) per
// wave set, several per block, blocks balanced within a stream so that the
// grid is about four rounds of resident blocks.
template <int D, bool ENC>
int launch_rvq_small(const fkv_rvq_desc* dsc, int ns, const uint16_t* x, const uint16_t* books,
                     const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad,
                     const EncArgs& enc, hipStream_t stream)
{
    constexpr int TOK = Cfg<D, false>::WAVES * 32;
    const int Kp = 64;
    const int64_t Ta = dsc->t_end - dsc->t_begin;
    int64_t tpi = TOK;
    if (ENC) {
        int a = enc.L, b = dsc->S;
        while (b) {
            const int t = a % b;
            a = b;
            b = t;
        }
        const int unit = enc.L / a;
        if (unit > TOK) return FKV_ERR_UNSUPPORTED;
        tpi = (int64_t)(TOK / unit) * unit;
    }
    const int64_t ips = (Ta + tpi - 1) / tpi;                   // items per stream
    const int64_t target = 256 * kSmallBlocks * 4;             // about four rounds of resident blocks
    const int64_t want = std::min<int64_t>(kSmallMaxItems, std::max<int64_t>(1, (dsc->n_streams * ips + target - 1) / target));
    const int64_t bps = (ips + want - 1) / want;               // blocks per stream
    const int64_t ipb = (ips + bps - 1) / bps;                 // items per block
    const int64_t nblk = bps * dsc->n_streams;
    if (nblk > 0x7fffffff) return FKV_ERR_UNSUPPORTED;
    const int64_t n_spans = ENC ? (Ta * dsc->S + enc.L - 1) / enc.L : 0;
    const size_t shm = 2 * buf_bytes_of(Shape<D>::ROW_P, Kp) + (ENC ? 256 * 16 + (size_t)kSmallMaxItems * TOK * 2 : 0);
    hipLaunchKernelGGL((rvq_small_kernel<D, ENC>), dim3((unsigned)nblk), dim3(Cfg<D, false>::THREADS), shm, stream,
                       (const _Float16*)x, (const _Float16*)books, stream_book, symbols, residual, n_bad, dsc->T,
                       dsc->t_begin, Ta, dsc->S, ns, dsc->K, Kp, dsc->n_books, bps, tpi, ipb, enc.points, enc.vtab, enc.r,
                       enc.N, enc.L, n_spans);
    return launch_status();
}

// Whether two wide blocks fit a compute unit: 16 waves' registers (at most 128 each
// up to d = 80) and two pairs of book buffers.
template <int D>
bool two_wide(const fkv_rvq_desc* dsc)
{
    return D <= 80 && 2 * lds_bytes<D, true>((dsc->K + 63) / 64 * 64) <= kLdsBudget;
}

// Whether a call of at most 32 tokens per work item takes rvq_few_kernel.  It
// does once there are more items than the staged form has resident blocks (one
// or two per compute unit): that form then runs them in rounds.  Below that,
// the staged form starts all its copies at once and only loses at d <= 64,
// where it scans 64 columns for a few tokens.  Measured, staged
// and few (us): d = 128, S = 3, K = 256, 512 items of 4 tokens 36.0 and 21.4,
// 300 of 16 31.7 and 22.3, 144 of 16 13.6 and 14.9; 2048 streams of 32 tokens
// 160 and 79.  d = 64, S = 2, K = 256, 288 items of 1 token 7.0 and 6.1, 144 of
// 16 9.9 and 8.5, 300 of 32 11.7 and 13.1.  Small books keep their own kernel
// in the per-stream form (K = 64, 2304 streams of 32 tokens: 14.0 and 15.8).
//
// A small book gives a block few waves, which then split many tokens' residuals
// between them (from a third stage on, chunk by chunk): there the staged form is
// the faster one up to about two rounds of its blocks, the more so where a wave
// without tokens skips its scan (groups) or two wide blocks fit a compute unit.
// Staged and few (us), groups: d = 80, S = 3, 300 items: K = 64, 32 tokens 7.9 and
// 13.6, 8 tokens 7.9 and 8.5, K = 256, 32 tokens 18.6 and 15.6; d = 128, S = 4, K = 32,
// 300 items of 32 20.0 and 28.2; d = 192, S = 4, K = 32, 1500 of 32 86 and 117; d = 16,
// S = 4, K = 32, 600 of 32 8.5 and 12.3.  One stage of a large book has no second load
// to overlap either: d = 192, S = 1, K = 192, 300 items 10.4 and 12.7.  Books of 129 to
// 192 codewords give it six waves where the staged form has eight: d = 16, S = 3,
// 1500 groups of 32 16.8 and 21.1; d = 144, S = 2, 300 of 32 18.1 and 21.0.
template <int D>
bool few_tokens(const fkv_rvq_desc* dsc, int ns, const GroupArgs& grp)
{
    const int64_t Ta = dsc->t_end - dsc->t_begin, n_items = grp.on ? grp.n_groups : dsc->n_streams;
    if (Ta > kFewTokens || (grp.on && grp.G * Ta > kFewTokens)) return false;
    const int K = dsc->K;
    const int64_t tokens = (grp.on ? grp.G : 1) * Ta;
    if (!grp.on && D <= 64 && K <= kSmallK && ns <= 2) return false;
    if (n_items <= (D <= 64 ? 512 : 256) && (D > 64 || tokens > 16)) return false;
    if (ns >= 3 && tokens > 16) {
        if (grp.on && D <= 32 && n_items <= 1024) return false;
        if (K <= 64 && (grp.on ? D <= 208 && n_items <= 1024 : D <= 144 && n_items <= 512)) return false;
    }
    if (!grp.on) return true;
    if (D == 80 && two_wide<D>(dsc) && tokens > (ns >= 3 && n_items <= 512 ? 8 : 16) && (ns >= 3 || n_items <= 512))
        return false;
    if (D <= 64 && ns >= 3 && tokens > 8 && K <= 64 && n_items <= 1024) return false;
    if (D <= 208 && ns == 2 && tokens > 16 && K <= 64 && n_items <= 512) return false;
    if (D > 128 && D <= 208 && ns >= 3 && tokens > 16 && K <= 32) return false;
    if (D <= 208 && tokens > 16 && K > 128 && K <= 192 && (D <= 32 || (D > 128 && (ns <= 2 || n_items <= 512)))) return false;
    if (ns > 1 || K <= 128) return true;
    if (D <= 64) return n_items > 512;
    return D <= 128 || !(D <= 208 ? n_items <= 512 || tokens >= 16 : n_items <= 1024 && tokens >= 16);
}

// Whether the staged form's blocks are narrow (d <= 128): with more than one full
// item per compute unit they are.  At d <= 64 two wide blocks fit one, and with at
// most two stages their second book buffer wins up to 1536 items (d = 64, S = 2,
// wide and narrow: 288 items 14.1 and 15.6 us, 1152 33.8 and 35.5, 1536 45.2 and 45.4,
// 4608 117.9 and 116.4; S = 4, 512: 36.6 and 34.5).  Items of at most half a block's
// tokens leave half of a narrow block's waves idle, while the wide shape's
// eight all have a tile, and copy the books twice as fast: S = 4, K = 256, wide and
// narrow (us): d = 64, 300 items of 128 tokens 18.5 and 28.9; d = 128, 300 of 128 44.7 and
// 50.9, 1600 of 128 162 and 175; S = 3, 2500 of 64 192 and 185.  At d = 80 two wide
// blocks fit a compute unit up to K = 192, and only full items make up for one book
// buffer: S = 3, K = 128, 1600 items of 128 tokens 46 and 64, of 200 68 and 73.
template <int D>
bool narrow_blocks(const fkv_rvq_desc* dsc, int ns, const GroupArgs& grp)
{
    if (D > 128) return false;
    const int64_t Ta = dsc->t_end - dsc->t_begin, units = grp.on ? grp.n_groups : dsc->n_streams;
    const int64_t tokens = grp.on ? grp.G * Ta : Ta, per_unit = (tokens + kItemTokens - 1) / kItemTokens;
    const int64_t items = units * per_unit;
    if (D <= 64) return items > (ns <= 2 ? 1536 : tokens > 200 * per_unit ? 256 : 512);
    if (D == 80 && two_wide<D>(dsc)) return items > 256 && tokens > 240 * per_unit;
    if (2 * tokens <= kItemTokens && (ns >= 4 ? items <= 2048 : ns == 3 && items <= 1024)) return false;
    return items > 256;
}

template <int D, bool GRP>
int launch_rvq_few(const fkv_rvq_desc* dsc, int ns, const uint16_t* x, const uint16_t* books,
                   const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad,
                   const GroupArgs& grp, hipStream_t stream)
{
    const int waves = (dsc->K + 31) / 32;
    const int64_t n_items = GRP ? grp.n_groups : dsc->n_streams;
    hipLaunchKernelGGL((rvq_few_kernel<D, GRP>), dim3((unsigned)std::min<int64_t>(n_items, 1 << 20)), dim3(64 * waves),
                       0, stream, (const _Float16*)x, (const _Float16*)books, stream_book, symbols, residual, n_bad,
                       dsc->T, dsc->t_begin, dsc->t_end - dsc->t_begin, dsc->S, ns, dsc->K, dsc->n_books, grp.groups,
                       grp.G, dsc->n_streams, n_items);
    return launch_status();
}

template <int D, bool WIDE>
int launch_rvq_w(const fkv_rvq_desc* dsc, int ns, const uint16_t* x, const uint16_t* books,
                 const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad, const EncArgs& enc,
                 const GroupArgs& grp, hipStream_t stream)
{
    if (grp.on)
        return launch_rvq_t<D, WIDE, false, true, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc,
                                                         grp, stream);
    if (enc.points)
        return launch_rvq_t<D, WIDE, true, false, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc,
                                                         grp, stream);
    // Blocks that can take several items, above d = 128 (in the narrow shape the
    // other block's scans cover an item's first wait).  With at most two stages the
    // prefetched rows only cost registers.  Without and with them (us), K = 256: d =
    // 256, 600 streams of 512, S = 1 71 and 109; 1000 of 988, S = 2 544 and 595; S = 4,
    // K = 200, 600 of 300 341 and 327; d = 192, S = 1 55 and 72.  (At d = 208 the form
    // without them spills inside the scan: S = 2 781 and 470.)
    if constexpr (WIDE && D > 128)
        if (ns > 2 || (D == 208 && ns == 2))
            return launch_rvq_t<D, WIDE, false, false, true>(dsc, ns, x, books, stream_book, symbols, residual, n_bad,
                                                             enc, grp, stream);
    return launch_rvq_t<D, WIDE, false, false, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc, grp,
                                                      stream);
}

template <int D>
int launch_rvq(const fkv_rvq_desc* dsc, int ns, const uint16_t* x, const uint16_t* books,
               const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad,
               const EncArgs& enc, const GroupArgs& grp, hipStream_t stream)
{
    // ns stages are assigned (the first ns of the S in the layout)
    if (!enc.points && few_tokens<D>(dsc, ns, grp)) {
        if (grp.on)
            return launch_rvq_few<D, true>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, grp, stream);
        return launch_rvq_few<D, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, grp, stream);
    }
    if constexpr (D <= 64) {
        if (!grp.on && dsc->K <= kSmallK && ns <= 2) {
            if (enc.points)
                return launch_rvq_small<D, true>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc, stream);
            return launch_rvq_small<D, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc, stream);
        }
    }
    if constexpr (D <= 128)
        if (narrow_blocks<D>(dsc, ns, grp))
            return launch_rvq_w<D, false>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc, grp, stream);
    return launch_rvq_w<D, true>(dsc, ns, x, books, stream_book, symbols, residual, n_bad, enc, grp, stream);
}

int rvq_dispatch(const fkv_rvq_desc* desc, int ns, const uint16_t* x_f16, const uint16_t* books_f16,
                 const int32_t* stream_book, uint8_t* symbols, float* residual, uint32_t* n_bad_streams,
                 const EncArgs& enc, void* stream, const GroupArgs& grp = GroupArgs{false, nullptr, 0, 0})
{
    if (!desc) return FKV_ERR_INVALID_ARG;
    const fkv_rvq_desc& d = *desc;
    if (d.n_streams < 0 || d.T < 0 || d.t_begin < 0 || d.t_end < d.t_begin || d.t_end > d.T)
        return FKV_ERR_INVALID_ARG;
    if (d.d < 16 || d.d > 256 || d.d % 16 != 0) return FKV_ERR_INVALID_ARG;
    if (d.S < 1 || d.S > 8 || d.K < 1 || d.K > 256 || d.n_books < 1) return FKV_ERR_INVALID_ARG;
    if (ns < 1 || ns > d.S || (enc.points && ns != d.S)) return FKV_ERR_INVALID_ARG;
    if (grp.on && (grp.n_groups < 0 || grp.G < 1 || grp.G > kMaxGroup || enc.points)) return FKV_ERR_INVALID_ARG;
    if (grp.on && grp.n_groups > 0 && (!grp.groups || !aligned(grp.groups, 4))) return FKV_ERR_INVALID_ARG;
    if (d.n_streams == 0 || d.t_end == d.t_begin || (grp.on && grp.n_groups == 0)) return FKV_OK;
    if (!x_f16 || !books_f16 || !stream_book || !symbols) return FKV_ERR_INVALID_ARG;
    if (!aligned(x_f16, 16) || !aligned(books_f16, 16) || !aligned(stream_book, 4))
        return FKV_ERR_INVALID_ARG;
    if (residual && !aligned(residual, 16)) return FKV_ERR_INVALID_ARG;
    if (n_bad_streams && !aligned(n_bad_streams, 4)) return FKV_ERR_INVALID_ARG;
    const hipStream_t st = (hipStream_t)stream;
#define FKV_RVQ_CASE(DD) \
    case DD: return launch_rvq<DD>(desc, ns, x_f16, books_f16, stream_book, symbols, residual, n_bad_streams, enc, grp, st);
    switch (d.d) {
        FKV_RVQ_CASE(16) FKV_RVQ_CASE(32) FKV_RVQ_CASE(48) FKV_RVQ_CASE(64)
        FKV_RVQ_CASE(80) FKV_RVQ_CASE(96) FKV_RVQ_CASE(112) FKV_RVQ_CASE(128)
        FKV_RVQ_CASE(144) FKV_RVQ_CASE(160) FKV_RVQ_CASE(176) FKV_RVQ_CASE(192)
        FKV_RVQ_CASE(208) FKV_RVQ_CASE(224) FKV_RVQ_CASE(240) FKV_RVQ_CASE(256)
    default: return FKV_ERR_INVALID_ARG;
    }
#undef FKV_RVQ_CASE
}

// From this many head vectors per call on, fkv_rvq_assign_encode runs the
// assignment and then the span encode as two kernels.  Small calls gain from the
// one launch and the symbols never read back (GPT-2 shape: 37 us fused against 41
// us); in large ones the encode's tail and its LDS cost the fused kernel more than
// the separate encode takes, by little since two or three blocks share a compute
// unit.  Fused and separate (us), K = 256: d = 128, S = 3, 2.0 M vectors 624 and 601, 7.7
// M 2270 and 2220, 16.8 M 4934 and 4803; d = 64, S = 2, 2.0 M 216 and 208, 16.8 M 1722 and
// 1663; S = 4, 9.2 M 1968 and 1948.  Small books are 2% faster fused at every size
// (K = 64, 16.8 M 617 and 627), and d = 256 is from 4 M on (9.2 M 7380 and 8416: the
// separate assignment keeps more scratch).
constexpr int64_t kSplitHeadVectors = (int64_t)1 << 23;

bool encode_split(const fkv_rvq_desc* desc, const uint8_t* symbols)
{
    return desc && desc->n_streams > 0 && desc->t_end > desc->t_begin &&
           desc->n_streams * (desc->t_end - desc->t_begin) >= kSplitHeadVectors && aligned(symbols, 4);
}

}  // namespace
}  // namespace fkv

using namespace fkv;

extern "C" int fkv_rvq_assign_encode_fused(const fkv_rvq_desc* desc, const uint8_t* symbols)
{
    if (!desc) return FKV_ERR_INVALID_ARG;
    return encode_split(desc, symbols) ? 0 : 1;
}

extern "C" int fkv_rvq_assign(const fkv_rvq_desc* desc, const uint16_t* x_f16, const uint16_t* books_f16,
                              const int32_t* stream_book, uint8_t* symbols, float* residual,
                              uint32_t* n_bad_streams, void* stream)
{
    const EncArgs none = {nullptr, nullptr, 0.0, 0, 1};
    return rvq_dispatch(desc, desc ? desc->S : 0, x_f16, books_f16, stream_book, symbols, residual, n_bad_streams,
                        none, stream);
}

extern "C" int fkv_rvq_assign_stages(const fkv_rvq_desc* desc, int32_t n_stages, const uint16_t* x_f16,
                                     const uint16_t* books_f16, const int32_t* stream_book, uint8_t* symbols,
                                     float* residual, uint32_t* n_bad_streams, void* stream)
{
    const EncArgs none = {nullptr, nullptr, 0.0, 0, 1};
    return rvq_dispatch(desc, n_stages, x_f16, books_f16, stream_book, symbols, residual, n_bad_streams, none,
                        stream);
}

extern "C" int fkv_rvq_assign_encode(const fkv_rvq_desc* desc, const uint16_t* x_f16, const uint16_t* books_f16,
                                     const int32_t* stream_book, const fkv_codec* c, const void* dev_table,
                                     uint8_t* symbols, double* points, float* residual, uint32_t* n_bad_streams,
                                     void* stream)
{
    if (!c || c->N < 3 || c->N > 256 || c->L < 1 || c->L > 64 || !(c->r > 0.0 && c->r < 1.0) ||
        !(c->r_max > 0.0 && c->r <= c->r_max * (1.0 + 1e-12)))
        return FKV_ERR_INVALID_ARG;
    if (!dev_table || !points || !aligned(dev_table, 16) || !aligned(points, 16)) return FKV_ERR_INVALID_ARG;
    if (encode_split(desc, symbols)) {
        // assignment, then the encode of its symbols on the same stream: the
        // same symbols and points as the fused kernel, bit for bit (an invalid
        // stream's 0xFF symbols encode to NaN points there too)
        const EncArgs none = {nullptr, nullptr, 0.0, 0, 1};
        const int rc = rvq_dispatch(desc, desc->S, x_f16, books_f16, stream_book, symbols, residual, n_bad_streams,
                                    none, stream);
        if (rc != FKV_OK) return rc;
        return fkv_cgr_encode_spans(c, dev_table, symbols, desc->n_streams, (desc->t_end - desc->t_begin) * desc->S,
                                    points, stream);
    }
    const EncArgs enc = {(double2*)points, (const double2*)((const uint8_t*)dev_table + table_off_V(c->N)), c->r,
                         c->N, c->L};
    return rvq_dispatch(desc, desc ? desc->S : 0, x_f16, books_f16, stream_book, symbols, residual, n_bad_streams,
                        enc, stream);
}

extern "C" int fkv_rvq_assign_groups(const fkv_rvq_desc* desc, const int32_t* groups, int64_t n_groups,
                                     int32_t group_size, const uint16_t* x_f16, const uint16_t* books_f16,
                                     const int32_t* stream_book, uint8_t* symbols, float* residual,
                                     uint32_t* n_bad_groups, void* stream)
{
    const EncArgs none = {nullptr, nullptr, 0.0, 0, 1};
    const GroupArgs grp = {true, groups, n_groups, group_size};
    return rvq_dispatch(desc, desc ? desc->S : 0, x_f16, books_f16, stream_book, symbols, residual, n_bad_groups,
                        none, stream, grp);
}
