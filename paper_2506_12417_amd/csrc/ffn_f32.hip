// Grouped fp32 GEMM on the matrix cores: the two products of an expert FFN (section 4.4: x W1 W2)
// in full precision, driven by the tile table (tiles of at most 64 rows).
//
//   out[r, n] = epilogue( sum_k a[r, k] * w_e[n, k] )      r in a tile of expert e
//
// Two kernels.  gemm_f32_split_kernel multiplies by bf16 matrix instructions, which run at 16 times the rate of the fp32 ones:
// every operand is cut into three bf16 parts that add up to it exactly, and eight of the nine products of parts are summed in
// fp32 (the ninth, of the smallest parts, is below 2^-33 of a term).  gemm_f32_rows_kernel, for calls too small for that,
// multiplies by v_mfma_f32_16x16x4_f32, the contraction in four or eight parts.
//
// Items in both: a tile and a block of weight rows, one work-group each, which the hardware starts where one has finished; the
// plan's bins, equal in rows but not in tiles, play no role (28 % of the CU time was idle with them).
#include <type_traits>
#include "common.h"
#include "ffn_kernels.h"
#include "ffn_f32_rule.h"

namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int BM = 64, BK = 32, PIECES = BK / 4;

__device__ __forceinline__ float silu_f(float z) { return z / (1.f + __expf(-z)); }

// Few multiply-adds, or few rows per expert: a call's time is the latency of one item, or the fetch of the weights.  An item is
// 16 NSUB weight rows of a tile; its KS wavefronts share the contraction out, a run of whole 128-byte lines each, UNROLL lines
// of every operand row in flight and sixteen wavefronts on a CU.  The lines are turned into the matrix instruction's fragments
// in a piece of LDS of the wavefront's own (no barrier), and the partial sums meet in LDS in a fixed order.
// (A work-group that staged 32 terms of all rows at a time, the next ones on their way, spent 0.55 us a stage however little was
// in it.  Measured, that -> this: one token, d=296 F=1984, E=8, k=2: 8.5 + 30 -> 4.9 + 7.5 us; 79 tokens, d=72 F=1408, E=4 7.2 + 29
// -> 6.5 + 13; 200 tokens, d=1024 F=2048, E=8 39 + 57 -> 31 + 31; 12 tokens, d=816 F=576, E=4, SwiGLU 18 + 12.6 -> 8.2 + 4.8.)
// Bound by latency in small calls; with tens of rows per expert by the fp32 instructions on ragged tiles, 58 TFLOP/s (full tiles, 6144
// rows of K = 768 and of 4096: 119 and 125).  Tried: sixteen wavefronts per item, tiles in parts of 16 or 32 rows: no faster, twice as
// slow where there are many items.
// Error of a layer against 64 bits 1.2 - 2.0e-7 of the result's norm; by a single chain of each wavefront's terms 1.5 - 3e-7.
//
// LDS: a row's line is eight 16-byte pieces, piece p at position p ^ (row & 7) (no bank conflicts).  Lane (l16, lq) reads pieces
// lq and 4 + lq and feeds their four terms to four matrix instructions each (both operands agree on the order of the terms).
template <int EPI, int KS, int NSUB>
__global__ __launch_bounds__(KS * 64, 4) void gemm_f32_rows_kernel(const float* __restrict__ a_mat, int K, int N,
                                                                   const void* const* __restrict__ w_ptrs,
                                                                   const moe_tile* __restrict__ tiles,
                                                                   const int32_t* __restrict__ hdr, float* __restrict__ out, int ld_out,
                                                                   const int32_t* __restrict__ row_src, int src_div) {
    constexpr bool GLU = EPI == MOE_EPI_SWIGLU;
    constexpr int NTH = KS * 64, COLS = 16 * NSUB, OUT = GLU ? 16 : COLS;
    static_assert(!GLU || NSUB == 2, "a gate and an up block");
    // (a wave-uniform base and 32-bit byte offsets: the launch sees to it that they suffice)
    auto fetch = [](const float* base, unsigned offset) __attribute__((always_inline)) {
        typedef const __attribute__((address_space(1))) unsigned char* gbytes;
        return *(const __attribute__((address_space(1))) f32x4*)((gbytes)(uintptr_t)base + offset);
    };
    __shared__ __attribute__((aligned(16))) float part[KS][BM][COLS + 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int st_row = lane >> 3, st_p = lane & 7, st_at = st_row * PIECES + (st_p ^ st_row), rd_at = l16 * PIECES + (lq ^ (l16 & 7));
    f32x4* const turn = (f32x4*)&part[wave][0][0];
    static_assert(sizeof part[0] >= 16 * 2 * NSUB * 128 && sizeof part[0] % 16 == 0, "a wavefront's lines turn where its sums will be");
    const int n_cb = GLU ? N / 32 : (N + COLS - 1) / COLS;
    const int n_lines = (K + BK - 1) / BK, per = (n_lines + KS - 1) / KS;
    const int s0 = wave * per < n_lines ? wave * per : n_lines, s1 = s0 + per < n_lines ? s0 + per : n_lines;
    const bool ragged = K % BK != 0;

    const int n_items = hdr[0] * n_cb;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int ti = item / n_cb, cb = item - ti * n_cb;
        const moe_tile t = tiles[ti];
        const int rc = __builtin_amdgcn_readfirstlane(t.row_count < BM ? t.row_count : BM);
        if (rc <= 0) continue;
        // SwiGLU: blocks of 32 gate and 32 up rows alternate; an item takes a half of each
        const int p0 = GLU ? (cb >> 1) * 64 + (cb & 1) * 16 : cb * COLS, w_step = GLU ? 32 : 16;
        const float* w_mat = (const float*)w_ptrs[__builtin_amdgcn_readfirstlane(t.expert)];
        unsigned w_src[NSUB][2];
#pragma unroll
        for (int h = 0; h < NSUB; ++h)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = p0 + h * w_step + i * 8 + st_row;
                w_src[h][i] = (unsigned)(r < N ? r : N - 1) * (unsigned)K * 4u;
            }
        auto multiply = [&](auto groups, auto unroll) __attribute__((always_inline)) {
            constexpr int RG = decltype(groups)::value, UNROLL = decltype(unroll)::value;
            unsigned a_src[RG][2];
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = g * 16 + i * 8 + st_row;
                    int row = t.row_begin + (r < rc ? r : rc - 1);
                    if (row_src) row = (int)((unsigned)row_src[row] / (unsigned)src_div);
                    a_src[g][i] = (unsigned)row * (unsigned)K * 4u;
                }
            f32x4 acc[RG][NSUB];
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int h = 0; h < NSUB; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[g][h][r] = 0.f;
            for (int s = s0; s < s1; s += UNROLL) {
                f32x4 wl[UNROLL][NSUB][2], al[UNROLL][RG][2];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    const int line = s + u < s1 ? s + u : s1 - 1;       // (past the end: the last line again, not multiplied)
                    const int k = line * BK + st_p * 4, at = (k < K ? k : K - 4) * 4;
#pragma unroll
                    for (int h = 0; h < NSUB; ++h)
#pragma unroll
                        for (int i = 0; i < 2; ++i) wl[u][h][i] = fetch(w_mat, w_src[h][i] + (unsigned)at);
#pragma unroll
                    for (int g = 0; g < RG; ++g)
#pragma unroll
                        for (int i = 0; i < 2; ++i) al[u][g][i] = fetch(a_mat, a_src[g][i] + (unsigned)at);
                }
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    if (s + u >= s1) continue;
                    if (ragged && s + u + 1 == n_lines) {               // (terms past K count as zero on both sides)
                        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                        const bool past = (s + u) * BK + st_p * 4 >= K;
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
#pragma unroll
                            for (int h = 0; h < NSUB; ++h) wl[u][h][i] = past ? zero : wl[u][h][i];
#pragma unroll
                            for (int g = 0; g < RG; ++g) al[u][g][i] = past ? zero : al[u][g][i];
                        }
                    }
#pragma unroll
                    for (int h = 0; h < NSUB; ++h)
#pragma unroll
                        for (int i = 0; i < 2; ++i) turn[(h * 16 + i * 8) * PIECES + st_at] = wl[u][h][i];
                    f32x4 wf[2][NSUB];
#pragma unroll
                    for (int v = 0; v < 2; ++v)
#pragma unroll
                        for (int h = 0; h < NSUB; ++h) wf[v][h] = turn[h * 16 * PIECES + (rd_at ^ (4 * v))];
#pragma unroll
                    for (int g = 0; g < RG; ++g) {
                        f32x4* const at = turn + 16 * NSUB * PIECES + (NSUB == 2 ? g & 1 : 0) * 16 * PIECES;
#pragma unroll
                        for (int i = 0; i < 2; ++i) at[i * 8 * PIECES + st_at] = al[u][g][i];
#pragma unroll
                        for (int v = 0; v < 2; ++v) {
                            // (16 terms at a time, added to the sum as one: half the rounding error of a single chain)
                            const f32x4 af = at[rd_at ^ (4 * v)];
                            f32x4 sixteen[NSUB];
#pragma unroll
                            for (int h = 0; h < NSUB; ++h) sixteen[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int j = 0; j < 4; ++j)
#pragma unroll
                                for (int h = 0; h < NSUB; ++h)
                                    sixteen[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[j], wf[v][h][j], sixteen[h], 0, 0, 0);
#pragma unroll
                            for (int h = 0; h < NSUB; ++h)
#pragma unroll
                                for (int r = 0; r < 4; ++r) acc[g][h][r] += sixteen[h][r];
                        }
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int h = 0; h < NSUB; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) part[wave][g * 16 + 4 * lq + r][h * 16 + l16] = acc[g][h][r];
        };
        // (lines in flight as the registers allow: 128 of them, with sixteen wavefronts on a CU)
        constexpr int ONE = NSUB == 1;
        if (rc <= 16) multiply(std::integral_constant<int, 1>{}, std::integral_constant<int, 3 + ONE>{});
        else if (rc <= 32) multiply(std::integral_constant<int, 2>{}, std::integral_constant<int, 2 + ONE>{});
        else if (rc <= 48) multiply(std::integral_constant<int, 3>{}, std::integral_constant<int, 1 + ONE>{});
        else multiply(std::integral_constant<int, 4>{}, std::integral_constant<int, 1 + ONE>{});
        __syncthreads();
        auto total = [&](int r, int c) __attribute__((always_inline)) {
            float v = part[0][r][c];
#pragma unroll
            for (int p = 1; p < KS; ++p) v += part[p][r][c];
            return v;
        };
        for (int i = tid; i < rc * OUT; i += NTH) {
            const int r = i / OUT, c = i % OUT, col = GLU ? cb * 16 + c : p0 + c;
            float v = total(r, c);
            if constexpr (GLU) v = silu_f(v) * total(r, 16 + c);
            else if constexpr (EPI == MOE_EPI_RELU) v = fmaxf(v, 0.f);
            if (GLU || col < N) out[(size_t)(t.row_begin + r) * ld_out + col] = v;
        }
        __syncthreads();
    }
}

// Eight fp32 values times 2^32 as three bf16 parts, v 2^32 = part[0] + part[1] + part[2] exactly (round to nearest, then the same of
// what is left: 8 + 8 + 8 bits of 24).  The factor lifts fp32's last bit, 2^-149, to 2^-117, so that no part of any value is below
// bf16's smallest numbers; values from 2^95 on become infinite.  Converted and subtracted by plain vector instructions, which
// run beside matrix instructions; v_dot2_f32_bf16 would subtract in one instead of two, but takes the matrix cores' time.
__device__ __forceinline__ void split3(f32x4 lo, f32x4 hi, bf16x8 (&part)[3]) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = lo[i] * 0x1p32f;
        v[4 + i] = hi[i] * 0x1p32f;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            const bf16x2 h = __builtin_convertvector((f32x2){v[i], v[i + 1]}, bf16x2);
            part[p][i] = h[0];
            part[p][i + 1] = h[1];
            if (p < 2) {
                const uint32_t u = __builtin_bit_cast(uint32_t, h);
                v[i] -= __builtin_bit_cast(float, u << 16);
                v[i + 1] -= __builtin_bit_cast(float, u & 0xffff0000u);
            }
        }
}

__device__ const f32x4 zeros = {0.f, 0.f, 0.f, 0.f};      // (fetched as one piece of 16 bytes, and aligned to it)

// An item is a tile and BN = 64 CB weight rows: each of the four wavefronts multiplies all rows of the tile with 16 CB weight rows of
// its own, in blocks of 16 x 16; blocks of 16 rows past the tile's end are left out.  Stages of 32 terms.  The rows' parts are made
// by the whole work-group and shared through two LDS buffers; the weights are fetched in whole lines, turned in a piece of
// LDS of the wavefront's own and cut in registers.  While a stage is multiplied, the next one is cut and the one after it
// is on its way; one barrier per stage.
//
// The term's large products (first parts) and its seven small ones are summed apart and added at the end: the large sum is
// rounded once per 32 terms, and a sum of one term once.  (Without the products of second and third parts, 2^-25 of a term each at
// most, single terms were off by up to 2^-24 more than their rounding; the products of 1501 x 768, F = 2048 took 252 us, 275 now.)
// Error of an fp32 layer (1501 x 768, F = 2048) against 64 bits: 3.85e-7 of the result's norm; the fp32 instructions' chain has 9.5e-7, a single
// sum of all products 8.2e-7.
//
// The sums are of values times 2^64 (split3).  An infinity or NaN, an operand of 2^95 or more and a sum of 2^64 or more make
// infinities or NaNs of them: a wavefront with a sum that is not finite does its block again by fp32 matrix instructions from global
// memory, so that such values come out as they do in fp32.  Everything else is exact in its parts, however small.
// (2048 tokens twice, d=1024 F=2048 E=16, both products: 335 us, with one infinite token 413, all of them 848; by fp32 instructions alone
// 393 always.  Fetching four bytes a lane and term, that second pass took 822 and 2740.)
//
// Bound by issue and latency as much as by the matrix cores: cutting takes as many vector instructions as the products take
// matrix instructions' cycles.  Full tiles (6144 rows, K = 768, N = 4096) 148 TFLOP/s of fp32 work, 1.2 PFLOP/s of bf16; a quarter goes into
// an item's way in (header, tile, addresses, first stage) and out.  Measured (fp32 instructions -> this): 3002 rows, d=768 F=2048 E=16
// SwiGLU 208 + 124 -> 183 + 114 us; 4000 rows, d=1000 F=2048 E=8 181 + 191 -> 138 + 159; 1501 tokens twice, d=768 F=2048 E=16, SwiGLU, a
// layer 348 -> 290.
// Tried, all within 3 %: weights' parts shared through LDS too, two tiles of an expert at a time (twice the registers), the
// next two stages in flight, two blocks of rows multiplied at a time.  v_dot2_f32_bf16 would take a part off in one instruction instead of two, but runs on the matrix
// cores: no faster.
//
// LDS: a row's 32 terms are four groups of 8 (terms 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3: fetched as two pieces of 16 bytes), group g of
// row r at position g ^ (-(r / 4) & 3); the weights' pieces p at p ^ (r & 7).  (No bank conflicts: the LDS serves lanes 0-3,
// 12-15, 20-23 and 24-27 of a 16-byte read together.)
template <int EPI, int CB>
__global__ __launch_bounds__(256, CB == 2 ? 2 : 3) void gemm_f32_split_kernel(const float* __restrict__ a_mat, int K, int N,
                                                           const void* const* __restrict__ w_ptrs,
                                                           const moe_tile* __restrict__ tiles,
                                                           const int32_t* __restrict__ hdr, float* __restrict__ out, int ld_out,
                                                           const int32_t* __restrict__ row_src, int src_div) {
    constexpr int NW = 4, NTH = NW * 64, BN = 16 * CB * NW, GROUPS = BK / 8, RB = BM / 16;
    constexpr int AL = BM * GROUPS / NTH, ROWS = NTH / GROUPS;
    constexpr bool GLU = EPI == MOE_EPI_SWIGLU;
    __shared__ bf16x8 lds[2][3][BM * GROUPS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int ld_row = tid / GROUPS, ld_g = tid % GROUPS;
    static_assert(ROWS % 16 == 0, "the swizzle repeats every 16 rows");
    const int st_at = ld_row * GROUPS + (ld_g ^ (-(ld_row >> 2) & 3));
    const int rd_at = l16 * GROUPS + (lq ^ (-(l16 >> 2) & 3));
    __shared__ f32x4 w_lds[NW][16 * CB * PIECES];
    f32x4* const w_own = w_lds[wave];
    const int w_row = lane >> 3, w_p = lane & 7, w_st = w_row * PIECES + (w_p ^ w_row), w_rd = l16 * PIECES + (lq ^ (l16 & 7));
    const int n_cb = (N + BN - 1) / BN, KT = (K + BK - 1) / BK;

    const int n_items = hdr[0] * n_cb;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int ti = item / n_cb, cb = item - ti * n_cb;
        const moe_tile t = tiles[ti];
        const int rc = __builtin_amdgcn_readfirstlane(t.row_count < BM ? t.row_count : BM);
        if (rc <= 0) continue;
        const int n0 = cb * BN + wave * (16 * CB);                      // the wavefront's first weight row
        const float* w_mat = (const float*)w_ptrs[t.expert];
        auto row_of = [&](int r) __attribute__((always_inline)) {
            int row = t.row_begin + (r < rc ? r : rc - 1);
            if (row_src) row = (int)((unsigned)row_src[row] / (unsigned)src_div);
            return a_mat + (size_t)row * K;
        };
        auto weights_of = [&](int h) __attribute__((always_inline)) {
            const int r = n0 + h;
            return w_mat + (size_t)(r < N ? r : N - 1) * K;
        };
        const float *a_src[AL], *b_src[2 * CB];
#pragma unroll
        for (int i = 0; i < AL; ++i) a_src[i] = row_of(ld_row + i * ROWS);
#pragma unroll
        for (int h = 0; h < 2 * CB; ++h) b_src[h] = weights_of(h * 8 + w_row);
        f32x4 av[AL][2], bv[2 * CB];
        bf16x8 b[2][CB][3];
        // (K is a multiple of 4; activations past K count as zero, and weights past K are the last ones again)
        auto fetch = [&](const float* at) __attribute__((always_inline)) { return *(const __attribute__((address_space(1))) f32x4*)(uintptr_t)at; };
        auto load = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < AL; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int k = kt * BK + j * 16 + ld_g * 4;
                    av[i][j] = fetch(k < K ? a_src[i] + k : (const float*)&zeros);
                }
            const int k = kt * BK + w_p * 4;
#pragma unroll
            for (int h = 0; h < 2 * CB; ++h) bv[h] = fetch(b_src[h] + (k < K ? k : K - 4));
        };
        auto store = [&](int kt) __attribute__((always_inline)) {
            bf16x8 part[3];
#pragma unroll
            for (int i = 0; i < AL; ++i) {
                split3(av[i][0], av[i][1], part);
#pragma unroll
                for (int p = 0; p < 3; ++p) lds[kt & 1][p][st_at + i * ROWS * GROUPS] = part[p];
            }
        };
        // (own rows only: no barrier)
        auto turn = [&](f32x4 (&raw)[CB][2]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2 * CB; ++h) w_own[h * 8 * PIECES + w_st] = bv[h];
#pragma unroll
            for (int h = 0; h < CB; ++h)
#pragma unroll
                for (int j = 0; j < 2; ++j) raw[h][j] = w_own[h * 16 * PIECES + (w_rd ^ (4 * j))];
        };
        f32x4 acc[RB][CB], low[RB][CB];
#pragma unroll
        for (int m = 0; m < RB; ++m)
#pragma unroll
            for (int h = 0; h < CB; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[m][h][r] = low[m][h][r] = 0.f;
        load(0);
        store(0);
        {
            f32x4 raw[CB][2];
            turn(raw);
#pragma unroll
            for (int h = 0; h < CB; ++h) split3(raw[h][0], raw[h][1], b[0][h]);
        }
        load(1 < KT ? 1 : 0);
        __syncthreads();
        auto multiply = [&](auto blocks) __attribute__((always_inline)) {
            constexpr int NB = decltype(blocks)::value;
            auto step = [&](int kt, bf16x8 (&b)[CB][3], bf16x8 (&next)[CB][3]) __attribute__((always_inline)) {
                bf16x8 a[3];
                auto products = [&](int m) __attribute__((always_inline)) {
#pragma unroll
                    for (int p = 0; p < 3; ++p) a[p] = lds[kt & 1][p][m * 16 * GROUPS + rd_at];
                    auto mul = [&](int pa, int pb, f32x4 (&c)[RB][CB]) __attribute__((always_inline)) {
#pragma unroll
                        for (int h = 0; h < CB; ++h) c[m][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[pa], b[h][pb], c[m][h], 0, 0, 0);
                    };
                    mul(2, 1, low);
                    mul(0, 0, acc);
                    mul(1, 2, low);
                    mul(2, 0, low);
                    mul(1, 1, low);
                    mul(0, 2, low);
                    mul(1, 0, low);
                    mul(0, 1, low);
                };
                f32x4 raw[CB][2];
                turn(raw);
                store(kt + 1);
                load(kt + 2 < KT ? kt + 2 : KT - 1);
                products(0);
#pragma unroll
                for (int h = 0; h < CB; ++h) split3(raw[h][0], raw[h][1], next[h]);
#pragma unroll
                for (int m = 1; m < NB; ++m) products(m);
                __syncthreads();
            };
            int kt = 0;
            for (; kt + 1 < KT; kt += 2) {
                step(kt, b[0], b[1]);
                step(kt + 1, b[1], b[0]);
            }
            if (kt < KT) step(kt, b[0], b[1]);
        };
        if (rc > 48) multiply(std::integral_constant<int, 4>{});
        else if (rc > 32) multiply(std::integral_constant<int, 3>{});
        else if (rc > 16) multiply(std::integral_constant<int, 2>{});
        else multiply(std::integral_constant<int, 1>{});
        bool redo = false;
#pragma unroll
        for (int m = 0; m < RB; ++m)
#pragma unroll
            for (int h = 0; h < CB; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    acc[m][h][r] = (acc[m][h][r] + low[m][h][r]) * 0x1p-64f;
                    redo = redo || !(__builtin_fabsf(acc[m][h][r]) < __builtin_inff());
                }
        if (__any(redo)) {
#pragma unroll
            for (int m = 0; m < RB; ++m)
#pragma unroll
                for (int h = 0; h < CB; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[m][h][r] = 0.f;
            const float *a[RB], *w[CB];
#pragma unroll
            for (int m = 0; m < RB; ++m) a[m] = row_of(m * 16 + l16) + lq * 4;
#pragma unroll
            for (int h = 0; h < CB; ++h) w[h] = weights_of(h * 16 + l16) + lq * 4;
            // (16 terms at a time, four of a lane's to four instructions each, the next 16 on their way; past K both sides count as zero)
            f32x4 an[RB], wn[CB];
            auto ask = [&](int k) __attribute__((always_inline)) {
                const bool in = k + lq * 4 < K;
#pragma unroll
                for (int m = 0; m < RB; ++m) an[m] = fetch(in ? a[m] + k : (const float*)&zeros);
#pragma unroll
                for (int h = 0; h < CB; ++h) wn[h] = fetch(in ? w[h] + k : (const float*)&zeros);
            };
            ask(0);
            for (int k = 0; k < K; k += 16) {
                f32x4 av[RB], wv[CB];
#pragma unroll
                for (int m = 0; m < RB; ++m) av[m] = an[m];
#pragma unroll
                for (int h = 0; h < CB; ++h) wv[h] = wn[h];
                ask(k + 16);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int m = 0; m < RB; ++m)
#pragma unroll
                        for (int h = 0; h < CB; ++h)
                            acc[m][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[m][j], wv[h][j], acc[m][h], 0, 0, 0);
            }
        }
        // acc[m][h][r]: row 16 m + 4 lq + r, weight row 16 h + l16 of the wavefront's
        bool keep = true;
        int col = n0 + l16;
        if constexpr (GLU) {
            // blocks of 32 gate and 32 up rows alternate: their wavefronts meet in LDS
            constexpr int PER = 2 / CB;
            const int pair = CB == 2 ? wave >> 1 : wave & 1;
            keep = !(wave & PER);
            col = cb * (BN / 2) + pair * (16 * CB) + l16;
            float* meet = (float*)&lds[0][0][0] + pair * (RB * CB * 4 * 64) + lane;
            static_assert((NW / 2) * RB * CB * 4 * 64 * 4 <= (int)sizeof lds, "");
            if (!keep) {
#pragma unroll
                for (int i = 0; i < RB * CB * 4; ++i) meet[i * 64] = acc[i / (4 * CB)][(i >> 2) % CB][i & 3];
            }
            __syncthreads();
            if (keep) {
#pragma unroll
                for (int m = 0; m < RB; ++m)
#pragma unroll
                    for (int h = 0; h < CB; ++h)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[m][h][r] = silu_f(acc[m][h][r]) * meet[((m * CB + h) * 4 + r) * 64];
            }
        }
        if (keep) {
#pragma unroll
            for (int h = 0; h < CB; ++h) {
                if (n0 + h * 16 + l16 < N) {
#pragma unroll
                    for (int m = 0; m < RB; ++m)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int row = m * 16 + 4 * lq + r;
                            if (row < rc) out[(size_t)(t.row_begin + row) * ld_out + col + h * 16] = EPI == MOE_EPI_RELU ? fmaxf(acc[m][h][r], 0.f) : acc[m][h][r];
                        }
                }
            }
        }
        __syncthreads();
    }
}

struct Args {
    const void* a;
    int A, K, N, E;
    const void* const* w;
    const moe_tile* tiles;
    const int32_t* hdr;
    void* out;
    int ld_out;
    const int32_t* row_src;
    int src_div;
};

// one work-group per item of the tiles there usually are (the device alone knows; they loop if there are more)
long long tiles_there_are(const Args& g) { return g.A < g.E + g.A / BM ? g.A : g.E + g.A / BM; }
unsigned grid_of(const Args& g, int bn) {
    const long long items = tiles_there_are(g) * ((g.N + bn - 1) / bn);
    return (unsigned)(items < (1 << 20) ? (items + 7) / 8 * 8 : 1 << 20);
}

template <int EPI, int CB>
int launch_split(const Args& g, hipStream_t st) {
    hipLaunchKernelGGL((gemm_f32_split_kernel<EPI, CB>), dim3(grid_of(g, 64 * CB)), dim3(256), 0, st, (const float*)g.a, g.K, g.N, g.w, g.tiles,
                       g.hdr, (float*)g.out, g.ld_out, g.row_src, g.src_div);
    MOE_CHECK_LAUNCH("moe_grouped_ffn (fp32 GEMM)");
    return MOE_OK;
}

template <int EPI>
int launch_rows(const Args& g, hipStream_t st) {
    auto go = [&](auto ks, auto nsub) {
        constexpr int KS = decltype(ks)::value, NSUB = decltype(nsub)::value;
        hipLaunchKernelGGL((gemm_f32_rows_kernel<EPI, KS, NSUB>), dim3(grid_of(g, 16 * NSUB)), dim3(KS * 64), 0, st, (const float*)g.a, g.K, g.N,
                           g.w, g.tiles, g.hdr, (float*)g.out, g.ld_out, g.row_src, g.src_div);
    };
    const std::integral_constant<int, 1> one{};
    const std::integral_constant<int, 2> two{};
    const std::integral_constant<int, 4> four{};
    const std::integral_constant<int, 8> eight{};
    // Items of 32 weight rows where those of 16 would be four per CU and more (304 tokens, K = 80, N = 1600 13.4 us by 16, 10.6 by 32;
    // 306 items of K = 1696 25 by 32, 19 by 16).  Eight wavefronts where they have two lines each at least and few items (19 items,
    // K = 1984: 7.9 and 6.8; N = 64, K = 2048: 14.0 and 11.3) or SwiGLU's wide items (K = 1000: 57 and 55; K = 256: 30 and 39).
    if constexpr (EPI == MOE_EPI_SWIGLU) {
        if (g.K >= 512) go(eight, two);
        else go(four, two);
    } else {
        const long long items = tiles_there_are(g) * ((g.N + 15) / 16);
        if (items < 64 && g.K >= 1024) go(eight, one);
        else if (items < 4 * 256) go(four, one);
        else go(four, two);
    }
    MOE_CHECK_LAUNCH("moe_grouped_ffn (fp32 GEMM)");
    return MOE_OK;
}

}  // namespace

int moe_launch_gemm_f32(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                        const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src, int src_div) {
    const Args g = {a, A, K, N, E, w, tiles, hdr, out, ld_out, row_src, src_div};
    const bool glu = epi == MOE_EPI_SWIGLU;
    const int kernel = moe_f32_kernel(glu, A, K, N, E);
    const bool narrow = kernel == MOE_F32_SPLIT_64;
    if (kernel == MOE_F32_ROWS) {
        if (glu) return launch_rows<MOE_EPI_SWIGLU>(g, st);
        return epi == MOE_EPI_RELU ? launch_rows<MOE_EPI_RELU>(g, st) : launch_rows<MOE_EPI_STORE>(g, st);
    }
    if (glu) return narrow ? launch_split<MOE_EPI_SWIGLU, 1>(g, st) : launch_split<MOE_EPI_SWIGLU, 2>(g, st);
    if (epi == MOE_EPI_RELU) return narrow ? launch_split<MOE_EPI_RELU, 1>(g, st) : launch_split<MOE_EPI_RELU, 2>(g, st);
    return narrow ? launch_split<MOE_EPI_STORE, 1>(g, st) : launch_split<MOE_EPI_STORE, 2>(g, st);
}
