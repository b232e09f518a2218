// Grouped fp32 GEMM on the matrix cores: the two products of an expert FFN (section 4.4: x W1 W2)
// in full precision, driven by the tile table (tiles of at most 64 rows).
//
//   out[r, n] = epilogue( sum_k a[r, k] * w_e[n, k] )      r in a tile of expert e
//
// Two kernels.  gemm_f32_split_kernel multiplies by bf16 matrix instructions, which run at 16 times the rate of the fp32 ones:
// every operand is cut into three bf16 parts that add up to it exactly, and six of the nine products of parts are summed in
// fp32 (the other three are below 2^-26 of a term).  gemm_f32_kernel, for items too few and small for that, multiplies by
// v_mfma_f32_32x32x2_f32 like an fma chain.
//
// Items in both: a tile and a block of weight rows, one work-group each, which the hardware starts where one has finished; the
// plan's bins, equal in rows but not in tiles, play no role (28 % of the CU time was idle with them).
#include <type_traits>
#include "common.h"
#include "ffn_kernels.h"

namespace {

typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int BM = 64, BK = 32, PIECES = BK / 4;

__device__ __forceinline__ float silu_f(float z) { return z / (1.f + __expf(-z)); }

// Items of 32 weight rows whose stages of 32 terms are shared by four wavefronts, a quarter of the terms each (their sums meet in
// LDS): for products whose wider items would leave CUs idle, where a stage's latency is what counts.  A stage is held in two
// LDS buffers, the next one on its way in registers; one barrier per stage.  A wavefront takes both 32-row blocks of the tile.
//
// LDS: a row holds 32 terms in eight 16-byte pieces, piece p at position p ^ ((row / 2) & 7): 16
// consecutive rows' pieces touch every bank once.  Lane (l32, lhi) reads piece 2 q + lhi and feeds its
// four terms to four matrix instructions: which term goes to which of the two k slots is free as
// long as both operands agree.
template <int EPI>
__global__ __launch_bounds__(256, 3) void gemm_f32_kernel(const float* __restrict__ a_mat, int K, int N,
                                                           const void* const* __restrict__ w_ptrs,
                                                           const moe_tile* __restrict__ tiles,
                                                           const int32_t* __restrict__ hdr, float* __restrict__ out, int ld_out,
                                                           const int32_t* __restrict__ row_src, int src_div) {
    constexpr int KSP = 4, NTH = KSP * 64, BN = 32;
    constexpr int AL = BM * PIECES / NTH, BL = BN * PIECES / NTH;       // 16-byte pieces per thread and stage
    __shared__ f32x4 lds[2][(BM + BN) * PIECES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int wk = wave;
    const int ld_row = tid / PIECES, ld_p = tid % PIECES;               // pass i: row ld_row + i * NTH / PIECES
    constexpr int ROWS = NTH / PIECES;
    static_assert(ROWS % 16 == 0, "the swizzle repeats every 16 rows");
    const int st_at = ld_row * PIECES + (ld_p ^ ((ld_row >> 1) & 7));
    const int rd_swz = (l32 >> 1) & 7;
    const int n_cb = (N + BN - 1) / BN, KT = (K + BK - 1) / BK;

    const int n_items = hdr[0] * n_cb;
    for (int item = blockIdx.x; item < n_items; item += gridDim.x) {
        const int ti = item / n_cb, cb = item - ti * n_cb;
        const moe_tile t = tiles[ti];
        const int rc = __builtin_amdgcn_readfirstlane(t.row_count < BM ? t.row_count : BM);
        if (rc <= 0) continue;
        const int n0 = cb * BN;
        // (rows past the tile's end and weight rows past N are the last ones again: never stored)
        const float* a_src[AL];
        const float* b_src[BL];
#pragma unroll
        for (int i = 0; i < AL; ++i) {
            const int r = ld_row + i * ROWS;
            int row = t.row_begin + (r < rc ? r : rc - 1);
            if (row_src) row = (int)((unsigned)row_src[row] / (unsigned)src_div);     // (the rows of x brought into expert order here)
            a_src[i] = a_mat + (size_t)row * K;
        }
#pragma unroll
        for (int i = 0; i < BL; ++i) {
            const int r = n0 + ld_row + i * ROWS;
            b_src[i] = (const float*)w_ptrs[t.expert] + (size_t)(r < N ? r : N - 1) * K;
        }
        f32x4 av[AL], bv[BL];
        auto load = [&](int kt) __attribute__((always_inline)) {
            const int k = kt * BK + ld_p * 4, at = k < K ? k : K - 4;   // (K is a multiple of 4)
#pragma unroll
            for (int i = 0; i < AL; ++i) av[i] = *(const __attribute__((address_space(1))) f32x4*)(uintptr_t)(a_src[i] + at);
#pragma unroll
            for (int i = 0; i < BL; ++i) bv[i] = *(const __attribute__((address_space(1))) f32x4*)(uintptr_t)(b_src[i] + at);
        };
        auto store = [&](int kt) __attribute__((always_inline)) {
            f32x4* buf = lds[kt & 1];
            if (kt + 1 == KT && kt * BK + ld_p * 4 >= K) {              // (terms past K count as zero on both sides)
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < AL; ++i) av[i] = zero;
#pragma unroll
                for (int i = 0; i < BL; ++i) bv[i] = zero;
            }
#pragma unroll
            for (int i = 0; i < AL; ++i) buf[st_at + i * ROWS * PIECES] = av[i];
#pragma unroll
            for (int i = 0; i < BL; ++i) buf[(BM + i * ROWS) * PIECES + st_at] = bv[i];
        };
        f32x16 acc[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[m][r] = 0.f;
        load(0);
        store(0);
        auto multiply = [&](auto second) __attribute__((always_inline)) {
            for (int kt = 0; kt < KT; ++kt) {
                __syncthreads();                                        // stage kt is complete, stage kt - 1 has been read
                load(kt + 1 < KT ? kt + 1 : kt);                        // (without a condition: the last step's is not used)
                const f32x4* buf = lds[kt & 1];
#pragma unroll
                for (int q0 = 0; q0 < PIECES / 2 / KSP; ++q0) {
                    const int at = (2 * (wk * (PIECES / 2 / KSP) + q0) + lhi) ^ rd_swz;
                    const f32x4 b = buf[(BM + l32) * PIECES + at];
                    const f32x4 a0 = buf[l32 * PIECES + at], a1 = buf[(32 + l32) * PIECES + at];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[j], b[j], acc[0], 0, 0, 0);
                        if constexpr (decltype(second)::value)
                            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[j], b[j], acc[1], 0, 0, 0);
                    }
                }
                // (nothing of the store may move up: it would wait for loads that have this whole step to arrive)
                __builtin_amdgcn_sched_barrier(0);
                store(kt + 1);
            }
        };
        if (rc > 32) multiply(std::true_type{});                        // (the second 32-row block holds rows)
        else multiply(std::false_type{});
        // acc[m][r]: row 32 m + 8 (r / 4) + 4 lhi + r % 4, weight row l32
        float* meet = (float*)&lds[0][0];                               // (the stages have been read)
        static_assert((KSP - 1) * 32 * 64 * 4 <= (int)sizeof lds, "the parts meet in the stages' memory");
        __syncthreads();
        if (wk) {
#pragma unroll
            for (int r = 0; r < 32; ++r) meet[(wk - 1) * (32 * 64) + r * 64 + lane] = acc[r >> 4][r & 15];
        }
        __syncthreads();
        if (!wk) {
#pragma unroll
            for (int p = 0; p < KSP - 1; ++p)
#pragma unroll
                for (int r = 0; r < 32; ++r) acc[r >> 4][r & 15] += meet[p * (32 * 64) + r * 64 + lane];
        }
        if (n0 + l32 < N && !wk) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = m * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
                    if (row < rc)
                        out[(size_t)(t.row_begin + row) * ld_out + n0 + l32] = EPI == MOE_EPI_RELU ? fmaxf(acc[m][r], 0.f) : acc[m][r];
                }
        }
        __syncthreads();                                                // the next item refills the first buffer
    }
}

// Eight fp32 values as three bf16 parts, v = part[0] + part[1] + part[2] exactly (round to nearest, then the same of what is
// left: 8 + 8 + 8 bits of 24; parts below bf16's 2^-133 are lost).  Converted and subtracted by plain vector instructions, which
// run beside matrix instructions; v_dot2_f32_bf16 would subtract in one instead of two, but takes the matrix cores' time.
__device__ __forceinline__ void split3(f32x4 lo, f32x4 hi, bf16x8 (&part)[3]) {
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = lo[i];
        v[4 + i] = hi[i];
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

__device__ const float zeros[4] = {0.f, 0.f, 0.f, 0.f};

// An item is a tile and BN = 64 CB weight rows: each of the four wavefronts multiplies all rows of the tile with 16 CB weight rows of
// its own, in blocks of 16 x 16; blocks of 16 rows past the tile's end are left out.  Stages of 32 terms.  The rows' parts are made
// by the whole work-group and shared through two LDS buffers; the weights are fetched in whole lines, turned in a piece of
// LDS of the wavefront's own and cut in registers.  While a stage is multiplied, the next one is cut and the one after it
// is on its way; one barrier per stage.
//
// The term's large products (first parts) and its five small ones are summed apart and added at the end: the large sum is
// rounded once per 32 terms.  Error of an fp32 layer (1501 x 768, F = 2048) against 64 bits: 3.8e-7 of the result's norm; the
// fp32 instructions' chain has 9.5e-7, a single sum of all six products 8.2e-7.
//
// An infinity or NaN, or an operand that rounds to a bf16 infinity, makes NaNs of the parts' products, and parts below 2^-133
// are lost: a wavefront with a sum that is not finite, or not zero and below 2^-60, does its block again by fp32 matrix
// instructions from global memory, so that such values come out as they do in fp32.
//
// Bound by issue and latency more than by the matrix cores: cutting takes as many vector instructions as the products take
// matrix instructions' cycles.  Full tiles (6144 rows, K = 768, N = 4096) 150 TFLOP/s of fp32 work, 1.0 PFLOP/s of bf16, 1.3 within
// the stages of an item: a quarter goes into an item's way in (header, tile, addresses, first stage) and out.  Measured
// (fp32 instructions -> this): 3002 rows, d=768 F=2048 E=16 SwiGLU 208 + 124 -> 160 + 97 us; 4000 rows, d=1000 F=2048 E=8
// 181 + 191 -> 133 + 145; 400 tokens, d=512 F=1024 E=16, first product 40 -> 28; 1000 rows of 32 experts 1024 x 2048 97 + 104 -> 84 + 92.
// Tried, all within 3 %: weights' parts shared through LDS too, two tiles of an expert at a time (twice the registers), the
// next two stages in flight.  v_dot2_f32_bf16 would take a part off in one instruction instead of two, but runs on the matrix
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
                    av[i][j] = fetch(k < K ? a_src[i] + k : zeros);
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
                    mul(2, 0, low);
                    mul(0, 0, acc);
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
                    acc[m][h][r] += low[m][h][r];
                    const float v = __builtin_fabsf(acc[m][h][r]);
                    redo = redo || !(v < __builtin_inff()) || (v < 0x1p-60f && v > 0.f);
                }
        if (__any(redo)) {
#pragma unroll
            for (int m = 0; m < RB; ++m)
#pragma unroll
                for (int h = 0; h < CB; ++h)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[m][h][r] = 0.f;
            typedef const __attribute__((address_space(1))) float* gptr;
            gptr a[RB], w[CB];
#pragma unroll
            for (int m = 0; m < RB; ++m) a[m] = (gptr)(uintptr_t)row_of(m * 16 + l16);
#pragma unroll
            for (int h = 0; h < CB; ++h) w[h] = (gptr)(uintptr_t)weights_of(h * 16 + l16);
            for (int k = lq; k < K; k += 4)
#pragma unroll
                for (int m = 0; m < RB; ++m)
#pragma unroll
                    for (int h = 0; h < CB; ++h)
                        acc[m][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][k], w[h][k], acc[m][h], 0, 0, 0);
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
unsigned grid_of(const Args& g, int bn) {
    const long long tiles_est = g.A < g.E + g.A / BM ? g.A : g.E + g.A / BM;
    const long long items = tiles_est * ((g.N + bn - 1) / bn);
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
int launch_fma(const Args& g, hipStream_t st) {
    hipLaunchKernelGGL((gemm_f32_kernel<EPI>), dim3(grid_of(g, 32)), dim3(256), 0, st, (const float*)g.a, g.K, g.N, g.w, g.tiles,
                       g.hdr, (float*)g.out, g.ld_out, g.row_src, g.src_div);
    MOE_CHECK_LAUNCH("moe_grouped_ffn (fp32 GEMM)");
    return MOE_OK;
}

}  // namespace

int moe_launch_gemm_f32(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                        const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src, int src_div) {
    // Column blocks of 128 weight rows read the activations half as often; of 64 where 128 would leave fewer than four items
    // per CU; of 32 by fp32 instructions where 64 would leave fewer than two (without SwiGLU, which needs a gate and an up block): 256
    // rows, second product of K = 512, N = 256 14.6 us by 64 weight rows, 10.9 by 32; 60 rows of 32 experts, K = 512, N = 504
    // 18 us by the split kernel with 32 weight rows, 13; 400 tokens twice, K = 1024, N = 512 36 and 34.
    const Args g = {a, A, K, N, E, w, tiles, hdr, out, ld_out, row_src, src_div};
    const long long tiles_est = (A + BM - 1) / BM + E / 2;
    const bool narrow = tiles_est * ((N + 127) / 128) < 4 * 256, narrowest = tiles_est * ((N + 63) / 64) < 2 * 256;
    if (epi == MOE_EPI_SWIGLU) return narrow ? launch_split<MOE_EPI_SWIGLU, 1>(g, st) : launch_split<MOE_EPI_SWIGLU, 2>(g, st);
    if (narrowest) return epi == MOE_EPI_RELU ? launch_fma<MOE_EPI_RELU>(g, st) : launch_fma<MOE_EPI_STORE>(g, st);
    if (epi == MOE_EPI_RELU) return narrow ? launch_split<MOE_EPI_RELU, 1>(g, st) : launch_split<MOE_EPI_RELU, 2>(g, st);
    return narrow ? launch_split<MOE_EPI_STORE, 1>(g, st) : launch_split<MOE_EPI_STORE, 2>(g, st);
}
