// Grouped fp32 GEMM on the matrix cores: the two products of an expert FFN (section 4.4: x W1 W2)
// in full precision, driven by the tile table (tiles of at most 64 rows).
//
//   out[r, n] = epilogue( sum_k a[r, k] * w_e[n, k] )      r in a tile of expert e
//
// v_mfma_f32_32x32x2_f32 multiplies and adds in fp32 like an fma chain and runs at twice the rate of
// the vector unit's plain fma (157 against 79 TFLOP/s); one instruction takes 64 cycles for two
// registers of operands, so LDS and issue slots are far from binding and the kernel can be simple:
// a work-group holds 64 rows x BN weight rows, 32 terms at a time in two LDS buffers, the next
// 32 on their way in registers; one barrier per 32 terms.  A wavefront takes both 32-row blocks of
// the tile, so that a ragged tile leaves all wavefronts the same work (an empty block is
// skipped), and one block of 32 weight rows; with SwiGLU a gate block and its up block lie on
// neighbouring wavefronts, which meet in LDS at the end.  Four wavefronts: one per SIMD.  The narrow
// forms hold two blocks of weight rows, or one, and give each wavefront half (a quarter) of every stage's
// terms (their sums meet in LDS), so that their items are smaller and still busy every SIMD.
//
// Bound by the matrix cores, and then by how evenly the items fall on the CUs: an item is a
// work-group of its own, which the hardware starts where one has finished; the plan's bins, equal in
// rows but not in tiles, play no role (28 % of the CU time was idle with them; equal runs of tiles per XCD,
// which differ in ragged tiles: 236 us for the first product below, every tile shared by all XCDs 220).
// 3002 rows, d=768 F=2048 E=16 SwiGLU: 496 + 292 us with vector fma tiles of 64 x 64, 207 + 120 here (layer after layer); 12288
// rows in full tiles, d=1024 F=4096: 128 TFLOP/s.
//
// LDS: a row holds 32 terms in eight 16-byte pieces, piece p at position p ^ ((row / 2) & 7): 16
// consecutive rows' pieces touch every bank once.  Lane (l32, lhi) reads piece 2 q + lhi and feeds its
// four terms to four matrix instructions: which term goes to which of the two k slots is free as
// long as both operands agree.
#include <type_traits>
#include "common.h"
#include "ffn_kernels.h"

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int BM = 64, BK = 32, PIECES = BK / 4;

__device__ __forceinline__ float silu_f(float z) { return z / (1.f + __expf(-z)); }

// NWN wavefronts along the weight rows, KSP along the terms
template <int EPI, int NWN, int KSP>
__global__ __launch_bounds__(NWN * KSP * 64, 3) void gemm_f32_kernel(const float* __restrict__ a_mat, int K, int N,
                                                           const void* const* __restrict__ w_ptrs,
                                                           const moe_tile* __restrict__ tiles,
                                                           const int32_t* __restrict__ hdr, float* __restrict__ out, int ld_out,
                                                           const int32_t* __restrict__ row_src, int src_div) {
    constexpr int NTH = NWN * KSP * 64, BN = 32 * NWN;
    constexpr int AL = BM * PIECES / NTH, BL = BN * PIECES / NTH;       // 16-byte pieces per thread and stage
    __shared__ f32x4 lds[2][(BM + BN) * PIECES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int wn = wave % NWN, wk = wave / NWN;
    const int ld_row = tid / PIECES, ld_p = tid % PIECES;               // pass i: row ld_row + i * NTH / PIECES
    constexpr int ROWS = NTH / PIECES;
    static_assert(ROWS % 16 == 0, "the swizzle repeats every 16 rows");
    const int st_at = ld_row * PIECES + (ld_p ^ ((ld_row >> 1) & 7));
    const int rd_swz = (l32 >> 1) & 7;
    const int n_cb = (N + BN - 1) / BN, KT = (K + BK - 1) / BK;

    // Items in the order of the plan's tiles, a tile's column blocks one after the other: the XCDs, to which
    // work-groups are dealt in turn, share every tile's column blocks evenly.  (With a multiple of eight column blocks
    // each XCD meets the same slices of an expert's weights in all of its tiles.)
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
                    const f32x4 b = buf[(BM + wn * 32 + l32) * PIECES + at];
                    const f32x4 a0 = buf[l32 * PIECES + at], a1 = buf[(32 + l32) * PIECES + at];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[j], b[j], acc[0], 0, 0, 0);
                        if constexpr (decltype(second)::value)
                            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[j], b[j], acc[1], 0, 0, 0);
                    }
                }
                // (the compiler asks for the next stage near the end of this one; pinning the loads or all fragment reads
                // to its start was slower, 128 -> 107 - 120 TFLOP/s on full tiles, three work-groups on a CU covering the latency)
                // (nothing of the store may move up: it would wait for loads that have this whole step to arrive)
                __builtin_amdgcn_sched_barrier(0);
                store(kt + 1);
            }
        };
        if (rc > 32) multiply(std::true_type{});                        // (the second 32-row block holds rows)
        else multiply(std::false_type{});
        // acc[m][r]: row 32 m + 8 (r / 4) + 4 lhi + r % 4, weight row l32 of the wavefront's block
        float* meet = (float*)&lds[0][0] + wn * (32 * 64);              // (the stages have been read)
        static_assert((KSP - 1) * NWN * 32 * 64 * 4 <= (int)sizeof lds, "the parts meet in the stages' memory");
        if constexpr (KSP > 1) {
            __syncthreads();
            if (wk) {
#pragma unroll
                for (int r = 0; r < 32; ++r) meet[(wk - 1) * (NWN * 32 * 64) + r * 64 + lane] = acc[r >> 4][r & 15];
            }
            __syncthreads();
            if (!wk) {
#pragma unroll
                for (int p = 0; p < KSP - 1; ++p)
#pragma unroll
                    for (int r = 0; r < 32; ++r) acc[r >> 4][r & 15] += meet[p * (NWN * 32 * 64) + r * 64 + lane];
            }
        }
        if constexpr (EPI == MOE_EPI_SWIGLU) {
            // even blocks are gate blocks, odd ones the up block of their neighbour
            __syncthreads();
            if ((wn & 1) && !wk) {
#pragma unroll
                for (int r = 0; r < 32; ++r) meet[r * 64 + lane] = acc[r >> 4][r & 15];
            }
            __syncthreads();
            if (!(wn & 1) && !wk) {
#pragma unroll
                for (int r = 0; r < 32; ++r) acc[r >> 4][r & 15] = silu_f(acc[r >> 4][r & 15]) * meet[32 * 64 + r * 64 + lane];
            }
        }
        const int p = n0 + wn * 32;                                    // packed row of the block
        const int col = (EPI == MOE_EPI_SWIGLU ? p / 2 : p) + l32;
        if (p + (EPI == MOE_EPI_SWIGLU ? 0 : l32) < N && !wk && !(EPI == MOE_EPI_SWIGLU && (wn & 1))) {
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = m * 32 + 8 * (r >> 2) + 4 * lhi + (r & 3);
                    if (row < rc)
                        out[(size_t)(t.row_begin + row) * ld_out + col] = EPI == MOE_EPI_RELU ? fmaxf(acc[m][r], 0.f) : acc[m][r];
                }
        }
        __syncthreads();                                                // the next item refills the first buffer
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

template <int EPI, int NWN, int KSP>
int launch(const Args& g, hipStream_t st) {
    // one work-group per item of the tiles there usually are (the device alone knows; they loop if there are more)
    const long long tiles_est = g.A < g.E + g.A / BM ? g.A : g.E + g.A / BM;
    const long long items = tiles_est * ((g.N + 32 * NWN - 1) / (32 * NWN));
    const unsigned grid = (unsigned)(items < (1 << 20) ? (items + 7) / 8 * 8 : 1 << 20);
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, NWN, KSP>), dim3(grid), dim3(NWN * KSP * 64), 0, st, (const float*)g.a, g.K, g.N, g.w, g.tiles,
                       g.hdr, (float*)g.out, g.ld_out, g.row_src, g.src_div);
    MOE_CHECK_LAUNCH("moe_grouped_ffn (fp32 GEMM)");
    return MOE_OK;
}

}  // namespace

int moe_launch_gemm_f32(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                        const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src, int src_div) {
    // Column blocks of 128 weight rows read the activations half as often; of 64 where 128 would
    // leave fewer than four items per CU; of 32, all four wavefronts on a stage's terms, where 64 would leave
    // fewer than two (without SwiGLU, which needs a gate and an up block): 256 rows, second product of K = 512,
    // N = 256 14.6 -> 10.9 us, first of K = 256, N = 512 9.3 -> 7.8; 1024 rows, K = 1024, N = 512 32.6 -> 26.1;
    // with two to four items per CU it makes no difference (3002 rows, K = 2048, N = 768: 119 and 120).
    const Args g = {a, A, K, N, E, w, tiles, hdr, out, ld_out, row_src, src_div};
    const long long tiles_est = (A + BM - 1) / BM + E / 2;
    const bool narrow = tiles_est * ((N + 127) / 128) < 4 * 256, narrowest = tiles_est * ((N + 63) / 64) < 2 * 256;
    if (epi == MOE_EPI_SWIGLU) return narrow ? launch<MOE_EPI_SWIGLU, 2, 2>(g, st) : launch<MOE_EPI_SWIGLU, 4, 1>(g, st);
    if (narrowest) return epi == MOE_EPI_RELU ? launch<MOE_EPI_RELU, 1, 4>(g, st) : launch<MOE_EPI_STORE, 1, 4>(g, st);
    if (epi == MOE_EPI_RELU) return narrow ? launch<MOE_EPI_RELU, 2, 2>(g, st) : launch<MOE_EPI_RELU, 4, 1>(g, st);
    return narrow ? launch<MOE_EPI_STORE, 2, 2>(g, st) : launch<MOE_EPI_STORE, 4, 1>(g, st);
}
