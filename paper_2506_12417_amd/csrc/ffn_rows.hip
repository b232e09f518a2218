// Grouped 16-bit GEMM for experts that hold a handful of rows each (decode steps, short batches):
// the products of ffn_bf16.hip in the regime where a product costs the fetch of its weights
// (section 4.4, rows per expert far below q), so that the fetch has to use the whole chip.
//
//   out[r, n] = epilogue( sum_k a[r, k] * w_e[n, k] )      r in a tile of expert e
//
// What bounds it: HBM, and the latency of a launch that moves only some tens of MB.  The tile
// kernels give an expert to one XCD (its bin) and 128 or 256 weight rows to a work-group: with
// eight active experts most of the chip idles.  Here a work item is 32 weight rows of one tile,
// whatever its bin: a work-group of KS wavefronts takes it, each wavefront a KS-th of the
// contraction.  Weights and activation rows are fetched in whole 128-byte lines, eight rows a load, UNROLL slices
// in flight per wavefront and sixteen wavefronts per CU, and turned into the matrix instruction's fragment layout in a piece
// of LDS of the wavefront's own (no barrier: a wavefront's LDS accesses keep their order).  The KS partial sums
// are added in a fixed order through LDS.  No item shares weights with another one, so XCDs and
// bins play no role and the grid is plain: the hardware hands out work-groups as CUs become free.
//
// Fetched straight into fragment registers, 16 rows x 64 bytes a load, the four lanes that the vector cache serves
// together lay on four rows: 64 look-ups a load instead of 16, which held a CU to 11 - 13 bytes a clock and the chip to
// 5.3 TB/s at best, less wherever the items fell unevenly or an expert had more than a few rows.
//
// Measured (fragments from global memory -> lines through LDS): d=2048 F=1408, 46 experts of 1..23 rows and a shared expert
// F=5632 with 33 rows 107 + 69 -> 93 + 57 us (6.2 and 5.0 TB/s of weights); d=4096 F=14336, three rows' experts 116 + 75 -> 105 + 60
// (6.5 and 5.5); d=768 F=3072, six experts 11 + 11.5 -> 9.4 + 8.7; four experts d=1024 F=2048 of 32 rows each 10.7 + 12.6 -> 9.2 + 7.6.
//
// A matrix instruction takes 16 activation rows; lanes past the tile's last row load that row
// again (rows of the product are independent, nothing is stored for them).
#include <type_traits>
#include "common.h"
#include "ffn_kernels.h"
#include "gemm_util.h"

namespace {

// 16 bytes at a wave-uniform address plus a per-lane byte offset.  (Global address space spelled
// out: a pointer read from the expert table is generic to the compiler, and flat loads would be
// waited for together with LDS traffic.)
typedef const __attribute__((address_space(1))) unsigned char* gptr;
typedef const __attribute__((address_space(1))) bf16x8* gfrag;
__device__ __forceinline__ bf16x8 load_frag(const void* base, unsigned offset) { return *(gfrag)((gptr)(uintptr_t)base + offset); }

// acc[g][h] = (16 activation rows of group g) x (16 weight rows of block h) over the slices [s0, s1)
// of 32 terms, UNROLL slices at a time: all their loads, then their products (the other wavefronts
// of the SIMD keep the memory busy meanwhile).  turn: 16 NSUB rows of 128 bytes of the wavefront's own.
template <bool HALF_IN, int RG, int NSUB, int UNROLL>
__device__ __forceinline__ void rows_product(const uint16_t* __restrict__ a_mat, const unsigned (&a_off)[RG][2],
                                             const uint16_t* w, size_t w_step, unsigned w_off, size_t w_eight, int s0, int s1,
                                             f32x4 (&acc)[RG][NSUB], bf16x8* turn) {
    static_assert(UNROLL % 2 == 0, "a line holds two slices");
    const int lane = threadIdx.x & 63, l16 = lane & 15, lq = lane >> 4;
    const int st_at = (lane >> 3) * 8 + ((lane & 7) ^ (lane >> 3)), rd_at = l16 * 8 + (lq ^ (l16 & 7));
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int h = 0; h < NSUB; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[g][h][r] = 0.f;
    for (int s = s0; s < s1; s += UNROLL) {
        bf16x8 wl[UNROLL / 2][NSUB][2], al[UNROLL / 2][RG][2];
#pragma unroll
        for (int u = 0; u < UNROLL; u += 2) {
            const int at = (s + u < s1 ? s + u : s1 - 2) * 32;   // (past the end: the last line again, not multiplied)
#pragma unroll
            for (int h = 0; h < NSUB; ++h)
#pragma unroll
                for (int i = 0; i < 2; ++i) wl[u / 2][h][i] = load_frag(w + h * w_step + i * w_eight + at, w_off);
#pragma unroll
            for (int g = 0; g < RG; ++g)
#pragma unroll
                for (int i = 0; i < 2; ++i) al[u / 2][g][i] = load_frag(a_mat + at, a_off[g][i]);
        }
#pragma unroll
        for (int u = 0; u < UNROLL; u += 2) {
            if (s + u < s1) {
#pragma unroll
                for (int h = 0; h < NSUB; ++h)
#pragma unroll
                    for (int i = 0; i < 2; ++i) turn[(h * 16 + i * 8) * 8 + st_at] = wl[u / 2][h][i];
                bf16x8 wf[2][NSUB];
#pragma unroll
                for (int v = 0; v < 2; ++v)
#pragma unroll
                    for (int h = 0; h < NSUB; ++h) wf[v][h] = turn[h * 16 * 8 + (rd_at ^ (4 * v))];
                // (two groups' lines side by side where the wavefront's piece holds them)
#pragma unroll
                for (int g = 0; g < RG; ++g) {
                    bf16x8* const at = turn + 16 * NSUB * 8 + (NSUB == 2 ? g & 1 : 0) * 16 * 8;
#pragma unroll
                    for (int i = 0; i < 2; ++i) at[i * 8 * 8 + st_at] = al[u / 2][g][i];
#pragma unroll
                    for (int v = 0; v < 2; ++v) {
                        const bf16x8 af = at[rd_at ^ (4 * v)];
#pragma unroll
                        for (int h = 0; h < NSUB; ++h)
                            if constexpr (HALF_IN)
                                acc[g][h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, af),
                                                                                   __builtin_bit_cast(f16x8, wf[v][h]), acc[g][h], 0, 0, 0);
                            else
                                acc[g][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, wf[v][h], acc[g][h], 0, 0, 0);
                    }
                }
            }
        }
    }
}

__device__ __forceinline__ uint16_t half_bits(float v) {     // saturating, nearest-even
    return __builtin_bit_cast(uint16_t, (_Float16)__builtin_amdgcn_fmed3f(v, -65504.f, 65504.f));
}

// One product: what a launch is given for it (moe_launch_gemm_rows).
struct Job {
    const uint16_t* a_mat;
    const void* const* w_ptrs;
    const moe_tile* tiles;
    const int32_t* hdr;
    void* out;
    const int32_t* row_token;
    const float* row_gate;
    int K, N, ld_out, a_div;
};

// Two products can share a launch: the first n_other work-groups serve `other`, the rest `main`.  (The
// shared expert beside the routed ones, whose own two launches leave the chip half idle.)
template <int EPI, bool GATHER, int KS, int NSUB, int UNROLL>
__global__ __launch_bounds__(KS * 64, 4) void gemm_rows_kernel(Job main, Job other, unsigned n_other) {
    constexpr bool SCAT = EPI == MOE_EPI_SCATTER, HALF_IN = SCAT || EPI == MOE_EPI_STORE, GLU = EPI == MOE_EPI_SWIGLU;
    constexpr int NTH = KS * 64, RGMAX = 4, COLS = 16 * NSUB;
    static_assert(NSUB == 2 || (NSUB == 1 && !GLU), "SwiGLU needs a gate and an up block");
    // partial sums [wavefront][row][weight row of the item]; the pitch puts a lane group's four rows and
    // the readers' rows on different banks
    __shared__ __attribute__((aligned(16))) float part[KS][RGMAX * 16][COLS + 4];
    const int tid = threadIdx.x, lane = tid & 63, wave = sgpr(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const bool second = blockIdx.x < n_other;
    const uint16_t* __restrict__ a_mat = second ? other.a_mat : main.a_mat;
    const void* const* __restrict__ w_ptrs = second ? other.w_ptrs : main.w_ptrs;
    const moe_tile* __restrict__ tiles = second ? other.tiles : main.tiles;
    const int32_t* __restrict__ hdr = second ? other.hdr : main.hdr;
    void* __restrict__ out = second ? other.out : main.out;
    const int32_t* __restrict__ row_token = second ? other.row_token : main.row_token;
    const float* __restrict__ row_gate = second ? other.row_gate : main.row_gate;
    const int K = second ? other.K : main.K, N = second ? other.N : main.N, ld_out = second ? other.ld_out : main.ld_out;
    const int a_div = second ? other.a_div : main.a_div;
    const int n_cb = N / COLS;                   // (N is a multiple of 64)
    // (whole lines: a wavefront's part is an even number of 64-byte slices, K being a multiple of 64.  K = 1408 by
    // four wavefronts in parts of 11 slices read 20 % more than the weights: 315 MB from memory for the second product of
    // 33 rows and E = 60; with the shared expert's 23 MB it reads 287 now.)
    const int n_slices = K / 32, per = (n_slices / 2 + KS - 1) / KS * 2;
    const int s0 = wave * per < n_slices ? wave * per : n_slices, s1 = s0 + per < n_slices ? s0 + per : n_slices;
    const unsigned w_off = ((unsigned)(lane >> 3) * (unsigned)K + (unsigned)(lane & 7) * 8u) * 2u;      // eight rows' lines a load
    // (a wavefront's lines turn where its sums will be.  Rows of eight 16-byte pieces, piece p of row r at position p ^ (r & 7):
    // no bank conflicts either way)
    bf16x8* const turn = (bf16x8*)&part[wave][0][0];
    static_assert(sizeof part[0] >= (16 * NSUB + 16 * NSUB) * 128 && sizeof part[0] % 16 == 0, "");

    // (The tile is read after the number of tiles, although both latencies pass before the weights can
    // be asked for: a table kept by its owner may end with its last tile.)
    const int n_items = sgpr(hdr[0]) * n_cb, step = (int)(second ? n_other : gridDim.x - n_other);
    for (int item = (int)(second ? blockIdx.x : blockIdx.x - n_other); item < n_items; item += step) {
        const int ti = item / n_cb, cb = item - ti * n_cb;
        const moe_tile t = tiles[ti];
        const int rc = sgpr(t.row_count), row0 = sgpr(t.row_begin), expert = sgpr(t.expert);
        // The item's blocks of 16 packed weight rows.  Packed rows 16 h + j of a block of 32 are outputs
        // 2 j + h (moe_pack_weights): an item of two blocks gives 32 adjacent outputs, an item of one
        // block the h-th of each pair.  With SwiGLU blocks of 32 gate and 32 up rows alternate, and the
        // item takes the h-th half of a gate block and of its up block (outputs 2 j + h of 32).
        const int p0 = GLU ? (cb >> 1) * 64 + (cb & 1) * 16 : cb * COLS;
        const int col = GLU || NSUB == 1 ? (cb >> 1) * 32 + (cb & 1) : cb * 32;        // + 2 j
        const uint16_t* w = (const uint16_t*)sgpr_ptr(w_ptrs[expert]) + (size_t)p0 * K;
        const size_t w_step = (size_t)(GLU ? 32 : 16) * K;
        for (int r0 = 0; r0 < rc; r0 += RGMAX * 16) {
            const int left = rc - r0;
            auto multiply = [&](auto groups, auto unroll) __attribute__((always_inline)) {
                constexpr int RG = decltype(groups)::value;
                unsigned a_off[RG][2];
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int at = g * 16 + i * 8 + (lane >> 3), r = at < left ? at : left - 1;
                        unsigned src = (unsigned)(row0 + r0 + r);
                        if constexpr (GATHER) {
                            if (row_token) src = (unsigned)row_token[src] / (unsigned)a_div;
                        }
                        a_off[g][i] = (src * (unsigned)K + (unsigned)(lane & 7) * 8u) * 2u;
                    }
                f32x4 acc[RG][NSUB];
                rows_product<HALF_IN, RG, NSUB, decltype(unroll)::value>(a_mat, a_off, w, w_step, w_off, (size_t)8 * K, s0, s1, acc, turn);
#pragma unroll
                for (int g = 0; g < RG; ++g)
#pragma unroll
                    for (int h = 0; h < NSUB; ++h)
#pragma unroll
                        for (int r = 0; r < 4; ++r) part[wave][g * 16 + 4 * lq + r][h * 16 + l16] = acc[g][h][r];
            };
            if (left <= 16) multiply(std::integral_constant<int, 1>{}, std::integral_constant<int, UNROLL>{});
            else if (left <= 32) multiply(std::integral_constant<int, 2>{}, std::integral_constant<int, UNROLL / 4 * 2>{});
            else if (left <= 48) multiply(std::integral_constant<int, 3>{}, std::integral_constant<int, UNROLL / 4 * 2>{});
            else multiply(std::integral_constant<int, 4>{}, std::integral_constant<int, UNROLL / 4 * 2>{});
            // (fetched while the other wavefronts finish: the place of this thread's first row)
            const int rows = left < RGMAX * 16 ? left : RGMAX * 16;
            unsigned tok = 0;
            float gate = 1.f;
            auto place = [&](int r) __attribute__((always_inline)) {
                tok = (unsigned)row_token[row0 + r0 + r];
                if (row_gate) gate = row_gate[tok];
            };
            if constexpr (SCAT) place((tid >> 4) < rows ? tid >> 4 : rows - 1);
            __syncthreads();
            auto total = [&](int r, int c) __attribute__((always_inline)) {
                float v = part[0][r][c];
#pragma unroll
                for (int p = 1; p < KS; ++p) v += part[p][r][c];
                return v;
            };
            // one column j of the item's block or blocks per thread and step
            for (int i = tid; i < rows * 16; i += NTH) {
                const int r = i >> 4, j = i & 15, row = row0 + r0 + r;
                float v0 = total(r, j), v1 = NSUB == 2 ? total(r, COLS - 16 + j) : 0.f;
                if constexpr (!HALF_IN) {
                    uint16_t* to = (uint16_t*)out + (size_t)row * ld_out + col + 2 * j;
                    if constexpr (GLU) *to = half_bits(silu_f(v0) * v1);
                    else if constexpr (NSUB == 1) *to = half_bits(fmaxf(v0, 0.f));
                    else *(uint32_t*)to = half_bits(fmaxf(v0, 0.f)) | ((uint32_t)half_bits(fmaxf(v1, 0.f)) << 16);
                } else {
                    if constexpr (SCAT) {
                        if (i >= NTH) place(r);
                        v0 *= gate;
                        v1 *= gate;
                    }
                    float* to = (float*)out + (size_t)(SCAT ? tok : (unsigned)row) * ld_out + col + 2 * j;
                    if constexpr (NSUB == 1) *to = v0;
                    else *(float2*)to = make_float2(v0, v1);
                }
            }
            __syncthreads();
        }
    }
}

// The number of tiles is known on the device only: at most one per row, about one per expert.
// A table with more tiles makes the work-groups loop, a shorter one lets some leave at once.
long long tiles_estimate(int A, int E) { return A < E + A / 128 ? A : E + A / 128; }

template <int EPI, bool GATHER>
int launch(const Job& main, int A, int E, hipStream_t st, const Job* other = nullptr, int other_A = 0) {
    const int dev_ok = moe_check_gemm_device();
    if (dev_ok != MOE_OK) return dev_ok;
    const int K = main.K, N = main.N;
    const long long tiles_est = tiles_estimate(A, E);
    const long long items = tiles_est * (N / 32);
    auto go = [&](auto ks, auto nsub, auto unroll) {
        constexpr int KS = decltype(ks)::value, NSUB = decltype(nsub)::value, UNROLL = decltype(unroll)::value;
        const long long n = tiles_est * (N / (16 * NSUB));
        const unsigned n_other = other ? (unsigned)(tiles_estimate(other_A, 1) * (other->N / (16 * NSUB))) : 0u;
        hipLaunchKernelGGL((gemm_rows_kernel<EPI, GATHER, KS, NSUB, UNROLL>), dim3((unsigned)(n < 32768 ? n : 32768) + n_other), dim3(KS * 64), 0,
                           st, main, other ? *other : main, n_other);
    };
    auto go_unroll = [&](auto ks, auto nsub) {
        // Slices per round of loads: eight, or six where that leaves fewer loads unused (K = 768:
        // 91 -> 76 us at 78 experts; K = 1408: 71 -> 60 us at 46).
        const int per = (K / 64 + decltype(ks)::value - 1) / decltype(ks)::value * 2;
        if ((per + 5) / 6 * 6 < (per + 7) / 8 * 8) go(ks, nsub, std::integral_constant<int, 6>{});
        else go(ks, nsub, std::integral_constant<int, 8>{});
    };
    const std::integral_constant<int, 1> one{};
    const std::integral_constant<int, 2> two{};
    const std::integral_constant<int, 4> four{};
    const std::integral_constant<int, 8> eight{};
    // Four wavefronts per item, eight where a long contraction meets fewer than four items per CU
    // (second products of one to three rows: K = 3072 with 72 items 14.3 -> 12.1 us, K = 14336 with
    // 256 items 55 -> 50 us; with K = 1024 or many items eight are slower, 25.6 against 41.3 us),
    // and items of 16 weight rows where there would be less than one per CU.
    if (items < 4 * MOE_GEMM_GRID && K >= 2048) {
        if constexpr (EPI != MOE_EPI_SWIGLU) {
            if (items < MOE_GEMM_GRID) {
                go_unroll(eight, one);
                MOE_CHECK_LAUNCH("moe_grouped_ffn (few-row GEMM)");
                return MOE_OK;
            }
        }
        go_unroll(eight, two);
    } else {
        go_unroll(four, two);
    }
    MOE_CHECK_LAUNCH("moe_grouped_ffn (few-row GEMM)");
    return MOE_OK;
}

}  // namespace

int moe_launch_gemm_rows(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                         const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_token, const float* row_gate) {
    const bool scatter = epi == MOE_EPI_SCATTER;
    const Job j = {(const uint16_t*)a, w, tiles, hdr, out, scatter ? row_token : nullptr, scatter ? row_gate : nullptr, K, N, ld_out, 1};
    if (epi == MOE_EPI_RELU) return launch<MOE_EPI_RELU, false>(j, A, E, st);
    if (epi == MOE_EPI_SWIGLU) return launch<MOE_EPI_SWIGLU, false>(j, A, E, st);
    if (scatter) return launch<MOE_EPI_SCATTER, false>(j, A, E, st);
    return launch<MOE_EPI_STORE, false>(j, A, E, st);
}

int moe_launch_gemm_rows_gather(int epi, const void* x, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                                const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src, int src_div) {
    const Job j = {(const uint16_t*)x, w, tiles, hdr, out, row_src, nullptr, K, N, ld_out, src_div};
    if (epi == MOE_EPI_SWIGLU) return launch<MOE_EPI_SWIGLU, true>(j, A, E, st);
    return launch<MOE_EPI_RELU, true>(j, A, E, st);
}

int moe_launch_gemm_rows_shared(int phase, const void* x, int T, int d, int F, int E, int k, const void* const* w, const moe_tile* tiles,
                                const int32_t* hdr, void* h, float* y_perm, const int32_t* perm, int shared_F,
                                const void* const* s_w, const moe_tile* s_tiles, const int32_t* s_hdr, void* s_h, float* s_y,
                                hipStream_t st) {
    if (phase == 1) {
        const Job j = {(const uint16_t*)x, w, tiles, hdr, h, perm, nullptr, d, 2 * F, F, k};
        const Job o = {(const uint16_t*)x, s_w, s_tiles, s_hdr, s_h, nullptr, nullptr, d, 2 * shared_F, shared_F, 1};
        return launch<MOE_EPI_SWIGLU, true>(j, T * k, E, st, &o, T);
    }
    const Job j = {(const uint16_t*)h, w, tiles, hdr, y_perm, nullptr, nullptr, F, d, d, 1};
    const Job o = {(const uint16_t*)s_h, s_w, s_tiles, s_hdr, s_y, nullptr, nullptr, shared_F, d, d, 1};
    return launch<MOE_EPI_STORE, false>(j, T * k, E, st, &o, T);
}
