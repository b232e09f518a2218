// moe_grouped_ffn: the expert FFNs over rows grouped by expert (Alg. 1 step 5; section 2: two
// dense layers with an activation between; section 4.4: x W1 W2, no biases).
//
// Two grouped GEMMs, each one persistent launch driven by the tile table of moe_plan_tiles:
//   G1  H = act(x_perm . W_in^T)     (ReLU, or SiLU(gate)*up on interleaved gate/up rows)
//   G2  y_perm = H . W_out^T         (fp32 out)
// This file holds the entry points and the choice of the kernel family (ffn_bf16.hip, ffn_wide.hip,
// ffn_rows.hip, ffn_stream.hip for 16 bits, ffn_f32.hip for fp32).
#include "common.h"
#include "ffn_kernels.h"

namespace {

constexpr int FM = 64;         // tile height of the fp32 kernel (ffn_f32.hip)

}  // namespace

extern "C" int moe_ffn_tile_m(moe_dtype dt) { return dt == MOE_BF16 ? 128 : FM; }

// bf16 has two tile heights: 256 rows pay off when the experts hold many rows each
extern "C" int moe_ffn_pick_tile_m(moe_dtype dt, int A, int E) {
    if (dt != MOE_BF16) return FM;
    return (E >= 1 && A / E >= 1024) ? 256 : 128;
}

// top1: step 6 folded into the second product (perm: output row of every row; gate_w may be null)
struct Top1 {
    const int32_t* perm = nullptr;
    const float* gate_w = nullptr;
    bool on = false;
};
// gather: step 4's row gather folded into the first product (x [x_rows, d]; row r is x[perm[r] / k])
struct Gather {
    const int32_t* perm = nullptr;
    int x_rows = 0, k = 1;
    bool on = false;
};

// which 16-bit kernels run: 0 the default (128-row tiles: the few-row kernels where they serve the
// call, the four-wavefront kernels two tiles at a time where wide_pairs says so, else the LDS-ring kernels; 256-row
// tiles: the four-wavefront kernels), 1 the LDS-ring kernels, 2 the four-wavefront kernels for 256-row
// tiles and for 128-row tiles the register-streaming kernels wherever they cover the call, else the LDS-ring kernels
static int g_kernel_mode = 0;

extern "C" int moe_ffn_kernel_mode(int mode) {
    MOE_REQUIRE(mode >= -1 && mode <= 2, MOE_ERR_ARG, "moe_ffn_kernel_mode: mode %d", mode);
    const int before = g_kernel_mode;
    if (mode >= 0) g_kernel_mode = mode;
    return before;
}

// Whether the few-row kernels (ffn_rows.hip) serve a plan of 128-row tiles.  The tile kernels fetch an expert through one XCD, one
// stage of 64 terms after the other: both products last about (d + F) / 64 stages of 0.35 us, however small they are.  The few-row
// kernels fetch it through the whole chip, but read the rows again for every 32 weight rows and the weights for every 64 rows: beyond the
// fetch of the weights they take 360 TFLOP/s.  So they serve calls that they multiply within those stages, 2 MFLOP per term of d + F,
// unless as many experts as XCDs have matrices of 32 MB and more, whose fetch outlasts the stages (4096 x 14336, E=8, SwiGLU 12 rows each 475 : 473,
// ReLU 12 rows 315 : 297; 3072 x 8192, E=16 8 rows 303 : 273);
// where both stream the weights at the memory's rate, calls of few rows per expert (a few hot ones make up for the bins); and with
// fewer experts than XCDs, up to the rows at which the idle XCDs are made up for.  flops: of both products.
// Measured (both products in us, few-row against tile kernels; the line in GFLOP or rows):
//   flops   256 x 512 (1.5): E=4 2.0 GFLOP 21 : 22, E=8 SwiGLU 4.0 28 : 25, E=16 3.0 23 : 23, E=64 3.0 27 : 24; 512 x 1024 (3.1): E=2 2.0 21 : 27, 4.0 38 : 27,
//           E=8 2.0 22 : 25, 4.0 28 : 26, E=32 3.0 23 : 27, 4.5 32 : 29; 768 x 768 (3.1): E=1 2.0 18 : 27, E=4 4.0 24 : 26, 6.0 34 : 28; 1024 x 1024
//           (4.1): E=2 4.0 25 : 33, 6.0 38 : 31, E=4 SwiGLU 4.0 27 : 32, 12 39 : 35; 1024 x 2048 (6.1): E=10 4.5 28 : 35, 8.0 45 : 37, E=16 6.0 34 : 37,
//           8.0 41 : 38; 2048 x 1408 (6.9): E=10 6.0 32 : 37, 8.0 45 : 39; 2048 x 5632 SwiGLU (15): E=4 13 63 : 81, E=8 13 110 : 114
//   rows    768 x 3072 SwiGLU, E=128, Zipf 0.7 and 1.2: 4.5 rows 1.00 and 0.78 of the tile kernels' time, 8 1.07 and 0.82; 2048 x 1408 SwiGLU, E=64: 8 rows
//           0.96 and 0.83; 2560 x 2560, E=64 1.09 and 0.95
//   XCDs    4096 x 14336 SwiGLU: one expert of 64 rows 111 : 175, 128 198 : 210; two of 64 177 : 212, 96 287 : 234; three of 48 257 : 297, 64 325 : 304;
//           four of 32 280 : 328, 64 416 : 341; six of 8 357 : 364, 32 422 : 408
static bool few_rows_per_expert(int A, int d, int F, int E, bool glu) {
    const double flops = 2.0 * A * d * F * (glu ? 3 : 2);
    if ((flops <= 2e6 * ((double)d + F) && (E < 8 || (long long)d * F < (1 << 24))) || A <= (long long)(glu ? 8 : 3) * E) return true;
    return E < 8 && A <= 64 * E && A <= 32 * (8 - E);
}

// the plan's tile height of a tile_m argument
static int tile_height(int tile_m) { return tile_m & ~MOE_TILE_WHOLE_PLAN; }

// Whether a product over 128-row tiles is better done two tiles at a time by the four-wavefront kernels (for a plan of all A
// rows only, MOE_TILE_WHOLE_PLAN: four of 32 experts, judged by all 12000 rows, took 41 us by single tiles and 64 in pairs).
// An item of 256 rows takes them as long whether its second tile is there or not, 1.5 to 2 times what one of 128 rows takes
// the eight-wavefront kernels, and a contraction of 1408 terms is long enough for a work-group's longer way in and out.
//   MOE_PAIRS_ONE_ROUND  the CUs then need one round of items instead of two
//   MOE_PAIRS_MANY       many rounds of a long contraction, nearly every tile with a partner: the matrix cores then run at
//                        their power limit, where a multiply-add of a larger tile is cheaper
// The table is on the device: an expert whose rows are split over bins, or are no multiple of 128, adds ragged tiles, one
// half per expert on average.  The bounds (three eighths for the table, five eighths for the pairs, and there of few experts
// at least the eight bins' share) are where the gain over Zipf loads of 2 to 48 experts is largest: seven or more of
// eight tables that the rule picks then have their second round, and their pairs one.
// Measured (one product, eight-wavefront kernels -> this; items per CU before, after): one round K=14336 (1.1, 0.7) 418 -> 380 us, (1.3,
// 0.8) 532 -> 366; K=2048 (1.2, 0.7) 77 -> 58, one expert; K=3968 (1.1, 0.6) 125 -> 103; K=1472 (1.1, 0.7) 59 -> 50.  Many rounds,
// launches one after the other, K=4096, 8 experts, means over Zipf 0 - 2: 425 rows each (14, 8) 1.02 of the time, 525 (17, 10) 0.98,
// 650 (20, 11) 0.97, 750 (23, 13) 0.93, 960 (29, 16) 0.92.  Where the rule says no: a single round before, K=2048 (0.2, 0.2) 38 -> 51, K=5632 (0.2, 0.2) 60 -> 124; more than
// one after, K=14336 (1.7, 1.1) 510 -> 630, (3.7, 2.1) 868 -> 903, K=3200 (4.7, 2.9) 325 -> 370; nothing to pair, 128 experts of 27 rows,
// K=3072 (1.6, 1.5) 138 -> 173.
static int wide_pairs(int A, int E, int K, int N) {
    const long long cb = (N + 255) / 256, rows = A;
    const long long ragged = E == 1 ? 0 : E < 8 ? 8 : E;
    const long long before = (rows + 127) / 128 + 3ll * E / 8, after = (rows + 255) / 256 + 5 * ragged / 8;
    if (K >= 1408 && before * cb > MOE_GEMM_GRID && after * cb <= MOE_GEMM_GRID) return MOE_PAIRS_ONE_ROUND;
    if (K >= 4096 && rows >= 500ll * E && rows / 128 + E <= MOE_PAIRS_MAX_TILES && after * cb >= 8 * MOE_GEMM_GRID) return MOE_PAIRS_MANY;
    return 0;
}

// (A product that moe_ffn_pairs says is taken in pairs is: 130 rows of one expert on very wide matrices could be either's.  With
// MOE_TILE_WHOLE_PLAN or without, so that it changes no bits.)
static bool few_rows_call(int A, int d, int F, int E, moe_act act, int tile_m) {
    if (tile_height(tile_m) != 128 || g_kernel_mode != 0 || (long long)A * (d > F ? d : F) >= (1ll << 31)) return false;
    const int n1 = act == MOE_SWIGLU ? 2 * F : F;
    if (wide_pairs(A, E, d, n1) || wide_pairs(A, E, F, d)) return false;
    return few_rows_per_expert(A, d, F, E, act == MOE_SWIGLU);
}

extern "C" int moe_ffn_pairs(int tile_m, int A, int E, int K, int N) {
    return tile_m == (128 | MOE_TILE_WHOLE_PLAN) && A >= 1 && E >= 1 && K % 64 == 0 && N >= 1 && wide_pairs(A, E, K, N) != 0;
}

// Whether nearly every expert fits one 128-row tile, so that the tile kernels read its weights once.
// Measured with and without the hint (both products): 128 experts of 768 x 3072, Zipf 1.0: 8 rows
// each 213 : 228 us, 16 rows 257 : 267, 32 rows 284 : 278; 60 of 2048 x 1408, Zipf 1.2: 13 rows 203 :
// 219, 27 rows 234 : 245, 53 rows 261 : 251.  Only where the matrices are larger than the memory-side
// cache (256 MB): smaller ones may be found there by the next call (16 of 1024 x 2048: 46 : 43 us).
static bool moe_weights_once(int A, int E, long long weights_bytes) { return A <= 24ll * E && weights_bytes > (256ll << 20); }

static int grouped_ffn_impl(int phases, const void* x_perm, int A, int d, int F, int E, moe_act act, moe_dtype dt,
                            const void* const* w_in, const void* const* w_out, const moe_tile* tiles,
                            int32_t* plan_hdr, int tile_m, void* h_scratch, float* y_perm, void* stream,
                            const Top1& top1 = Top1(), const Gather& gather = Gather()) {
    MOE_REQUIRE(moe_dtype_ok(dt), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn: dtype %d", (int)dt);
    MOE_REQUIRE(act == MOE_RELU || act == MOE_SWIGLU, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn: activation %d", (int)act);
    MOE_REQUIRE(A >= 0 && d >= 1 && F >= 1 && E >= 1, MOE_ERR_ARG, "moe_grouped_ffn: A=%d d=%d F=%d E=%d", A, d, F, E);
    const bool whole_plan = tile_m & MOE_TILE_WHOLE_PLAN;
    if (dt == MOE_BF16) {
        tile_m = tile_height(tile_m);
        MOE_REQUIRE(tile_m == 128 || tile_m == 256, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn: bf16 tile_m=%d, must be 128 or 256", tile_m);
        MOE_REQUIRE(d % 64 == 0 && F % 64 == 0, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn: bf16 needs d and F multiples of 64 (d=%d F=%d)", d, F);
    } else {
        MOE_REQUIRE(tile_m == FM, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn: fp32 tile_m=%d, the kernel's is %d", tile_m, FM);
        MOE_REQUIRE(d % 4 == 0 && F % 4 == 0 && (act != MOE_SWIGLU || F % 32 == 0), MOE_ERR_UNSUPPORTED,
                    "moe_grouped_ffn: fp32 needs d and F multiples of 4 (32 for SwiGLU) (d=%d F=%d)", d, F);
    }
    if (A == 0) return MOE_OK;
    MOE_REQUIRE(tiles && plan_hdr && h_scratch, MOE_ERR_ARG, "moe_grouped_ffn: null pointer");
    MOE_REQUIRE(!(phases & 1) || (x_perm && w_in), MOE_ERR_ARG, "moe_grouped_ffn: null pointer");
    MOE_REQUIRE(!(phases & 2) || (y_perm && w_out), MOE_ERR_ARG, "moe_grouped_ffn: null pointer");
    hipStream_t st = (hipStream_t)stream;
    const int n1 = act == MOE_SWIGLU ? 2 * F : F;
    int rc;
    if (dt == MOE_BF16) {
        // Work items are (tile, column block), handed to the work-groups as they become free.
        // Wide column blocks read an activation tile fewer times; only when there would not be
        // two items per CU does a GEMM take narrower ones.  The number of tiles is known on the
        // device only; this is its expected value.
        const long long tiles_est = (A + tile_m - 1) / tile_m + E / 2;
        auto narrow = [&](int N) { return tile_m == 128 && tiles_est * ((N + 255) / 256) < 2 * MOE_GEMM_GRID; };
        // The kernels that stream the weights into registers (ffn_stream.hip) run on request only
        // (moe_ffn_kernel_mode 2): on the workloads measured so far the LDS-ring kernels are faster.
        // They take items of 128 weight rows, two work-groups per CU, unless there are four wide
        // items per CU.
        const bool streaming = tile_m == 128 && g_kernel_mode == 2;
        auto stream = [&](int epi, int K) { return streaming && moe_gemm_stream_supports(epi, K); };
        auto stream_narrow = [&](int N) { return tiles_est * ((N + 255) / 256) < 4 * MOE_GEMM_GRID; };
        const bool rows = few_rows_call(A, d, F, E, act, tile_m);
        // 256-row tiles (many rows per expert: the arithmetic-bound case) go to the four-wavefront
        // kernels of ffn_wide.hip unless the LDS-ring kernels are asked for (moe_ffn_kernel_mode 1), 128-row
        // tiles where taking them in pairs pays.
        auto pairs = [&](int K, int N) {
            return tile_m == 128 && whole_plan && g_kernel_mode == 0 && !rows ? wide_pairs(A, E, K, N) : 0;
        };
        auto wide = [&](int epi, int K, int N) {
            return g_kernel_mode != 1 && moe_gemm_wide_supports(epi, K) && (tile_m == 256 || pairs(K, N));
        };
        // (the eight XCDs' L2s hold 32 MB)
        auto cache = [&](long long weights, size_t out_bytes) {
            return moe_weights_once(A, E, weights * E * 2) ? MOE_CACHE_WEIGHTS_ONCE
                   : out_bytes > (32u << 20)               ? MOE_CACHE_LARGE_OUT
                                                           : MOE_CACHE_PLAIN;
        };
        const int cache_h = cache((long long)d * n1, (size_t)A * F * 2), cache_y = cache((long long)F * d, (size_t)A * d * 4);
        if (phases & 1) {
            const int epi = act == MOE_SWIGLU ? MOE_EPI_SWIGLU : MOE_EPI_RELU;
            if (rows && gather.on)
                rc = moe_launch_gemm_rows_gather(epi, x_perm, A, d, n1, E, w_in, tiles, plan_hdr, h_scratch, F, st, gather.perm,
                                                 gather.k);
            else if (rows)
                rc = moe_launch_gemm_rows(epi, x_perm, A, d, n1, E, w_in, tiles, plan_hdr, h_scratch, F, st);
            else if (gather.on && stream(epi, d))
                rc = moe_launch_gemm_stream_gather(stream_narrow(n1), x_perm, gather.x_rows, d, n1, w_in, tiles, plan_hdr,
                                                   h_scratch, F, st, gather.perm, gather.k);
            else if (gather.on && wide(epi, d, n1))
                // (with 256-row tiles fused_impl has checked that these kernels are in use and cover d)
                rc = moe_launch_gemm_wide_gather(epi, pairs(d, n1), x_perm, gather.x_rows, d, n1, w_in, tiles, plan_hdr, h_scratch, F, st,
                                                 gather.perm, gather.k);
            else if (gather.on)
                rc = moe_launch_gemm_bf16_gather(epi, cache_h, x_perm, gather.x_rows, d, n1,
                                                 w_in, tiles, plan_hdr, h_scratch, F, st, gather.perm, gather.k);
            else if (stream(epi, d))
                rc = moe_launch_gemm_stream(epi, stream_narrow(n1), x_perm, d, n1, w_in, tiles, plan_hdr, h_scratch, F, st);
            else if (wide(epi, d, n1))
                rc = moe_launch_gemm_wide(epi, pairs(d, n1), x_perm, d, n1, w_in, tiles, plan_hdr, h_scratch, F, st);
            else
                rc = moe_launch_gemm_bf16(epi, tile_m, narrow(n1), cache_h, x_perm, d, n1,
                                          w_in, tiles, plan_hdr, h_scratch, F, st);
            if (rc != MOE_OK) return rc;
        }
        if (phases & 2) {
            const int epi = top1.on ? MOE_EPI_SCATTER : MOE_EPI_STORE;
            if (rows)
                rc = moe_launch_gemm_rows(epi, h_scratch, A, F, d, E, w_out, tiles, plan_hdr, (void*)y_perm, d, st, top1.perm,
                                          top1.gate_w);
            else if (stream(epi, F))
                rc = moe_launch_gemm_stream(epi, stream_narrow(d), h_scratch, F, d, w_out, tiles, plan_hdr, (void*)y_perm, d, st,
                                            top1.perm, top1.gate_w, top1.on ? A : 0);
            else if (wide(epi, F, d))
                rc = moe_launch_gemm_wide(epi, pairs(F, d), h_scratch, F, d, w_out, tiles, plan_hdr, (void*)y_perm, d, st, top1.perm,
                                          top1.gate_w, top1.on ? A : 0);
            else if (top1.on)
                rc = moe_launch_gemm_bf16(MOE_EPI_SCATTER, tile_m, narrow(d), cache_y, h_scratch, F, d, w_out, tiles, plan_hdr,
                                          (void*)y_perm, d, st, top1.perm, top1.gate_w, A);
            else
                rc = moe_launch_gemm_bf16(MOE_EPI_STORE, tile_m, narrow(d), cache_y, h_scratch, F, d, w_out, tiles, plan_hdr,
                                          (void*)y_perm, d, st);
            if (rc != MOE_OK) return rc;
        }
    } else {
        if (phases & 1) {
            rc = moe_launch_gemm_f32(act == MOE_SWIGLU ? MOE_EPI_SWIGLU : MOE_EPI_RELU, x_perm, A, d, n1, E, w_in, tiles, plan_hdr,
                                     h_scratch, F, st, gather.on ? gather.perm : nullptr, gather.k);
            if (rc != MOE_OK) return rc;
        }
        if (phases & 2) {
            rc = moe_launch_gemm_f32(MOE_EPI_STORE, h_scratch, A, F, d, E, w_out, tiles, plan_hdr, y_perm, d, st);
            if (rc != MOE_OK) return rc;
        }
    }
    return MOE_OK;
}

extern "C" int moe_grouped_ffn(const void* x_perm, int A, int d, int F, int E, moe_act act, moe_dtype dt,
                               const void* const* w_in, const void* const* w_out, const moe_tile* tiles,
                               int32_t* plan_hdr, int tile_m, void* h_scratch, float* y_perm, void* stream) {
    return grouped_ffn_impl(3, x_perm, A, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y_perm, stream);
}

extern "C" int moe_grouped_ffn_phase(int phase, const void* x_perm, int A, int d, int F, int E, moe_act act,
                                     moe_dtype dt, const void* const* w_in, const void* const* w_out,
                                     const moe_tile* tiles, int32_t* plan_hdr, int tile_m, void* h_scratch,
                                     float* y_perm, void* stream) {
    MOE_REQUIRE(phase == 1 || phase == 2, MOE_ERR_ARG, "moe_grouped_ffn_phase: phase %d", phase);
    return grouped_ffn_impl(phase, x_perm, A, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y_perm, stream);
}

static int top1_impl(int phases, const void* x_perm, int T, int d, int F, int E, moe_act act, moe_dtype dt,
                     const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                     int tile_m, void* h_scratch, const int32_t* perm, const float* gate_w, float* y, void* stream) {
    MOE_REQUIRE(dt == MOE_BF16, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_top1: MOE_BF16 only (dtype %d)", (int)dt);
    MOE_REQUIRE(F >= 512, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_top1: needs F >= 512 (F=%d)", F);
    MOE_REQUIRE(T == 0 || !(phases & 2) || (perm && y), MOE_ERR_ARG, "moe_grouped_ffn_top1: null pointer");
    MOE_REQUIRE((long long)T * d * 4 < (1ll << 31), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_top1: y must be smaller than 2 GiB (T=%d d=%d)", T, d);
    Top1 t;
    t.perm = perm;
    t.gate_w = gate_w;
    t.on = true;
    return grouped_ffn_impl(phases, x_perm, T, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y, stream, t);
}

extern "C" int moe_grouped_ffn_top1(const void* x_perm, int T, int d, int F, int E, moe_act act, moe_dtype dt,
                                    const void* const* w_in, const void* const* w_out, const moe_tile* tiles,
                                    int32_t* plan_hdr, int tile_m, void* h_scratch, const int32_t* perm,
                                    const float* gate_w, float* y, void* stream) {
    return top1_impl(3, x_perm, T, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, gate_w, y, stream);
}

extern "C" int moe_grouped_ffn_top1_phase(int phase, const void* x_perm, int T, int d, int F, int E, moe_act act,
                                          moe_dtype dt, const void* const* w_in, const void* const* w_out,
                                          const moe_tile* tiles, int32_t* plan_hdr, int tile_m, void* h_scratch,
                                          const int32_t* perm, const float* gate_w, float* y, void* stream) {
    MOE_REQUIRE(phase == 1 || phase == 2, MOE_ERR_ARG, "moe_grouped_ffn_top1_phase: phase %d", phase);
    return top1_impl(phase, x_perm, T, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, gate_w, y, stream);
}

static int fused_impl(int phases, const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                      const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                      int tile_m, void* h_scratch, const int32_t* perm, const float* gate_w, float* y_out, void* stream) {
    MOE_REQUIRE(dt == MOE_BF16, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: MOE_BF16 only (dtype %d)", (int)dt);
    MOE_REQUIRE(T >= 0 && k >= 1, MOE_ERR_ARG, "moe_grouped_ffn_fused: T=%d k=%d", T, k);
    MOE_REQUIRE((long long)T * k < (1ll << 30), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: T*k too large");
    const int height = tile_height(tile_m);
    MOE_REQUIRE(height == 128 || height == 256, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: bf16 tile_m=%d, must be 128 or 256", height);
    MOE_REQUIRE(height == 128 || (g_kernel_mode != 1 && moe_gemm_wide_supports(MOE_EPI_RELU, d)), MOE_ERR_UNSUPPORTED,
                "moe_grouped_ffn_fused: with 256-row tiles the row gather is done by the four-wavefront kernels only "
                "(moe_ffn_kernel_mode %d, d=%d)", g_kernel_mode, d);
    MOE_REQUIRE(d >= 256, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: needs d >= 256 (d=%d)", d);
    MOE_REQUIRE((long long)T * d * 2 < (1ll << 32), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: x must be smaller than 4 GiB (T=%d d=%d)", T, d);
    MOE_REQUIRE(T == 0 || perm, MOE_ERR_ARG, "moe_grouped_ffn_fused: null pointer");
    Gather g;
    g.perm = perm;
    g.x_rows = T;
    g.k = k;
    g.on = true;
    if (k == 1) {
        MOE_REQUIRE(F >= 512, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: top-1 needs F >= 512 (F=%d)", F);
        MOE_REQUIRE(T == 0 || !(phases & 2) || y_out, MOE_ERR_ARG, "moe_grouped_ffn_fused: null pointer");
        MOE_REQUIRE((long long)T * d * 4 < (1ll << 31), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_fused: y must be smaller than 2 GiB (T=%d d=%d)", T, d);
        Top1 t;
        t.perm = perm;
        t.gate_w = gate_w;
        t.on = true;
        return grouped_ffn_impl(phases, x, T, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y_out, stream, t, g);
    }
    return grouped_ffn_impl(phases, x, T * k, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y_out, stream, Top1(), g);
}

extern "C" int moe_grouped_ffn_fused(const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                                     const void* const* w_in, const void* const* w_out, const moe_tile* tiles,
                                     int32_t* plan_hdr, int tile_m, void* h_scratch, const int32_t* perm,
                                     const float* gate_w, float* y_out, void* stream) {
    return fused_impl(3, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, gate_w, y_out, stream);
}

extern "C" int moe_grouped_ffn_fused_phase(int phase, const void* x, int T, int d, int F, int E, int k, moe_act act,
                                           moe_dtype dt, const void* const* w_in, const void* const* w_out,
                                           const moe_tile* tiles, int32_t* plan_hdr, int tile_m, void* h_scratch,
                                           const int32_t* perm, const float* gate_w, float* y_out, void* stream) {
    MOE_REQUIRE(phase == 1 || phase == 2, MOE_ERR_ARG, "moe_grouped_ffn_fused_phase: phase %d", phase);
    return fused_impl(phase, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, gate_w, y_out, stream);
}

static int gather_impl(int phases, const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                       const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                       int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, void* stream) {
    MOE_REQUIRE(dt == MOE_F32, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_gather: MOE_F32 only (dtype %d)", (int)dt);
    MOE_REQUIRE(T >= 0 && k >= 1, MOE_ERR_ARG, "moe_grouped_ffn_gather: T=%d k=%d", T, k);
    MOE_REQUIRE((long long)T * k < (1ll << 30), MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_gather: T*k too large");
    MOE_REQUIRE(T == 0 || !(phases & 1) || perm, MOE_ERR_ARG, "moe_grouped_ffn_gather: null pointer");
    Gather g;
    g.perm = perm;
    g.x_rows = T;
    g.k = k;
    g.on = true;
    return grouped_ffn_impl(phases, x, T * k, d, F, E, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, y_perm, stream, Top1(), g);
}

extern "C" int moe_grouped_ffn_gather(const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                                      const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                                      int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, void* stream) {
    return gather_impl(3, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, y_perm, stream);
}

extern "C" int moe_grouped_ffn_gather_phase(int phase, const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                                            const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                                            int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, void* stream) {
    MOE_REQUIRE(phase == 1 || phase == 2, MOE_ERR_ARG, "moe_grouped_ffn_gather_phase: phase %d", phase);
    return gather_impl(phase, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, y_perm, stream);
}

// moe_grouped_ffn_fused and the shared expert's moe_grouped_ffn.  Where the few-row kernels serve both, each
// product of the shared expert shares the launch of the routed experts' one (33 rows of 2048 x 1408, E = 60, and
// 5632: 94 + 56 + 25 + 26 us in four launches, 108 + 70 in two): one expert's product has too few items to keep
// the memory busy by itself.  Everywhere else the calls follow one another.  phases: bits of moe_grouped_ffn_shared_phase.
static int shared_impl(int phases, const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                       const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                       int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, int shared_F,
                       const void* const* s_w_in, const void* const* s_w_out, const moe_tile* s_tiles,
                       int32_t* s_plan_hdr, int s_tile_m, void* s_h_scratch, float* s_y, void* stream) {
    MOE_REQUIRE(k >= 2, MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_shared: needs k >= 2 (k=%d)", k);
    const bool rows = dt == MOE_BF16 && act == MOE_SWIGLU && T >= 1 && E >= 1 && k >= 2 && (long long)T * k < (1ll << 30) &&
                      few_rows_call(T * k, d, F, E, act, tile_m) && few_rows_call(T, d, shared_F, 1, MOE_SWIGLU, s_tile_m);
    MOE_REQUIRE(T <= 0 || (x && w_in && w_out && y_perm && s_w_in && s_w_out && s_y), MOE_ERR_ARG, "moe_grouped_ffn_shared: null pointer");
    auto routed = [&](int p) {
        return fused_impl(p, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, nullptr, y_perm, stream);
    };
    auto shared = [&](int p) {
        return grouped_ffn_impl(p, x, T, d, shared_F, 1, MOE_SWIGLU, dt, s_w_in, s_w_out, s_tiles, s_plan_hdr, s_tile_m, s_h_scratch, s_y,
                                stream);
    };
    // (phase 0 checks the other arguments and enqueues nothing)
    int rc = routed(0);
    if (rc == MOE_OK) rc = shared(0);
    for (int p = 1; p <= 2 && rc == MOE_OK; ++p) {
        if (!(phases & p)) continue;
        rc = rows ? moe_launch_gemm_rows_shared(p, x, T, d, F, E, k, p == 1 ? w_in : w_out, tiles, plan_hdr, h_scratch, y_perm, perm, shared_F,
                                                p == 1 ? s_w_in : s_w_out, s_tiles, s_plan_hdr, s_h_scratch, s_y, (hipStream_t)stream)
                  : routed(p);
    }
    if (rc == MOE_OK && (phases & 4) && !rows) rc = shared(3);
    return rc;
}

extern "C" int moe_grouped_ffn_shared(const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                                      const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                                      int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, int shared_F,
                                      const void* const* s_w_in, const void* const* s_w_out, const moe_tile* s_tiles,
                                      int32_t* s_plan_hdr, int s_tile_m, void* s_h_scratch, float* s_y, void* stream) {
    return shared_impl(7, x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, y_perm, shared_F, s_w_in,
                       s_w_out, s_tiles, s_plan_hdr, s_tile_m, s_h_scratch, s_y, stream);
}

extern "C" int moe_grouped_ffn_shared_phase(int phase, const void* x, int T, int d, int F, int E, int k, moe_act act, moe_dtype dt,
                                            const void* const* w_in, const void* const* w_out, const moe_tile* tiles, int32_t* plan_hdr,
                                            int tile_m, void* h_scratch, const int32_t* perm, float* y_perm, int shared_F,
                                            const void* const* s_w_in, const void* const* s_w_out, const moe_tile* s_tiles,
                                            int32_t* s_plan_hdr, int s_tile_m, void* s_h_scratch, float* s_y, void* stream) {
    MOE_REQUIRE(phase >= 1 && phase <= 3, MOE_ERR_ARG, "moe_grouped_ffn_shared_phase: phase %d", phase);
    return shared_impl(1 << (phase - 1), x, T, d, F, E, k, act, dt, w_in, w_out, tiles, plan_hdr, tile_m, h_scratch, perm, y_perm,
                       shared_F, s_w_in, s_w_out, s_tiles, s_plan_hdr, s_tile_m, s_h_scratch, s_y, stream);
}
