// Internal interface between the FFN entry points (ffn.hip) and the bf16 MFMA kernels (ffn_bf16.hip).
#pragma once
#include "common.h"

enum { MOE_EPI_RELU = 0, MOE_EPI_SWIGLU = 1, MOE_EPI_STORE = 2, MOE_EPI_SCATTER = 3 };

// persistent grid: one work-group per CU (256 CUs; 32 per XCD, dealt round-robin)
constexpr int MOE_GEMM_GRID = 256;

// out = epilogue(a . w_e^T) over the tile table.  epi: RELU / SWIGLU write half, STORE writes fp32,
// SCATTER writes fp32 row r to out[row_token[r]] times row_gate[row_token[r]] (row_gate may be null;
// out has out_rows rows).
// tile_m: 128 or 256 (the tile height the table was planned with).  narrow: with tile_m = 128,
// use column blocks of 128 instead of 256 outputs (ignored for SWIGLU).  cache: a hint for 128-row tiles.
enum {
    MOE_CACHE_PLAIN = 0,
    MOE_CACHE_WEIGHTS_ONCE = 1,    // an expert's weights are hardly shared between work items
    MOE_CACHE_LARGE_OUT = 2        // the output is larger than the L2s
};
int moe_launch_gemm_bf16(int epi, int tile_m, int narrow, int cache, const void* a, int K, int N, const void* const* w,
                         const moe_tile* tiles, int32_t* hdr, void* out, int ld_out, hipStream_t st,
                         const int32_t* row_token = nullptr, const float* row_gate = nullptr, int out_rows = 0);

// The first product with the row gather folded in (128-row tiles, RELU or SWIGLU; K / 64 >= 4):
// row r of the table's row space is row row_src[r] / src_div of x [x_rows, K].
int moe_launch_gemm_bf16_gather(int epi, int cache, const void* x, int x_rows, int K, int N, const void* const* w,
                                const moe_tile* tiles, int32_t* hdr, void* out, int ld_out, hipStream_t st,
                                const int32_t* row_src, int src_div);

// The same products by the kernels of ffn_stream.hip (128-row tiles; weights streamed global ->
// registers: for experts that hold few rows each, where a product's time is the fetch of its
// weights).  Same results, bit for bit.  narrow: items of 128 instead of 256 weight rows, two
// work-groups per CU.  moe_gemm_stream_supports: whether those kernels cover (epilogue, K).
bool moe_gemm_stream_supports(int epi, int K);
int moe_launch_gemm_stream(int epi, int narrow, const void* a, int K, int N, const void* const* w, const moe_tile* tiles,
                           int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_token = nullptr,
                           const float* row_gate = nullptr, int out_rows = 0);
int moe_launch_gemm_stream_gather(int narrow, const void* x, int x_rows, int K, int N, const void* const* w,
                                  const moe_tile* tiles, int32_t* hdr, void* out, int ld_out, hipStream_t st,
                                  const int32_t* row_src, int src_div);

// The same products for 256-row tiles, or (pairs) neighbouring 128-row tiles of an expert taken two at a time, by the
// kernels of ffn_wide.hip (four wavefronts of 128 x 128 per work-group instead of eight of 128 x 64: less
// LDS traffic per multiply-add, which is what the power-bound case pays for).  Same results, bit for bit; all four epilogues, and the first
// product with the row gather folded in (arguments as for the launchers above).
enum { MOE_PAIRS_ONE_ROUND = 1, MOE_PAIRS_MANY = 2 };
constexpr int MOE_PAIRS_MAX_TILES = 3068;      // single tiles of a work-group's share that can be paired
bool moe_gemm_wide_supports(int epi, int K);
int moe_launch_gemm_wide(int epi, int pairs, const void* a, int K, int N, const void* const* w, const moe_tile* tiles,
                         const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_token = nullptr,
                         const float* row_gate = nullptr, int out_rows = 0);
int moe_launch_gemm_wide_gather(int epi, int pairs, const void* x, int x_rows, int K, int N, const void* const* w,
                                const moe_tile* tiles, const int32_t* hdr, void* out, int ld_out, hipStream_t st,
                                const int32_t* row_src, int src_div);

// The same products for experts that hold a handful of rows each, by the kernels of ffn_rows.hip
// (tiles of at most 128 rows; the fetch of the weights is the work and uses the whole chip,
// whatever the plan's bins).  All four epilogues, and the first product with the row gather folded
// in (arguments as for the launchers above; A rows in the table).
int moe_launch_gemm_rows(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                         const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_token = nullptr,
                         const float* row_gate = nullptr);
int moe_launch_gemm_rows_gather(int epi, const void* x, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                                const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src, int src_div);

// The same for the routed SwiGLU experts (rows gathered from x, k > 1) and a shared SwiGLU expert over all
// T rows of x (one expert's plan) in one launch per product (phase 1, 2); the shared expert has the same d.
int moe_launch_gemm_rows_shared(int phase, const void* x, int T, int d, int F, int E, int k, const void* const* w, const moe_tile* tiles,
                                const int32_t* hdr, void* h, float* y_perm, const int32_t* perm, int shared_F,
                                const void* const* s_w, const moe_tile* s_tiles, const int32_t* s_hdr, void* s_h, float* s_y,
                                hipStream_t st);

// The fp32 products (ffn_f32.hip; tiles of at most 64 rows, RELU / SWIGLU / STORE, all of fp32).  row_src: row r
// of the table's row space is row row_src[r] / src_div of a.
int moe_launch_gemm_f32(int epi, const void* a, int A, int K, int N, int E, const void* const* w, const moe_tile* tiles,
                        const int32_t* hdr, void* out, int ld_out, hipStream_t st, const int32_t* row_src = nullptr, int src_div = 1);

// MOE_OK if the current device is the GPU the persistent launches are laid out for (256 compute
// units in 8 XCDs), else MOE_ERR_UNSUPPORTED.
int moe_check_gemm_device();
