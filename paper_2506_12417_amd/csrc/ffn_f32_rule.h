// Which of the fp32 kernels (ffn_f32.hip) serves a product of A rows, K terms and N weight rows of E experts, and with what items.
// Plain C++, so that the host can say which kernels a set of sizes takes.
//
// Column blocks of 128 weight rows read the activations half as often; of 64 where 128 would leave fewer than four items
// per CU.  The few-row kernel where 64 would leave fewer than two (one with SwiGLU), or the experts hold few rows.  By the split
// kernel and by it, in us: 600 tokens, K = N = 1024, E = 4, k = 2 (320 items of 64) 55 and 42; 2000 tokens twice, K = 1024, N = 128, E = 4 28 and 25;
// 1300 tokens, K = N = 1024, E = 8 38 and 38; 1501 tokens twice, K = 2048, N = 768, E = 16 (660 items) 112 and 118.  Rows per expert:
// 1000 tokens of 32 experts, K = 1024, N = 2048 89 and 74; 900 of 16, K = 768, N = 1536 39 and 33; 2048 of 32 (64 rows each), K = 512, N = 2048 56 and
// 58; 4096 of 32, K = N = 1024 100 and 102.  With SwiGLU (N: gate and up) 250 tokens, K = 1024, N = 1024, E = 4 27 and 15; 40 tokens twice, K = 1024,
// N = 4096, E = 32 110 and 74; 300 of 16 77 and 57, 600 85 and 77; 240 tokens twice, K = 1000, N = 3072, E = 16 74 and 66; 2000, K = 512, N = 640, E = 8
// (360 items) 23 and 22; 1501 twice, K = 768, N = 4096, E = 16 177 and 211.
#pragma once

enum { MOE_F32_ROWS = 0, MOE_F32_SPLIT_64 = 1, MOE_F32_SPLIT_128 = 2 };     // (split: weight rows of an item)

inline int moe_f32_kernel(bool glu, long long A, long long K, long long N, long long E) {
    const long long tiles = (A + 63) / 64 + E / 2, items = tiles * ((N + 63) / 64);
    const bool in_reach = A * K < 1ll << 30 && N * K < 1ll << 30;           // of the few-row kernel's 32-bit byte offsets
    if (in_reach && (glu ? items < 256 || A <= 32 * E : items < 2 * 256 || A <= 48 * E)) return MOE_F32_ROWS;
    return tiles * ((N + 127) / 128) < 4 * 256 ? MOE_F32_SPLIT_64 : MOE_F32_SPLIT_128;
}
