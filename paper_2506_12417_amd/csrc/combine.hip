// moe_unpermute_combine: original token order restored, the k expert outputs of a token
// weighted by the router's values and summed (Alg. 1 step 6, "reconstruct"; section 2).
// One float4 of one output row per thread; j ascending, so the sum has a fixed order.
// HBM bound: A*d*4 bytes read (+ T*d*4 for the shared expert), T*d*4 written, every byte once: all
// of it bypasses the caches' keeping (nontemporal), and a thread asks for its k rows together.
// 20011 x 8 rows of 1032: 4.3 -> 5.8 TB/s; 8192 x 2 rows of 4096: 5.4 -> 6.2 TB/s.
// An assignment without a row (inv_perm negative) adds nothing if its weight is zero and makes its
// token NaN otherwise; the first row is fetched in its place and not used.
#include "common.h"

namespace {
constexpr int NTH = 256, MAXK = MOE_MAX_TOPK;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// K: experts per token, 0 for more than MAXK (in groups of MAXK)
template <int K>
__global__ __launch_bounds__(NTH) void combine_kernel(const f32x4* __restrict__ y_perm, const int32_t* __restrict__ inv_perm,
                                                      const float* __restrict__ gate_w, const f32x4* __restrict__ shared,
                                                      unsigned total, unsigned vpr, int k_any, f32x4* __restrict__ y) {
    const unsigned i = blockIdx.x * NTH + threadIdx.x;
    if (i >= total) return;
    const unsigned t = i / vpr, v = i - t * vpr;
    const int k = K ? K : k_any;
    const size_t a0 = (size_t)t * k;
    constexpr int G = K ? K : MAXK;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int j0 = 0; j0 < k; j0 += G) {
        f32x4 r[G];
        float w[G];
        int row[G];
#pragma unroll
        for (int j = 0; j < G; ++j) {
            const int jj = K ? j : (j0 + j < k ? j0 + j : k - 1);
            w[j] = gate_w ? gate_w[a0 + jj] : 1.f;
            row[j] = inv_perm[a0 + jj];
            r[j] = __builtin_nontemporal_load(y_perm + (size_t)(row[j] < 0 ? 0 : row[j]) * vpr + v);
        }
#pragma unroll
        for (int j = 0; j < G; ++j)
            if (K || j0 + j < k) {
                const float none = w[j] == 0.f ? 0.f : __builtin_nanf("");
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] = fmaf(w[j], row[j] < 0 ? none : r[j][c], acc[c]);
            }
    }
    if (shared) {
        const f32x4 s = __builtin_nontemporal_load(shared + i);
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] += s[c];
    }
    __builtin_nontemporal_store(acc, y + i);
}
}  // namespace

extern "C" int moe_unpermute_combine(const float* y_perm, const int32_t* inv_perm, const float* gate_w,
                                     const float* shared, int T, int d, int k, float* y, void* stream) {
    MOE_REQUIRE(T >= 0 && d >= 1 && k >= 1, MOE_ERR_ARG, "moe_unpermute_combine: T=%d d=%d k=%d", T, d, k);
    MOE_REQUIRE(d % 4 == 0, MOE_ERR_UNSUPPORTED, "moe_unpermute_combine: d=%d is not a multiple of 4", d);
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(y_perm && inv_perm && y, MOE_ERR_ARG, "moe_unpermute_combine: null pointer");
    // (slices of whole tokens whose float4s a 32-bit index counts)
    const unsigned vpr = (unsigned)d / 4;
    const long long slice = (1ll << 31) / vpr;
    for (long long t0 = 0; t0 < T; t0 += slice) {
        const unsigned total = (unsigned)((T - t0 < slice ? T - t0 : slice) * vpr);
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3((total + NTH - 1) / NTH), dim3(NTH), 0, (hipStream_t)stream, (const f32x4*)y_perm,
                               inv_perm + (size_t)t0 * k, gate_w ? gate_w + (size_t)t0 * k : nullptr,
                               shared ? (const f32x4*)shared + (size_t)t0 * vpr : nullptr, total, vpr, k,
                               (f32x4*)y + (size_t)t0 * vpr);
        };
        switch (k) {
            case 1: go(combine_kernel<1>); break;
            case 2: go(combine_kernel<2>); break;
            case 3: go(combine_kernel<3>); break;
            case 4: go(combine_kernel<4>); break;
            case 5: go(combine_kernel<5>); break;
            case 6: go(combine_kernel<6>); break;
            case 7: go(combine_kernel<7>); break;
            case 8: go(combine_kernel<8>); break;
            default: go(combine_kernel<0>); break;
        }
    }
    MOE_CHECK_LAUNCH("moe_unpermute_combine");
    return MOE_OK;
}
