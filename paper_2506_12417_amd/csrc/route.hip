// moe_route_topk: router logits, softmax, top-k selection (Alg. 1 step 1; section 2).
// This file: argument checks, and the kernel for fp32 inputs (and for bf16 with fewer than eight
// experts); other bf16 inputs go to route_mfma.hip.
//
// The logits are computed in fp64 on the matrix cores (v_mfma_f64_16x16x4_f64, 79 TFLOP/s: products
// of two fp32 values are exact in fp64), so the selection needs no error bound and no second
// look.  A work-group takes 16 tokens; its eight wavefronts split the experts into groups of up to two
// 16-column blocks and the contraction into 8 / GROUPS parts, whose sums are added in a fixed order
// through LDS.  Operands go straight
// from global memory to registers: a lane reads four consecutive terms of its token and the four
// matching entries of its expert's column (16 neighbouring columns per load), and gives one of
// the four to each of four matrix instructions.
// (fp32 fma tiles whose column norms were summed by an LDS atomic per entry of W_g took 111 us for
// 1501 tokens x 768, E = 16; this takes 9.  64 tokens per work-group, which fetch W_g a quarter as
// often, were no faster at any size: 33000 tokens x 768, E = 128 219 against 166 us.)
#include "common.h"
#include <climits>

namespace {

typedef __attribute__((ext_vector_type(4))) double f64x4;

__device__ __forceinline__ bool beats(double av, int ae, double bv, int be) { return av > bv || (av == bv && ae < be); }
// reductions over a group of SPAN neighbouring lanes
template <int SPAN> __device__ __forceinline__ void group_best(double& v, int& e) {
#pragma unroll
    for (int off = SPAN / 2; off >= 1; off >>= 1) {
        const double ov = __shfl_xor(v, off);
        const int oe = __shfl_xor(e, off);
        if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    }
}
template <int SPAN> __device__ __forceinline__ double group_sum(double v) {
#pragma unroll
    for (int off = SPAN / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}
template <int SPAN> __device__ __forceinline__ double group_max(double v) {
#pragma unroll
    for (int off = SPAN / 2; off >= 1; off >>= 1) { const double o = __shfl_xor(v, off); v = o > v ? o : v; }
    return v;
}
constexpr double NEG_INF = -__builtin_huge_val();

// SPAN neighbouring lanes hold one token's logits, lane l of them owning experts l, l + SPAN, ...  Picks
// the k largest (ties to the lower expert id), forms their softmax values and writes the choice.
// A chosen expert gives up its id, not only its logit: -inf is a logit that others may hold (experts
// masked by their bias), and the chosen one must not come up among those again.
template <int SPAN, int NE>
__device__ __forceinline__ void choose(const double (&v)[NE], int l, int E, int k, int renorm, int32_t* idx_row, float* w_row) {
    static_assert(SPAN >= MOE_MAX_TOPK, "lane r writes choice r");
    double m = NEG_INF, s = 0.0;
    int id[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        id[j] = l + SPAN * j < E ? l + SPAN * j : INT_MAX;
        if (id[j] != INT_MAX) m = v[j] > m ? v[j] : m;
    }
    m = group_max<SPAN>(m);
#pragma unroll
    for (int j = 0; j < NE; ++j) if (id[j] != INT_MAX) s += exp(v[j] - m);
    const double denom = group_sum<SPAN>(s);
    double p[MOE_MAX_TOPK], tot = 0.0, first = 0.0;
    int sel[MOE_MAX_TOPK];
#pragma unroll
    for (int r = 0; r < MOE_MAX_TOPK; ++r) {
        if (r < k) {
            double bv = NEG_INF;
            int be = INT_MAX;
#pragma unroll
            for (int j = 0; j < NE; ++j)
                if (id[j] != INT_MAX && beats(v[j], id[j], bv, be)) { bv = v[j]; be = id[j]; }
            group_best<SPAN>(bv, be);
#pragma unroll
            for (int j = 0; j < NE; ++j) if (id[j] == be) id[j] = INT_MAX;
            if (r == 0) first = bv;
            sel[r] = be;
            p[r] = exp(bv - first) / denom;
            tot += p[r];
        }
    }
#pragma unroll
    for (int r = 0; r < MOE_MAX_TOPK; ++r) {
        if (r < k && l == r) {
            idx_row[r] = sel[r];
            w_row[r] = (float)(renorm ? p[r] / tot : p[r]);
        }
    }
}

// (the copies state no alignment beyond the element's: x may be a view that starts anywhere)
__device__ __forceinline__ void load4(const float* p, double (&v)[4]) {
    float4 f;
    __builtin_memcpy(&f, p, sizeof f);
    v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
}
__device__ __forceinline__ void load4(const uint16_t* p, double (&v)[4]) {
    uint2 u;
    __builtin_memcpy(&u, p, sizeof u);
    v[0] = __uint_as_float(u.x << 16); v[1] = __uint_as_float(u.x & 0xffff0000u);
    v[2] = __uint_as_float(u.y << 16); v[3] = __uint_as_float(u.y & 0xffff0000u);
}

// GROUPS expert groups of NT blocks of 16 columns
template <typename XT, int GROUPS, int NT>
__global__ __launch_bounds__(512) void route_kernel(const XT* __restrict__ x, const XT* __restrict__ wg,
                                                    const float* __restrict__ bias, int T, int d, int E, int k, int renorm,
                                                    int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                                    float* __restrict__ logits_out) {
    constexpr int KSP = 8 / GROUPS, EP = GROUPS * NT * 16, TB = 16, NC = 2;
    __shared__ double part[KSP * TB * EP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const int grp = wave / KSP, ks = wave % KSP;
    const int t0 = blockIdx.x * TB;
    f64x4 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[n][r] = 0.0;
    // (tokens past T and columns past E are the last ones again: never looked at)
    const XT* xr = x + (size_t)(t0 + l16 < T ? t0 + l16 : T - 1) * d;
    int col[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) col[n] = (grp * NT + n) * 16 + l16 < E ? (grp * NT + n) * 16 + l16 : E - 1;
    // chunks of 16 terms, NC of a wavefront's chunks in flight together
    for (int k0 = ks * 16; k0 < d; k0 += KSP * 16 * NC) {
        double xv[NC][4];
        float wv[NC][NT][4];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            // (d is a multiple of 8: a lane's four terms are all inside or all past the end, where x counts
            // as zero and W_g's last entries stand in)
            const int at = k0 + c * KSP * 16 + lq * 4, in = at < d ? at : d - 4;
            load4(xr + in, xv[c]);
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int j = 0; j < 4; ++j) wv[c][n][j] = load_as_f32<XT>(wg + (size_t)(in + j) * E + col[n]);
            if (at >= d) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    xv[c][j] = 0.0;
#pragma unroll
                    for (int n = 0; n < NT; ++n) wv[c][n][j] = 0.f;
                }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int n = 0; n < NT; ++n)
                    acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[c][j], (double)wv[c][n][j], acc[n], 0, 0, 0);
    }
    // acc[n][r]: token 4 r + lq, column l16 of the block
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(ks * TB + 4 * r + lq) * EP + (grp * NT + n) * 16 + l16] = acc[n][r];
    __syncthreads();
    // A token's experts lie across SPAN lanes; with few experts a wavefront takes several tokens at once
    // (the selection is a chain of exchanges and 64-bit exponentials: with one token per wavefront,
    // two in turn, 16384 tokens x 64, E = 4 took 22 us, with four at once 9).
    constexpr int SPAN = EP < 64 ? EP : 64, NE = EP / SPAN, PER = 64 / SPAN;
    const int l = lane % SPAN;
    for (int tok = wave * PER + lane / SPAN; tok < TB; tok += 8 * PER) {
        const int t = t0 + tok;
        if (t >= T) break;
        double v[NE];
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = l + SPAN * j;
            v[j] = 0.0;
            if (e < E) {
                double s = part[tok * EP + e];
#pragma unroll
                for (int p = 1; p < KSP; ++p) s += part[(p * TB + tok) * EP + e];
                v[j] = s + (bias ? (double)bias[e] : 0.0);
                if (logits_out) logits_out[(size_t)t * E + e] = (float)v[j];
            }
        }
        choose<SPAN, NE>(v, l, E, k, renorm, idx_out + (size_t)t * k, w_out + (size_t)t * k);
    }
}

template <typename XT, int GROUPS, int NT>
int launch_route(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm,
                 int32_t* idx, float* w, float* logits, hipStream_t st) {
    hipLaunchKernelGGL((route_kernel<XT, GROUPS, NT>), dim3((T + 15) / 16), dim3(512), 0, st, (const XT*)x, (const XT*)wg, bias, T, d, E,
                       k, renorm, idx, w, logits);
    MOE_CHECK_LAUNCH("moe_route_topk");
    return MOE_OK;
}

int route_f32(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm, int32_t* idx, float* w,
              float* logits, hipStream_t st) {
    if (E <= 16) return launch_route<float, 1, 1>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 32) return launch_route<float, 1, 2>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 64) return launch_route<float, 2, 2>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 128) return launch_route<float, 4, 2>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    return launch_route<float, 8, 2>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
}

}  // namespace

// fewer than eight experts in bf16: a row of W_g is shorter than a 16-byte load
int moe_route_small(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm, int32_t* idx, float* w,
                    float* logits, hipStream_t st) {
    return launch_route<uint16_t, 1, 1>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
}

// bf16 inputs: the MFMA kernel of route_mfma.hip
int moe_route_bf16_mfma(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm,
                        int32_t* idx, float* w, float* logits, hipStream_t st);

int moe_route_bf16_packed(const void* x, const void* wgt, const float* w_norm2, const float* bias, int T, int d, int E,
                          int k, int renorm, int32_t* idx, float* w, float* logits, hipStream_t st);

extern "C" int moe_route_topk_packed(const void* x, const void* w_gate_t, const float* w_norm2, const float* bias, int T,
                                     int d, int E, int k, int renorm, moe_dtype dt, int32_t* expert_idx, float* gate_w,
                                     float* logits_out, void* stream) {
    MOE_REQUIRE(dt == MOE_BF16, MOE_ERR_UNSUPPORTED, "moe_route_topk_packed: dtype %d (bf16 only)", (int)dt);
    MOE_REQUIRE(T >= 0 && d >= 1 && E >= 1, MOE_ERR_ARG, "moe_route_topk_packed: T=%d d=%d E=%d", T, d, E);
    MOE_REQUIRE(k >= 1 && k <= E, MOE_ERR_ARG, "moe_route_topk_packed: k=%d outside [1, E=%d]", k, E);
    MOE_REQUIRE(k <= MOE_MAX_TOPK, MOE_ERR_UNSUPPORTED, "moe_route_topk_packed: k=%d > %d", k, MOE_MAX_TOPK);
    MOE_REQUIRE(E <= MOE_MAX_EXPERTS, MOE_ERR_UNSUPPORTED, "moe_route_topk_packed: E=%d > %d", E, MOE_MAX_EXPERTS);
    MOE_REQUIRE(d % 64 == 0, MOE_ERR_UNSUPPORTED, "moe_route_topk_packed: d=%d is not a multiple of 64", d);
    MOE_REQUIRE((long long)d * MOE_MAX_EXPERTS * 2 < (1ll << 31), MOE_ERR_UNSUPPORTED, "moe_route_topk_packed: d=%d too large", d);
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(x && w_gate_t && w_norm2 && expert_idx && gate_w, MOE_ERR_ARG, "moe_route_topk_packed: null pointer");
    return moe_route_bf16_packed(x, w_gate_t, w_norm2, bias, T, d, E, k, renorm, expert_idx, gate_w, logits_out,
                                 (hipStream_t)stream);
}

extern "C" int moe_route_topk(const void* x, const void* w_gate, const float* bias, int T, int d, int E, int k,
                              int renorm, moe_dtype dt, int32_t* expert_idx, float* gate_w, float* logits_out,
                              void* stream) {
    MOE_REQUIRE(moe_dtype_ok(dt), MOE_ERR_UNSUPPORTED, "moe_route_topk: dtype %d", (int)dt);
    MOE_REQUIRE(T >= 0 && d >= 1 && E >= 1, MOE_ERR_ARG, "moe_route_topk: T=%d d=%d E=%d", T, d, E);
    MOE_REQUIRE(k >= 1 && k <= E, MOE_ERR_ARG, "moe_route_topk: k=%d outside [1, E=%d]", k, E);
    MOE_REQUIRE(k <= MOE_MAX_TOPK, MOE_ERR_UNSUPPORTED, "moe_route_topk: k=%d > %d", k, MOE_MAX_TOPK);
    MOE_REQUIRE(E <= MOE_MAX_EXPERTS, MOE_ERR_UNSUPPORTED, "moe_route_topk: E=%d > %d", E, MOE_MAX_EXPERTS);
    MOE_REQUIRE(d % 8 == 0, MOE_ERR_UNSUPPORTED, "moe_route_topk: d=%d is not a multiple of 8", d);
    if (T == 0) return MOE_OK;
    MOE_REQUIRE(x && w_gate && expert_idx && gate_w, MOE_ERR_ARG, "moe_route_topk: null pointer");
    hipStream_t st = (hipStream_t)stream;
    if (dt == MOE_BF16)
        return moe_route_bf16_mfma(x, w_gate, bias, T, d, E, k, renorm, expert_idx, gate_w, logits_out, st);
    return route_f32(x, w_gate, bias, T, d, E, k, renorm, expert_idx, gate_w, logits_out, st);
}
