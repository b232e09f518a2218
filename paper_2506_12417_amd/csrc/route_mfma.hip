// moe_route_topk and moe_route_topk_packed for bf16 inputs: the router product on the matrix cores
// (Alg. 1 step 1).
//
// One work-group takes 32 tokens.  Logits x.W_g are accumulated by v_mfma_f32_32x32x16_bf16 in
// chunks of KACC terms (bf16 x bf16 products are exact in fp32); each chunk's fp32 result is added
// into fp64 accumulators, so only the rounding inside a chunk counts: |error| <= c * |x_t| * |w_e|
// with c = (2*KACC+6) * 2^-24 (two roundings per term allowed for, since the accumulation order
// inside the instruction is not specified).  A token whose deciding gaps are all wider than twice
// that bound keeps its fp32 selection; the others get the logits of every expert that could still
// reach the top k recomputed in fp64, so expert indices and their order are those of exact
// arithmetic (ties to the lower index).
//
// The wavefronts of a work-group split the experts into blocks of 32 (NB blocks) and, when there
// are fewer than four blocks, also the contraction (KSP parts); the partial sums of the parts are
// added in a fixed order through LDS.  The two kernels differ in how the operands reach LDS:
// route_packed_kernel reads a W_g prepared by moe_pack_router, route_plain_kernel W_g as given.
//
// Selection: eight or sixteen threads scan one token's logits from LDS, keep a sorted top-(k+1)
// list in registers, and merge the lists with DPP exchanges inside their group of lanes.
#include "common.h"
#include "route_stage.h"
#include <climits>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef u32x4 frag_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

// the two bf16 values of a 32-bit word.  (A value, not an expression: __builtin_bit_cast of a vector's
// element written in place, `v[i]`, takes the vector's first element whatever i is.)
__device__ __forceinline__ bf16x2 bf16_pair(unsigned word) { return __builtin_bit_cast(bf16x2, word); }

constexpr int KC = 64;                 // terms per chunk (four MFMAs)
// Terms per fp32 accumulation.  Fewer make the bound on a logit's error tighter, and with it the share
// of tokens that the exact path has to look at again (which is what a work-group then waits for):
// 256 terms: 34.3 us for 8192 tokens x 2048, E = 60, k = 4, 51 us at E = 256, k = 8; 64 terms: 26.7 and 38.
constexpr int KACC = 64;
constexpr int MAXR = MOE_MAX_TOPK + 1;
constexpr float NEG_INF = -__builtin_huge_valf();

__device__ __forceinline__ bool beats(float av, int ae, float bv, int be) { return av > bv || (av == bv && ae < be); }
__device__ __forceinline__ bool beats(double av, int ae, double bv, int be) { return av > bv || (av == bv && ae < be); }

// exchange inside groups of 4 (steps 0, 1), 8 (step 2) and 16 (step 3) neighbouring lanes
template <int STEP> __device__ __forceinline__ int dpp_xchg(int v) {
    if (STEP == 0) return __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, false);    // quad_perm [1,0,3,2]
    if (STEP == 1) return __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, false);    // quad_perm [2,3,0,1]
    if (STEP == 2) return __builtin_amdgcn_update_dpp(v, v, 0x141, 0xf, 0xf, false);   // row_half_mirror
    return __builtin_amdgcn_update_dpp(v, v, 0x140, 0xf, 0xf, false);                  // row_mirror
}
template <int STEP> __device__ __forceinline__ float dpp_xchg(float v) {
    return __int_as_float(dpp_xchg<STEP>(__float_as_int(v)));
}
template <int TPT> __device__ __forceinline__ float group_max(float v) {
    v = fmaxf(v, dpp_xchg<0>(v));
    v = fmaxf(v, dpp_xchg<1>(v));
    if (TPT >= 8) v = fmaxf(v, dpp_xchg<2>(v));
    if (TPT == 16) v = fmaxf(v, dpp_xchg<3>(v));
    return v;
}
// fixed pairing order, so every lane of the group gets the same bits
template <int TPT> __device__ __forceinline__ float group_sum(float v) {
    v += dpp_xchg<0>(v);
    v += dpp_xchg<1>(v);
    if (TPT >= 8) v += dpp_xchg<2>(v);
    if (TPT == 16) v += dpp_xchg<3>(v);
    return v;
}
template <int TPT> __device__ __forceinline__ void group_best(float& v, int& e) {
    float ov; int oe;
    ov = dpp_xchg<0>(v); oe = dpp_xchg<0>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    ov = dpp_xchg<1>(v); oe = dpp_xchg<1>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    if (TPT >= 8) { ov = dpp_xchg<2>(v); oe = dpp_xchg<2>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; } }
    if (TPT == 16) { ov = dpp_xchg<3>(v); oe = dpp_xchg<3>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; } }
}

// the same for doubles: exchanges inside a row of 16 lanes stay in the vector unit (a __shfl goes through
// LDS and takes ten times as long)
template <int STEP> __device__ __forceinline__ double dpp_xchg(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)dpp_xchg<STEP>((int)(unsigned)u), hi = (unsigned)dpp_xchg<STEP>((int)(unsigned)(u >> 32));
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double lane_f64(double v, int lane) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
__device__ __forceinline__ double row_sum_f64(double v) {
    v += dpp_xchg<0>(v);
    v += dpp_xchg<1>(v);
    v += dpp_xchg<2>(v);
    v += dpp_xchg<3>(v);
    return v;
}
__device__ __forceinline__ double wave_sum_f64(double v) {
    v = row_sum_f64(v);
    return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
// the best of each row of 16 lanes, or (all) of the wavefront
__device__ __forceinline__ void row_best_f64(double& v, int& e, bool all) {
    double ov; int oe;
    ov = dpp_xchg<0>(v); oe = dpp_xchg<0>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    ov = dpp_xchg<1>(v); oe = dpp_xchg<1>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    ov = dpp_xchg<2>(v); oe = dpp_xchg<2>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    ov = dpp_xchg<3>(v); oe = dpp_xchg<3>(e); if (beats(ov, oe, v, e)) { v = ov; e = oe; }
    if (all) {
#pragma unroll
        for (int off = 16; off <= 32; off <<= 1) {
            ov = __shfl_xor(v, off);
            oe = __shfl_xor(e, off);
            if (beats(ov, oe, v, e)) { v = ov; e = oe; }
        }
    }
}

// exp(v) = 2^t for t = v log2(e), with what the rounding of t took away put back (v is up to tens, so t alone costs several
// units in the last place of the result).
__device__ __forceinline__ float gate_exp(float v) {
    constexpr float L = 1.44269504088896340736f, L_REST = (float)(1.44269504088896340736 - (double)L), LN2 = 0.69314718055994530942f;
    const float t = v * L, rest = fmaf(v, L_REST, fmaf(v, L, -t)), e = __builtin_amdgcn_exp2f(t);
    return e > 0.f ? fmaf(e, rest * LN2, e) : e;     // (rest is no number for an infinite v)
}

// LDS of the phases after the product (it reuses the memory of the operand staging).
template <int NB, int KSP>
struct RouteLds {
    static constexpr int NWV = NB * KSP, NTHR = NWV * 64, TB = 32, EPT = 32 * NB;
    static constexpr int PL = EPT + 4;               // pitch of a logit row (floats)
    static constexpr int LIST = MOE_MAX_EXPERTS + 32;    // entries of a wavefront's candidate list
    static constexpr int SLAB = KSP > 1 ? KSP * TB * EPT * 8 : 0;
    static constexpr int CAND = NWV * LIST * 12;
    static constexpr int REGION0 = SLAB > CAND ? SLAB : CAND;
    static constexpr size_t BYTES = REGION0 + (size_t)TB * PL * 4 + KSP * TB * 4 + 4 * TB * 4 + 2 * NWV * 4 + NWV * 4 + 16;
};

// What a thread needs of the bias: fetched before the product, so that its latency passes under it.
struct RouteBias {
    float column;          // of the logits that this thread forms
    float largest;         // |bias| of expert `tid`: this thread's share of the largest one
};
template <int NB, int KSP>
__device__ __forceinline__ RouteBias route_bias(const float* __restrict__ bias, int E) {
    typedef RouteLds<NB, KSP> L;
    static_assert(L::NTHR % L::EPT == 0, "one thread per expert at least, and one column per thread");
    const int tid = threadIdx.x;
    const int e = KSP > 1 ? tid % L::EPT : (tid >> 6) * 32 + (tid & 31);
    RouteBias b = {0.f, 0.f};
    if (bias && e < E) b.column = bias[e];
    if (bias && tid < E) b.largest = fmaxf(0.f, fabsf(bias[tid]));       // (a NaN does not count)
    return b;
}

// Logits, softmax, top-k and the exact path, from the wavefronts' fp64 sums: acc64[r] = token
// 8*(r/4) + 4*lhi + r%4, expert nbi*32 + l32, contraction part ksi.  xsq: this lane's share of the token
// norms (wavefronts of expert block 0).  w2: this thread's share of the largest squared column
// norm.  All threads of the work-group arrive with the staging memory no longer in use.
template <int NB, int KSP, int RMAX, bool PACKED>
__device__ __forceinline__ void route_finish(unsigned char* smem, const double (&acc64)[16], float xsq, float w2, const RouteBias& mine_b,
                                             const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg,
                                             const float* __restrict__ bias, int T, int d, int E, int k, int renorm,
                                             int32_t* __restrict__ idx_out, float* __restrict__ w_out,
                                             float* __restrict__ logits_out) {
    typedef RouteLds<NB, KSP> L;
    constexpr int NWV = L::NWV, NTHR = L::NTHR, TB = L::TB, EPT = L::EPT, PL = L::PL;
    constexpr int TPT = NTHR / TB >= 16 && EPT >= 64 ? 16 : 8;    // threads per token in the selection
    double* slab = reinterpret_cast<double*>(smem);  // [KSP][32][EPT], later the candidate lists
    float* ls = reinterpret_cast<float*>(smem + L::REGION0);     // logits [32][PL]
    float* xn2p = ls + TB * PL;                      // [KSP][32]
    int* flag_tok = reinterpret_cast<int*>(xn2p + KSP * TB);
    float* flag_thr = reinterpret_cast<float*>(flag_tok + TB);
    float* flag_max = flag_thr + TB;
    float* flag_den = flag_max + TB;
    float* red = flag_den + TB;                      // [2 * NWV]
    int* n_cand = reinterpret_cast<int*>(red + 2 * NWV);         // [NWV]
    int* n_flag = n_cand + NWV;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nbi = wave / KSP, ksi = wave % KSP;
    const int t0 = blockIdx.x * TB;

    if (tid == 0) *n_flag = 0;

    // ---- logits.  acc64[r]: token 8*(r/4) + 4*lhi + r%4, expert nbi*32 + l32.
    if (KSP > 1) {                                   // the partial sums of the contraction parts, fixed order
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int tok = 8 * (r >> 2) + 4 * lhi + (r & 3);
            slab[(ksi * TB + tok) * EPT + nbi * 32 + l32] = acc64[r];
        }
        __syncthreads();
        for (int i = tid; i < TB * EPT; i += NTHR) {
            const int tok = i / EPT, e = i % EPT;
            if (e < E) {
                double v = slab[i];
#pragma unroll
                for (int p = 1; p < KSP; ++p) v += slab[p * TB * EPT + i];
                const float l = (float)(v + (double)mine_b.column);
                ls[tok * PL + e] = l;
                if (logits_out && t0 + tok < T) logits_out[(size_t)(t0 + tok) * E + e] = l;
            }
        }
    } else {
        const int e = nbi * 32 + l32;
        const double be = (double)mine_b.column;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int tok = 8 * (r >> 2) + 4 * lhi + (r & 3);
            const float l = (float)(acc64[r] + be);
            if (e < E) {
                ls[tok * PL + e] = l;
                if (logits_out && t0 + tok < T) logits_out[(size_t)(t0 + tok) * E + e] = l;
            }
        }
    }
    // token norms: the two k-halves of a token sit in lanes l and l+32; the parts are added in a fixed order
    xsq += __shfl_xor(xsq, 32);
    if (nbi == 0 && lhi == 0) xn2p[ksi * TB + l32] = xsq;
    {   // largest column norm and largest |bias|
        w2 = moe_wave_max_nonneg(w2);
        const float bm = moe_wave_max_nonneg(mine_b.largest);
        if (lane == 0) { red[wave] = w2; red[NWV + wave] = bm; }
    }
    __syncthreads();
    float wmax2 = 0.f, bmax = 0.f;
#pragma unroll
    for (int w = 0; w < NWV; ++w) { wmax2 = fmaxf(wmax2, red[w]); bmax = fmaxf(bmax, red[NWV + w]); }
    const float wn_max = sqrtf(wmax2) * 1.0001f;
    const int rounds = (k + 1 < E) ? k + 1 : E;
    const float u = 5.9604645e-8f;   // 2^-24

    // ---- selection: TPT threads per token; thread `sub` takes the CPT
    // consecutive experts from sub * CPT on, fetched with four-float reads before the scan (a read
    // per expert inside the scan made it wait for LDS at every step)
    if (tid < TB * TPT) {
        constexpr int CPT = EPT / TPT;
        static_assert(CPT % 4 == 0 && PL % 4 == 0, "four-float reads of a logit row");
        const int tok = tid / TPT, sub = tid % TPT, t = t0 + tok;
        const float* row = ls + tok * PL;
        float mine[CPT];
#pragma unroll
        for (int j = 0; j < CPT; j += 4) {
            const float4 q = *reinterpret_cast<const float4*>(row + sub * CPT + j);
            mine[j] = q.x; mine[j + 1] = q.y; mine[j + 2] = q.z; mine[j + 3] = q.w;
        }
        float lv[RMAX];
        int le[RMAX];
#pragma unroll
        for (int r = 0; r < RMAX; ++r) { lv[r] = NEG_INF; le[r] = INT_MAX; }
        float m = NEG_INF;
#pragma unroll
        for (int j = 0; j < CPT; ++j) {
            const int ve = sub * CPT + j;
            const float v = ve < E ? mine[j] : NEG_INF;          // (columns past E hold nothing)
            mine[j] = v;
            m = fmaxf(m, v);
            // sorted insertion, static indices (rising experts: among equals the one before stays ahead;
            // an entry that holds nothing yet gives way to anything, a logit of -inf included).  The
            // entries behind its place all move down one, equal ones too: every place compares the new
            // logit with its own entry and the one above it, from the last place up.
            if (v > lv[RMAX - 1] || (le[RMAX - 1] == INT_MAX && v == v && ve < E)) {
#pragma unroll
                for (int r = RMAX - 1; r >= 0; --r) {
                    const bool here = v > lv[r] || le[r] == INT_MAX;
                    const bool above = r > 0 && (v > lv[r > 0 ? r - 1 : 0] || le[r > 0 ? r - 1 : 0] == INT_MAX);
                    lv[r] = above ? lv[r > 0 ? r - 1 : 0] : here ? v : lv[r];
                    le[r] = above ? le[r > 0 ? r - 1 : 0] : here ? ve : le[r];
                }
            }
        }
        m = group_max<TPT>(m);
        float s[4] = {0.f, 0.f, 0.f, 0.f};                       // (four short sums: half the rounding of one)
#pragma unroll
        for (int j = 0; j < CPT; ++j) s[j & 3] += sub * CPT + j < E ? gate_exp(mine[j] - m) : 0.f;
        const float denom = group_sum<TPT>((s[0] + s[1]) + (s[2] + s[3]));
        float sel_v[RMAX];
        int sel_e[RMAX];
#pragma unroll
        for (int r = 0; r < RMAX; ++r) {
            sel_v[r] = NEG_INF; sel_e[r] = INT_MAX;
            if (r < rounds) {
                float bv = lv[0];
                int be = le[0];
                group_best<TPT>(bv, be);
                sel_v[r] = bv;
                sel_e[r] = be;
                if (le[0] == be) {                               // the winner's owner pops its head
#pragma unroll
                    for (int i = 0; i + 1 < RMAX; ++i) { lv[i] = lv[i + 1]; le[i] = le[i + 1]; }
                    lv[RMAX - 1] = NEG_INF; le[RMAX - 1] = INT_MAX;
                }
            }
        }
        float xs2 = xn2p[tok];
#pragma unroll
        for (int p = 1; p < KSP; ++p) xs2 += xn2p[p * TB + tok];
        const float xn = sqrtf(xs2) * 1.0001f;
        const float tau = 2.1f * u * ((2 * KACC + 6) * xn * wn_max + bmax);
        bool near = false;
#pragma unroll
        for (int r = 0; r + 1 < RMAX; ++r)
            if (r + 1 < rounds && sel_v[r] - sel_v[r + 1] < tau) near = true;
        if (t < T && sub == 0) {
            if (!near) {
                float p[RMAX], tot = 0.f;
#pragma unroll
                for (int r = 0; r < RMAX; ++r)
                    if (r < k) { p[r] = gate_exp(sel_v[r] - m); tot += p[r]; }
                const float over = renorm && denom == denom ? tot : denom;     // (a logit that is no number: nor is any gate)
#pragma unroll
                for (int r = 0; r < RMAX; ++r)
                    if (r < k) {
                        idx_out[(size_t)t * k + r] = sel_e[r];
                        w_out[(size_t)t * k + r] = p[r] / over;     // (one rounding; renormalised, the sum over all cancels)
                    }
            } else {
                float last = sel_v[0];                           // the k-th choice: what lies tau below it cannot be among them
#pragma unroll
                for (int r = 1; r < RMAX; ++r) if (r < k) last = sel_v[r];
                const int f = atomicAdd(n_flag, 1);
                flag_tok[f] = tok;
                flag_thr[f] = last - tau;
                flag_max[f] = m;
                flag_den[f] = denom;
            }
        }
    }
    __syncthreads();

    // ---- exact path for the flagged tokens: every expert whose fp32 logit could still reach the top k is recomputed in fp64, for
    // the decision and for its gate.  A round takes as many flagged tokens as there are wavefronts: each wavefront lists one token's
    // candidates, then all of them share out the (token, candidate) pairs, a memory latency each, and each selects for its token: up
    // to 64 candidates a lane each, which counts those that beat its own.  What it costs is a chain of latencies (256 experts, k = 8: 20
    // to 30 us of a work-group's time where a token is flagged), so the sums go through the vector unit's lane exchanges
    // (through LDS: 8 us more).  Sharing a candidate's terms out over the wavefronts was slower (64-lane sums for everybody), and so
    // were 32 instead of 16 loads in flight (20011 tokens, E = 256: 17 us more).  (Candidates down from the k-th instead of the k + 1-th
    // choice, chosen at once instead of one after the other: 20011 x 1032, E = 256, k = 8 112 -> 102 us; 619 x 1792, E = 83, k = 6 71 -> 64;
    // 8192 x 2048, E = 256, k = 8, W_g prepared, 45 -> 41.  Recomputing only the candidates with another one within tau, which decide
    // just as well, takes 82, 44 and 36, but leaves the other choices' gates to fp32 logits.)
    constexpr int CJ = (MOE_MAX_EXPERTS + 63) / 64;
    double* cand_v = slab;                                       // [NWV][LIST]
    int* cand_e = reinterpret_cast<int*>(slab + NWV * L::LIST);  // [NWV][LIST]
    const int nf = *n_flag;
    for (int f0 = 0; f0 < nf; f0 += NWV) {
        const int f = f0 + wave;
        int nc = 0;
        if (f < nf) {
            const int tok = flag_tok[f];
            const float thr = flag_thr[f];
            for (int e0 = 0; e0 < E; e0 += 64) {
                const int e = e0 + lane;
                const bool in = e < E && ls[tok * PL + e] >= thr;
                const unsigned long long mask = __ballot(in);
                if (in) cand_e[wave * L::LIST + nc + __popcll(mask & ((1ull << lane) - 1ull))] = e;
                nc += __popcll(mask);
            }
        }
        if (lane == 0) n_cand[wave] = nc;
        __syncthreads();
        for (int s = 0, p = wave; s < NWV; ++s) {
            const int n = __builtin_amdgcn_readfirstlane(n_cand[s]);
            for (; p < n; p += NWV) {
                const int t = t0 + flag_tok[f0 + s], ce = __builtin_amdgcn_readfirstlane(cand_e[s * L::LIST + p]);
                const uint16_t* xr = x + (size_t)t * d;
                double psum = 0.0, psum1 = 0.0;
                if constexpr (PACKED) {                      // both operand rows are contiguous
                    const uint16_t* wr = wg + (size_t)ce * d;
                    for (int i0 = lane * 8; i0 < d; i0 += 4 * 64 * 8) {   // 8 terms per lane and 16-byte load, eight loads in flight
                        frag_t xv[4], wv[4];
#pragma unroll
                        for (int u2 = 0; u2 < 4; ++u2) {
                            xv[u2] = wv[u2] = frag_t{0u, 0u, 0u, 0u};
                            if (i0 + u2 * 512 < d) {
                                xv[u2] = *(const frag_t*)(xr + i0 + u2 * 512);
                                wv[u2] = *(const frag_t*)(wr + i0 + u2 * 512);
                            }
                        }
#pragma unroll
                        for (int u2 = 0; u2 < 4; ++u2)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const unsigned xw = xv[u2][i], ww = wv[u2][i];
                                psum = fma((double)__uint_as_float(xw << 16), (double)__uint_as_float(ww << 16), psum);
                                psum1 = fma((double)__uint_as_float(xw & 0xffff0000u), (double)__uint_as_float(ww & 0xffff0000u), psum1);
                            }
                    }
                } else {
                    for (int i0 = lane; i0 < d; i0 += 64 * 8) {        // 16 loads in flight per lane
                        float xa[8], wa[8];
#pragma unroll
                        for (int u2 = 0; u2 < 8; ++u2) {
                            const int i = i0 + 64 * u2;
                            xa[u2] = i < d ? bf16_to_f32(xr[i]) : 0.f;
                            wa[u2] = i < d ? bf16_to_f32(wg[(size_t)i * E + ce]) : 0.f;
                        }
#pragma unroll
                        for (int u2 = 0; u2 < 8; ++u2) psum = fma((double)xa[u2], (double)wa[u2], psum);
                    }
                }
                const double tot = wave_sum_f64(psum + psum1) + (bias ? (double)bias[ce] : 0.0);
                if (lane == 0) cand_v[s * L::LIST + p] = tot;
            }
            p -= n;
        }
        __syncthreads();
        if (f < nf && nc <= 64) {                                // a candidate's place: how many beat it
            const int t = t0 + flag_tok[f], at = wave * L::LIST + lane;
            const double v = lane < nc ? cand_v[at] : -__builtin_huge_val();
            const int e = lane < nc ? cand_e[at] : INT_MAX;
            int place = 0;
            for (int j = 0; j < nc; ++j) place += beats(lane_f64(v, j), __builtin_amdgcn_readlane(e, j), v, e) ? 1 : 0;
            // (logits that are no numbers are no candidates: with fewer than k others, the places behind them name no expert)
            if (lane >= nc) place = lane;
            const bool chosen = place < k;
            const double p = exp(v - (double)flag_max[f]) / (double)flag_den[f];
            if (chosen) cand_v[wave * L::LIST + place] = p;      // (every lane has read its own)
            double tot = 0.0;
            for (int r = 0; r < k; ++r) tot += cand_v[wave * L::LIST + r];
            if (chosen) {
                idx_out[(size_t)t * k + place] = e;
                w_out[(size_t)t * k + place] = (float)(renorm ? p / tot : p);
            }
        } else if (f < nf) {
            const int t = t0 + flag_tok[f];
            double cv[CJ];
            int ce_[CJ];
#pragma unroll
            for (int j = 0; j < CJ; ++j) {
                const int c = lane + 64 * j;
                cv[j] = c < nc ? cand_v[wave * L::LIST + c] : -__builtin_huge_val();
                ce_[j] = c < nc ? cand_e[wave * L::LIST + c] : INT_MAX;
            }
            // (lane r < k of the first row keeps the r-th choice: one exponential for all of them)
            double mine = 0.0;
            int mine_e = 0;
            for (int r = 0; r < k; ++r) {
                double bv = -__builtin_huge_val();
                int be = INT_MAX;
#pragma unroll
                for (int j = 0; j < CJ; ++j)
                    if (beats(cv[j], ce_[j], bv, be)) { bv = cv[j]; be = ce_[j]; }
                row_best_f64(bv, be, nc > 16);               // (up to 16 candidates sit in the first row)
#pragma unroll
                for (int j = 0; j < CJ; ++j)
                    if (ce_[j] == be) { cv[j] = -__builtin_huge_val(); ce_[j] = INT_MAX; }
                if (lane == r) { mine = bv; mine_e = be; }
            }
            const double p = exp(mine - (double)flag_max[f]) / (double)flag_den[f];
            double tot = 0.0;
            for (int r = 0; r < k; ++r) tot += lane_f64(p, r);
            if (lane < k) {
                idx_out[(size_t)t * k + lane] = mine_e;
                w_out[(size_t)t * k + lane] = (float)(renorm ? p / tot : p);
            }
        }
        __syncthreads();                                     // (the lists are reused)
    }
}


// =========================================================================================
// Router with a prepared W_g (moe_pack_router): W_g^T [E,d], so the contraction index is
// contiguous for both operands.  Both are staged through LDS by global -> LDS loads of whole
// 128-byte lines (a stage = 64 * KSP contraction terms of the 32 tokens and of all experts; three or
// four stages in flight, one barrier per stage), and the MFMA fragments are read from there.
// (Fetching the fragments straight from global memory, 16 bytes per lane, touched 32 lines per
// load for 32 bytes each and left the kernel waiting on the vector cache: 20 us of its 34 on
// 16384 tokens x 768.)
//
// One work-group = 32 tokens.  Its wavefronts split the experts into blocks of 32 (NB blocks)
// and, when there are fewer than four blocks, also the contraction (KSP parts): wavefront
// (block, part) takes the 64-term chunks part, part+KSP, ... for its 32 experts.  A wavefront's
// fp32 MFMA accumulator collects up to KACC terms before it is added into fp64 sums (same error
// model as above, with KACC-term chunks); the KSP partial sums are added in a fixed order
// through LDS.  The staging ring shares its LDS with the buffers of the later phases.
typedef __attribute__((address_space(3))) void lds_void_t;
constexpr int ROUTE_RING = 3;          // stages of the prepared-router kernel's staging ring
// s_waitcnt on vmcnt only (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[15:14])
#define MOE_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))

// (the body is a __device__ function: buffer-descriptor types exist on the device side only)
template <int NB, int KSP, int RMAX>   // expert blocks, contraction parts, depth of the top list (>= k + 1)
__device__ __forceinline__ void route_packed_body(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wgt,
                                                  const float* __restrict__ w_norm2, const float* __restrict__ bias,
                                                  int T, int d, int E, int k, int renorm, int32_t* __restrict__ idx_out,
                                                  float* __restrict__ w_out, float* __restrict__ logits_out) {
    constexpr int NWV = NB * KSP, TB = 32, EPT = 32 * NB;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nbi = wave / KSP, ksi = wave % KSP;    // this wavefront's expert block and contraction part
    const int t0 = blockIdx.x * TB;
    const int n_chunks = d / KC;
    const int rows = T - t0 < TB ? T - t0 : TB;
    float xsq = 0.f;
    const RouteBias mine = route_bias<NB, KSP>(bias, E);
    const float w2 = tid < E ? fmaxf(0.f, w_norm2[tid]) : 0.f;           // this thread's share of the largest column norm

    double acc64[16];
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc64[r] = 0.0; acc[r] = 0.f; }
    static_assert(KACC == KC, "a chunk is what one fp32 accumulation holds");

    // ---- staging (route_stage.h).  With one or two wavefronts on a SIMD the loop is bound by the instructions a
    // wavefront issues (one every five cycles), so a wavefront's loads are the same in every stage, their
    // per-lane offsets formed once, the stage only in the scalar offset.  (Deciding in every stage which rows
    // a load brings took 0.6 us a stage.)  Chunks past the end bring earlier terms again and are not
    // multiplied; past the last stage its loads go out again, so that the count of outstanding loads that
    // guarantees a stage is a constant.
    using S = RouteStage<NB, KSP>;
    constexpr int STAGE = S::BYTES, LPW = S::LPW, RING = ROUTE_RING;
    static_assert(S::TB == TB && S::EPT == EPT && S::CHUNK == KC * 2, "route_stage.h");
    static_assert(LPW * (RING - 1) < 64 && RING * STAGE + 1024 <= 150 * 1024, "staging ring");
    unsigned char* ring = smem;
    const int n_stages = (n_chunks + KSP - 1) / KSP;
    const __amdgpu_buffer_rsrc_t rx =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(wgt), 0, E * d * 2, 0x00020000);
    unsigned voff[LPW], to[LPW], last[LPW];                  // byte offsets: in the matrix, and (scalar) in the stage and at most
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        voff[i] = S::lane_offset(wave, i, lane, d);
        to[i] = (unsigned)__builtin_amdgcn_readfirstlane((int)S::lds(wave, i));
        last[i] = (unsigned)__builtin_amdgcn_readfirstlane((int)S::last_offset(wave, i, n_chunks));
        if (S::spare(wave, i)) { voff[i] = 0x80000000u; to[i] = RING * STAGE; }   // (zeros to the 1 KB behind the ring)
    }
    auto issue_stage = [&](int st) {
        const unsigned buf = (unsigned)(st % RING) * STAGE;
#pragma unroll
        for (int i = 0; i < LPW; ++i) {
            const bool spare = S::XL * NWV > TB / 8 * KSP && S::is_x(i);     // (its place does not move with the stage)
            lds_void_t* at = (lds_void_t*)(ring + (spare && to[i] == (unsigned)(RING * STAGE) ? to[i] : buf + to[i]));
            const unsigned soff = S::offset(st, last[i]);
            if (S::is_x(i)) __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, at, 16, voff[i], soff, 0, 0);
            else __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, at, 16, voff[i], soff, 0, 0);
        }
    };
#pragma unroll
    for (int st = 0; st < RING - 1; ++st) issue_stage(st);
    const int frag_at = l32 * 128;
    const int frag_sw = (l32 >> 1) & 7;
    for (int st = 0; st < n_stages; ++st) {
        // stage st has landed once only the RING-2 younger stages are outstanding
        MOE_WAIT_VMCNT((RING - 2) * LPW);
        // ... for every wavefront after the barrier; and stage st-1 has been read by all.  (A bare
        // barrier: __syncthreads would first wait for every load in flight, the prefetched stages too.)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        const int c = st * KSP + ksi;
        const unsigned char* xb = ring + (st % RING) * STAGE + ksi * (TB + EPT) * 128;
        const unsigned char* wb_ = xb + (TB + nbi * 32) * 128;
        frag_t xa[KC / 16], wb[KC / 16];
#pragma unroll
        for (int ks = 0; ks < KC / 16; ++ks) {
            const int pos = ((ks * 2 + lhi) ^ frag_sw) << 4;
            xa[ks] = *(const frag_t*)(xb + frag_at + pos);
            wb[ks] = *(const frag_t*)(wb_ + frag_at + pos);
        }
        issue_stage(st + RING - 1);                          // into the buffer of stage st-1
        // (the sums of the chunk before: they pass while this one's fragments arrive)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc64[r] += (double)acc[r];
        const frag_t none = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < KC / 16; ++ks) {
            if (c >= n_chunks) xa[ks] = none;                // (a stage's last chunks may be past the end)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa[ks]),
                                                          __builtin_bit_cast(bf16x8, c < n_chunks ? wb[ks] : none), acc, 0, 0, 0);
            if (nbi == 0) {                                  // the token norms, once per contraction part
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bf16x2 p2 = bf16_pair(xa[ks][i]);
                    xsq = __builtin_amdgcn_fdot2_f32_bf16(p2, p2, xsq, false);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc64[r] += (double)acc[r];
    MOE_WAIT_VMCNT(0);                                       // (the trailing loads, the last stage's again, still target this LDS)
    __syncthreads();                                         // the ring's memory is reused below
    route_finish<NB, KSP, RMAX, true>(smem, acc64, xsq, w2, mine, x, wgt, bias, T, d, E, k, renorm, idx_out, w_out, logits_out);
}

template <int NB, int KSP, int RMAX>
__global__ __launch_bounds__(NB * KSP * 64, 2) void route_packed_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wgt,
                                                                        const float* __restrict__ w_norm2,
                                                                        const float* __restrict__ bias, int T, int d, int E, int k,
                                                                        int renorm, int32_t* __restrict__ idx_out,
                                                                        float* __restrict__ w_out, float* __restrict__ logits_out) {
    route_packed_body<NB, KSP, RMAX>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx_out, w_out, logits_out);
}

// =========================================================================================
// Router with W_g as given, [d,E]: the expert index is contiguous, the matrix instruction wants the
// contraction index contiguous for both operands.  W_g is transposed on its way into LDS: a
// thread fetches eight terms of eight neighbouring experts (eight 16-byte loads), swaps them into
// eight runs of eight terms with byte permutes, and writes those as 16-byte pieces.  (Two-byte
// loads and LDS writes, one term of one expert each, kept the kernel at 1257 us for 20011 tokens x
// 1032, E = 256; this takes 102 us, 64 of them before the exact path.)  A stage is 128 terms per contraction part of the 32 tokens and
// all experts; its loads are in flight while the previous stage is multiplied.
//
// LDS rows hold 16 pieces (128 terms); piece p of row r sits at position p ^ swz(r), chosen so that
// both the fragment reads (16 consecutive rows, one piece) and the transposed writes (every
// eighth row, one piece) touch all banks once.
constexpr int KPLAIN = 128;            // terms per stage and contraction part

__device__ __forceinline__ int plain_swz(int r) { return (((r & 7) << 1) ^ (r >> 3)) & 15; }

template <int NB, int KSP, int RMAX>
__global__ __launch_bounds__(NB * KSP * 64, NB >= 4 ? 4 : NB == 2 ? 3 : 2) void route_plain_kernel(const uint16_t* __restrict__ x, const uint16_t* __restrict__ wg,
                                                                       const float* __restrict__ bias, int T, int d, int E, int k,
                                                                       int renorm, int32_t* __restrict__ idx_out,
                                                                       float* __restrict__ w_out, float* __restrict__ logits_out) {
    constexpr int NWV = NB * KSP, NTHR = NWV * 64, TB = 32, EPT = 32 * NB;
    constexpr int PART = (TB + EPT) * KPLAIN * 2;            // bytes of one contraction part of a stage: token rows, expert rows
    constexpr int XN = TB * 16 * KSP / NTHR;                 // 16-byte pieces of x per thread
    constexpr int GROUPS = EPT / 8;                          // groups of eight experts
    static_assert(GROUPS * 16 * KSP == NTHR, "one block of 8 experts x 8 terms per thread and stage");
    static_assert(XN >= 1 && TB * 16 * KSP % NTHR == 0, "x pieces");
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, lhi = lane >> 5;
    const int nbi = wave / KSP, ksi = wave % KSP;
    const int t0 = blockIdx.x * TB;

    // This thread's block of W_g: experts 8 g .. 8 g + 7, terms 8 kg .. 8 kg + 7 of the stage.  The loads
    // carry no conditions: groups past E, tokens past T and terms past d fetch the last ones again
    // (columns and tokens that do not exist are never looked at, terms past d are cleared below).
    // Rows are 2-byte aligned only when E is odd: the copies state no alignment.
    const int g = tid % GROUPS, kg = tid / GROUPS;
    const int g_in = g * 8 < E ? g : (E - 1) / 8;
    // Entries of this group past its row's end belong to the next row; the last row has none: there
    // the eight last entries of the matrix are read and moved into place (E >= 8).
    const int over = g_in * 8 + 8 > E ? g_in * 8 + 8 - E : 0;
    u32x4 wv[8], xv[XN];
    auto load_stage = [&](int st) {
        const int k0 = st * (KPLAIN * KSP);
#pragma unroll
        for (int u2 = 0; u2 < XN; ++u2) {
            const int p = tid + u2 * NTHR, kk = k0 + (p % (16 * KSP)) * 8, tok = t0 + p / (16 * KSP);
            xv[u2] = *(const u32x4*)(x + (size_t)(tok < T ? tok : T - 1) * d + (kk < d ? kk : d - 8));
        }
        const int kk = k0 + kg * 8 < d ? k0 + kg * 8 : d - 8;    // (d is a multiple of 8)
        const uint16_t* src = wg + (size_t)kk * E + g_in * 8;
#pragma unroll
        for (int j = 0; j < 7; ++j) __builtin_memcpy(&wv[j], src + (size_t)j * E, 16);
        __builtin_memcpy(&wv[7], src + (size_t)7 * E - (kk + 8 == d ? over : 0), 16);
    };
    auto mend_last_stage = [&](int st) {
        const int k0 = st * (KPLAIN * KSP);
        const u32x4 zero = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int u2 = 0; u2 < XN; ++u2)
            if (k0 + ((tid + u2 * NTHR) % (16 * KSP)) * 8 >= d) xv[u2] = zero;
        if (k0 + kg * 8 + 8 >= d)
            wv[7] = __builtin_bit_cast(u32x4, __builtin_bit_cast(unsigned __int128, wv[7]) >> (16 * over));
        if (k0 + kg * 8 >= d) {
#pragma unroll
            for (int j = 0; j < 8; ++j) wv[j] = zero;
        }
    };

    const RouteBias mine = route_bias<NB, KSP>(bias, E);
    double acc64[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) acc64[r] = 0.0;
    float xsq = 0.f, wsq = 0.f;                              // this lane's share of the norm of its token row and expert row
    const int n_stages = (d + KPLAIN * KSP - 1) / (KPLAIN * KSP);
    // Swizzled LDS offsets: piece c * 2 + lhi of a fragment row, and expert e of this thread's block, are
    // the offset of piece lhi / expert 0 with bits flipped.
    int xb_at = ksi * PART + l32 * 256 + ((lhi ^ plain_swz(l32)) << 4);
    int wb_at = ksi * PART + (TB + nbi * 32 + l32) * 256 + ((lhi ^ plain_swz(nbi * 32 + l32)) << 4);
    int wr_at = (kg >> 4) * PART + (TB + g * 8) * 256 + (((kg ^ g) & 15) << 4);
    load_stage(0);
    for (int st = 0; st < n_stages; ++st) {
        if (st) __syncthreads();                             // the previous stage has been read
        // (the empty asm keeps the compiler from forming all flipped offsets once, outside the loop)
        asm volatile("" : "+v"(xb_at), "+v"(wb_at), "+v"(wr_at));
        if (st + 1 == n_stages) mend_last_stage(st);
#pragma unroll
        for (int u2 = 0; u2 < XN; ++u2) {
            const int p = tid + u2 * NTHR, tok = p / (16 * KSP), pc = p % (16 * KSP);
            *(u32x4*)(smem + (pc >> 4) * PART + tok * 256 + (((pc & 15) ^ plain_swz(tok)) << 4)) = xv[u2];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {                        // expert g * 8 + e: its eight terms
            u32x4 piece;
#pragma unroll
            for (int m = 0; m < 4; ++m)
                piece[m] = __builtin_amdgcn_perm(wv[2 * m + 1][e >> 1], wv[2 * m][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
            *(u32x4*)(smem + (wr_at ^ (e << 5)) + e * 256) = piece;
        }
        __syncthreads();
        if (st + 1 < n_stages) load_stage(st + 1);
#pragma unroll
        for (int h = 0; h < KPLAIN / KACC; ++h) {
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KACC / 16; ++ks) {
                const int flip = (h * (KACC / 16) + ks) << 5;
                const frag_t xa = *(const frag_t*)(smem + (xb_at ^ flip)), wa = *(const frag_t*)(smem + (wb_at ^ flip));
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, xa), __builtin_bit_cast(bf16x8, wa), acc, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const bf16x2 w2 = bf16_pair(wa[i]);
                    wsq = __builtin_amdgcn_fdot2_f32_bf16(w2, w2, wsq, false);
                    if (nbi == 0) {                          // (wave-uniform)
                        const bf16x2 x2 = bf16_pair(xa[i]);
                        xsq = __builtin_amdgcn_fdot2_f32_bf16(x2, x2, xsq, false);
                    }
                }
                if (ks & 1) __builtin_amdgcn_sched_barrier(0);     // (two slices' fragments in registers at a time)
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) acc64[r] += (double)acc[r];
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // squared column norms (a little rounded up): the halves of a row's terms sit in lanes l and l + 32, the
    // contraction parts in the wavefronts that share an expert block
    wsq += __shfl_xor(wsq, 32);
    __syncthreads();
    float* wn = reinterpret_cast<float*>(smem);              // [KSP][EPT]
    if (lhi == 0) wn[ksi * EPT + nbi * 32 + l32] = wsq;
    __syncthreads();
    float w2 = 0.f;
    for (int e = tid; e < E; e += NTHR) {
        float v = wn[e];
#pragma unroll
        for (int p = 1; p < KSP; ++p) v += wn[p * EPT + e];
        w2 = fmaxf(w2, v * 1.002f);
    }
    __syncthreads();                                         // the staging memory is free now
    route_finish<NB, KSP, RMAX, false>(smem, acc64, xsq, w2, mine, x, wg, bias, T, d, E, k, renorm, idx_out, w_out, logits_out);
}

template <int NB, int KSP, int RMAX>
int launch_packed_r(const void* x, const void* wgt, const float* w_norm2, const float* bias, int T, int d, int E, int k,
                    int renorm, int32_t* idx, float* w, float* logits, hipStream_t st) {
    constexpr int NWV = NB * KSP, EPT = 32 * NB;
    const size_t later = RouteLds<NB, KSP>::BYTES;
    const size_t ring = (size_t)ROUTE_RING * (32 + EPT) * KSP * 128 + 1024;       // the staging ring and the later buffers share LDS
    const size_t smem = ring > later ? ring : later;
    auto kern = route_packed_kernel<NB, KSP, RMAX>;
    if (smem > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return moe_fail(MOE_ERR_HIP, "moe_route_topk_packed: shared memory attribute: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, dim3((T + 31) / 32), dim3(NWV * 64), smem, st, (const uint16_t*)x, (const uint16_t*)wgt, w_norm2,
                       bias, T, d, E, k, renorm, idx, w, logits);
    MOE_CHECK_LAUNCH("moe_route_topk_packed");
    return MOE_OK;
}

template <int NB, int KSP>
int launch_packed(const void* x, const void* wgt, const float* w_norm2, const float* bias, int T, int d, int E, int k,
                  int renorm, int32_t* idx, float* w, float* logits, hipStream_t st) {
    // the depth of the per-thread top list follows k (a shorter list is less work per logit)
    if (k <= 1) return launch_packed_r<NB, KSP, 2>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (k <= 2) return launch_packed_r<NB, KSP, 3>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (k <= 4) return launch_packed_r<NB, KSP, 5>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    return launch_packed_r<NB, KSP, MAXR>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
}

template <int NB, int KSP, int RMAX>
int launch_plain_r(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm, int32_t* idx, float* w,
                   float* logits, hipStream_t st) {
    constexpr size_t stage = (size_t)KSP * (32 + 32 * NB) * KPLAIN * 2, later = RouteLds<NB, KSP>::BYTES;
    constexpr size_t smem = stage > later ? stage : later;
    auto kern = route_plain_kernel<NB, KSP, RMAX>;
    if (smem > 48 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return moe_fail(MOE_ERR_HIP, "moe_route_topk: shared memory attribute: %s", hipGetErrorString(e));
    }
    hipLaunchKernelGGL(kern, dim3((T + 31) / 32), dim3(NB * KSP * 64), smem, st, (const uint16_t*)x, (const uint16_t*)wg, bias, T, d, E,
                       k, renorm, idx, w, logits);
    MOE_CHECK_LAUNCH("moe_route_topk");
    return MOE_OK;
}

template <int NB, int KSP>
int launch_plain(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm, int32_t* idx, float* w,
                 float* logits, hipStream_t st) {
    // (two depths of the per-thread top list: the selection is a small part of this kernel)
    if (k <= 2) return launch_plain_r<NB, KSP, 3>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    return launch_plain_r<NB, KSP, MAXR>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
}

}  // namespace

// the general kernel of route.hip (fewer than eight experts: a row of W_g is shorter than a 16-byte load)
int moe_route_small(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm, int32_t* idx, float* w,
                    float* logits, hipStream_t st);

// bf16 path of moe_route_topk (arguments already validated by the caller)
int moe_route_bf16_mfma(const void* x, const void* wg, const float* bias, int T, int d, int E, int k, int renorm,
                        int32_t* idx, float* w, float* logits, hipStream_t st) {
    if (E < 8) return moe_route_small(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 32) return launch_plain<1, 4>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 64) return launch_plain<2, 2>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 128) return launch_plain<4, 1>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
    return launch_plain<8, 1>(x, wg, bias, T, d, E, k, renorm, idx, w, logits, st);
}

// bf16 path of moe_route_topk_packed (arguments already validated by the caller)
int moe_route_bf16_packed(const void* x, const void* wgt, const float* w_norm2, const float* bias, int T, int d, int E,
                          int k, int renorm, int32_t* idx, float* w, float* logits, hipStream_t st) {
    if (E <= 32) return launch_packed<1, 4>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 64) return launch_packed<2, 2>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    if (E <= 128) return launch_packed<4, 1>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
    return launch_packed<8, 1>(x, wgt, w_norm2, bias, T, d, E, k, renorm, idx, w, logits, st);
}
