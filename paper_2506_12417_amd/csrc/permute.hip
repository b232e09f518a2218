// moe_permute: stable counting sort of the A = T*k assignments by expert, and the row gather
// (one-GPU form of Alg. 1 step 4; counts[] is the one-GPU slice of S_initial, step 3).
//
// Four launches, no float atomics, no ordering left to chance:
//   1. per-block histogram of expert ids (1024 assignments per work-group, LDS integer adds)
//   2. one wavefront per expert: exclusive prefix over the blocks -> counts
//   3. per-block stable rank: inside a wavefront the peers of an assignment (same expert) are
//      found with one ballot per bit of the expert id; popcount of the lower lanes is the rank;
//      per-64-chunk counts are prefix-summed in LDS -> offsets, perm, inv_perm
//   4. rows x_perm[inv_perm[t*k+j]] = x[t]: every row of x is read once and written k times
#include "common.h"
#include "permute_rank.h"
#include <mutex>

namespace {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
using moe_rank::CHUNKS;
using moe_rank::NTH;
constexpr int COUNT_BLOCKS = 2;
using moe_rank::PB;   // assignments per work-group in steps 1 and 3

__global__ __launch_bounds__(NTH) void hist_kernel(const int32_t* __restrict__ idx, int A, int E,
                                                   int32_t* __restrict__ block_hist) {
    __shared__ int h[MOE_MAX_EXPERTS];
    for (int e = threadIdx.x; e < E; e += NTH) h[e] = 0;
    __syncthreads();
    const int base = blockIdx.x * PB;
    int mine[PB / NTH];                                     // (all loads first: one memory latency, not PB / NTH)
#pragma unroll
    for (int j = 0; j < PB / NTH; ++j) {
        const int a = base + j * NTH + threadIdx.x;
        mine[j] = a < A ? idx[a] : -1;
    }
#pragma unroll
    for (int j = 0; j < PB / NTH; ++j)
        if ((unsigned)mine[j] < (unsigned)E) atomicAdd(&h[mine[j]], 1);
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += NTH) block_hist[(size_t)blockIdx.x * E + e] = h[e];
}

// One wavefront per expert: block_hist[b][e] becomes the number of assignments of expert e in
// blocks < b.  (One work-group for all experts, each thread walking its expert's blocks, took 18 us
// for 157 blocks and 256 experts; this takes 5.)
__global__ __launch_bounds__(NTH) void scan_kernel(int32_t* __restrict__ block_hist, int nb, int A, int E,
                                                   int32_t* __restrict__ counts, int32_t* __restrict__ offsets) {
    constexpr int NB = 4;                                  // 64-block groups whose loads are in flight together
    const int e = blockIdx.x * (NTH / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (e >= E) return;
    int run = 0;
    for (int b0 = 0; b0 < nb; b0 += 64 * NB) {
        int v[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int b = b0 + j * 64 + lane;
            v[j] = b < nb ? block_hist[(size_t)b * E + e] : 0;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int b = b0 + j * 64 + lane;
            int incl = v[j];
#pragma unroll
            for (int step = 1; step < 64; step <<= 1) {
                const int o = __shfl_up(incl, step);
                incl += lane >= step ? o : 0;
            }
            if (b < nb) block_hist[(size_t)b * E + e] = run + incl - v[j];
            run += __shfl(incl, 63);
        }
    }
    if (lane == 0) {
        counts[e] = run;
        if (A == 0) {                                      // (otherwise the rank kernel writes them)
            offsets[e] = 0;
            if (e == E - 1) offsets[E] = 0;
        }
    }
}

template <int MODE>
__global__ __launch_bounds__(NTH) void rank_kernel(const int32_t* __restrict__ idx, int A, int E, int nbits, int nb,
                                                   const int32_t* __restrict__ block_hist,
                                                   int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                                                   int32_t* __restrict__ perm, int32_t* __restrict__ inv_perm) {
    moe_rank::rank_body<MODE>(idx, A, E, nbits, nb, block_hist, counts, offsets, perm, inv_perm);
}

// x_perm row inv_perm[t*k+j] <- x row t, in 16-byte pieces (vpr pieces per row), one piece of one
// token per thread; an assignment without a row (inv_perm -1) is skipped.  HBM bound, and by its scattered stores at that: x is read once (gathering through
// perm read it k times through the L2 and the row's address at the end of a chain of two loads).
// 20011 x 8 rows of 2064 bytes: 96 -> 84 us back to back (4.5 TB/s), 95 -> 91 in a dispatch pass, where it
// writes 335 MB for 330 of rows: the lines that two rows share cost nothing extra.  Nontemporal
// stores were slower for them.
__global__ __launch_bounds__(NTH) void spread_rows_kernel(const u32x4* __restrict__ x, const int32_t* __restrict__ inv_perm,
                                                          unsigned total, unsigned A, unsigned k, unsigned vpr,
                                                          u32x4* __restrict__ x_perm) {
    const unsigned i = blockIdx.x * NTH + threadIdx.x;
    if (i >= total) return;
    const unsigned t = i / vpr, v = i - t * vpr;
    const u32x4 piece = x[i];
    const int32_t* to = inv_perm + (size_t)t * k;
    for (unsigned j0 = 0; j0 < k; j0 += 4) {
        unsigned row[4];
#pragma unroll
        for (unsigned j = 0; j < 4; ++j) row[j] = j0 + j < k ? (unsigned)to[j0 + j] : A;       // (-1 is past A)
#pragma unroll
        for (unsigned j = 0; j < 4; ++j)
            if (row[j] < A) x_perm[(size_t)row[j] * vpr + v] = piece;
    }
}

}  // namespace

// Scratch of moe_permute_static: the block histograms, in the library's own device memory (each
// GPU the library runs on holds a copy of this array until the process ends).  Host code never
// passes the array's name to a kernel: it asks the runtime for the array's address on the
// current device, once per device, and uses that pointer.
static __device__ __align__(256) unsigned char scratch[MOE_PERMUTE_STATIC_BYTES];

static int32_t* g_scratch_ptr[64] = {};          // per device, set on first use
static std::mutex g_scratch_mutex;

static int scratch_on_current_device(int32_t** out) {
    int dev = -1;
    MOE_CHECK_HIP(hipGetDevice(&dev));
    MOE_REQUIRE(dev >= 0 && dev < 64, MOE_ERR_UNSUPPORTED, "moe_permute_static: device %d", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        MOE_CHECK_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        MOE_REQUIRE(p != nullptr, MOE_ERR_HIP, "moe_permute_static: no address for the scratch array");
        g_scratch_ptr[dev] = (int32_t*)p;
    }
    *out = g_scratch_ptr[dev];
    return MOE_OK;
}

// Argument checks shared by the two entry points (nothing is enqueued on an error).
static int permute_check(const char* who, const void* x, const int32_t* expert_idx, int T, int d, int E, int k,
                         moe_dtype dt, const int32_t* counts, const int32_t* offsets, const int32_t* perm,
                         const int32_t* inv_perm, const void* x_perm) {
    MOE_REQUIRE(moe_dtype_ok(dt), MOE_ERR_UNSUPPORTED, "%s: dtype %d", who, (int)dt);
    MOE_REQUIRE(T >= 0 && E >= 1 && k >= 1 && d >= 1, MOE_ERR_ARG, "%s: T=%d d=%d E=%d k=%d", who, T, d, E, k);
    MOE_REQUIRE(E <= MOE_MAX_EXPERTS, MOE_ERR_UNSUPPORTED, "%s: E=%d > %d", who, E, MOE_MAX_EXPERTS);
    MOE_REQUIRE((long long)T * k < (1ll << 30), MOE_ERR_UNSUPPORTED, "%s: T*k too large", who);
    MOE_REQUIRE((x == nullptr) == (x_perm == nullptr), MOE_ERR_ARG, "%s: x and x_perm must both be given or both be null", who);
    MOE_REQUIRE(((size_t)d * moe_elem_size(dt)) % 16 == 0, MOE_ERR_UNSUPPORTED, "%s: row of %d elements is not a multiple of 16 bytes", who, d);
    MOE_REQUIRE(counts && offsets, MOE_ERR_ARG, "%s: null pointer", who);
    MOE_REQUIRE((long long)T * k == 0 || (expert_idx && perm && inv_perm), MOE_ERR_ARG, "%s: null pointer", who);
    return MOE_OK;
}

// The launches of the sort; block_hist holds one histogram of E counters per block of PB
// assignments (every entry is written by hist_kernel before anything reads it).
static int permute_launch(const void* x, const int32_t* expert_idx, int T, int d, int E, int k, moe_dtype dt,
                          int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm, void* x_perm,
                          int32_t* block_hist, hipStream_t st) {
    const int A = T * k;
    const int nb = A == 0 ? 1 : (A + PB - 1) / PB;
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;

    // With one or two blocks every rank work-group counts all ids itself (a launch less, which is what
    // such a call pays for: 512 assignments 7.2 -> 6.7 us back to back, an fp32 layer of 512
    // assignments 51 -> 46; from three blocks on the reading costs as much, 4096 assignments 7.1 : 8.2);
    // with some more it repeats the scan over the blocks' histograms; with many blocks, or nothing to
    // rank, the scan is a launch of its own.
    const bool count_in_rank = A > 0 && nb <= COUNT_BLOCKS;
    const bool fused_scan = A > 0 && nb <= 64;
    if (!count_in_rank) {
        hipLaunchKernelGGL(hist_kernel, dim3(nb), dim3(NTH), 0, st, expert_idx, A, E, block_hist);
        MOE_CHECK_LAUNCH("moe_permute/hist");
    }
    if (!fused_scan) {
        hipLaunchKernelGGL(scan_kernel, dim3((E + NTH / 64 - 1) / (NTH / 64)), dim3(NTH), 0, st, block_hist, nb, A, E, counts, offsets);
        MOE_CHECK_LAUNCH("moe_permute/scan");
    }
    if (A == 0) return MOE_OK;
    auto rank = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(NTH), sizeof(int) * CHUNKS * E, st, expert_idx, A, E, nbits, nb, block_hist, counts, offsets,
                           perm, inv_perm);
    };
    if (count_in_rank) rank(rank_kernel<2>);
    else if (fused_scan) rank(rank_kernel<1>);
    else rank(rank_kernel<0>);
    MOE_CHECK_LAUNCH("moe_permute/rank");
    if (x) {
        // (slices of whole tokens whose pieces a 32-bit index counts)
        const unsigned vpr = (unsigned)((size_t)d * moe_elem_size(dt) / 16);
        const long long slice = (1ll << 31) / vpr;
        for (long long t0 = 0; t0 < T; t0 += slice) {
            const unsigned total = (unsigned)((T - t0 < slice ? T - t0 : slice) * vpr);
            hipLaunchKernelGGL(spread_rows_kernel, dim3((total + NTH - 1) / NTH), dim3(NTH), 0, st,
                               (const u32x4*)x + (size_t)t0 * vpr, inv_perm + (size_t)t0 * k, total, (unsigned)A, (unsigned)k, vpr,
                               (u32x4*)x_perm);
        }
        MOE_CHECK_LAUNCH("moe_permute/rows");
    }
    return MOE_OK;
}

extern "C" int moe_permute(const void* x, const int32_t* expert_idx, int T, int d, int E, int k, moe_dtype dt,
                           int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm, void* x_perm,
                           void* ws, size_t ws_bytes, void* stream) {
    const int rc = permute_check("moe_permute", x, expert_idx, T, d, E, k, dt, counts, offsets, perm, inv_perm, x_perm);
    if (rc != MOE_OK) return rc;
    MOE_REQUIRE(ws, MOE_ERR_ARG, "moe_permute: null pointer");
    MOE_REQUIRE(ws_bytes >= moe_workspace_bytes(MOE_OP_PERMUTE, T, d, 0, E, k, dt), MOE_ERR_WORKSPACE,
                "moe_permute: workspace %zu < %zu bytes", ws_bytes, moe_workspace_bytes(MOE_OP_PERMUTE, T, d, 0, E, k, dt));
    return permute_launch(x, expert_idx, T, d, E, k, dt, counts, offsets, perm, inv_perm, x_perm, (int32_t*)ws,
                          (hipStream_t)stream);
}

extern "C" int moe_permute_static(const void* x, const int32_t* expert_idx, int T, int d, int E, int k, moe_dtype dt,
                                  int32_t* counts, int32_t* offsets, int32_t* perm, int32_t* inv_perm, void* x_perm,
                                  void* stream) {
    const int rc = permute_check("moe_permute_static", x, expert_idx, T, d, E, k, dt, counts, offsets, perm, inv_perm, x_perm);
    if (rc != MOE_OK) return rc;
    const size_t need = moe_workspace_bytes(MOE_OP_PERMUTE, T, d, 0, E, k, dt);
    MOE_REQUIRE(need <= MOE_PERMUTE_STATIC_BYTES, MOE_ERR_CAPACITY,
                "moe_permute_static: T*k = %lld with E = %d needs %zu bytes of scratch, the built-in array holds %u "
                "(use moe_permute with a workspace)", (long long)T * k, E, need, MOE_PERMUTE_STATIC_BYTES);
    int32_t* block_hist = nullptr;
    const int rs = scratch_on_current_device(&block_hist);
    if (rs != MOE_OK) return rs;
    return permute_launch(x, expert_idx, T, d, E, k, dt, counts, offsets, perm, inv_perm, x_perm, block_hist,
                          (hipStream_t)stream);
}
