// Device-side helpers shared by the 16-bit grouped GEMM kernels (ffn_bf16.hip, ffn_stream.hip).
#pragma once
#include "common.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((address_space(3))) void lds_void_t;

// s_waitcnt on vmcnt only (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[15:14])
#define MOE_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (0x7 << 4) | (0xF << 8))
// s_waitcnt on lgkmcnt only
#define MOE_WAIT_LGKMCNT(n) __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4) | (((n) & 0xF) << 8))

// cache policy of a buffer access: nontemporal
constexpr int CACHE_NT = 2;

__device__ __forceinline__ float silu_f(float z) { return z / (1.f + __expf(-z)); }

// raw buffer descriptor over [p, p + bytes): offsets beyond `bytes` read 0 / are not written
// (pointer and size are wave-uniform; readfirstlane tells the compiler so)
__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const void* sgpr_ptr(const void* p) {
    const uint64_t u = (uint64_t)p;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    return (const void*)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(sgpr_ptr(p)), 0, sgpr((int)bytes), 0x00020000);
}

// Which tiles a work-group of a persistent launch shares with which others: those of its bin, on the
// bin's XCD -- or, where a small call leaves most XCDs idle, all tiles with all work-groups.  The
// plan places experts, not work: Alg. 2 moves no block below q rows, so an expert of 300 rows
// stays on one XCD of eight.  All work-groups see the same header and decide alike, by the rounds of
// items that the fullest bin and the whole chip would take: flat up to two rounds if that is fewer, up
// to four if it is fewer by two fifths; beyond, sharing an XCD's L2 is worth more than the idle CUs.
// One expert of 2048 x 5632 (both products): 512 rows 259 -> 94 us, 1100 rows 530 -> 179; four
// experts, 1024 rows 230 -> 154, 2048 rows (6 rounds against 4) 232 by bins, 242 flat.
// one_round_of_pairs: the launch takes the tiles two at a time, and the whole chip then has one round: by bins
// if the fullest one has too (its tiles count for five eighths, some having no partner), else flat.  32 experts, 12000 rows
// of 768 x 3072, second product: 94 us by bins, 106 flat; 16000 rows (two rounds by bins): 162 and 122.
struct WorkShare {
    int bin, first, stride, bin_start, n_tiles;   // bin: whose work counter hands out the items
};
__device__ __forceinline__ WorkShare work_share(const int32_t* __restrict__ hdr, int n_col_blocks, bool one_round_of_pairs = false) {
    // (the bins' starts are fetched with the number of bins, not after it: one memory latency)
    const int grid = (int)gridDim.x, lane = threadIdx.x & 63;
    const int at = lane < MOE_MAX_BINS ? lane : MOE_MAX_BINS - 1;
    const int start = hdr[4 + at], end = hdr[5 + at];
    const int G = hdr[1];
    const int fullest = (int)moe_wave_max_u32(lane < G ? (unsigned)(end - start) : 0u);
    const int first_tile = __builtin_amdgcn_readlane(start, 0), all = __builtin_amdgcn_readlane(end, G - 1) - first_tile;
    const int rounds_flat = one_round_of_pairs ? 1 : (all * n_col_blocks + grid - 1) / grid;
    const int per_bin = grid / G, rounds_bin = ((one_round_of_pairs ? (5 * fullest + 7) / 8 : fullest) * n_col_blocks + per_bin - 1) / per_bin;
    WorkShare w;
    if (rounds_flat < rounds_bin && (rounds_flat <= 2 || (rounds_flat <= 4 && 3 * rounds_bin >= 5 * rounds_flat))) {
        w.bin = 0;
        w.first = (int)blockIdx.x;
        w.stride = grid;
        w.bin_start = first_tile;
        w.n_tiles = all;
    } else {
        w.bin = (int)blockIdx.x % G;
        w.first = (int)blockIdx.x / G;
        w.stride = (grid - w.bin + G - 1) / G;
        w.bin_start = __builtin_amdgcn_readlane(start, w.bin);
        w.n_tiles = __builtin_amdgcn_readlane(end, w.bin) - w.bin_start;
    }
    return w;
}

// take_ticket: lane 0 adds one to *ctr; the old value arrives some time later, like a load, in
// register v250.  read_ticket fetches it from there; the caller does so only after a vmcnt wait
// that covers the request.  Written as assembly with a fixed register, because the compiler would
// wait for the answer on the spot (draining the whole queue of operand loads in flight), and
// because a result register it knows of gets copied around before the answer is in it.  This is
// sound only in kernels whose own code never touches v250: the kernels that use it stay well
// below 250 registers, and a unit test compiles this file and checks that v250 appears in these
// two instructions only.
#define MOE_TICKET_REG "v250"
__device__ __forceinline__ void take_ticket(int32_t* ctr) {
    unsigned long long saved;
    asm volatile(
        "s_mov_b64 %0, exec\n\t"
        "s_mov_b64 exec, 1\n\t"
        "global_atomic_add " MOE_TICKET_REG ", %1, %2, %3 sc0\n\t"
        "s_mov_b64 exec, %0"
        : "=&s"(saved)
        : "v"(0), "v"(1), "s"(ctr)
        : "memory", MOE_TICKET_REG);
}
__device__ __forceinline__ int read_ticket() {
    int v;
    asm volatile("v_readfirstlane_b32 %0, " MOE_TICKET_REG : "=s"(v) : : MOE_TICKET_REG);
    return v;
}

}  // namespace
