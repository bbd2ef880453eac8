// What the two bf16 attention kernels (attention_bf16.hip, attention_wide.hip)
// share: tile geometry, LDS swizzles, direct-to-LDS loads and the schedule of
// a launch.
#pragma once

#include "common.h"
#include "kernels.h"

namespace pcpp {
namespace attn {

constexpr int D = 64;
constexpr int KT = 64;                      // keys per tile
constexpr int TILE_BYTES = KT * D * 2;      // 8 KB of K or of V
constexpr float P_LIMIT = 1048576.0f;       // 2^20: bound on a lane's probability sum per half-tile
constexpr int WIDE_QUERIES = 256;           // queries per block of attention_wide.hip

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

template <int V>
struct Int {
    static constexpr int value = V;
};

// 16 bytes per lane from global memory straight into LDS: lane l's bytes land
// at lds + 16 l (lds is the wave-uniform LDS byte address).  Written as inline
// assembly so that the compiler does not track the LDS write: its own tracking
// of such writes covers at most a few LDS buffers and otherwise waits for every
// staging load in flight before any LDS read.  The kernel orders these writes
// before the reads itself, with vmcnt waits and barriers.  Loads complete in
// order, so the compiler's own vmcnt waits for register loads stay safe: they
// only become more conservative.
__device__ __forceinline__ void dma16(const void* g, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "{m0}"(lds) : "memory");
}

// The same with a wave-uniform 64-bit base in SGPRs and a 32-bit per-lane
// byte offset (the load's saddr form): no per-lane address arithmetic.
// lds is the wave-uniform LDS byte address.
__device__ __forceinline__ void dma16_s(uint64_t base, uint32_t voff, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
}

// A wave-uniform value known to the compiler as such (kept in SGPRs).
__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// LDS swizzles: 16-byte chunk c of tile row r is stored at slot c ^ mask(r).
// K rows are read 16 bytes per lane by 32 consecutive rows at one chunk; V
// rows by four rows x 32 bytes per 16 lanes (transposing read).  Both masks
// repeat every 16 rows, so a half-tile (32 rows) offset keeps them.
__device__ __forceinline__ int k_mask(int r) { return (r >> 1) & 7; }
__device__ __forceinline__ int v_mask(int r) { return ((r >> 1) & 3) << 1; }

struct Sched {
    int32_t n_xcd;      // XCDs; workgroup w runs on XCD w % n_xcd
    int32_t bpx;        // blocks per XCD (the last XCD may hold fewer)
    int32_t k;          // pieces per block
    int32_t n_tiles;    // key tiles per block
    int32_t nqb;        // blocks per (image, head)
    int32_t n_blocks;   // blocks in total
    int* counters;      // [n_blocks]: zero at launch, left zero (split launches only)
    float* part_o;      // [grid][block queries * D] partial outputs of pieces
    float* part_ml;     // [grid][block queries][2] their row statistics
};

__device__ __forceinline__ int64_t pick(int j, int end0, int end1, int64_t a0, int64_t a1, int64_t a2) {
    const int64_t a12 = j < end1 ? a1 : a2;
    return j < end0 ? a0 : a12;
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// Two transposing reads (rows p and p + 8 of a V tile) form one V^T operand.
__device__ __forceinline__ bf16x8 read_vt(const char* p) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 1024));
    const short __attribute__((ext_vector_type(8))) w = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, w);
}

// Value of lanes l and l ^ 32 combined, without an LDS round trip.
__device__ __forceinline__ float max_xor32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xor32(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// (1, 1) in a register the compiler cannot see through: the row-sum dots then
// take it as an operand, and the first dot of a half can take the inline
// constant 0 as its addend instead of a register cleared by a move.
__device__ __forceinline__ bf16x2 opaque_ones() {
    const bf16x2 one = {(bf16)1.0f, (bf16)1.0f};
    uint32_t u = __builtin_bit_cast(uint32_t, one);
    asm volatile("" : "+v"(u));
    return __builtin_bit_cast(bf16x2, u);
}

// acc + pk[0] + pk[1]; the first of a chain starts from the inline constant 0.
__device__ __forceinline__ float dot_sum(bf16x2 pk, bf16x2 ones, float acc, bool first) {
    if (first) {
        asm("v_dot2_f32_bf16 %0, %1, %2, 0"
            : "=v"(acc)
            : "v"(__builtin_bit_cast(uint32_t, pk)), "v"(__builtin_bit_cast(uint32_t, ones)));
        return acc;
    }
    return __builtin_amdgcn_fdot2_f32_bf16(pk, ones, acc, false);
}

// s_waitcnt immediate for vmcnt(v) alone.
constexpr int vm_imm(int v) { return 0xF70 | (v & 15) | ((v >> 4) << 14); }

}  // namespace attn

// The 256-query kernel (attention_wide.hip) with a schedule for its blocks.
hipError_t launch_attention_wide(const AttnParams& p, const attn::Sched& sc, int grid, hipStream_t stream);

}  // namespace pcpp
