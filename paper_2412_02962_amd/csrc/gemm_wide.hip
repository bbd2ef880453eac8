// bf16 GEMM and implicit 3x3 convolution on wide tiles (gfx950 MFMA).
//
// What bounds these products is first the L2: it delivers about 18 TB/s to
// the 256 compute units (33 bytes a clock each), so a BM x BN tile can not
// run above BM BN / (BM + BN) flops per byte times that: 576 TFLOP/s for the
// 64 x 64 tiles of gemm_dma_kernel, 1280 for 128 x 160, 1770 for 256 x 160.
// At 16384 x 320 x 8640 (a level-0 convolution) the 64 x 64 tiles moved 17.5
// TB/s and took 157 us; 128 x 160 tiles take 93 us (980 TFLOP/s; the same
// loop without its loads 65 us, without its products 70).  At 7200 x 1280 x
// 5120: 173 us on 64 x 64 tiles, 107 us on 256 x 160.
//
// One workgroup of eight wavefronts, 4 (tokens) x 2 (W rows), two per SIMD.
// Y^T = W X^T with 16x16x32 MFMAs: a lane ends up with four consecutive
// outputs of one token.  X and W tiles (64 of K) go straight into LDS, NS
// stages (rows of 128 bytes, 16-byte chunk c of row r at slot c ^ (r / 2 %
// 8): 16 consecutive rows read at one chunk are conflict-free).  Loads take
// a wave-uniform base in scalar registers plus per-lane offsets fixed before
// the loop.  One barrier per k-tile; the operands of a tile's second 32-long
// step are held in registers across it, so that every LDS read is issued
// behind one half of the products and waited for after them (256 x 160: 5 %
// over reading both halves first).
//
// Products with fewer tiles than compute units split K: the pieces of a
// tile run on one XCD, exchange their sums (fp32) through its L2, and each
// finishes its share of the tile's outputs when all have arrived, adding the
// pieces in order (so results do not depend on timing).  The sums of an XCD's
// 32 workgroups are 2 MB for 128 x 128 tiles and 2.6 for 128 x 160, which its
// 4 MB of L2 hold, but 5.2 MB for 256 x 160, of which some go to memory and
// back (the merge of 9 us in kShapes).  A piece waits a bounded time for the
// others; if it gives up, the last one to arrive does its share too.

#include <math.h>

#include "common.h"
#include "gelu.h"
#include "gemm.h"
#include "kernels.h"

namespace pcpp {

namespace {

constexpr int KT = 64;        // K per tile
constexpr int WN = 2;         // wavefronts along the W rows

typedef __attribute__((address_space(3))) void* lptr;

// 16 bytes per lane from global memory into LDS at lds + 16 lane; base is
// wave-uniform, voff the lane's byte offset.  Inline assembly, so that the
// compiler does not wait for loads in flight before every LDS read: the
// kernel orders them itself with vmcnt waits and barriers.
__device__ __forceinline__ void dma16(uint64_t base, uint32_t voff, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "{m0}"(lds) : "memory");
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// s_waitcnt immediate for vmcnt(v) alone.
constexpr int vm_imm(int v) { return 0xF70 | (v & 15) | ((v >> 4) << 14); }

// Waits until at most later * PT of this wavefront's loads are in flight (later <= L).
template <int PT, int L>
__device__ __forceinline__ void wait_tiles(int later) {
    if constexpr (L == 0) {
        __builtin_amdgcn_s_waitcnt(vm_imm(0));
    } else {
        if (later >= L)
            __builtin_amdgcn_s_waitcnt(vm_imm(L * PT));
        else
            wait_tiles<PT, L - 1>(later);
    }
}

template <int V>
struct Int {
    static constexpr int value = V;
};

__device__ __forceinline__ int l2_add(int* p, int v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

template <int BM, int BN, int WM, int NS, bool CONV, bool GEGLU>
__global__ __launch_bounds__(64 * WM * WN) void gemm_wide_kernel(GemmParams p) {
    constexpr int NWV = WM * WN;
    constexpr int THREADS = 64 * NWV;
    constexpr int STAGE = (BM + BN) * KT * 2;
    constexpr int TM = BM / WM, TN = BN / WN;  // tokens and W rows per wavefront
    constexpr int MB = TM / 16, NB = TN / 16;  // its 16 x 16 blocks
    constexpr int Q = NB * MB;
    constexpr int PIECES = (BM + BN) / 8;  // 1 KB loads (8 rows) per k-tile
    constexpr int PT = (PIECES + NWV - 1) / NWV;
    constexpr int REM = PIECES % NWV;  // wavefronts below REM load PT of them, the others PT - 1
    static_assert(BM % 64 == 0 && TN % 16 == 0 && (NS - 2) * PT <= 63, "tile shape");
    __shared__ __attribute__((aligned(16))) char lds[NS * STAGE];
    __shared__ int flag_lds;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lr = lane & 15, lq = lane >> 4;

    // Workgroup w runs on XCD w % n_xcd; an XCD's tiles are a contiguous
    // range, the pieces of a tile follow each other within it.
    const int xcd = blockIdx.x % p.n_xcd;
    const int jj = blockIdx.x / p.n_xcd;
    const int tl = jj / p.splitk;
    const int piece = jj - tl * p.splitk;
    const int tile = xcd * p.tpx + tl;
    if (tl >= p.tpx || tile >= p.n_tiles) return;  // idle slot of the last XCD (uniform)
    constexpr int BNO = GEGLU ? BN / 2 : BN;  // outputs per tile
    // groups of m_group token tiles, n-major within a group
    const int mt = (p.M + BM - 1) / BM;
    const int grp = tile / (p.m_group * (p.N / BNO));
    const int in_grp = tile - grp * (p.m_group * (p.N / BNO));
    const int gm = min(p.m_group, mt - grp * p.m_group);
    const int n_tile = in_grp / gm;
    const int m_tile = grp * p.m_group + (in_grp - n_tile * gm);
    const int m0 = m_tile * BM, n0 = n_tile * BNO;
    const int nk_all = p.K / KT;
    const int kt0 = (int)((int64_t)nk_all * piece / p.splitk);
    const int nkt = (int)((int64_t)nk_all * (piece + 1) / p.splitk) - kt0;

    // Byte offset of token m's row of X (convolution: of its tap (0, 0) in
    // the framed band).
    const int cin = CONV ? p.K / 9 : 0;
    auto row_off = [&](int m) -> int64_t {
        if constexpr (CONV) {
            const int st = p.conv_stride;
            const int wo = p.conv_W / st;
            const int per = (p.conv_rows / st) * wo;
            const int b = m / per, rem = m - b * per;
            const int y = rem / wo, x = rem - y * wo;
            return ((int64_t)(b * (p.conv_rows + 2) + st * y) * (p.conv_W + 2) + st * x) * cin * 2;
        } else {
            return (int64_t)m * p.lda * 2;
        }
    };
    const int64_t x0 = row_off(m0);
    const uint64_t xbase = uniform64((uint64_t)(uintptr_t)p.a + (uint64_t)x0);
    const __bf16* wmat = p.w;
    int wrow0 = n0;
    if (!GEGLU && p.w_seg_rows > 0) {  // a tile's rows never straddle two matrices
        const int j = n0 / p.w_seg_rows;
        wmat = p.w_seg[j];
        wrow0 = n0 - j * p.w_seg_rows;
    }
    const uint64_t wbase = uniform64((uint64_t)(uintptr_t)wmat + (uint64_t)wrow0 * p.K * 2);
    uint32_t voff[PT];
#pragma unroll
    for (int q = 0; q < PT; ++q) {
        const int r = 8 * (wave + NWV * q) + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        if (r < BM) {
            voff[q] = (uint32_t)(row_off(min(m0 + r, p.M - 1)) - x0) + 16 * c;
        } else {
            int wr = min(r - BM, BN - 1);
            if (GEGLU && wr >= BN / 2) wr += p.F - BN / 2;
            voff[q] = (uint32_t)wr * (uint32_t)(p.K * 2) + 16 * c;
        }
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lptr)lds);
    // Convolution: the nine taps of 64 channels follow each other, so that a
    // tile's X rows are read nine times within a short while (from the L2;
    // with the channels inside the taps they came from beyond it each time).
    int iss_t = 0, iss_kx = 0;
    int64_t iss_x = 0, iss_w = 0;
    if constexpr (CONV) {
        const int cb = kt0 / 9;
        iss_t = kt0 - 9 * cb;
        iss_kx = iss_t % 3;
        iss_x = ((int64_t)(iss_t / 3 * (p.conv_W + 2) + iss_kx) * cin + cb * KT) * 2;
        iss_w = ((int64_t)iss_t * cin + cb * KT) * 2;
    } else {
        iss_x = iss_w = (int64_t)kt0 * KT * 2;
    }
    const bool more = REM == 0 || wave < REM;
    auto issue = [&](int slot) {  // the next k-tile into `slot`
        const uint64_t xb = xbase + (uint64_t)iss_x, wb = wbase + (uint64_t)iss_w;
        if constexpr (CONV) {
            iss_w += 2 * cin;
            iss_x += 2 * cin;
            if (++iss_kx == 3) {
                iss_kx = 0;
                iss_x += (int64_t)(p.conv_W - 1) * cin * 2;
            }
            if (++iss_t == 9) {
                iss_t = 0;
                iss_w += KT * 2 - 18 * (int64_t)cin;
                iss_x += KT * 2 - 6 * (int64_t)(p.conv_W + 2) * cin;
            }
        } else {
            iss_x += KT * 2;
            iss_w += KT * 2;
        }
        const uint32_t l = lds0 + slot * STAGE + wave * 1024;
#pragma unroll
        for (int q = 0; q < PT; ++q)
            if (q < PT - 1 || more) dma16((wave + NWV * q) * 8 < BM ? xb : wb, voff[q], l + q * NWV * 1024);
    };

    // Operands of k-step s (32 of K): rows lr of each block, chunk 4 s + lq.
    const int swz = (lr >> 1) & 7;
    const uint32_t coff[2] = {(uint32_t)(((lq ^ swz) << 4) + lr * 128), (uint32_t)((((4 + lq) ^ swz) << 4) + lr * 128)};
    struct Ops {
        bf16x8 x[MB], w[NB];
    };
    auto read_ops = [&](int slot, int s, Ops& o) {
        const char* b = lds + slot * STAGE + coff[s];
#pragma unroll
        for (int j = 0; j < MB; ++j) o.x[j] = *(const bf16x8*)(b + (wm * TM + 16 * j) * 128);
#pragma unroll
        for (int i = 0; i < NB; ++i) o.w[i] = *(const bf16x8*)(b + (BM + wn * TN + 16 * i) * 128);
    };
    f32x4 acc[NB][MB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto mma = [&](const Ops& o) {
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) acc[i][j] = mfma16(o.w[i], o.x[j], acc[i][j]);
    };

#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < nkt) issue(s);
    Ops o0, o1;
    int slot = 0;
    for (int i = 0; i < nkt; ++i) {
        const int later = min(nkt - 1 - i, NS - 2);  // k-tiles issued after this one
        if (more)
            wait_tiles<PT, NS - 2>(later);
        else
            wait_tiles<PT - 1, NS - 2>(later);
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this wavefront has read the previous tile
        // Everyone's pieces of this tile have landed, and the previous tile's slot is free.
        __builtin_amdgcn_s_barrier();
        if (i + NS - 1 < nkt) issue(slot == 0 ? NS - 1 : slot - 1);
        read_ops(slot, 0, o0);
        __builtin_amdgcn_sched_barrier(0);
        if (i > 0) mma(o1);
        __builtin_amdgcn_sched_barrier(0);
        read_ops(slot, 1, o1);
        __builtin_amdgcn_sched_barrier(0);
        mma(o0);
        __builtin_amdgcn_sched_barrier(0);
        slot = slot == NS - 1 ? 0 : slot + 1;
    }
    mma(o1);

    // The output segment is the whole tile's (the plan sees to it): picked
    // per lane it would be a load from the kernel's arguments for every store.
    char* out = (char*)p.out[0];
    int nseg = n0;  // the tile's first column within it
    if (p.seg < p.N) {
        const int seg = n0 / p.seg;
        nseg = n0 - seg * p.seg;
        if (p.seg_stride > 0)
            out += (int64_t)seg * p.seg_stride * (p.out_f32 ? 4 : 2);
        else
            out = (char*)(seg == 0 ? p.out[0] : (seg == 1 ? p.out[1] : p.out[2]));
    }
    // bias2's row, where the whole tile lies in one image
    const int b2_lo = p.bias2 != nullptr ? m0 / p.bias2_rows : 0;
    const bool b2_one = p.bias2 != nullptr && (min(m0 + BM, p.M) - 1) / p.bias2_rows == b2_lo;
    auto widen = [](bf16x4 b) -> f32x4 {
        return f32x4{bf16_to_f32(b[0]), bf16_to_f32(b[1]), bf16_to_f32(b[2]), bf16_to_f32(b[3])};
    };
    auto bias_at = [&](int n) -> bf16x4 {
        bf16x4 b = {};
        if (p.bias != nullptr) b = *(const bf16x4*)(p.bias + n);
        return b;
    };
    // Residual plus the per-image bias of outputs n .. n + 3 of token m.
    auto resid_at = [&](int m, int n) -> f32x4 {
        m = min(m, p.M - 1);
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (p.resid != nullptr) {
            const int64_t at = (int64_t)m * p.ldr + n;
            if (p.resid_f32)
                v = *(const f32x4*)((const float*)p.resid + at);
            else
                v = widen(*(const bf16x4*)((const bf16*)p.resid + at));
        }
        if (p.bias2 != nullptr)
            v += *(const f32x4*)(p.bias2 + (int64_t)(b2_one ? b2_lo : m / p.bias2_rows) * p.N + n);
        return v;
    };
    auto to_bf16 = [](f32x4 v) -> bf16x4 {
        return bf16x4{f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
    };

    if (GEGLU || p.splitk == 1) {
        // Through LDS, so that loads and stores run along the rows: straight
        // from the accumulators a store touches 16 rows for 32 bytes each,
        // about 80 cycles, and a 256 x 160 tile took 8 us for its outputs.
        // Passes of ROWS tokens; a thread takes eight outputs of every RPI-th.
        constexpr int ROWS = BM > 128 ? 128 : BM;
        constexpr int PASSES = BM / ROWS;
        constexpr int LDF = BN + 4;  // floats per row: 16 rows written at one column on distinct banks
        constexpr int C8 = BNO / 8;
        constexpr int RPI = THREADS / C8;  // tokens per iteration (the last THREADS % C8 threads idle)
        constexpr int ITER = (ROWS + RPI - 1) / RPI;
        static_assert(ROWS * LDF * 4 <= NS * STAGE && ROWS % TM == 0, "a pass fits the stages");
        float* tab = (float*)lds;
        const int r0 = tid / C8, c = 8 * (tid - r0 * C8), n = n0 + c;
        const bool active = tid < RPI * C8;
        bf16x4 bias[2], bias_g[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            bias[h] = bias_at(n + 4 * h);
            if constexpr (GEGLU) bias_g[h] = bias_at(p.F + n + 4 * h);
        }
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
            const int mp = m0 + ROWS * ps + r0;
            f32x4 res[ITER][2];
            if constexpr (!GEGLU) {  // all of a pass's loads before its first store: the output may be the residual
#pragma unroll
                for (int it = 0; it < ITER; ++it) {
                    res[it][0] = resid_at(mp + RPI * it, n);
                    res[it][1] = resid_at(mp + RPI * it, n + 4);
                }
            }
            __syncthreads();  // the stages, or the previous pass, have been read
            if (wm * TM / ROWS == ps) {
                float* at = tab + (wm * TM - ROWS * ps + lr) * LDF + wn * TN + 4 * lq;
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int j = 0; j < MB; ++j) *(f32x4*)(at + 16 * j * LDF + 16 * i) = acc[i][j];
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < ITER; ++it) {
                const int r = r0 + RPI * it, m = mp + RPI * it;
                if (!active || r >= ROWS || m >= p.M) continue;
                f32x4 v[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v[h] = *(const f32x4*)(tab + r * LDF + c + 4 * h) + widen(bias[h]);
                    if constexpr (GEGLU) {
                        const f32x4 g = *(const f32x4*)(tab + r * LDF + BNO + c + 4 * h) + widen(bias_g[h]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[h][e] *= gelu_erf(g[e]);
                    } else {
                        v[h] += res[it][h];
                    }
                }
                const bf16x4 b0 = to_bf16(v[0]), b1 = to_bf16(v[1]);
                const bf16x8 b = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
                const int64_t at = (int64_t)m * p.ldo + c;
                if (p.out_f32) {
                    float* o = (float*)out + nseg + at;
                    *(f32x4*)o = v[0];
                    *(f32x4*)(o + 4) = v[1];
                } else {
                    *(bf16x8*)((bf16*)out + nseg + at) = b;
                }
                if (p.out_bf16 != nullptr) *(bf16x8*)((bf16*)p.out_bf16 + n0 + at) = b;
            }
        }
        return;
    }

    // Block (i, j) of a wavefront: token m_of(j) of this lane, outputs n0 + c_of(i) .. + 3.
    auto m_of = [&](int j) { return m0 + wm * TM + 16 * j + lr; };
    auto c_of = [&](int i) { return wn * TN + 16 * i + 4 * lq; };
    auto put = [&](int m, int c, f32x4 v) {
        if (m >= p.M) return;
        const bf16x4 b = to_bf16(v);
        const int64_t at = (int64_t)m * p.ldo + c;
        if (p.out_f32)
            *(f32x4*)((float*)out + nseg + at) = v;
        else
            *(bf16x4*)((bf16*)out + nseg + at) = b;
        if (p.out_bf16 != nullptr) *(bf16x4*)((bf16*)p.out_bf16 + n0 + at) = b;
    };

    // Split K.  tile's two counters: bits 0-7 arrivals, bit 8 + s set when
    // piece s gave up; and the pieces that are done with the first.
    const int k = p.splitk;
    auto part_of = [&](int pc) {
        return (float*)p.split_ws + GEMM_SPLIT_COUNTERS +
               ((int64_t)((tl * k + pc) * p.n_xcd + xcd) * NWV + wave) * (Q * 256) + lane * 4;
    };
    {
        float* dst = part_of(piece);
#pragma unroll
        for (int q = 0; q < Q; ++q) *(f32x4*)(dst + q * 256) = acc[q / MB][q % MB];
    }
    __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0): this thread's stores reached the L2
    __syncthreads();
    if (tid == 0) {
        int* cnt = (int*)p.split_ws + 2 * tile;
        int todo = 0;
        const int was = l2_add(cnt, 1);
        if ((was & 255) == k - 1) {
            todo = (was >> 8) | (1 << piece);  // the last: its own share and those given up
        } else {
            // An addend that the compiler does not know to be zero: it would
            // turn the read into a load, which may hit in the L1.
            int zero = 0;
            asm volatile("" : "+v"(zero));
            bool all = false;
            for (int it = 0; !all && it < p.max_polls; ++it) {
                __builtin_amdgcn_s_sleep(1);
                all = (l2_add(cnt, zero) & 255) == k;
            }
            // Giving up and the last arrival are ordered by the counter: either
            // the last one sees the bit, or all had arrived.
            if (!all) all = (l2_add(cnt, 256 << piece) & 255) == k;
            if (all) todo = 1 << piece;
        }
        flag_lds = todo;
        if (l2_add(cnt + 1, 1) == k - 1) {  // nobody looks at the first counter any more
            __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(cnt + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    __syncthreads();
    const int todo = __builtin_amdgcn_readfirstlane(flag_lds);
    // Share s of the tile: of every wavefront's blocks, those from Q s / k on.
    auto share = [&](auto ktag, int s) {
        constexpr int K = decltype(ktag)::value;
        constexpr int QS = (Q + K - 1) / K;  // blocks, at most
        constexpr int G = QS < 16 / K ? QS : 16 / K;  // blocks in flight at once
        const int q0 = Q * s / K, q1 = Q * (s + 1) / K;
#pragma unroll 1
        for (int g = q0; g < q1; g += G) {
            f32x4 v[K][G], res[G];
            bf16x4 bias[G];
#pragma unroll
            for (int pc = 0; pc < K; ++pc)
#pragma unroll
                for (int r = 0; r < G; ++r) v[pc][r] = *(const f32x4*)(part_of(pc) + min(g + r, q1 - 1) * 256);
#pragma unroll
            for (int r = 0; r < G; ++r) {
                const int q = min(g + r, q1 - 1), n = n0 + c_of(q / MB);
                bias[r] = bias_at(n);
                res[r] = resid_at(m_of(q % MB), n);
            }
#pragma unroll
            for (int r = 0; r < G; ++r) {
                f32x4 sum = v[0][r];
#pragma unroll
                for (int pc = 1; pc < K; ++pc) sum += v[pc][r];
                const int q = g + r;
                if (q < q1) put(m_of(q % MB), c_of(q / MB), (sum + widen(bias[r])) + res[r]);
            }
        }
    };
    for (int s = 0; s < k; ++s) {
        if (!(todo >> s & 1)) continue;
        switch (k) {
            case 2: share(Int<2>{}, s); break;
            case 3: share(Int<3>{}, s); break;
            case 4: share(Int<4>{}, s); break;
            case 5: share(Int<5>{}, s); break;
            case 6: share(Int<6>{}, s); break;
            case 7: share(Int<7>{}, s); break;
            default: share(Int<8>{}, s); break;
        }
    }
}

template <int BM, int BN, int WM, int NS>
hipError_t launch_shape(const GemmParams& p, hipStream_t s) {
    constexpr int THREADS = 64 * WM * WN;
    const dim3 grid((unsigned)((int64_t)p.n_xcd * p.tpx * p.splitk));
    if (p.geglu)
        gemm_wide_kernel<BM, BN, WM, NS, false, true><<<grid, THREADS, 0, s>>>(p);
    else if (p.conv_W > 0)
        gemm_wide_kernel<BM, BN, WM, NS, true, false><<<grid, THREADS, 0, s>>>(p);
    else
        gemm_wide_kernel<BM, BN, WM, NS, false, false><<<grid, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

// The tiles, with the measured microseconds of one round of workgroups: ends
// (first loads, stores), per k-tile (of a launch with at most one workgroup
// per compute unit, and with more), and the merge of split pieces.
struct Shape {
    int bm, bn, share;  // share: workgroups on a compute unit
    double ends, ktile, ktile_shared, merge;
};
constexpr Shape kShapes[] = {
    {256, 160, 1, 8.5, 0.98, 0.98, 9.0},  // 156 KB of LDS, three stages
    {128, 160, 1, 4.0, 0.68, 0.68, 8.5},  // 144 KB, four stages
    {128, 128, 1, 4.0, 0.57, 0.57, 5.0},  // 128 KB, four stages
    {64, 128, 2, 3.3, 0.40, 0.77, 5.0},   // 72 KB, three stages, four wavefronts
};
// GEGLU, fitted to 100 products of 65 to 40000 tokens and K = 64 to 1280
// (launch 2 us; the estimate's choice is on average 1 % over the fastest
// tile). It never splits. Short K and several rounds of workgroups want
// small tiles, whose ends hide behind other workgroups of the unit: with two
// stages of 64 x 128 (48 KB) three of them share one. 2072 x 1280 x 320: 16.2 us
// on 256 x 160, 12.4 there; 8219 x 1024 x 256: 30.4 on 128 x 128, 22.4; 23864 x
// 2048 x 512: 206 and 155. (Plain products and convolutions keep the first
// four: they have the 64 x 64 and 64 x 80 tiles of gemm.hip beside them.)
constexpr Shape kGegluShapes[] = {
    {256, 160, 1, 7.5, 0.92, 1.12, 0.0},
    {128, 160, 1, 4.1, 0.64, 0.73, 0.0},
    {128, 128, 1, 3.6, 0.51, 0.56, 0.0},
    {64, 128, 2, 2.8, 0.36, 0.62, 0.0},
    {64, 128, 3, 3.0, 0.48, 0.88, 0.0},  // two stages
};
constexpr double kLaunch = 4.0, kGegluLaunch = 2.0;
constexpr int kMaxSplit = 8;
constexpr int kMinPieceTiles = 4;  // k-tiles per piece

struct Choice {
    int shape, splitk;
    double us;
    size_t bytes;
};

// The estimated fastest tile and split: rounds of workgroups, each the ends
// plus its k-tiles.  A split launch is one round (its pieces wait for each
// other) and needs `bytes` of workspace.
Choice choose(int M, int outs, int K, bool geglu, int seg, int w_seg_rows, size_t ws, const DeviceLayout& dl) {
    Choice best{-1, 1, 1e30, 0};
    const int nk = K / KT;
    const int n_xcd = dl.xcd_merge ? dl.n_xcd : 1;
    const int n_shapes = geglu ? sizeof(kGegluShapes) / sizeof(Shape) : sizeof(kShapes) / sizeof(Shape);
    for (int i = 0; i < n_shapes; ++i) {
        const Shape& sh = geglu ? kGegluShapes[i] : kShapes[i];
        const int bno = geglu ? sh.bn / 2 : sh.bn;
        if (outs % bno != 0 || (w_seg_rows > 0 && w_seg_rows % sh.bn != 0) || (seg < outs && seg % bno != 0)) continue;
        const int64_t tiles = (int64_t)((M + sh.bm - 1) / sh.bm) * (outs / bno);
        const int64_t tpx = (tiles + n_xcd - 1) / n_xcd;
        if (tiles < 1 || n_xcd * tpx * kMaxSplit > INT32_MAX) continue;
        const int64_t slots = (int64_t)dl.cus * sh.share;
        for (int k = 1; k <= kMaxSplit; ++k) {
            const int64_t wgs = n_xcd * tpx * k;
            size_t bytes = 0;
            if (k > 1) {
                bytes = (size_t)GEMM_SPLIT_COUNTERS * 4 + (size_t)wgs * sh.bm * sh.bn * 4;
                if (geglu || !dl.xcd_merge || sh.share > 1 || wgs > dl.cus || nk / k < kMinPieceTiles || bytes > ws ||
                    2 * tiles > GEMM_SPLIT_COUNTERS)
                    break;
            }
            const double rounds = (double)((wgs + slots - 1) / slots);
            const double ktile = wgs > dl.cus ? sh.ktile_shared : sh.ktile;
            const double us = (geglu ? kGegluLaunch : kLaunch) + rounds * (sh.ends + ktile * ((nk + k - 1) / k)) + (k > 1 ? sh.merge : 0.0);
            if (us < best.us) best = Choice{i, k, us, bytes};
        }
    }
    return best;
}

// Bound on the byte offsets of the largest tile's rows of X from its first
// row.  Convolution: 256 tokens reach (255 / wo + 1) output rows further,
// each `stride` framed rows, and two framed rows more per image boundary;
// one row for the place within a row.  (A bound that gives every token a row
// of its own refuses the 3840 px ResNets: 1920 -> 640 on 60 rows of 240 columns
// 885 us on 64 x 64 and 128 x 128 tiles, 541 on these; 960 -> 320 on 60 rows of
// 480: 683 and 331.)
int64_t x_span(const GemmParams& p) {
    if (p.conv_W <= 0) return (int64_t)256 * p.lda * 2;
    const int64_t wo = p.conv_W / p.conv_stride, per = (p.conv_rows / p.conv_stride) * wo;
    const int64_t rows = (255 / wo + 1) * p.conv_stride + (255 / per + 1) * 2 + 1;
    return rows * (p.conv_W + 2) * (p.K / 9) * 2;
}

}  // namespace

void wide_tile(int shape, bool geglu, int32_t& tokens, int32_t& outputs, int32_t& per_cu) {
    const Shape& sh = geglu ? kGegluShapes[shape] : kShapes[shape];
    tokens = sh.bm;
    outputs = geglu ? sh.bn / 2 : sh.bn;
    per_cu = sh.share;
}

size_t wide_split_bytes(int M, int N, int K, const DeviceLayout& dl) {
    if (M < 1 || N < 1 || K % KT != 0) return 0;
    return choose(M, N, K, false, N, 0, SIZE_MAX, dl).bytes;
}

bool plan_wide(GemmParams& p, const DeviceLayout& dl, double& limit_us, int& shape) {
    if (p.a_f32 || p.xa_T != 0 || p.gn_N != 0 || p.K % KT != 0 || p.M < 1 || p.ldo % 8 != 0 ||
        (p.resid != nullptr && p.ldr % 8 != 0))
        return false;
    if (p.geglu && (p.resid != nullptr || p.out_bf16 != nullptr || p.bias2 != nullptr || p.seg < p.N ||
                    p.w_seg_rows != 0 || p.seg_stride != 0))
        return false;
    // 32-bit offsets within a tile's rows of W and X
    const int64_t w_span = ((p.geglu ? (int64_t)p.F : 0) + 160) * p.K * 2;
    if (w_span >= INT32_MAX || x_span(p) >= INT32_MAX) return false;
    const bool ws_ok = p.split_ws != nullptr && ((uintptr_t)p.split_ws & 15u) == 0;
    const Choice c = choose(p.M, p.N, p.K, p.geglu != 0, p.seg, p.w_seg_rows, ws_ok ? p.split_ws_bytes : 0, dl);
    if (c.shape < 0 || c.us >= limit_us) return false;
    const Shape& sh = p.geglu ? kGegluShapes[c.shape] : kShapes[c.shape];
    const int mt = (p.M + sh.bm - 1) / sh.bm, nt = p.N / (p.geglu ? sh.bn / 2 : sh.bn);
    p.n_tiles = mt * nt;
    p.splitk = c.splitk;
    p.n_xcd = dl.xcd_merge ? dl.n_xcd : 1;
    p.tpx = (p.n_tiles + p.n_xcd - 1) / p.n_xcd;
    // Order of the tiles: groups of token tiles whose range of tpx tiles on an
    // XCD covers the fewest rows of X and W, which its L2 takes in.
    int64_t fewest = INT64_MAX;
    for (int g = 1; g <= mt && g <= 64; g = g < mt && 2 * g > mt ? mt : 2 * g) {
        const int64_t per = (int64_t)g * nt;  // tiles of a group
        const int64_t mr = p.tpx <= g ? p.tpx : g * ((p.tpx + per - 1) / per);
        const int64_t nr = p.tpx >= per ? nt : (p.tpx + g - 1) / g;
        const int64_t rows = (mr < mt ? mr : mt) * sh.bm + nr * sh.bn;
        if (rows < fewest) {
            fewest = rows;
            p.m_group = g;
        }
    }
    shape = c.shape;
    limit_us = c.us;
    return true;
}

hipError_t launch_gemm_wide(const GemmParams& p, int shape, hipStream_t s) {
    switch (shape) {
        case 0: return launch_shape<256, 160, 4, 3>(p, s);
        case 1: return launch_shape<128, 160, 4, 4>(p, s);
        case 2: return launch_shape<128, 128, 4, 4>(p, s);
        case 3: return launch_shape<64, 128, 2, 3>(p, s);
        default: {  // GEGLU's own
            const dim3 grid((unsigned)((int64_t)p.n_xcd * p.tpx));
            gemm_wide_kernel<64, 128, 2, 2, false, true><<<grid, 64 * 2 * WN, 0, s>>>(p);
            return hipGetLastError();
        }
    }
}

}  // namespace pcpp
