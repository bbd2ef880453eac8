// Partially conditioned self-attention, bf16, 256 queries per workgroup: the
// form for launches with enough queries to fill the compute units
// (attention_bf16.hip has the 128-query form, the mathematics and the key
// sources; the softmax, its rounding and the merge of key pieces are the
// same here).
//
// What bounds both forms is how the wavefronts of a SIMD share its issue: a
// 32-key half-tile costs 32 queries 256 cycles of matrix products and about
// 270 of vector work (an exponential 8 to 10 cycles, the rest 4 to 5, at two
// wavefronts per SIMD; one alone issues only every 8 to 16 cycles), and the
// 128-query form takes 484.  Here a wavefront holds 64 queries, two blocks A
// and B of 32, half a half-tile apart:
//   phase 1 of half-tile h   products  O_B += V(h-1)^T P_B(h-1),  S_B(h) = K(h) Q_B
//                            softmax   S_A(h) -> P_A(h)
//   phase 2                  products  O_A += V(h)^T P_A(h),  S_A(h+1) = K(h+1) Q_A
//                            softmax   S_B(h) -> P_B(h)
// Nothing in a phase's softmax waits for its products: they are issued in one
// run, which the other wavefront of the SIMD fills with its softmax.  K and V
// operands are read once for both blocks (half the LDS reads and half the
// staging per query), into the registers whose last use has just been
// issued.  About 400 cycles: 28800 x 37440 x 10 heads 2780 -> 2664 us, 7200 x
// 9360 x 20 heads 453 -> 374 us (replayed in turn on one card).  (One workgroup per compute unit: 3660 us;
// products and softmax interleaved one by one: 2816; products at high
// priority or not, in runs of two, four or eight: within 1 %.)
//
// K and V tiles (64 keys, 8 KB each) go straight into a ring of LDS slots,
// AHEAD tiles ahead; one barrier per tile.

#include <math.h>

#include "attention_bf16.h"
#include "common.h"
#include "kernels.h"

namespace pcpp {

namespace {

using namespace attn;

constexpr int QW = 64;                  // queries per wavefront
constexpr int NW = 4;
constexpr int QB = QW * NW;
constexpr int NTHREADS = 64 * NW;
constexpr int AHEAD = 2;                // tiles in flight or landed beyond the current one
constexpr int SLOTS = AHEAD + 2;        // V of the tile before is still being read
constexpr int PIECES = TILE_BYTES / 1024 / NW;
constexpr int TILE_LOADS = 2 * PIECES;  // per thread
static_assert(QB == WIDE_QUERIES, "block size");

#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#define INLINE __attribute__((always_inline))  // a closure left as a call would live in scratch memory

__global__ __launch_bounds__(NTHREADS, 2) void attn_wide_kernel(AttnParams p, Sched sc) {
    __shared__ __attribute__((aligned(16))) char lds[SLOTS * 2 * TILE_BYTES];  // slot: K tile, V tile
    __shared__ int flag_lds;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31;
    const int half = lane >> 5;
    const int C = p.C;
    const int kv_end = p.kv.n_kv;
    const int end0 = p.kv.end0, end1 = p.kv.end1;
    const float sl2 = p.scale_log2;
    const bf16x2 ones = opaque_ones();
    const int n_tiles = sc.n_tiles;

    const int x = blockIdx.x % sc.n_xcd;
    const int jx = blockIdx.x / sc.n_xcd;
    const int bl = jx / sc.k;  // block, XCD-local
    const int piece = jx - bl * sc.k;
    const int blk = x * sc.bpx + bl;
    if (bl >= sc.bpx || blk >= sc.n_blocks) return;  // idle slot of the last XCD (uniform)
    const int t0 = (int)((int64_t)n_tiles * piece / sc.k);
    const int t1 = (int)((int64_t)n_tiles * (piece + 1) / sc.k);

    const int qb = blk % sc.nqb;
    const int bh = blk / sc.nqb;
    const int head = bh % p.heads;
    const int b = bh / p.heads;
    const int head_off = head * D;

    // Staging: wavefront w fills the 1 KB parts 2 w and 2 w + 1 of a tile.
    int ld_row[PIECES];
    uint32_t ld_koff[PIECES], ld_voff[PIECES];
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
        const int r = 8 * (PIECES * wave + i) + (lane >> 3);
        ld_row[i] = r;
        ld_koff[i] = (uint32_t)(r * C * 2 + (((lane & 7) ^ k_mask(r)) << 4));
        ld_voff[i] = (uint32_t)(r * C * 2 + (((lane & 7) ^ v_mask(r)) << 4));
    }
    const int64_t o0 = (int64_t)b * p.kv.bstride[0] + head_off;
    const int64_t o1 = (int64_t)b * p.kv.bstride[1] - (int64_t)end0 * C + head_off;
    const int64_t o2 = (int64_t)b * p.kv.bstride[2] - (int64_t)end1 * C + head_off;
    const uint64_t sk0 = uniform64((uint64_t)(uintptr_t)p.kv.k[0] + (uint64_t)(o0 * 2));
    const uint64_t sk1 = uniform64((uint64_t)(uintptr_t)p.kv.k[1] + (uint64_t)(o1 * 2));
    const uint64_t sk2 = uniform64((uint64_t)(uintptr_t)p.kv.k[2] + (uint64_t)(o2 * 2));
    const uint64_t sv0 = uniform64((uint64_t)(uintptr_t)p.kv.v[0] + (uint64_t)(o0 * 2));
    const uint64_t sv1 = uniform64((uint64_t)(uintptr_t)p.kv.v[1] + (uint64_t)(o1 * 2));
    const uint64_t sv2 = uniform64((uint64_t)(uintptr_t)p.kv.v[2] + (uint64_t)(o2 * 2));
    const uint32_t lds_w = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lptr_t)lds) +
                           (uint32_t)(PIECES * wave * 1024);
    // Stage K and V of tile t into its slot.
    auto issue = [&](int t_in, int slot) INLINE {
        const int t = __builtin_amdgcn_readfirstlane(t_in);
        const uint32_t dst = lds_w + slot * (2 * TILE_BYTES);
        const int j0 = t * KT, j1 = j0 + KT;
        if (j1 <= kv_end && (j1 <= end0 || j0 >= end0) && (j1 <= end1 || j0 >= end1)) {  // one source
            const uint64_t at = (uint64_t)j0 * (uint64_t)(C * 2);
            const uint64_t kb = (uint64_t)pick(j0, end0, end1, sk0, sk1, sk2) + at;
            const uint64_t vb = (uint64_t)pick(j0, end0, end1, sv0, sv1, sv2) + at;
#pragma unroll
            for (int i = 0; i < PIECES; ++i) dma16_s(kb, ld_koff[i], dst + i * 1024);
#pragma unroll
            for (int i = 0; i < PIECES; ++i) dma16_s(vb, ld_voff[i], dst + TILE_BYTES + i * 1024);
            return;
        }
        // A tile across two sources, or past the end (clamped; its scores are masked): row by row.
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            int jk = j0 + ld_row[i];
            jk = jk < kv_end ? jk : kv_end - 1;
            const int64_t at = ((int64_t)jk - ld_row[i]) * C * 2;
            dma16((const char*)(uintptr_t)(pick(jk, end0, end1, sk0, sk1, sk2) + at) + ld_koff[i], dst + i * 1024);
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            int jk = j0 + ld_row[i];
            jk = jk < kv_end ? jk : kv_end - 1;
            const int64_t at = ((int64_t)jk - ld_row[i]) * C * 2;
            dma16((const char*)(uintptr_t)(pick(jk, end0, end1, sv0, sv1, sv2) + at) + ld_voff[i],
                  dst + TILE_BYTES + i * 1024);
        }
    };

    // Operand reads within a half-tile (32 keys): K rows col, chunks 2 kk +
    // half; V through the transposing read, 32-dim block mb.
    int k_rel[4], v_rel[2];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) k_rel[kk] = col * 128 + (((2 * kk + half) ^ k_mask(col)) << 4);
    {
        const int jj = lane & 15;
        const int tr_row = 4 * half + (jj >> 2);
        const int tr_e = 16 * ((lane >> 4) & 1) + 4 * (jj & 3);
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            const int e = 32 * mb + tr_e;
            v_rel[mb] = TILE_BYTES + tr_row * 128 + (((e >> 3) ^ v_mask(tr_row)) << 4) + ((e & 7) << 1);
        }
    }

#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
        if (t0 + t < t1) issue(t0 + t, t);

    // Q^T operands of the two blocks.
    const int q_base = qb * QB + QW * wave;
    bf16x8 qop[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int qrow = min(q_base + 32 * u + col, p.nq - 1);
        const bf16* qp = (const bf16*)p.q + (int64_t)b * p.q_bstride + (int64_t)qrow * C + head_off + 8 * half;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qop[u][kk] = *(const bf16x8*)(qp + 16 * kk);
    }

    f32x16 o[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[u][mb][r] = 0.f;
    float m_run[2] = {-INFINITY, -INFINITY}, l_run[2] = {0.f, 0.f};
    f32x16 s[2];
    bf16x8 pr[2][2], kop[4], vop[2][2];
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            pr[0][st][e] = pr[1][st][e] = (bf16)0.0f;
            vop[0][st][e] = vop[1][st][e] = (bf16)0.0f;
        }

    // Scores of half h past the last key are -inf.
    auto mask_half = [&](int h, f32x16& sv) INLINE {
        if ((h >> 1) * KT + KT > kv_end) {
            int hl = 4 * half;
            asm volatile("" : "+v"(hl));  // (not computed ahead of the branch)
#pragma unroll
            for (int rr = 0; rr < 16; ++rr) {
                const int jk = (h >> 1) * KT + 32 * (h & 1) + 8 * (rr >> 2) + hl + (rr & 3);
                if (jk >= kv_end) sv[rr] = -INFINITY;
            }
        }
    };

    // One phase.  Products: O_w += V^T P_w (vop), S_w = K Q_w (kop), w =
    // WB; softmax of block 1 - w.  FILL: after a K or V operand's use its
    // registers take the operand at the given LDS addresses.  QK: with the
    // score products.
    auto phase = [&](auto wtag, auto fill_tag, auto qk_tag, const char* knext, const char* vnext) INLINE {
        constexpr int W = decltype(wtag)::value, A = 1 - W;
        constexpr bool FILL = decltype(fill_tag)::value, QK = decltype(qk_tag)::value;
        float acc0 = 0.f;
        float mneg = -m_run[A];
        // Probabilities of scores 2 i, 2 i + 1 and their sum, as bf16.
        auto pair = [&](int i) INLINE {
            const float e0 = fast_exp2(fmaf(s[A][2 * i], sl2, mneg));
            const float e1 = fast_exp2(fmaf(s[A][2 * i + 1], sl2, mneg));
            const bf16x2 pk = {f32_to_bf16(e0), f32_to_bf16(e1)};
            pr[A][i >> 2][2 * (i & 3)] = pk[0];
            pr[A][i >> 2][2 * (i & 3) + 1] = pk[1];
            acc0 = dot_sum(pk, ones, acc0, i == 0);
        };
        SCHED_FENCE();
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int st = i >> 2, mb = (i >> 1) & 1, kk = i >> 1;
            if ((i & 1) == 0) {
                if constexpr (QK) s[W] = mfma32x32x16(kop[kk], qop[W][kk], kk == 0 ? f32x16{} : s[W]);
            } else {
                o[W][mb] = mfma32x32x16(vop[mb][st], pr[W][st], o[W][mb]);
            }
            SCHED_FENCE();
            if constexpr (FILL) {
                if ((i & 1) == 0)
                    kop[kk] = *(const bf16x8*)(knext + k_rel[kk]);
                else
                    vop[mb][st] = read_vt(vnext + v_rel[mb] + st * 2048);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        SCHED_FENCE();
#pragma unroll
        for (int i = 0; i < 8; ++i) pair(i);
        SCHED_FENCE();
        float lt = acc0;
        if (__any(!(lt < P_LIMIT))) {
            // As in the 128-query form: the half's maximum is taken only when a
            // lane's probabilities sum to 2^20 or more (or to inf or NaN).
            float m4[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                m4[i] = fmaxf(fmaxf(s[A][4 * i], s[A][4 * i + 1]), fmaxf(s[A][4 * i + 2], s[A][4 * i + 3]));
            const float mx = max_xor32(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]))) * sl2;
            const float m_new = fmaxf(m_run[A], mx);
            // A query whose scores so far are all -inf: the maxima are equal and
            // their difference no number; its probabilities are exp2(-inf) = 0.
            const float alpha = m_new == m_run[A] ? 1.f : fast_exp2(m_run[A] - m_new);
            m_run[A] = m_new;
            l_run[A] *= alpha;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[A][mb][r] *= alpha;
            mneg = m_new == -INFINITY ? 0.f : -m_new;
#pragma unroll
            for (int i = 0; i < 8; ++i) pair(i);
            lt = acc0;
        }
        l_run[A] += lt;
    };
    constexpr Int<0> kA{};
    constexpr Int<1> kB{};
    constexpr Int<0> no{};
    constexpr Int<1> yes{};
    auto k_at = [&](int slot, int hh) INLINE { return (const char*)lds + slot * (2 * TILE_BYTES) + hh * (TILE_BYTES / 2); };
    // Half-tile h: phase 1 reads K(h + 1) and V(h).
    auto half_step = [&](int h, auto last_tag, int k_slot, int k_half, int v_slot, int v_half) INLINE {
        constexpr bool LAST = decltype(last_tag)::value;
        phase(kB, yes, yes, k_at(k_slot, k_half), k_at(v_slot, v_half));
        mask_half(h, s[1]);
        if constexpr (LAST) {
            phase(kA, no, no, nullptr, nullptr);
        } else {
            phase(kA, no, yes, nullptr, nullptr);
            mask_half(h + 1, s[0]);
        }
    };
    // Tile t has landed when at most the loads of the tiles issued after it
    // (`later` of them) are in flight.
    auto wait_tile = [&](int later) INLINE {
        if (later >= 1)
            __builtin_amdgcn_s_waitcnt(vm_imm(TILE_LOADS));
        else
            __builtin_amdgcn_s_waitcnt(vm_imm(0));
    };
    static_assert(AHEAD == 2, "wait_tile");

    __builtin_amdgcn_s_waitcnt(vm_imm(0));  // the first tiles and Q
    __builtin_amdgcn_s_barrier();
    if (t0 + AHEAD < t1) issue(t0 + AHEAD, AHEAD);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kop[kk] = *(const bf16x8*)(k_at(0, 0) + k_rel[kk]);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) s[0] = mfma32x32x16(kop[kk], qop[0][kk], kk == 0 ? f32x16{} : s[0]);
    mask_half(2 * t0, s[0]);
    half_step(2 * t0, no, 0, 1, 0, 0);
    int slot = 0;  // of tile t - 1
    for (int t = t0 + 1; t < t1; ++t) {
        const int nslot = slot == SLOTS - 1 ? 0 : slot + 1;
        // K and V of tile t (its loads, issued AHEAD tiles ago, and all before them).
        wait_tile(min(t1 - 1 - t, AHEAD - 1));
        // Everyone's loads have landed, and nobody reads V of tile t - 2 any more.
        __builtin_amdgcn_s_barrier();
        if (t + AHEAD < t1) issue(t + AHEAD, nslot + AHEAD >= SLOTS ? nslot + AHEAD - SLOTS : nslot + AHEAD);
        half_step(2 * t - 1, no, nslot, 0, slot, 1);
        half_step(2 * t, no, nslot, 1, nslot, 0);
        slot = nslot;
    }
    half_step(2 * t1 - 1, yes, slot, 1, slot, 1);
    // Drain: O_B += V^T P_B of the last half.
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) o[1][mb] = mfma32x32x16(vop[mb][st], pr[1][st], o[1][mb]);

    // ---- block epilogue: as in the 128-query form, for each of the two blocks ----
    float l_tot[2] = {sum_xor32(l_run[0]), sum_xor32(l_run[1])};
    auto store_out = [&](int u, const f32x16 (&a)[2], float scale) {
        const int q_out = q_base + 32 * u + col;
        if (q_out >= p.nq) return;
        bf16* out_row = (bf16*)p.out + (int64_t)b * p.q_bstride + (int64_t)q_out * C + head_off + 4 * half;
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = f32_to_bf16(a[mb][4 * g + e] * scale);
                *(bf16x4*)(out_row + 32 * mb + 8 * g) = v;
            }
    };
    if (sc.k == 1) {
#pragma unroll
        for (int u = 0; u < 2; ++u) store_out(u, o[u], 1.0f / l_tot[u]);
        return;
    }
    auto part_of = [&](int w, int u) INLINE {
        return sc.part_o + (int64_t)w * (QB * D) + (2 * wave + u) * (32 * D) + lane * 4;
    };
    auto ml_of = [&](int w, int u) INLINE { return sc.part_ml + ((int64_t)w * QB + QW * wave + 32 * u + col) * 2; };
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float* po = part_of(blockIdx.x, u);
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const f32x16& a = o[u][c >> 2];
            const int g = c & 3;
            *(f32x4*)(po + c * 256) = f32x4{a[4 * g], a[4 * g + 1], a[4 * g + 2], a[4 * g + 3]};
        }
        if (half == 0) {
            float* pml = ml_of(blockIdx.x, u);
            pml[0] = m_run[u];
            pml[1] = l_tot[u];
        }
    }
    __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0): this thread's stores reached the L2
    __syncthreads();
    if (tid == 0) {
        int* counter = sc.counters + blk;
        const int prev = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const int last = prev == sc.k - 1;
        if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        flag_lds = last;
    }
    __syncthreads();
    if (!flag_lds) return;
    // The last piece combines all of them in piece order, its own read back
    // like the others.
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float M = -INFINITY, L = 0.f;
        f32x16 res[2];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) res[mb][r] = 0.f;
        auto load_piece = [&](int pi, f32x4 (&pc)[8], float& mk, float& lk) {
            const int w = (bl * sc.k + pi) * sc.n_xcd + x;
            const float* pml = ml_of(w, u);
            mk = pml[0];
            lk = pml[1];
            const float* pk = part_of(w, u);
#pragma unroll
            for (int c = 0; c < 8; ++c) pc[c] = *(const f32x4*)(pk + c * 256);
        };
        auto combine = [&](const f32x4 (&pc)[8], float mk, float lk) {
            const float Mn = fmaxf(M, mk);
            const float a = M == Mn ? 1.f : fast_exp2(M - Mn);  // (both may be -inf)
            const float w = mk == Mn ? 1.f : fast_exp2(mk - Mn);
            L = __builtin_fmaf(lk, w, L * a);
#pragma unroll
            for (int c = 0; c < 8; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = 4 * (c & 3) + e;
                    res[c >> 2][r] = __builtin_fmaf(pc[c][e], w, res[c >> 2][r] * a);
                }
            M = Mn;
        };
        f32x4 pc_a[8], pc_b[8];
        float m_a, l_a, m_b, l_b;
        load_piece(0, pc_a, m_a, l_a);
        for (int pi = 0; pi < sc.k; pi += 2) {
            if (pi + 1 < sc.k) load_piece(pi + 1, pc_b, m_b, l_b);
            combine(pc_a, m_a, l_a);
            if (pi + 1 < sc.k) {
                if (pi + 2 < sc.k) load_piece(pi + 2, pc_a, m_a, l_a);
                combine(pc_b, m_b, l_b);
            }
        }
        store_out(u, res, 1.0f / L);
    }
}

}  // namespace

hipError_t launch_attention_wide(const AttnParams& p, const attn::Sched& sc, int grid, hipStream_t stream) {
    attn_wide_kernel<<<grid, NTHREADS, 0, stream>>>(p, sc);
    return hipGetLastError();
}

}  // namespace pcpp
