// bf16 GEMM on gfx950 MFMA for the transformer block's linear layers:
//   Y[m, n] = sum_k X[m, k] * W[n, k]  (+ bias[n]) (+ residual[m, n])
// with W in nn.Linear layout [out, in].  Optional GEGLU epilogue: the
// workgroup computes the value columns n and the gate columns F + n of the
// same outputs and writes value * GELU(gate) (exact erf GELU).
//
// The product is computed transposed, Y^T = W X^T, with 32x32x16 MFMAs so
// each lane ends up holding four consecutive output features of one token:
// stores are 8-byte (bf16) or 16-byte (fp32) vectors along the row.
// Tiles: BK = 32, LDS rows padded to 40 elements (conflict-free 16-byte
// operand reads), register-staged double buffering of the next K slice.
// X may be bf16 or fp32 (fp32 is rounded to bf16 while staging).

#include <math.h>

#include "common.h"
#include "gelu.h"
#include "gemm.h"
#include "kernels.h"

namespace pcpp {

namespace {

constexpr int BK = 32;
constexpr int LSTR = 40;  // LDS row stride in elements

typedef const __attribute__((address_space(1))) u32x4* gchunk;

template <int V>
struct IC {
    static constexpr int value = V;
};

// Output of column n (at most three segments) and its place in the segment.
// Compares and selects: an index computed per lane makes the compiler fetch
// p.out[.] from the kernel's arguments with a vector load before every store,
// and wait for it behind the store before.
__device__ __forceinline__ void* out_segment(const GemmParams& p, int n, int& ns) {
    void* const o0 = p.out[0];
    void* const o1 = p.out[1];
    void* const o2 = p.out[2];
    const bool in1 = n >= p.seg, in2 = n >= 2 * (int64_t)p.seg;
    ns = in2 ? n - 2 * p.seg : in1 ? n - p.seg : n;
    return in2 ? o2 : in1 ? o1 : o0;
}

// The same for segments seg_stride elements apart.
__device__ __forceinline__ void* strided_segment(const GemmParams& p, int n, int& ns) {
    const int seg = n / p.seg;
    ns = n - seg * p.seg;
    return (char*)p.out[0] + (int64_t)seg * p.seg_stride * (p.out_f32 ? 4 : 2);
}

template <int WMB, int WNB, bool AF32>
__global__ __launch_bounds__(256) void gemm_kernel(GemmParams p) {
    constexpr int BM = 2 * 32 * WMB;           // tokens per workgroup
    constexpr int BNW = 2 * 32 * WNB;          // W-tile rows per workgroup
    constexpr int A_CHUNKS = BM * BK / 8;      // 16-byte bf16 chunks of the X tile
    constexpr int W_CHUNKS = BNW * BK / 8;
    constexpr int A_PER = (A_CHUNKS + 255) / 256;
    constexpr int W_PER = (W_CHUNKS + 255) / 256;

    __shared__ __attribute__((aligned(16))) bf16 a_lds[2][BM * LSTR];
    __shared__ __attribute__((aligned(16))) bf16 w_lds[2][BNW * LSTR];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave & 1;
    const int wn = wave >> 1;
    const int col = lane & 31;
    const int half = lane >> 5;
    const int m0 = blockIdx.x * BM;
    // output columns per workgroup: BNW, or BNW/2 with the GEGLU pairing
    const int bn_out = p.geglu ? BNW / 2 : BNW;
    const int n0 = blockIdx.y * bn_out;

    // global W row of W-tile row r
    auto w_row = [&](int r) -> int {
        if (!p.geglu) return n0 + r;
        return r < BNW / 2 ? n0 + r : p.F + n0 + (r - BNW / 2);
    };

    u32x4 a_reg[A_PER * (AF32 ? 2 : 1)];
    u32x4 w_reg[W_PER];

    auto load = [&](int k0) {
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int c = tid + 256 * i;
            const int r = c >> 2, kc = (c & 3) * 8;
            const int m = m0 + r;
            const u32x4 z = {0u, 0u, 0u, 0u};
            if (c < A_CHUNKS && m < p.M) {
                if (AF32) {
                    gchunk src = (gchunk)((const float*)p.a + (int64_t)m * p.lda + k0 + kc);
                    a_reg[2 * i] = src[0];
                    a_reg[2 * i + 1] = src[1];
                } else {
                    a_reg[i] = *(gchunk)((const bf16*)p.a + (int64_t)m * p.lda + k0 + kc);
                }
            } else {
                if (AF32) {
                    a_reg[2 * i] = z;
                    a_reg[2 * i + 1] = z;
                } else {
                    a_reg[i] = z;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < W_PER; ++i) {
            const int c = tid + 256 * i;
            const int r = c >> 2, kc = (c & 3) * 8;
            if (c < W_CHUNKS) w_reg[i] = *(gchunk)(p.w + (int64_t)w_row(r) * p.K + k0 + kc);
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < A_PER; ++i) {
            const int c = tid + 256 * i;
            if (c >= A_CHUNKS) continue;
            const int r = c >> 2, kc = (c & 3) * 8;
            u32x4 v;
            if (AF32) {
                f32x4 lo = __builtin_bit_cast(f32x4, a_reg[2 * i]);
                f32x4 hi = __builtin_bit_cast(f32x4, a_reg[2 * i + 1]);
                bf16x8 b = {f32_to_bf16(lo[0]), f32_to_bf16(lo[1]), f32_to_bf16(lo[2]), f32_to_bf16(lo[3]),
                            f32_to_bf16(hi[0]), f32_to_bf16(hi[1]), f32_to_bf16(hi[2]), f32_to_bf16(hi[3])};
                v = __builtin_bit_cast(u32x4, b);
            } else {
                v = a_reg[i];
            }
            *(u32x4*)(a_lds[buf] + r * LSTR + kc) = v;
        }
#pragma unroll
        for (int i = 0; i < W_PER; ++i) {
            const int c = tid + 256 * i;
            if (c >= W_CHUNKS) continue;
            const int r = c >> 2, kc = (c & 3) * 8;
            *(u32x4*)(w_lds[buf] + r * LSTR + kc) = w_reg[i];
        }
    };

    f32x16 acc[WNB][WMB];
#pragma unroll
    for (int i = 0; i < WNB; ++i)
#pragma unroll
        for (int j = 0; j < WMB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    // W-tile row offset of this wave's n-block i
    auto wrow_off = [&](int i) -> int { return p.geglu ? 32 * wn + (BNW / 2) * i : (BNW / 2) * wn + 32 * i; };

    const int nk = p.K / BK;
    load(0);
    store(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load((kt + 1) * BK);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8 wop[WNB], aop[WMB];
#pragma unroll
            for (int i = 0; i < WNB; ++i)
                wop[i] = *(const bf16x8*)(w_lds[buf] + (wrow_off(i) + col) * LSTR + 16 * kk + 8 * half);
#pragma unroll
            for (int j = 0; j < WMB; ++j)
                aop[j] = *(const bf16x8*)(a_lds[buf] + (32 * WMB * wm + 32 * j + col) * LSTR + 16 * kk + 8 * half);
#pragma unroll
            for (int i = 0; i < WNB; ++i)
#pragma unroll
                for (int j = 0; j < WMB; ++j) acc[i][j] = mfma32x32x16(wop[i], aop[j], acc[i][j]);
        }
        if (kt + 1 < nk) store(buf ^ 1);
        __syncthreads();
    }

    // Epilogue: lane holds token m = m-block base + col and features
    // n-block base + 8*c + 4*half + (0..3) in registers 4c..4c+3.
    const int n_blocks_out = p.geglu ? 1 : WNB;
#pragma unroll
    for (int i = 0; i < n_blocks_out; ++i) {
#pragma unroll
        for (int j = 0; j < WMB; ++j) {
            const int m = m0 + 32 * WMB * wm + 32 * j + col;
            if (m >= p.M) continue;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int nloc = p.geglu ? 32 * wn + 8 * c + 4 * half : (BNW / 2) * wn + 32 * i + 8 * c + 4 * half;
                const int n = n0 + nloc;
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[i][j][4 * c + e];
                if (p.bias != nullptr) {
                    bf16x4 bv = *(const bf16x4*)(p.bias + n);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += bf16_to_f32(bv[e]);
                }
                if (WNB == 2 && p.geglu) {
                    float g[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) g[e] = acc[WNB - 1][j][4 * c + e];
                    if (p.bias != nullptr) {
                        bf16x4 bg = *(const bf16x4*)(p.bias + p.F + n);
#pragma unroll
                        for (int e = 0; e < 4; ++e) g[e] += bf16_to_f32(bg[e]);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] *= gelu_erf(g[e]);
                }
                if (p.resid != nullptr) {
                    if (p.resid_f32) {
                        f32x4 rv = *(const f32x4*)((const float*)p.resid + (int64_t)m * p.ldr + n);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += rv[e];
                    } else {
                        bf16x4 rv = *(const bf16x4*)((const bf16*)p.resid + (int64_t)m * p.ldr + n);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += bf16_to_f32(rv[e]);
                    }
                }
                int ns;
                void* dst = out_segment(p, n, ns);
                if (p.out_f32) {
                    f32x4 o = {v[0], v[1], v[2], v[3]};
                    *(f32x4*)((float*)dst + (int64_t)m * p.ldo + ns) = o;
                } else {
                    bf16x4 o = {f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
                    *(bf16x4*)((bf16*)dst + (int64_t)m * p.ldo + ns) = o;
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Pipelined variant for bf16 X and K % 64 == 0: X and W tiles (BK = 64) go
// straight from global memory into LDS (direct global->LDS loads, NS stages
// in flight), MFMA operands are read with explicit LDS waits one k-step
// ahead.  LDS rows are 128 bytes with the 16-byte chunk c of row r stored at
// slot c ^ ((r >> 1) & 7), so 32 consecutive rows read at one chunk are
// conflict-free.  64 x 64 tiles, 4 wavefronts in a 2 x 2 layout, each
// computing 32 tokens x 32 W rows.
// ---------------------------------------------------------------------------

constexpr int DBK = 64;
constexpr int DT = 64;                     // tokens and W rows of a tile
constexpr int DNS = 3;                     // stages
constexpr int DSTAGE = 2 * DT * DBK * 2;  // bytes per stage

typedef const __attribute__((address_space(1))) void* gvoid;
typedef __attribute__((address_space(3))) void* lvoid;

template <int OFF>
__device__ __forceinline__ u32x4 lds_b128(uint32_t a) {
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(a), "n"(OFF));
    return r;
}

// s_waitcnt immediate for vmcnt(v) alone (gfx9 layout: low four bits at
// [3:0], high two at [15:14]; expcnt and lgkmcnt left at their maxima).
constexpr int vmcnt_imm(int v) { return 0xF70 | (v & 15) | ((v >> 4) << 14); }

// Waits until at most later * PT vector loads of this thread are in flight:
// the k-tile `later` tiles before the newest issued one has landed.
template <int PT, int L>
__device__ __forceinline__ void wait_tiles_after(int later) {
    if constexpr (L == 0) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    } else {
        if (later >= L)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(L * PT));
        else
            wait_tiles_after<PT, L - 1>(later);
    }
}

// LDS floats of the cross-attention epilogue's K rows and transposed V, and
// of GroupNorm staging's scale and shift per channel and statistics per group.
constexpr int XA_TAB_FLOATS = (GEMM_XA_MAXT * 128 + 64 * 200) / 4;
constexpr int GN_TAB_FLOATS = 2 * GEMM_GN_MAXC + 2 * 256;

// What a pipelined launch does besides the product: nothing, an implicit
// convolution, the cross-attention epilogue, GroupNorm staging.
enum DmaForm { DMA_PLAIN, DMA_CONV, DMA_XATT, DMA_GN };
constexpr int tab_floats(int form) { return form == DMA_XATT ? XA_TAB_FLOATS : form == DMA_GN ? GN_TAB_FLOATS : 4; }

// One workgroup's tile of the product; (bx, by) is its place in the
// product's own grid (blockIdx of a single launch); lds holds DNS stages,
// tab tab_floats(FORM) floats.
template <int FORM>
__device__ __forceinline__ void gemm_dma_body(const GemmParams& p, const int bx, const int by, char* lds,
                                              float* tab) {
    constexpr bool CONV = FORM == DMA_CONV, XATT = FORM == DMA_XATT, AGN = FORM == DMA_GN;
    constexpr int XP = DT / 32;   // 1 KB pieces of X per wavefront per k-tile, and of W
    constexpr int PT = 2 * XP;    // loads per thread per k-tile
    static_assert(DNS == 3 && (DNS - 2) * PT <= 63, "wait_x; vmcnt holds at most 63 loads");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1;
    const int wn = wave >> 1;
    const int col = lane & 31;
    const int half = lane >> 5;
    // XCD-contiguous tiles (tpx > 0; always with split K): workgroup w runs
    // on XCD w % n_xcd; the tiles of an XCD are a contiguous range of tpx
    // tiles in n-major order (all token tiles of one W tile together), and
    // the splitk pieces of a tile follow each other within it, so all pieces
    // of a tile share one L2.
    int m_tile = bx, n_tile = by, piece = 0, tile = 0, xcd = 0, tl = 0;
    if (p.tpx > 0) {
        xcd = bx % p.n_xcd;
        const int j = bx / p.n_xcd;
        tl = j / p.splitk;
        piece = j - tl * p.splitk;
        tile = xcd * p.tpx + tl;
        if (tl >= p.tpx || tile >= p.n_tiles) return;  // idle slot of the last XCD (uniform)
        const int mt = (p.M + DT - 1) / DT;
        n_tile = tile / mt;
        m_tile = tile - n_tile * mt;
    }
    const int m0 = m_tile * DT;
    const int n0 = n_tile * DT;
    const int nk_all = p.K / DBK;
    const int kt0 = (int)((int64_t)nk_all * piece / p.splitk);
    const int kt1 = (int)((int64_t)nk_all * (piece + 1) / p.splitk);

    // Per-lane global source of each staged piece (row 8q + (lane >> 3),
    // chunk (lane & 7) ^ swizzle), k offset added per k-tile.
    const char* xsrc[XP];
    const char* wsrc[XP];
    const int cin = CONV ? p.K / 9 : 0;
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int r = 8 * (wave + 4 * i) + (lane >> 3);
        const int m = min(m0 + r, p.M - 1);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        int64_t row = (int64_t)m * p.lda;
        if constexpr (CONV) {  // the tap (0, 0) of output token (b, y, x) sits at framed (s y, s x)
            const int st = p.conv_stride;
            const int wo = p.conv_W / st;
            const int per = (p.conv_rows / st) * wo;
            const int b = m / per, rem = m - b * per;
            const int y = rem / wo, x = rem - y * wo;
            row = ((int64_t)(b * (p.conv_rows + 2) + st * y) * (p.conv_W + 2) + st * x) * cin;
        }
        xsrc[i] = (const char*)p.a + (row + 8 * c) * 2;
    }
    // Convolution: the k-tiles are issued in order, so the X offset of the
    // next one advances by 64 channels, then to the next tap (one token
    // right, or to the next framed row's first tap column).
    int iss_cb = 0, iss_kx = 0;
    int64_t iss_xoff = 0;
    if (CONV && kt0 > 0) {
        const int cbn = cin / DBK;
        const int t = kt0 / cbn, ky = t / 3;
        iss_cb = kt0 - t * cbn;
        iss_kx = t - 3 * ky;
        iss_xoff = ((int64_t)(ky * (p.conv_W + 2) + iss_kx) * cin + iss_cb * DBK) * 2;
    }
    // W of this tile: one of several matrices when w_seg_rows > 0 (a tile's
    // rows never straddle two of them).
    const __bf16* wmat = p.w;
    int wrow0 = n0;
    if (p.w_seg_rows > 0) {
        const int j = n0 / p.w_seg_rows;
        wmat = p.w_seg[j];
        wrow0 = n0 - j * p.w_seg_rows;
    }
#pragma unroll
    for (int i = 0; i < XP; ++i) {
        const int r = 8 * (wave + 4 * i) + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        wsrc[i] = (const char*)wmat + ((int64_t)(wrow0 + r) * p.K + 8 * c) * 2;
    }
    auto issue = [&](int kt, int stage) {
        char* st = lds + stage * DSTAGE;
        const int koff = kt * DBK * 2;
        const int64_t xoff = CONV ? iss_xoff : koff;
        if constexpr (CONV) {
            if (++iss_cb * DBK == cin) {
                iss_cb = 0;
                if (++iss_kx == 3) {
                    iss_kx = 0;
                    iss_xoff += ((int64_t)(p.conv_W + 2) * cin - 2 * cin - (cin - DBK)) * 2;
                } else {
                    iss_xoff += DBK * 2;
                }
            } else {
                iss_xoff += DBK * 2;
            }
        }
#pragma unroll
        for (int i = 0; i < XP; ++i)
            __builtin_amdgcn_global_load_lds((gvoid)(xsrc[i] + xoff), (lvoid)(st + (wave + 4 * i) * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < XP; ++i)
            __builtin_amdgcn_global_load_lds((gvoid)(wsrc[i] + koff), (lvoid)(st + DT * 128 + (wave + 4 * i) * 1024),
                                             16, 0, 0);
    };

    // Operand read addresses: row col of each 32-row block, chunk 2kk + half.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const int cmask = (col >> 1) & 7;
    uint32_t chunk_off[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) chunk_off[kk] = ((2 * kk + half) ^ cmask) << 4;
    const uint32_t w_row0 = DT * 128 + 32 * wn * 128 + col * 128;
    const uint32_t x_row0 = (32 * wm + col) * 128;

    struct Ops {
        u32x4 w, x;
    };
    // Both addresses before the first read: with the second between the reads
    // the compiler puts the third product behind the last operands' wait
    // (512 x 64 x 17280 as a convolution 74.6 -> 78 us).
    auto read_ops = [&](uint32_t sbase, int kk, Ops& o) {
        const uint32_t wa = sbase + w_row0 + chunk_off[kk];
        const uint32_t xa = sbase + x_row0 + chunk_off[kk];
        o.w = lds_b128<0>(wa);
        o.x = lds_b128<0>(xa);
    };
    auto wait_ops = [&](Ops& o, auto n_tag) {
        constexpr int N = decltype(n_tag)::value;
        asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(o.w), "+v"(o.x) : "n"(N));
    };

    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    // The MFMAs of the k-tile in the stage at LDS address sbase.
    auto mfma_tile = [&](uint32_t sbase) {
        Ops o[2];
        read_ops(sbase, 0, o[0]);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            Ops& cur = o[kk & 1];
            if (kk < 3) {
                read_ops(sbase, kk + 1, o[(kk + 1) & 1]);
                wait_ops(cur, IC<2>{});
            } else {
                wait_ops(cur, IC<0>{});
            }
            acc = mfma32x32x16(__builtin_bit_cast(bf16x8, cur.w), __builtin_bit_cast(bf16x8, cur.x), acc);
        }
    };

    // Cross-attention.  tab holds K_h as rows of 128 bytes (the
    // operand swizzle; keys past xa_T zero) and V_h transposed, a row of
    // 200 bytes per head dimension (keys along the row; 200 keeps the eight-
    // byte reads of 32 dimensions on distinct banks).
    constexpr int XA_VT_STRIDE = 200;
    char* xa = (char*)tab;
    char* xa_vt = xa + GEMM_XA_MAXT * 128;
    auto xatt_stage = [&]() {
        const int img = m0 / p.xa_N;
        const int64_t kvo = (int64_t)img * p.xa_T * p.xa_ldkv + n0;
#pragma unroll
        for (int it = 0; it < GEMM_XA_MAXT * 8 / 256; ++it) {
            const int i = tid + 256 * it;
            const int key = i >> 3, c = i & 7;
            u32x4 kv = {0u, 0u, 0u, 0u}, vv = {0u, 0u, 0u, 0u};
            if (key < p.xa_T) {
                kv = *(const u32x4*)(p.xa_k + kvo + (int64_t)key * p.xa_ldkv + 8 * c);
                vv = *(const u32x4*)(p.xa_v + kvo + (int64_t)key * p.xa_ldkv + 8 * c);
            }
            *(u32x4*)(xa + key * 128 + ((c ^ ((key >> 1) & 7)) << 4)) = kv;
            const bf16x8 v8 = __builtin_bit_cast(bf16x8, vv);
#pragma unroll
            for (int e = 0; e < 8; ++e) *(bf16*)(xa_vt + (8 * c + e) * XA_VT_STRIDE + key * 2) = v8[e];
        }
    };
    // After the product: Q (bf16, rows of 128 bytes) into the first stage,
    // then wavefront (qb, dh) = (w % 2, w / 2) computes S^T = K Q^T for
    // queries 32 qb .. + 31 over all keys (a lane holds one query), the
    // softmax in registers (the key halves meet across lanes l and l ^ 32),
    // and O^T = V^T P^T for head dimensions 32 dh .. + 31.  P^T feeds the
    // matrix product straight from the S^T registers: its k-slot e of lane
    // half h is key 16 u + 8 (e / 4) + 4 h + e % 4 of the step, and V^T is
    // read with the same key order.
    auto xatt_epilogue = [&]() {
        __syncthreads();  // every operand read of the last stage is done
        {
            const int t = 32 * wm + col;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int chunk = 4 * wn + c;  // head dimensions 32 wn + 8 c + 4 half + 0..3
                const bf16x4 q4 = {f32_to_bf16(acc[4 * c]), f32_to_bf16(acc[4 * c + 1]),
                                   f32_to_bf16(acc[4 * c + 2]), f32_to_bf16(acc[4 * c + 3])};
                *(bf16x4*)(lds + t * 128 + ((chunk ^ ((t >> 1) & 7)) << 4) + 8 * half) = q4;
            }
        }
        __syncthreads();
        const int qb = wave & 1, dh = wave >> 1;
        f32x16 sc[3];
#pragma unroll
        for (int kb = 0; kb < 3; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) sc[kb][r] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            const int ch = 2 * ks + half;
            const int qr = 32 * qb + col;
            const u32x4 qv = *(const u32x4*)(lds + qr * 128 + ((ch ^ ((qr >> 1) & 7)) << 4));
#pragma unroll
            for (int kb = 0; kb < 3; ++kb) {
                const int kr = 32 * kb + col;
                const u32x4 kv = *(const u32x4*)(xa + kr * 128 + ((ch ^ ((kr >> 1) & 7)) << 4));
                sc[kb] = mfma32x32x16(__builtin_bit_cast(bf16x8, kv), __builtin_bit_cast(bf16x8, qv), sc[kb]);
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 3; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = 32 * kb + 8 * (r >> 2) + 4 * half + (r & 3);
                if (key >= p.xa_T) sc[kb][r] = -INFINITY;
                mx = fmaxf(mx, sc[kb][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float cl = 1.4426950408889634f * 0.125f;  // log2(e) / sqrt(64)
        const float mcl = mx * cl;
        float l = 0.f;
        bf16x8 pb[3][2];
#pragma unroll
        for (int kb = 0; kb < 3; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bf16 pr = f32_to_bf16(fast_exp2(__builtin_fmaf(sc[kb][r], cl, -mcl)));
                pb[kb][r >> 3][r & 7] = pr;
                l += bf16_to_f32(pr);  // the weights the products use
            }
        l += __shfl_xor(l, 32);
        f32x16 o;
#pragma unroll
        for (int r = 0; r < 16; ++r) o[r] = 0.f;
        const int d = 32 * dh + col;
#pragma unroll
        for (int kb = 0; kb < 3; ++kb)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int k0 = 32 * kb + 16 * u + 4 * half;
                const u32x2 a0 = *(const u32x2*)(xa_vt + d * XA_VT_STRIDE + k0 * 2);
                const u32x2 a1 = *(const u32x2*)(xa_vt + d * XA_VT_STRIDE + (k0 + 8) * 2);
                const u32x4 av = {a0[0], a0[1], a1[0], a1[1]};
                o = mfma32x32x16(__builtin_bit_cast(bf16x8, av), pb[kb][u], o);
            }
        const int m = m0 + 32 * qb + col;
        if (m >= p.M) return;
        const float inv = 1.f / l;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bf16x4 ov = {f32_to_bf16(o[4 * q] * inv), f32_to_bf16(o[4 * q + 1] * inv),
                               f32_to_bf16(o[4 * q + 2] * inv), f32_to_bf16(o[4 * q + 3] * inv)};
            *(bf16x4*)((bf16*)p.out[0] + (int64_t)m * p.ldo + n0 + 32 * dh + 8 * q + 4 * half) = ov;
        }
    };

    // Epilogue: lane holds token m and W rows n_of(c) .. + 3 in registers 4c ..
    // 4c + 3.  Bias and residual are loaded after the products: in front of
    // them, in 42 more registers, they made the modules of 64 to 1024 x 1280 0.5
    // to 1 % slower.
    const int m = m0 + 32 * wm + col;
    auto n_of = [&](int c) { return n0 + 32 * wn + 8 * c + 4 * half; };
    bf16x4 bias_v[4] = {}, res_h[4] = {};
    f32x4 res_v[4] = {}, bias2_v[4] = {};
    auto load_addends = [&]() {
        const int64_t mc = min(m, p.M - 1);
        if (p.bias != nullptr) {
#pragma unroll
            for (int c = 0; c < 4; ++c) bias_v[c] = *(const bf16x4*)(p.bias + n_of(c));
        }
        if (p.resid != nullptr && p.resid_f32) {
#pragma unroll
            for (int c = 0; c < 4; ++c) res_v[c] = *(const f32x4*)((const float*)p.resid + mc * p.ldr + n_of(c));
        }
        if (p.resid != nullptr && !p.resid_f32) {
#pragma unroll
            for (int c = 0; c < 4; ++c) res_h[c] = *(const bf16x4*)((const bf16*)p.resid + mc * p.ldr + n_of(c));
        }
        if (p.bias2 != nullptr) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                bias2_v[c] = *(const f32x4*)(p.bias2 + (int64_t)((int)mc / p.bias2_rows) * p.N + n_of(c));
        }
    };

    // GroupNorm staging.  X arrives with the direct loads like W; after the
    // products of k-tile kt each lane rewrites in place the 16-byte pieces of
    // k-tile kt + 1 that its own loads brought (so that its own wait suffices),
    // published by the next barrier.  Piece i of the lane: row 8 (wave + 4 i)
    // + lane / 8, source chunk (lane % 8) ^ ((row / 2) % 8).
    float* const sc = tab;
    float* const sh = tab + GEMM_GN_MAXC;
    auto gn_rewrite = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            const int r = 8 * (wave + 4 * i) + (lane >> 3);
            const int c0 = kt * DBK + 8 * ((lane & 7) ^ ((r >> 1) & 7));
            bf16x8* at = (bf16x8*)(lds + stage * DSTAGE + (wave + 4 * i) * 1024 + lane * 16);
            const bf16x8 v = *at;
            bf16x8 y;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f32x4 a = *(const f32x4*)(sc + c0 + 4 * h), b = *(const f32x4*)(sh + c0 + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) y[4 * h + e] = f32_to_bf16(__builtin_fmaf((float)v[4 * h + e], a[e], b[e]));
            }
            *at = y;
        }
    };
    // X of the k-tile before the newest: behind it its own W and, if issued, a k-tile.
    auto wait_x = [&](bool one_more) {
        if (one_more)
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(XP + PT));
        else
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(XP));
    };

#pragma unroll
    for (int s = 0; s < DNS - 1; ++s)
        if (kt0 + s < kt1) issue(kt0 + s, s);
    if constexpr (XATT) xatt_stage();  // its loads wait behind the first k-tiles'
    if constexpr (AGN) {               // the statistics are merged while the first k-tiles are in flight
        const int img = m0 / p.gn_N;
        float* g_mean = tab + 2 * GEMM_GN_MAXC;
        float* g_rstd = g_mean + 256;
        gn_group_stats(p.gn, img, m0 == img * p.gn_N && n0 == 0, g_mean, g_rstd);
        const int cg = p.K / p.gn.G;
        for (int c = tid; c < p.K; c += 256) {
            const int g = c / cg;
            const float a = g_rstd[g] * bf16_to_f32(p.gn_gamma[c]);
            sc[c] = a;
            sh[c] = bf16_to_f32(p.gn_beta[c]) - g_mean[g] * a;
        }
        __syncthreads();
        wait_x(kt0 + 1 < kt1);
        gn_rewrite(kt0, 0);
    }
    // A convolution's loop at a fixed place within the 32 bytes that are fetched
    // at once (three instructions past a boundary): at that of the eight places
    // 512 x 64 x 17280 takes 74.6 us, at the others 77.1 to 78.3, and code elsewhere
    // in the kernel would decide which.  (The plain forms: no difference.)
    if constexpr (CONV) asm volatile(".p2align 5\n\ts_nop 0\n\ts_nop 0\n\ts_nop 0");
    for (int kt = kt0; kt < kt1; ++kt) {
        // k-tiles issued after kt so far: min(kt1 - 1 - kt, DNS - 2), PT loads each
        wait_tiles_after<PT, DNS - 2>(min(kt1 - 1 - kt, DNS - 2));
        if constexpr (AGN) __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this lane's rewrite of X(kt)
        __builtin_amdgcn_s_barrier();  // everyone's pieces of tile kt landed; the stage of tile kt-1 is free
        if (kt + DNS - 1 < kt1) issue(kt + DNS - 1, (kt - kt0 + DNS - 1) % DNS);
        mfma_tile(lds0 + ((kt - kt0) % DNS) * DSTAGE);
        if constexpr (AGN) {
            if (kt + 1 < kt1) {
                wait_x(kt + 2 < kt1);
                gn_rewrite(kt + 1, (kt - kt0 + 1) % DNS);
            }
        }
    }

    if constexpr (XATT) {
        xatt_epilogue();
        return;
    }

    // Split K: every piece stores its partial tile (fp32, 1 KB per wavefront
    // store); the last piece of a tile to arrive adds all of them in piece
    // order (its own from registers: the same values) and runs the epilogue.
    if (p.splitk > 1) {
        __shared__ int last_flag;
        auto part_of = [&](int wg) { return (float*)p.split_ws + GEMM_SPLIT_COUNTERS + (int64_t)wg * DT * DT; };
        {
            float* dst = part_of(bx) + (wave * 64 + lane) * 4;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(f32x4*)(dst + q * 1024) = f32x4{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        }
        __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0): this thread's stores reached the L2
        __syncthreads();
        if (tid == 0) {
            int* counter = (int*)p.split_ws + tile;
            const int prev = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const int last = prev == p.splitk - 1;
            if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            last_flag = last;
        }
        __syncthreads();
        if (!last_flag) return;
        const f32x16 own = acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (int pc = 0; pc < p.splitk; ++pc) {
            if (pc == piece) {
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] += own[r];
                continue;
            }
            const float* src = part_of((tl * p.splitk + pc) * p.n_xcd + xcd) + (wave * 64 + lane) * 4;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f32x4 v = *(const f32x4*)(src + q * 1024);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[4 * q + e] += v[e];
            }
        }
    }

    load_addends();
    if (m >= p.M) return;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int n = n_of(c);
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float rv = p.resid_f32 ? res_v[c][e] : bf16_to_f32(res_h[c][e]);
            if (p.bias2 != nullptr) rv += bias2_v[c][e];
            v[e] = (acc[4 * c + e] + bf16_to_f32(bias_v[c][e])) + rv;
        }
        const bf16x4 h = {f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
        int ns;
        void* dst = p.seg_stride > 0 ? strided_segment(p, n, ns) : out_segment(p, n, ns);
        if (p.out_f32)
            *(f32x4*)((float*)dst + (int64_t)m * p.ldo + ns) = v;
        else
            *(bf16x4*)((bf16*)dst + (int64_t)m * p.ldo + ns) = h;
        if (p.out_bf16 != nullptr) *(bf16x4*)((bf16*)p.out_bf16 + (int64_t)m * p.ldo + n) = h;
    }
}

template <int FORM>
__global__ __launch_bounds__(256) void gemm_dma_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(16))) char lds[DNS * DSTAGE];
    __shared__ __attribute__((aligned(16))) float tab[tab_floats(FORM)];
    gemm_dma_body<FORM>(p, blockIdx.x, blockIdx.y, lds, tab);
}

// Two independent products, the second plain, in one launch (so that neither
// pays a launch's fixed cost alone): workgroups [0, n_a) run `a`, [b0, b0 + n_b)
// run `b`, each product's grid linearised x-fastest; b0 is a multiple of the
// XCD count, so a product on XCD-ordered tiles keeps its workgroup-to-XCD
// map; the workgroups in between exit at once.
struct GemmPair {
    GemmParams a, b;
    int32_t gx_a, n_a, gx_b, b0;
};

template <int FORM_A>
__global__ __launch_bounds__(256) void gemm_dma_pair_kernel(GemmPair pp) {
    __shared__ __attribute__((aligned(16))) char lds[DNS * DSTAGE];
    __shared__ __attribute__((aligned(16))) float tab[tab_floats(FORM_A)];
    const int id = blockIdx.x;
    if (id < pp.n_a)
        gemm_dma_body<FORM_A>(pp.a, id % pp.gx_a, id / pp.gx_a, lds, tab);
    else if (id >= pp.b0)
        gemm_dma_body<DMA_PLAIN>(pp.b, (id - pp.b0) % pp.gx_b, (id - pp.b0) / pp.gx_b, lds, tab);
}

// ---------------------------------------------------------------------------
// Balanced tiles for products whose 64 x 64 tiles do not divide evenly over
// the compute units: 64 tokens x 80 W rows per workgroup, so that a
// 2048 x 640 product is 256 tiles, one per compute unit (64 x 64 tiles give
// 320: a quarter of the compute units would run two, and the launch lasts
// as long as they do).  Y^T = W X^T with 16x16x32 MFMAs (a lane ends up with
// four consecutive outputs of one token).  Eight wavefronts: wavefront w
// takes tokens 16 (w % 4) .. + 15 and k-step w / 4 of the two 32-long steps
// of every 64-long k-tile, for all 80 rows (five 16-row blocks); the two
// k-steps' sums meet through LDS at the end.  X and W go straight into LDS
// in the row layout and swizzle of the kernel above: 18 pieces of 1 KB per
// k-tile (8 of X, 10 of W), piece j loaded by wavefront j % 8; NS stages
// (4 with one tile per compute unit, 2 when several share one).
// ---------------------------------------------------------------------------
constexpr int G80_BM = 64, G80_BN = 80;
constexpr int G80_STAGE = (G80_BM + G80_BN) * DBK * 2;  // 18 KB

__device__ __forceinline__ f32x4 mfma16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

template <int NS>
__global__ __launch_bounds__(512, NS == 2 ? 6 : 2) void gemm80_kernel(GemmParams p) {
    __shared__ __attribute__((aligned(16))) char lds[NS * G80_STAGE];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tb = wave & 3, kg = wave >> 2;
    const int m0 = blockIdx.x * G80_BM, n0 = blockIdx.y * G80_BN;
    const int nk = p.K / DBK;

    // Pieces j = wave + 8 q of this wavefront: LDS rows 8 j .. 8 j + 7 of the
    // stage (X rows 0..63, then W rows 64..143); lane: row 8 j + lane / 8,
    // chunk (lane % 8) ^ ((row / 2) % 8).
    const char* src[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int j = wave + 8 * q;
        const int row = 8 * j + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        if (row < G80_BM) {
            const int m = min(m0 + row, p.M - 1);
            src[q] = (const char*)p.a + ((int64_t)m * p.lda + 8 * c) * 2;
        } else {
            src[q] = (const char*)p.w + ((int64_t)(n0 + min(row, G80_BM + G80_BN - 1) - G80_BM) * p.K + 8 * c) * 2;
        }
    }
    const bool three = wave < 2;  // 18 pieces: wavefronts 0 and 1 load a third
    auto issue = [&](int kt, int stage) {
        char* st = lds + stage * G80_STAGE;
        const int koff = kt * DBK * 2;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            __builtin_amdgcn_global_load_lds((gvoid)(src[q] + koff), (lvoid)(st + (wave + 8 * q) * 1024), 16, 0, 0);
        if (three)
            __builtin_amdgcn_global_load_lds((gvoid)(src[2] + koff), (lvoid)(st + (wave + 16) * 1024), 16, 0, 0);
    };

    // Operands of k-step kg: X rows 16 tb + lane % 16 (B, tokens), W rows
    // 64 + 16 fb + lane % 16 (A, W rows), k-octet lane / 16 of the step.
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    const int chunk = 4 * kg + (lane >> 4);
    const int xr = 16 * tb + (lane & 15);
    const uint32_t xoff = xr * 128 + ((chunk ^ ((xr >> 1) & 7)) << 4);
    uint32_t woff[5];
#pragma unroll
    for (int fb = 0; fb < 5; ++fb) {
        const int r = G80_BM + 16 * fb + (lane & 15);
        woff[fb] = r * 128 + ((chunk ^ ((r >> 1) & 7)) << 4);
    }
    f32x4 acc[5];
#pragma unroll
    for (int fb = 0; fb < 5; ++fb) acc[fb] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Wavefront (tb, 0) finishes blocks 0-2, (tb, 1) blocks 3-4: token
    // m0 + 16 tb + lane % 16, W rows n0 + 16 fb + 4 (lane / 16) + 0..3.  With one
    // tile per compute unit their bias and residual are loaded here, behind the
    // products: after them the loads' trip to memory adds to every launch
    // (1024 x 1280 x 1280 with a float32 residual 11.96 -> 11.56 us, 4096 x 640 x
    // 640 13.8 -> 13.1).  Held through the loop they take 17 registers, and with
    // two stages a third workgroup would no longer fit its compute unit (80
    // registers): 4096 x 960 x 320 8.9 -> 11.6 us; there they are loaded after it.
    auto owned = [&](int fb) { return kg == 0 ? fb < 3 : fb >= 3; };
    const int m = m0 + 16 * tb + (lane & 15);
    const int mc = min(m, p.M - 1);
    bf16x4 bias_v[3] = {}, res_h[3] = {};
    f32x4 res_v[3] = {};
    const int nl = n0 + 4 * (lane >> 4);
    auto row_of = [&](int i) { return nl + 16 * min(3 * kg + i, 4); };  // (tb, 1): its second block twice
    auto load_addends = [&]() {
        if (p.bias != nullptr) {
#pragma unroll
            for (int i = 0; i < 3; ++i) bias_v[i] = *(const bf16x4*)(p.bias + row_of(i));
        }
        if (p.resid != nullptr && p.resid_f32) {
            const float* r = (const float*)p.resid + (int64_t)mc * p.ldr;
#pragma unroll
            for (int i = 0; i < 3; ++i) res_v[i] = *(const f32x4*)(r + row_of(i));
        }
        if (p.resid != nullptr && !p.resid_f32) {
            const bf16* r = (const bf16*)p.resid + (int64_t)mc * p.ldr;
#pragma unroll
            for (int i = 0; i < 3; ++i) res_h[i] = *(const bf16x4*)(r + row_of(i));
        }
    };
    constexpr bool EARLY = NS > 2;
    if constexpr (EARLY) load_addends();

#pragma unroll
    for (int st = 0; st < NS - 1; ++st)
        if (st < nk) issue(st, st);
    for (int kt = 0; kt < nk; ++kt) {
        const int later = min(nk - 1 - kt, NS - 2);
        if (three)
            wait_tiles_after<3, NS - 2>(later);
        else
            wait_tiles_after<2, NS - 2>(later);
        __builtin_amdgcn_s_barrier();  // everyone's pieces of tile kt landed; the stage of tile kt-1 is free
        if (kt + NS - 1 < nk) issue(kt + NS - 1, (kt + NS - 1) % NS);
        const uint32_t sb = lds0 + (kt % NS) * G80_STAGE;
        u32x4 x = lds_b128<0>(sb + xoff);
        u32x4 w0 = lds_b128<0>(sb + woff[0]);
        u32x4 w1 = lds_b128<0>(sb + woff[1]);
        u32x4 w2 = lds_b128<0>(sb + woff[2]);
        u32x4 w3 = lds_b128<0>(sb + woff[3]);
        u32x4 w4 = lds_b128<0>(sb + woff[4]);
        asm volatile("s_waitcnt lgkmcnt(4)" : "+v"(x), "+v"(w0));
        acc[0] = mfma16x16x32(__builtin_bit_cast(bf16x8, w0), __builtin_bit_cast(bf16x8, x), acc[0]);
        asm volatile("s_waitcnt lgkmcnt(3)" : "+v"(w1));
        acc[1] = mfma16x16x32(__builtin_bit_cast(bf16x8, w1), __builtin_bit_cast(bf16x8, x), acc[1]);
        asm volatile("s_waitcnt lgkmcnt(2)" : "+v"(w2));
        acc[2] = mfma16x16x32(__builtin_bit_cast(bf16x8, w2), __builtin_bit_cast(bf16x8, x), acc[2]);
        asm volatile("s_waitcnt lgkmcnt(1)" : "+v"(w3));
        acc[3] = mfma16x16x32(__builtin_bit_cast(bf16x8, w3), __builtin_bit_cast(bf16x8, x), acc[3]);
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(w4));
        acc[4] = mfma16x16x32(__builtin_bit_cast(bf16x8, w4), __builtin_bit_cast(bf16x8, x), acc[4]);
    }

    if constexpr (!EARLY) load_addends();

    // The two k-steps' sums: each wavefront hands its partner the sums of the
    // partner's blocks.
    __syncthreads();  // every wavefront is past its last LDS operand read
    float* red = (float*)lds;  // [tb][block][lane] x 4 floats (20 KB)
#pragma unroll
    for (int fb = 0; fb < 5; ++fb)
        if (!owned(fb)) *(f32x4*)(red + ((tb * 5 + fb) * 64 + lane) * 4) = acc[fb];
    __syncthreads();
#pragma unroll
    for (int fb = 0; fb < 5; ++fb)
        if (owned(fb)) acc[fb] += *(const f32x4*)(red + ((tb * 5 + fb) * 64 + lane) * 4);

    if (m >= p.M) return;
    int ns0;
    void* const dst = out_segment(p, n0, ns0);  // of the whole tile (80 divides the segment width)
#pragma unroll
    for (int fb = 0; fb < 5; ++fb) {
        if (!owned(fb)) continue;
        const int n = nl + 16 * fb;
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {  // the 64 x 64 kernel's order; one of the two residuals is zero
            const int i = fb % 3;
            const float res = p.resid_f32 ? res_v[i][e] : bf16_to_f32(res_h[i][e]);
            v[e] = (acc[fb][e] + bf16_to_f32(bias_v[i][e])) + res;
        }
        const int ns = ns0 + (n - n0);
        if (p.out_f32) {
            *(f32x4*)((float*)dst + (int64_t)m * p.ldo + ns) = f32x4{v[0], v[1], v[2], v[3]};
        } else {
            const bf16x4 o = {f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
            *(bf16x4*)((bf16*)dst + (int64_t)m * p.ldo + ns) = o;
        }
        if (p.out_bf16 != nullptr) {
            const bf16x4 o = {f32_to_bf16(v[0]), f32_to_bf16(v[1]), f32_to_bf16(v[2]), f32_to_bf16(v[3])};
            *(bf16x4*)((bf16*)p.out_bf16 + (int64_t)m * p.ldo + n) = o;
        }
    }
}

// The 64 x 64 kernel at three stages.
hipError_t launch_dma64(const GemmParams& p, hipStream_t s) {
    dim3 grid((p.M + 63) / 64, p.N / 64);
    if (p.tpx > 0) grid = dim3((unsigned)(p.n_xcd * p.tpx * p.splitk), 1);
    if (p.xa_T > 0)
        gemm_dma_kernel<DMA_XATT><<<grid, 256, 0, s>>>(p);
    else if (p.gn_N > 0)
        gemm_dma_kernel<DMA_GN><<<grid, 256, 0, s>>>(p);
    else if (p.conv_W > 0)
        gemm_dma_kernel<DMA_CONV><<<grid, 256, 0, s>>>(p);
    else
        gemm_dma_kernel<DMA_PLAIN><<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

template <int WMB, int WNB>
hipError_t launch_shape(const GemmParams& p, hipStream_t s) {
    constexpr int BM = 64 * WMB;
    const int bn_out = p.geglu ? 32 * WNB : 64 * WNB;
    dim3 grid((p.M + BM - 1) / BM, p.N / bn_out);
    if (p.a_f32)
        gemm_kernel<WMB, WNB, true><<<grid, 256, 0, s>>>(p);
    else
        gemm_kernel<WMB, WNB, false><<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace

bool gemm_shape_ok(const GemmParams& p) {
    if (p.K % BK != 0 || p.M < 1 || p.N < 1) return false;
    if (p.bias2 != nullptr && (p.bias2_rows < 1 || p.N % 4 != 0)) return false;
    if (p.conv_W > 0) {
        const int st = p.conv_stride;
        if ((st != 1 && st != 2) || (st == 2 && (p.conv_rows % 2 != 0 || p.conv_W % 2 != 0))) return false;
        return !p.a_f32 && !p.geglu && p.conv_rows > 0 && p.K % (9 * DBK) == 0 && p.N % 64 == 0 &&
               p.seg % 4 == 0 && p.M % ((p.conv_rows / st) * (p.conv_W / st)) == 0;
    }
    if (p.geglu) return p.N % 64 == 0;  // two n-blocks of 32 per workgroup pair
    return p.N % 64 == 0 && p.seg % 4 == 0;
}

namespace {

struct SplitPlan {
    int splitk, n_xcd, tpx, n_tiles;
    size_t bytes;
};

// Split of a plain GEMM over 64 x 64 tiles when they are fewer than the
// compute units (one workgroup per compute unit and the rest idle): about
// kSplitTarget workgroups per compute unit, each piece at least
// kSplitMinTiles k-tiles long.  Measured at 512 x 1280 (2048 px level 2):
// K = 5120 in 3 pieces 21.4 us against 25.8 unsplit (4 or 5 pieces, from a
// target of 3 or 4 workgroups per compute unit: the level-2 block 4-8 us
// slower); K = 1280 in 2 pieces of 10 k-tiles 10.6 against 9.4, hence the
// minimum length.  A deeper LDS
// ring (4, 6 or 8 stages) for the unsplit small launches gained nothing.
constexpr int kSplitTarget = 2;
constexpr int kSplitMinTiles = 16;

SplitPlan split_plan_plain(int M, int N, int K, const DeviceLayout& d) {
    SplitPlan sp{1, 1, 0, 0, 0};
    const int cus = d.cus;
    if (!d.xcd_merge || N % 64 != 0 || K % DBK != 0) return sp;
    const int64_t tiles = (int64_t)((M + 63) / 64) * (N / 64);
    if (tiles < 1 || tiles >= cus || tiles > GEMM_SPLIT_COUNTERS) return sp;
    const int n_xcd = d.n_xcd;
    const int64_t tpx = (tiles + n_xcd - 1) / n_xcd;
    int64_t k = (int64_t)kSplitTarget * cus / (n_xcd * tpx);
    const int64_t k_max = (K / DBK) / kSplitMinTiles;
    if (k > k_max) k = k_max;
    if (k > 8) k = 8;
    if (k < 2) return sp;
    sp.splitk = (int)k;
    sp.n_xcd = n_xcd;
    sp.tpx = (int)tpx;
    sp.n_tiles = (int)tiles;
    sp.bytes = (size_t)GEMM_SPLIT_COUNTERS * 4 + (size_t)n_xcd * tpx * k * 64 * 64 * 4;
    return sp;
}

}  // namespace

// Sized for a launch that may use every compute unit (a CU-masked stream
// only ever needs less).
size_t gemm_split_ws_bytes(int M, int N, int K, bool conv) {
    const DeviceLayout d = device_layout_unmasked();
    const size_t narrow = conv ? 0 : split_plan_plain(M, N, K, d).bytes;
    const size_t wide = wide_split_bytes(M, N, K, d);
    return wide > narrow ? wide : narrow;
}

namespace {

// The kernel a product runs on.
enum GemmKind { GK_DMA_64, GK_G80, GK_REG_22, GK_REG_12, GK_REG_11, GK_WIDE };

// Validates p, picks its kernel among those of this file, and sets the
// fields of a split or XCD-ordered launch.
hipError_t plan_narrow(GemmParams& p, const DeviceLayout& dl, GemmKind& kind) {
    if (p.conv_W > 0 && !gemm_shape_ok(p)) return hipErrorInvalidValue;
    if (p.xa_T != 0) {  // cross-attention epilogue: the 64 x 64 pipelined kernel, unsplit
        if (p.a_f32 || p.geglu || p.conv_W > 0 || p.K % DBK != 0 || p.N % 64 != 0 || p.seg < p.N || p.out_f32 ||
            p.resid != nullptr || p.out_bf16 != nullptr || p.bias != nullptr || p.bias2 != nullptr ||
            p.w_seg_rows != 0 || p.seg_stride != 0 || p.xa_k == nullptr || p.xa_v == nullptr || p.xa_T < 1 ||
            p.xa_T > GEMM_XA_MAXT || p.xa_N <= 0 || p.xa_N % 64 != 0 || p.M % p.xa_N != 0 || p.xa_ldkv < p.N ||
            p.xa_ldkv % 8 != 0)
            return hipErrorInvalidValue;
    }
    if (p.gn_N != 0) {  // GroupNorm staging: the 64 x 64 pipelined kernel, unsplit
        if (p.a_f32 || p.geglu || p.conv_W > 0 || p.xa_T != 0 || p.K % DBK != 0 || p.K > GEMM_GN_MAXC ||
            p.N % 64 != 0 || p.seg % 4 != 0 || p.gn_N <= 0 || p.gn_N % 64 != 0 || p.M % p.gn_N != 0 || p.gn.G < 1 ||
            p.gn.G > 256 || p.K % p.gn.G != 0 || p.gn.stats == nullptr || p.gn_gamma == nullptr ||
            p.gn_beta == nullptr)
            return hipErrorInvalidValue;
    }
    if (p.w_seg_rows != 0 || p.seg_stride != 0) {  // the pipelined kernel's plain form only
        if (p.a_f32 || p.geglu || p.conv_W > 0 || p.K % DBK != 0 || p.seg % 4 != 0 || p.N % 64 != 0 ||
            p.seg_stride < 0 || p.w_seg_rows < 0)
            return hipErrorInvalidValue;
        if (p.w_seg_rows > 0 &&
            (p.w_seg_rows % 128 != 0 || p.N % p.w_seg_rows != 0 || p.N / p.w_seg_rows > GEMM_MAX_WSEG))
            return hipErrorInvalidValue;
    }
    p.splitk = 1;
    p.tpx = 0;
    // Unsplit launches: when W (rows x K) is at least four times X (M x K),
    // each XCD takes a contiguous n-major range of tiles, so a W tile is
    // fetched into one XCD's L2 (the hardware deals workgroups round-robin
    // over the XCDs, which with few token tiles sends every W tile to all of
    // them).  At 512 tokens (2048 px level 2): Q/K/V (3840 W rows) 16.4 ->
    // 13.6 us; at ratios of 1 to 2.5 it changed nothing measurable.
    auto map_xcd = [&]() {
        if (!dl.xcd_merge || p.N < 4 * (int64_t)p.M) return;
        const int64_t tiles = (int64_t)((p.M + 63) / 64) * (p.N / 64);
        const int n_xcd = dl.n_xcd;
        if (tiles < n_xcd || tiles > INT32_MAX / 2) return;
        p.n_xcd = n_xcd;
        p.tpx = (int)((tiles + n_xcd - 1) / n_xcd);
        p.n_tiles = (int)tiles;
    };
    // bf16 X with K % 64 == 0: the pipelined kernels.
    if (!p.a_f32 && p.K % DBK == 0 && p.seg % 4 == 0) {
        if (!p.geglu && p.conv_W == 0 && p.split_ws != nullptr && p.N % 64 == 0 && p.xa_T == 0 && p.gn_N == 0) {
            const SplitPlan sp = split_plan_plain(p.M, p.N, p.K, dl);
            if (sp.splitk > 1 && p.split_ws_bytes >= sp.bytes && ((uintptr_t)p.split_ws & 15u) == 0) {
                p.splitk = sp.splitk;
                p.n_xcd = sp.n_xcd;
                p.tpx = sp.tpx;
                p.n_tiles = sp.n_tiles;
                kind = GK_DMA_64;
                return hipSuccess;
            }
        }
        if (!p.geglu) {
            // 64x64 tiles at three stages (48 KB of LDS: three workgroups per
            // compute unit).  Balanced 64 x 80 tiles when the 64 x 64 ones would divide
            // unevenly over the compute units while the 80-row tiles come to
            // at most three per compute unit and fill at least three quarters
            // of them: a 2048 x 640 product is 256 tiles instead of 320, the
            // 2048 x 1920 Q/K/V product 768 instead of 960.  Not when W has
            // four times X's rows: those keep the XCD-contiguous 64 x 64 tiles.
            const int64_t mt64 = (p.M + 63) / 64;
            const int64_t t80 = p.N % 80 == 0 ? mt64 * (p.N / 80) : 0;
            const bool g80_form = p.xa_T == 0 && p.gn_N == 0 && p.conv_W == 0 && p.w_seg_rows == 0 && p.seg_stride == 0 &&
                                  p.bias2 == nullptr && (p.seg >= p.N || (p.seg % 80 == 0 && p.N / p.seg <= 3));
            if (g80_form && p.N < 4 * (int64_t)p.M && t80 > 0 && t80 <= 3 * dl.cus && 4 * t80 >= 3 * (int64_t)dl.cus &&
                mt64 * (p.N / 64) > dl.cus) {
                kind = GK_G80;
                return hipSuccess;
            }
            if (p.N % 64 == 0) {
                map_xcd();
                kind = GK_DMA_64;
                return hipSuccess;
            }
        }
    }
    // only the pipelined kernel writes a bf16 copy, adds bias2 or convolves
    if (p.out_bf16 != nullptr || p.bias2 != nullptr || p.conv_W > 0) return hipErrorInvalidValue;
    // 128x128 tiles when they still give about a workgroup per compute unit,
    // else 64x128 / 64x64.
    kind = GK_REG_11;
    if (p.geglu) kind = GK_REG_22;
    const int64_t t128 = (int64_t)((p.M + 127) / 128) * (p.N / 128);
    if (!p.geglu && p.N % 128 == 0 && t128 >= 200)
        kind = GK_REG_22;
    else if (!p.geglu && p.N % 128 == 0 && (int64_t)((p.M + 63) / 64) * (p.N / 128) >= 160)
        kind = GK_REG_12;
    return hipSuccess;
}

// Microseconds that a planned launch of this file takes, from the measured
// times per k-tile (64 of K) of its tiles: a 64 x 64 tile is bound by its
// compute unit's share of the L2 (0.30 us a k-tile, however many share the
// unit), a 64 x 80 tile 0.32 us alone on its unit and 0.26 shared;
// a launch's ends 5 to 7, a merge of split pieces 3.
double narrow_us(const GemmParams& p, GemmKind kind, int cus) {
    const double nk = (double)(p.K / DBK) / p.splitk;
    auto tiles = [&](int bm, int bn) { return (double)((p.M + bm - 1) / bm) * (p.N / bn) * p.splitk; };
    auto shared = [&](double t) { return t > cus ? t / cus : 1.0; };
    const double merge = p.splitk > 1 ? 3.0 : 0.0;
    switch (kind) {
        case GK_DMA_64: return 5.8 + merge + shared(tiles(64, 64)) * nk * 0.30;
        case GK_G80: return 7.0 + ceil(tiles(64, 80) / cus) * nk * (tiles(64, 80) > cus ? 0.26 : 0.32);
        default: return 1e9;
    }
}

// The narrow kernels' plan, or the wide tiles' where they are estimated to
// be faster (gemm_wide.hip).
struct GemmPlan {
    GemmKind kind;
    int shape;  // wide tile
    double us;  // estimated
};

hipError_t plan_gemm(GemmParams& p, const DeviceLayout& dl, GemmPlan& pl) {
    const GemmParams in = p;
    const hipError_t e = plan_narrow(p, dl, pl.kind);
    if (e != hipSuccess) return e;
    pl.us = narrow_us(p, pl.kind, dl.cus);
    GemmParams w = in;
    double wide_us = 0.97 * pl.us;
    if (plan_wide(w, dl, wide_us, pl.shape)) {
        p = w;
        pl.kind = GK_WIDE;
        pl.us = wide_us;
    }
    return hipSuccess;
}

hipError_t launch_planned(const GemmParams& p, const GemmPlan& pl, hipStream_t s) {
    switch (pl.kind) {
        case GK_WIDE: return launch_gemm_wide(p, pl.shape, s);
        case GK_DMA_64: return launch_dma64(p, s);
        case GK_G80: {
            // two stages (36 KB of LDS) when the tiles need several per compute unit
            const dim3 grid((unsigned)((p.M + G80_BM - 1) / G80_BM), (unsigned)(p.N / G80_BN));
            if ((int64_t)grid.x * grid.y > device_layout(s).cus)
                gemm80_kernel<2><<<grid, 512, 0, s>>>(p);
            else
                gemm80_kernel<4><<<grid, 512, 0, s>>>(p);
            return hipGetLastError();
        }
        case GK_REG_22: return launch_shape<2, 2>(p, s);
        case GK_REG_12: return launch_shape<1, 2>(p, s);
        default: return launch_shape<1, 1>(p, s);
    }
}

// Workgroups along x and y of a 64 x 64 pipelined launch (launch_dma64).
void dma64_grid(const GemmParams& p, int& gx, int& gy) {
    if (p.tpx > 0) {
        gx = p.n_xcd * p.tpx * p.splitk;
        gy = 1;
    } else {
        gx = (p.M + 63) / 64;
        gy = p.N / 64;
    }
}

}  // namespace

hipError_t launch_gemm(const GemmParams& p_in, hipStream_t s) {
    GemmParams p = p_in;
    GemmPlan pl;
    const hipError_t e = plan_gemm(p, device_layout(s), pl);
    return e != hipSuccess ? e : launch_planned(p, pl, s);
}

hipError_t gemm_plan_info(GemmParams p, const DeviceLayout& dl, GemmPlanInfo* info) {
    alignas(16) static char any[16];
    p.split_ws = any;  // only looked at for its alignment
    p.split_ws_bytes = SIZE_MAX;
    GemmPlan pl;
    const hipError_t e = plan_gemm(p, dl, pl);
    if (e != hipSuccess) return e;
    info->pieces = p.splitk;
    info->per_cu = 0;
    switch (pl.kind) {
        case GK_WIDE:
            wide_tile(pl.shape, p.geglu != 0, info->tile_tokens, info->tile_outputs, info->per_cu);
            break;
        case GK_DMA_64: info->tile_tokens = info->tile_outputs = 64; break;
        case GK_G80:
            info->tile_tokens = G80_BM;
            info->tile_outputs = G80_BN;
            break;
        default:
            info->tile_tokens = pl.kind == GK_REG_22 ? 128 : 64;
            info->tile_outputs = pl.kind == GK_REG_11 || p.geglu ? 64 : 128;
    }
    return hipSuccess;
}

hipError_t launch_gemm_pair(const GemmParams& a_in, const GemmParams& b_in, hipStream_t s) {
    GemmParams a = a_in, b = b_in;
    GemmPlan pa, pb;
    const DeviceLayout dl = device_layout(s);
    hipError_t e = plan_gemm(a, dl, pa);
    if (e != hipSuccess) return e;
    e = plan_gemm(b, dl, pb);
    if (e != hipSuccess) return e;
    // One launch on the 64 x 64 pipelined kernel where that is estimated to
    // be faster than the two planned ones: its workgroups share the compute
    // units and it has one launch's ends (proj_in of the 2048 x 640 band and
    // the two blocks' text K/V: 11 us against 8 + 10).  Neither carries the
    // cross-attention epilogue, and at most one splits K (the split region
    // holds one product's partials).
    GemmParams a64 = a;
    const bool plain_a = !a.a_f32 && !a.geglu && a.conv_W == 0 && a.K % DBK == 0 && a.N % 64 == 0 && a.seg % 4 == 0 &&
                         a.xa_T == 0;
    if (pa.kind != GK_DMA_64 && plain_a) {
        a64 = a_in;
        a64.splitk = 1;
        a64.tpx = 0;
    }
    if (pb.kind == GK_DMA_64 && b.conv_W == 0 && b.xa_T == 0 && b.gn_N == 0 && plain_a && !(a64.splitk > 1 && b.splitk > 1)) {
        auto work = [](const GemmParams& p) {
            return (double)((p.M + 63) / 64) * (p.N / 64) * (p.K / DBK);
        };
        const double wgs = (work(a64) / (a64.K / DBK)) * a64.splitk + (work(b) / (b.K / DBK)) * b.splitk;
        const double longest = fmax((double)(a64.K / DBK) / a64.splitk, (double)(b.K / DBK) / b.splitk);
        const double us = 5.8 + (a64.splitk > 1 || b.splitk > 1 ? 3.0 : 0.0) +
                          0.30 * (wgs > dl.cus ? fmax(longest, (work(a64) + work(b)) / dl.cus) : longest);
        if (us < pa.us + pb.us || a.gn_N > 0) {
            GemmPair pp;
            pp.a = a64;
            pp.b = b;
            int gy_a, gy_b;
            dma64_grid(a64, pp.gx_a, gy_a);
            dma64_grid(b, pp.gx_b, gy_b);
            pp.n_a = pp.gx_a * gy_a;
            const int n_xcd = dl.n_xcd > 0 ? dl.n_xcd : 1;
            pp.b0 = (pp.n_a + n_xcd - 1) / n_xcd * n_xcd;
            const int64_t total = (int64_t)pp.b0 + (int64_t)pp.gx_b * gy_b;
            if (total > INT32_MAX) return hipErrorInvalidValue;
            if (a.gn_N > 0)
                gemm_dma_pair_kernel<DMA_GN><<<dim3((unsigned)total), 256, 0, s>>>(pp);
            else
                gemm_dma_pair_kernel<DMA_PLAIN><<<dim3((unsigned)total), 256, 0, s>>>(pp);
            return hipGetLastError();
        }
    }
    e = launch_planned(a, pa, s);
    return e != hipSuccess ? e : launch_planned(b, pb, s);
}

}  // namespace pcpp
