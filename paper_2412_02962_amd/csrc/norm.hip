// GroupNorm and LayerNorm (bandwidth-bound).
//
// GroupNorm uses the statistics of the band's own tokens (each image, each
// group of C/G consecutive channels), or with `bands` the whole image's
// (synchronized GroupNorm, Sec. 3.3 of arXiv 2412.02962: every band's
// (count, mean, M2) merged in band order, this band's own in its place).
// Two kernels:
//   gn_stats_slab  a workgroup per chunk of tokens and slab of channels, held
//                  in registers, reduced to per-group (count, mean, M2) with
//                  two passes over the registers (sum, then squared
//                  deviations from the chunk mean).  gn_stats_rows takes all
//                  channels, for groups that no slab of whole 16-byte vectors
//                  up to 256 channels holds.
//   gn_apply       every workgroup first merges its image's chunk records with
//                  Chan et al.'s pairwise update in a fixed order (so all of
//                  them get the same statistics), then the bands, then applies
//                  the per-channel scale and shift to its rows with 16-byte
//                  vectors (optionally SiLU).  Workgroup 0 of an image writes
//                  the band's own statistics.  In framed mode (the input of a
//                  3x3 convolution) it writes into [B][rows+2][W+2][C], and
//                  the workgroups also fill the frame (neighbour edge rows or
//                  zeros) and export the band's own first and last rows.
// LayerNorm: one wavefront per fp32 row, 16-byte loads, two passes over
// registers (wavefront sums by DPP and lane swaps), 8-byte bf16 stores.

#include <math.h>

#include "common.h"
#include "gemm.h"
#include "gn_merge.h"
#include "kernels.h"

namespace pcpp {

namespace {

constexpr int GN_THREADS = 256;
constexpr int GN_MAX_C = 2560;     // channels (the U-Net's widest concatenation)
constexpr int GN_MAX_G = 256;
// Tokens per workgroup of gn_stats_rows: 32, or 8 when a band has fewer than
// 2048 tokens.
constexpr int GN_CHUNK_LONG = 32;
constexpr int GN_CHUNK_SHORT = 8;
__host__ __device__ inline int gn_chunk_tokens(int N) { return N >= 64 * GN_CHUNK_LONG ? GN_CHUNK_LONG : GN_CHUNK_SHORT; }

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Sum over T consecutive lanes (a power of two up to a wavefront, at a
// multiple of T), the same bits in each of them: quad permutes, the half-row
// and row mirrors (DPP), then the 16- and 32-lane swaps; no LDS round trip.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float lanes_sum(float v, int T) {
    if (T >= 2) v = dpp_add<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    if (T >= 4) v = dpp_add<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    if (T >= 8) v = dpp_add<0x141>(v);  // row_half_mirror
    if (T >= 16) v = dpp_add<0x140>(v);  // row_mirror
    if (T >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if (T >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}
__device__ __forceinline__ float wave_sum(float v) { return lanes_sum(v, 64); }

// Workspace of GroupNorm: [B][chunks][G] x (count, mean, M2).
size_t gn_part_bytes(int B, int G, int chunks) { return (size_t)B * G * chunks * 3 * sizeof(float); }

// The general kernel: a workgroup per chunk of tokens, all channels.
template <int GN_CHUNK_TOKENS, int PP>  // PP: channel pairs per thread, ceil(C / 2 / GN_THREADS)
__global__ __launch_bounds__(GN_THREADS) void gn_stats_rows(GroupNormParams p) {
    __shared__ float chan_acc[GN_MAX_C];
    __shared__ float g_mean[GN_MAX_G];
    const int ch = blockIdx.x, b = blockIdx.y;
    const int tid = threadIdx.x;
    if (ch == 0 && b == 0) {
        if (p.zero != nullptr)
            for (int i = tid; i < p.n_zero; i += GN_THREADS) p.zero[i] = 0;
        if (p.zero2 != nullptr)
            for (int i = tid; i < p.n_zero2; i += GN_THREADS) p.zero2[i] = 0;
    }
    const int C = p.C, G = p.G, cg = C / G, np = C / 2;
    const int t0 = ch * GN_CHUNK_TOKENS;
    const int nt = min(GN_CHUNK_TOKENS, p.N - t0);
    const bf16* xb = p.x + ((int64_t)b * p.N + t0) * C;

    // The chunk's rows, channel pairs per lane, held in registers for both
    // passes (GN_CHUNK_TOKENS tokens, PP pairs per thread): all loads of a
    // thread in flight together.
    bf16x2 xv[PP][GN_CHUNK_TOKENS];
#pragma unroll
    for (int k = 0; k < PP; ++k) {
        const int cp = tid + GN_THREADS * k;
#pragma unroll
        for (int t = 0; t < GN_CHUNK_TOKENS; ++t) {
            bf16x2 v = {};
            if (cp < np && t < nt) v = *(const bf16x2*)(xb + (int64_t)t * C + 2 * cp);
            xv[k][t] = v;
        }
    }
    // Pass 1: per channel, the sum over the chunk's tokens.
#pragma unroll
    for (int k = 0; k < PP; ++k) {
        const int cp = tid + GN_THREADS * k;
        if (cp >= np) break;
        float s0 = 0.f, s1 = 0.f;
#pragma unroll
        for (int t = 0; t < GN_CHUNK_TOKENS; ++t) {
            s0 += (float)xv[k][t][0];
            s1 += (float)xv[k][t][1];
        }
        chan_acc[2 * cp] = s0;
        chan_acc[2 * cp + 1] = s1;
    }
    __syncthreads();
    // Per group: T consecutive lanes (a power of two, within one wavefront)
    // each add every T-th channel of the group, then a fixed shuffle tree.
    const int T = gn_group_lanes(G);
    const int gg = tid / T, gu = tid % T;
    auto group_sum = [&]() {
        float v = 0.f;
        if (gg < G)
            for (int c = gg * cg + gu; c < (gg + 1) * cg; c += T) v += chan_acc[c];
        for (int o = 1; o < T; o <<= 1) v += __shfl_xor(v, o);
        return v;
    };
    const float n_chunk = (float)nt * (float)cg;
    {
        const float v = group_sum();
        if (gg < G && gu == 0) g_mean[gg] = v / n_chunk;
    }
    __syncthreads();
    // Pass 2: squared deviations from the chunk mean of the channel's group.
#pragma unroll
    for (int k = 0; k < PP; ++k) {
        const int cp = tid + GN_THREADS * k;
        if (cp >= np) break;
        const float m0 = g_mean[2 * cp / cg], m1 = g_mean[(2 * cp + 1) / cg];
        float q0 = 0.f, q1 = 0.f;
#pragma unroll
        for (int t = 0; t < GN_CHUNK_TOKENS; ++t) {
            if (t < nt) {
                const float d0 = (float)xv[k][t][0] - m0, d1 = (float)xv[k][t][1] - m1;
                q0 += d0 * d0;
                q1 += d1 * d1;
            }
        }
        chan_acc[2 * cp] = q0;
        chan_acc[2 * cp + 1] = q1;
    }
    __syncthreads();
    {
        const float q = group_sum();
        if (gg < G && gu == 0) {
            float* st = p.stats + (((int64_t)b * p.chunks + ch) * G + gg) * 3;
            st[0] = n_chunk;
            st[1] = g_mean[gg];
            st[2] = q;
        }
    }
}

// A slab launch: slabs of S channels (gs whole groups of cg, V whole 16-byte
// vectors) and chunks of ct tokens.  RP rows of the slab fit the workgroup
// side by side; T = 2^log_T lanes sum a group.  The kernel divides by cg and V through
// their inverses (ceil(2^16 / x), exact for the dividends below 256 that it
// has): a division by a kernel argument is 30 instructions.
struct Slab {
    int32_t S, ct, cg, gs, V, RP, log_T, inv_cg, inv_V;
};

// Statistics of a chunk of tokens and a slab of channels: a thread holds one
// vector of up to KR rows in registers.  Splitting the channels as well keeps
// the launch at about one workgroup per compute unit with 16 (32) chunks per
// image, whose records every consumer merges: with 64 to 256 chunks the merge
// was most of the apply's time (statistics and apply of 2 x 8192 x 960: 9.6 +
// 27.7 us, now 9.2 + 18.6; of 2 x 8192 x 320: 5.7 + 21.4, now 5.6 + 8.8; of 2048
// x 640: 6.9 + 6.7, now 4.8 + 5.7).  A small band's launch is the chain of one
// workgroup: the load, two sums over a thread's rows, the threads of a group
// (LDS) and the group's lanes (DPP), three barriers: 512 x 1280 4.5 us, 2 x
// 133 x 64 with 64 groups 3.7 (gn_stats_rows 5.2 and 3.6; with a sum over the
// threads of a channel first, LDS permutes and a division per channel 5.9
// and 14).
template <int KR>
__global__ __launch_bounds__(GN_THREADS) void gn_stats_slab(GroupNormParams p, Slab a) {
    __shared__ __attribute__((aligned(16))) float part[GN_THREADS * 8];  // [row of RP][channel of the slab]
    __shared__ float g_mean[GN_THREADS];
    const int ch = blockIdx.x, b = blockIdx.z;
    const int tid = threadIdx.x;
    const int r0 = (tid * a.inv_V) >> 16, v = tid - r0 * a.V;
    const int t0 = ch * a.ct, nt = min(a.ct, p.N - t0);
    const bf16* xb = p.x + ((int64_t)b * p.N + t0) * p.C + blockIdx.y * a.S + 8 * v;
    bf16x8 x[KR];
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int r = r0 + k * a.RP;
        x[k] = bf16x8{};
        if (r0 < a.RP && r < nt) x[k] = *(const bf16x8*)(xb + (int64_t)r * p.C);
    }
    if (ch == 0 && blockIdx.y == 0 && b == 0) {
        if (p.zero != nullptr)
            for (int i = tid; i < p.n_zero; i += GN_THREADS) p.zero[i] = 0;
        if (p.zero2 != nullptr)
            for (int i = tid; i < p.n_zero2; i += GN_THREADS) p.zero2[i] = 0;
    }
    // Lanes u = 0 .. T - 1 of group g add every T-th of its values in part,
    // row by row, and then theirs.
    const int T = 1 << a.log_T, g = tid >> a.log_T, u = tid & (T - 1);
    const int u_r = (u * a.inv_cg) >> 16, u_c = u - u_r * a.cg;
    const int step_r = (T * a.inv_cg) >> 16, step_c = T - step_r * a.cg;
    const int step_at = step_r * a.S + step_c;
    const int rows = min(a.RP, nt);  // (the others are zeros)
    const int n_sum = (rows * a.cg + T - 1) >> a.log_T;
    auto group_sum = [&](const float (&s)[8]) {
        if (r0 < a.RP) {
            *(f32x4*)(part + r0 * a.S + 8 * v) = f32x4{s[0], s[1], s[2], s[3]};
            *(f32x4*)(part + r0 * a.S + 8 * v + 4) = f32x4{s[4], s[5], s[6], s[7]};
        }
        __syncthreads();
        float sum = 0.f;
        int r = g < a.gs ? u_r : rows, c = u_c, at = g * a.cg + u_r * a.S + u_c;
        for (int k = 0; k < n_sum; k += 4) {  // four reads in flight
            float w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[j] = part[r < rows ? at : 0];
                if (r >= rows) w[j] = 0.f;
                const bool wrap = c + step_c >= a.cg;
                c += wrap ? step_c - a.cg : step_c;
                r += wrap ? step_r + 1 : step_r;
                at += step_at + (wrap ? a.S - a.cg : 0);
            }
            sum += (w[0] + w[1]) + (w[2] + w[3]);
        }
        return lanes_sum(sum, T);
    };
    const float n_chunk = (float)nt * (float)a.cg;
    float s[8] = {};
#pragma unroll
    for (int k = 0; k < KR; ++k)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += (float)x[k][e];  // rows past the end are zeros
    const float mean_g = group_sum(s) / n_chunk;
    if (g < a.gs && u == 0) g_mean[g] = mean_g;
    __syncthreads();
    // Second pass: squared deviations from the chunk mean of the channel's group.
    float mean[8];
    {
        int ge = (8 * v * a.inv_cg) >> 16, left = (ge + 1) * a.cg - 8 * v;  // channels left in group ge
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (left == 0) {
                ++ge;
                left = a.cg;
            }
            --left;
            mean[e] = g_mean[ge];
            s[e] = 0.f;
        }
    }
#pragma unroll
    for (int k = 0; k < KR; ++k)
        if (r0 + k * a.RP < nt) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = (float)x[k][e] - mean[e];
                s[e] += d * d;
            }
        }
    const float m2 = group_sum(s);
    if (g < a.gs && u == 0) {
        float* st = p.stats + (((int64_t)b * p.chunks + ch) * p.G + blockIdx.y * a.gs + g) * 3;
        st[0] = n_chunk;
        st[1] = mean_g;
        st[2] = m2;
    }
}

// A thread takes one 16-byte vector of channels (its scale and shift in
// registers) in KR rows, RPI rows of the workgroup side by side: 320 threads
// are whole rows of 320, 640, 1280 and 2560 channels.
constexpr int GA_THREADS = 320;
static_assert(GN_MAX_C / 8 <= GA_THREADS, "a row's vectors fit the workgroup");

template <int KR>
__global__ __launch_bounds__(GA_THREADS) void gn_apply(GroupNormParams p) {
    __shared__ float g_mean[GN_MAX_G], g_rstd[GN_MAX_G];
    const int b = blockIdx.y;
    const int tid = threadIdx.x;
    const int C = p.C, G = p.G, cg = C / G;
    const int vpr = C / 8;  // 16-byte vectors per token row
    const int RPI = GA_THREADS / vpr;
    const int r0 = tid / vpr, c = 8 * (tid - r0 * vpr);
    const bool active = r0 < RPI;
    const int tok0 = blockIdx.x * (RPI * KR) + r0;
    const bf16* xb = p.x + (int64_t)b * p.N * C + c;
    // The vectors, scale and shift are loaded first, the statistics merged meanwhile.
    bf16x8 xv[KR], gm = {}, bt = {};
#pragma unroll
    for (int k = 0; k < KR; ++k)
        if (active && tok0 + k * RPI < p.N) xv[k] = *(const bf16x8*)(xb + (int64_t)(tok0 + k * RPI) * C);
    if (active) {
        gm = *(const bf16x8*)(p.gamma + c);
        bt = *(const bf16x8*)(p.beta + c);
    }
    // The image's statistics (chunks, then bands).
    {
        GnStatsSrc src;
        src.stats = p.stats;
        src.chunks = p.chunks;
        src.G = G;
        src.B = p.B;
        src.eps = p.eps;
        src.bands = p.bands;
        src.n_bands = p.n_bands;
        src.band = p.band;
        src.own_out = p.own_out;
        gn_group_stats(src, b, blockIdx.x == 0, g_mean, g_rstd);
    }
    float sc[8], sh[8];
    {
        int g = min(c, C - 8) / cg, left = (g + 1) * cg - min(c, C - 8);  // channels left in group g
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (left == 0) {
                ++g;
                left = cg;
            }
            --left;
            sc[e] = g_rstd[g] * bf16_to_f32(gm[e]);
            sh[e] = bf16_to_f32(bt[e]) - g_mean[g] * sc[e];
        }
    }
    const int pad_rows = p.pad_W > 0 ? p.N / p.pad_W : 0;
#pragma unroll
    for (int k = 0; k < KR; ++k) {
        const int tok = tok0 + k * RPI;
        if (active && tok < p.N) {
            bf16x8 y;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = __builtin_fmaf((float)xv[k][e], sc[e], sh[e]);
                if (p.silu) v = v * __builtin_amdgcn_rcpf(1.f + __expf(-v));
                y[e] = f32_to_bf16(v);
            }
            if (p.pad_W > 0) {  // token (row, col) of image b at framed (row + 1, col + 1)
                const int row = tok / p.pad_W, col = tok - row * p.pad_W;
                const int64_t dst = ((int64_t)(b * (pad_rows + 2) + row + 1) * (p.pad_W + 2) + col + 1) * C;
                *(bf16x8*)(p.y + dst + c) = y;
                if (p.edges_out != nullptr) {  // the band's first and last rows, for its neighbours
                    if (row == 0) *(bf16x8*)(p.edges_out + ((int64_t)(2 * b) * p.pad_W + col) * C + c) = y;
                    if (row == pad_rows - 1)
                        *(bf16x8*)(p.edges_out + ((int64_t)(2 * b + 1) * p.pad_W + col) * C + c) = y;
                }
            } else {
                *(bf16x8*)(p.y + ((int64_t)b * p.N + tok) * C + c) = y;
            }
        }
    }
    // Framed mode: the frame of image b, spread over the image's workgroups:
    // framed row 0 (columns 1..W) from row 1 of frame_up [B][2][W][C] or
    // zeros, framed row rows+1 from row 0 of frame_dn or zeros, and zero
    // columns 0 and W+1 of every framed row.
    if (p.pad_W > 0) {
        const int W = p.pad_W;
        const int64_t halo = 2LL * W * vpr;
        const int64_t total = halo + 2LL * (pad_rows + 2) * vpr;
        bf16* fb = p.y + (int64_t)b * (pad_rows + 2) * (W + 2) * C;
        for (int64_t u = (int64_t)blockIdx.x * GA_THREADS + tid; u < total; u += (int64_t)gridDim.x * GA_THREADS) {
            u32x4 v = {0u, 0u, 0u, 0u};
            int64_t dst;
            if (u < halo) {
                const int side = (int)(u / ((int64_t)W * vpr));
                const int64_t jj = u - (int64_t)side * W * vpr;
                const int x = (int)(jj / vpr), c = (int)(jj - (int64_t)x * vpr) * 8;
                const bf16* src = side == 0 ? p.frame_up : p.frame_dn;
                if (src != nullptr) v = *(const u32x4*)(src + ((int64_t)(2 * b + (side == 0 ? 1 : 0)) * W + x) * C + c);
                dst = ((int64_t)(side == 0 ? 0 : pad_rows + 1) * (W + 2) + x + 1) * C + c;
            } else {
                const int64_t jj = u - halo;
                const int row = (int)(jj / (2 * vpr));
                const int rem = (int)(jj - (int64_t)row * 2 * vpr);
                const int col = rem < vpr ? 0 : W + 1;
                const int c = (rem < vpr ? rem : rem - vpr) * 8;
                dst = ((int64_t)row * (W + 2) + col) * C + c;
            }
            *(u32x4*)(fb + dst) = v;
        }
    }
}

constexpr int LN_MAX_VEC = 8;  // 16-byte fp32 vectors per lane: C <= 2048

template <int NV>  // 16-byte vectors per lane: C <= 256 * NV
__global__ __launch_bounds__(256) void ln_kernel(LayerNormParams p) {
    const int row = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= p.rows) return;
    const int nv = p.C / 4;
    const f32x4* xr = (const f32x4*)(p.x + (int64_t)row * p.C);
    // The row's loads first (all in flight together), then gamma and beta.
    f32x4 v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int j = lane + 64 * k;
        v[k] = j < nv ? xr[j] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x4 gm[NV], bt[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int j = lane + 64 * k;
        if (j < nv) {
            gm[k] = *(const bf16x4*)(p.gamma + 4 * j);
            bt[k] = *(const bf16x4*)(p.beta + 4 * j);
        }
    }
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) s += (v[k][0] + v[k][1]) + (v[k][2] + v[k][3]);
    const float mean = wave_sum(s) / (float)p.C;
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int j = lane + 64 * k;
        if (j < nv) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float d = v[k][e] - mean;
                q += d * d;
            }
        }
    }
    const float rstd = rsqrtf(wave_sum(q) / (float)p.C + p.eps);
    bf16* yr = p.y + (int64_t)row * p.C;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const int j = lane + 64 * k;
        if (j < nv) {
            bf16x4 y;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                y[e] = f32_to_bf16((v[k][e] - mean) * rstd * (float)gm[k][e] + (float)bt[k][e]);
            *(bf16x4*)(yr + 4 * j) = y;
        }
    }
}

// Chunks of the general statistics kernel, at least those of the other: the
// workspace is sized for it.
int gn_chunks(int N) {
    const int ct = gn_chunk_tokens(N);
    return N > 0 ? (N + ct - 1) / ct : 1;
}

// Plan of gn_stats_slab; S = 0 where the groups do not fit it (a multiple of
// whole groups and of 8 channels above 256).  16 chunks per image (32 from
// 4096 tokens on), more where a thread would hold over 16 rows; the widest
// slab that still gives a workgroup per compute unit.
struct SlabPlan {
    Slab a;
    int chunks, rows;  // rows: per thread
};
constexpr int GN_SLAB_ROWS = 16;

SlabPlan slab_plan(int B, int N, int C, int G, int cus) {
    SlabPlan sp{};
    const int cg = C / G;
    int unit = cg;
    while (unit % 8 != 0) unit += cg;  // C is a multiple of 8 and of cg: so is this of C
    if (unit > GN_THREADS) return sp;
    int chunks = N < 4096 ? 16 : 32;
    if (chunks > gn_chunks(N)) chunks = gn_chunks(N);
    int S = unit;
    for (int s = unit; s <= GN_THREADS; s += unit)
        if (C % s == 0 && (int64_t)chunks * B * (C / s) >= cus) S = s;
    Slab a{};
    a.V = S / 8;
    a.RP = GN_THREADS / a.V;
    a.ct = (N + chunks - 1) / chunks;
    if (a.ct > GN_SLAB_ROWS * a.RP) a.ct = GN_SLAB_ROWS * a.RP;
    sp.chunks = (N + a.ct - 1) / a.ct;
    if (sp.chunks > gn_chunks(N)) return sp;
    a.S = S;
    a.cg = cg;
    a.gs = S / cg;
    while ((1 << a.log_T) < gn_group_lanes(a.gs)) ++a.log_T;
    a.inv_cg = (65536 + cg - 1) / cg;
    a.inv_V = (65536 + a.V - 1) / a.V;
    sp.a = a;
    sp.rows = (a.ct + a.RP - 1) / a.RP;
    return sp;
}

}  // namespace

size_t group_norm_ws_bytes(int B, int G, int N) { return gn_part_bytes(B, G, gn_chunks(N)); }

bool gn_shapes_ok(int C, int G) {
    return C > 0 && C % 8 == 0 && C <= GN_MAX_C && G > 0 && G <= GN_MAX_G && C % G == 0;
}

bool norm_shapes_ok(int C, int G) { return gn_shapes_ok(C, G) && C <= 4 * 64 * LN_MAX_VEC; }

hipError_t launch_group_norm_stats(GroupNormParams& p, hipStream_t s) {
    if (!gn_shapes_ok(p.C, p.G)) return hipErrorInvalidValue;
    if (p.pad_W < 0 || (p.pad_W > 0 && p.N % p.pad_W != 0)) return hipErrorInvalidValue;
    const SlabPlan sp = slab_plan(p.B, p.N, p.C, p.G, device_layout(s).cus);
    if (sp.a.S > 0) {
        p.chunks = sp.chunks;
        const dim3 grid((unsigned)sp.chunks, (unsigned)(p.C / sp.a.S), (unsigned)p.B);
        if (sp.rows <= 2)
            gn_stats_slab<2><<<grid, GN_THREADS, 0, s>>>(p, sp.a);
        else if (sp.rows <= 4)
            gn_stats_slab<4><<<grid, GN_THREADS, 0, s>>>(p, sp.a);
        else if (sp.rows <= 8)
            gn_stats_slab<8><<<grid, GN_THREADS, 0, s>>>(p, sp.a);
        else
            gn_stats_slab<GN_SLAB_ROWS><<<grid, GN_THREADS, 0, s>>>(p, sp.a);
        return hipGetLastError();
    }
    p.chunks = gn_chunks(p.N);
    const dim3 grid(p.chunks, p.B);
    const bool lng = gn_chunk_tokens(p.N) == GN_CHUNK_LONG;
    switch ((p.C / 2 + GN_THREADS - 1) / GN_THREADS) {
#define PCPP_GN_STATS(PP)                                                                      \
    case PP:                                                                                   \
        if (lng)                                                                               \
            gn_stats_rows<GN_CHUNK_LONG, PP><<<grid, GN_THREADS, 0, s>>>(p);                    \
        else                                                                                   \
            gn_stats_rows<GN_CHUNK_SHORT, PP><<<grid, GN_THREADS, 0, s>>>(p);                   \
        break;
        PCPP_GN_STATS(1)
        PCPP_GN_STATS(2)
        PCPP_GN_STATS(3)
        PCPP_GN_STATS(4)
        PCPP_GN_STATS(5)
#undef PCPP_GN_STATS
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_group_norm(GroupNormParams p, hipStream_t s) {
    const hipError_t e = launch_group_norm_stats(p, s);
    if (e != hipSuccess) return e;
    // Rows per thread: the most of 8, 4, 2 and 1 that still give two
    // workgroups per compute unit (each merges the statistics records itself;
    // one per compute unit: level-0 ResNets 1 % slower).
    const int cus = device_layout(s).cus;
    const int rpi = GA_THREADS / (p.C / 8);
    auto blocks = [&](int kr) { return (unsigned)((p.N + rpi * kr - 1) / (rpi * kr)); };
    int kr = 8;
    while (kr > 1 && (int64_t)blocks(kr) * p.B < 2 * cus) kr /= 2;
    const dim3 grid(blocks(kr), (unsigned)p.B);
    switch (kr) {
        case 8: gn_apply<8><<<grid, GA_THREADS, 0, s>>>(p); break;
        case 4: gn_apply<4><<<grid, GA_THREADS, 0, s>>>(p); break;
        case 2: gn_apply<2><<<grid, GA_THREADS, 0, s>>>(p); break;
        default: gn_apply<1><<<grid, GA_THREADS, 0, s>>>(p); break;
    }
    return hipGetLastError();
}

hipError_t launch_layer_norm(const LayerNormParams& p, hipStream_t s) {
    if (p.C % 4 != 0 || p.C > 4 * 64 * LN_MAX_VEC) return hipErrorInvalidValue;
    // One row per wavefront; one wavefront per workgroup, so that short
    // launches still spread over every compute unit.
    const unsigned grid = (unsigned)p.rows;
    switch ((p.C + 255) / 256) {
        case 1: ln_kernel<1><<<grid, 64, 0, s>>>(p); break;
        case 2: ln_kernel<2><<<grid, 64, 0, s>>>(p); break;
        case 3: ln_kernel<3><<<grid, 64, 0, s>>>(p); break;
        case 4: ln_kernel<4><<<grid, 64, 0, s>>>(p); break;
        case 5: ln_kernel<5><<<grid, 64, 0, s>>>(p); break;
        case 6: ln_kernel<6><<<grid, 64, 0, s>>>(p); break;
        case 7: ln_kernel<7><<<grid, 64, 0, s>>>(p); break;
        default: ln_kernel<8><<<grid, 64, 0, s>>>(p); break;
    }
    return hipGetLastError();
}

}  // namespace pcpp
