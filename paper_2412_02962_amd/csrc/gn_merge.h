// GroupNorm statistics of one image from the chunk records of the
// statistics launch: Chan et al.'s pairwise update of (count, mean, M2) in a
// fixed order, then, for the synchronized form (Sec. 3.3 of arXiv
// 2412.02962, kept from DistriFusion), every band's statistics in band order
// with this band's own in its place.
#pragma once

#include "common.h"

namespace pcpp {

// Chan et al.'s pairwise update of (n, mean, M2) with (nb, mb, m2b).
__device__ __forceinline__ void chan_merge(float& n, float& mean, float& m2, float nb, float mb, float m2b) {
    if (nb <= 0.f) return;
    const float nn = n + nb;
    const float r = __builtin_amdgcn_rcpf(nn);  // statistics: a 1-ulp reciprocal is plenty
    const float d = mb - mean;
    mean += d * (nb * r);
    m2 += m2b + d * d * (n * nb * r);
    n = nn;
}

struct GnStatsSrc {
    const float* stats;  // [B][chunks][G] x (count, mean, M2)
    int32_t chunks, G, B;
    float eps;
    const float* bands;  // [n_bands][B][G] x (count, mean, M2), or null
    int32_t n_bands, band;
    float* own_out;      // [B][G] x (count, mean, M2) of this band, or null
};

// Lanes that share one group's work: the largest power of two with G of them
// in 256 threads, at most a wavefront.
__host__ __device__ inline int gn_group_lanes(int G) {
    int t = 1;
    while (2 * t * G <= 256 && 2 * t <= 64) t *= 2;
    return t;
}

// Statistics of image b for the calling workgroup (its first 256 threads do
// the work; all must call): S consecutive lanes per group merge chunks j, j +
// S, ... each and meet in a shuffle tree; the bands' statistics, a lane each
// and loaded before everything else, up to 2 S of them (a chain of eight
// dependent loads took 4 us), are then merged in band order by the group's
// first lane.  Writes g_mean[G] and g_rstd[G] (LDS) and the band's own
// statistics if write_own; ends with a workgroup barrier.
__device__ __forceinline__ void gn_group_stats(const GnStatsSrc& a, int b, bool write_own, float* g_mean,
                                               float* g_rstd) {
    const int tid = threadIdx.x;
    if (tid < 256) {
        const int G = a.G;
        const int S = gn_group_lanes(G);
        const int g = min(tid / S, G - 1), j = tid % S;
        const bool mine = tid / S < G;
        struct Band {
            float n, mean, m2;
        };
        Band cur = {}, next = {};  // this lane's of S bands, and of the S after them
        auto load_band = [&](int jb, Band& x) {
            const float* o = a.bands + (((int64_t)min(jb, a.n_bands - 1) * a.B + b) * G + g) * 3;
            x.n = o[0];
            x.mean = o[1];
            x.m2 = o[2];
        };
        if (a.bands != nullptr) {
            load_band(j, cur);
            load_band(S + j, next);
        }
        float n = 0.f, mean = 0.f, m2 = 0.f;
        const float* st = a.stats + ((int64_t)b * a.chunks * G + g) * 3;
        for (int k0 = j; k0 < a.chunks; k0 += 4 * S) {
            // Records past the last chunk read the last one (every load in
            // bounds, none behind a branch: all in flight together) and count
            // zero, which the update skips.
            float cn[4], cm[4], cq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int k = k0 + u * S;
                const float* r = st + (int64_t)(k < a.chunks ? k : a.chunks - 1) * G * 3;
                cn[u] = r[0];
                cm[u] = r[1];
                cq[u] = r[2];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (k0 + u * S >= a.chunks) cn[u] = 0.f;
#pragma unroll
            for (int u = 0; u < 4; ++u) chan_merge(n, mean, m2, cn[u], cm[u], cq[u]);
        }
        for (int o = 1; o < S; o <<= 1) {
            const float on = __shfl_xor(n, o), om = __shfl_xor(mean, o), oq = __shfl_xor(m2, o);
            chan_merge(n, mean, m2, on, om, oq);
        }
        if (mine && j == 0 && write_own && a.own_out != nullptr) {
            float* o = a.own_out + ((int64_t)b * G + g) * 3;
            o[0] = n;
            o[1] = mean;
            o[2] = m2;
        }
        if (a.bands != nullptr) {
            // (only the first lane's sums are used: its own statistics are the ones written above)
            const int lane0 = (tid & 63) - j;
            float tn = 0.f, tm = 0.f, tq = 0.f;
            for (int jb = 0; jb < a.n_bands; ++jb) {
                const int at = jb & (S - 1);
                if (jb > 0 && at == 0) {
                    cur = next;
                    if (jb + S < a.n_bands) load_band(jb + S + j, next);
                }
                const float on = __shfl(cur.n, lane0 + at), om = __shfl(cur.mean, lane0 + at),
                            oq = __shfl(cur.m2, lane0 + at);
                if (jb == a.band)
                    chan_merge(tn, tm, tq, n, mean, m2);
                else
                    chan_merge(tn, tm, tq, on, om, oq);
            }
            n = tn;
            mean = tm;
            m2 = tq;
        }
        if (mine && j == 0) {
            g_mean[g] = mean;
            g_rstd[g] = n > 0.f ? rsqrtf(m2 / n + a.eps) : 0.f;
        }
    }
    __syncthreads();
}

}  // namespace pcpp
