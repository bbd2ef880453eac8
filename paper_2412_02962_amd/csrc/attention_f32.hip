// Partially conditioned self-attention, float32 storage, float64 arithmetic.
//
// Same mathematics as the bf16 path (Sec. 3.3 and Eq. 1 of arXiv
// 2412.02962): per image and head, softmax(Q K_ctx^T / sqrt(64)) V_ctx over
// the fresh band plus the stale boundary rows of the neighbours, read in
// place from the three sources.  Logits, softmax weights, their sum and the
// weighted sum of values are float64 (the float32 inputs widen exactly), so
// the only float32 rounding is the final store.
//
// Bound by the float64 matrix rate (73 TFLOP/s in a large library product).  A
// workgroup computes 16 queries of one (image, head); its wavefronts take
// consecutive ranges of the 16-key tiles and their results meet in LDS.  Both
// products run on 16x16x4 float64 MFMAs, transposed (S^T = K Q^T, O^T = V^T
// P^T), so that a lane owns one query and S^T's accumulators are the second
// product's B operand as they stand.  The contractions are permuted so that
// every lane reads 16 consecutive bytes: lane group g = lane / 16 takes head
// dimensions 16 g .. 16 g + 15 of K and Q, and value row lane % 16 of block
// db is head dimension 4 (lane % 16) + db.  K and V go straight from the L2
// into registers, a tile ahead: 16 queries per read of a key give 8 flops a
// byte, 9 TB/s at the full rate, half of the 18 TB/s of the L2.
// The matrix and the vector unit share the float64 multipliers, so that a
// tile's exponentials and conversions (about 1000 cycles a wavefront) add to
// its 2048 cycles of products.  256 queries x 640 keys x 20 heads: 1163 us
// with one thread per query (40 workgroups of two wavefronts), 38 us here;
// 1024 x 1536 x 10: 2808 -> 123 us, 33 TFLOP/s.

#include <math.h>

#include "common.h"
#include "kernels.h"

namespace pcpp {

namespace {

constexpr int D = 64;
constexpr int BQ = 16;   // queries per workgroup
constexpr int BKV = 16;  // keys per tile
constexpr int NW = 4;    // wavefronts per workgroup (8: 45 us, 2: 71 us at the shape above)
constexpr double LIMIT = 256.0;

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ const float* kv_row_f32(const KvSource& s, bool v, int b, int j, int C, int head_off) {
    const int seg = j < s.end0 ? 0 : (j < s.end1 ? 1 : 2);
    const int begin = seg == 0 ? 0 : (seg == 1 ? s.end0 : s.end1);
    const void* p0 = v ? s.v[0] : s.k[0];
    const void* p1 = v ? s.v[1] : s.k[1];
    const void* p2 = v ? s.v[2] : s.k[2];
    const float* base = (const float*)(seg == 0 ? p0 : (seg == 1 ? p1 : p2));
    const int64_t bs = seg == 0 ? s.bstride[0] : (seg == 1 ? s.bstride[1] : s.bstride[2]);
    return base + (int64_t)b * bs + (int64_t)(j - begin) * C + head_off;
}

__device__ __forceinline__ double xor_max(double v, int m) { return fmax(v, __shfl_xor(v, m)); }
__device__ __forceinline__ double xor_sum(double v, int m) { return v + __shfl_xor(v, m); }

__global__ __launch_bounds__(64 * NW) void attn_f32_kernel(AttnParams p) {
    __shared__ double o_lds[NW][16][64];  // [wavefront][4 db + r][lane]
    __shared__ double ml_lds[NW][2][16];  // [wavefront][m, l][query]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int head = blockIdx.y, b = blockIdx.z;
    const int head_off = head * D;
    const int q0 = blockIdx.x * BQ;
    const int n_kv = p.kv.n_kv;
    const int n_tiles = (n_kv + BKV - 1) / BKV;
    const int t0 = (int)((int64_t)n_tiles * wave / NW), t1 = (int)((int64_t)n_tiles * (wave + 1) / NW);

    // Q^T operand: query c, head dimension 16 g + kk of step kk.
    double qv[16];
    {
        const f32x4* qp = (const f32x4*)((const float*)p.q + (int64_t)b * p.q_bstride +
                                         (int64_t)min(q0 + c, p.nq - 1) * p.C + head_off + 16 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x4 v = qp[u];
#pragma unroll
            for (int e = 0; e < 4; ++e) qv[4 * u + e] = (double)v[e];
        }
    }
    const double scale = (double)p.scale;

    // A tile's operands: K row c, dimensions 16 g .. + 15; V rows 4 i + g,
    // dimensions 4 c .. + 3.  Keys past the end read the last row (K's scores
    // are masked; V's are cleared when used).
    struct Tile {
        f32x4 k[4], v[4];
    };
    auto load = [&](int t, Tile& x) {
        const f32x4* kp = (const f32x4*)(kv_row_f32(p.kv, false, b, min(t * BKV + c, n_kv - 1), p.C, head_off) + 16 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u) x.k[u] = kp[u];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x.v[i] = *(const f32x4*)(kv_row_f32(p.kv, true, b, min(t * BKV + 4 * i + g, n_kv - 1), p.C, head_off) + 4 * c);
    };

    f64x4 o[4];
#pragma unroll
    for (int db = 0; db < 4; ++db) o[db] = f64x4{0.0, 0.0, 0.0, 0.0};
    double m_run = -INFINITY, l_run = 0.0;  // the weights' reference (query c), this lane's share of the sum

    // S^T of a tile: row 4 i + g (register i) is the key, column c the query;
    // two chains of products, so that none waits for the one before it.
    // Keys past the end: score -inf.
    auto scores = [&](int t, const Tile& x, double (&s)[4]) {
        f64x4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 16; kk += 2) {
            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x.k[kk >> 2][kk & 3], qv[kk], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x.k[kk >> 2][(kk + 1) & 3], qv[kk + 1], s1, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] = (s0[i] + s1[i]) * scale;
        if ((t + 1) * BKV > n_kv) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (t * BKV + 4 * i + g >= n_kv) s[i] = -INFINITY;
        }
    };
    // One tile: K and V of tile t + 1 were loaded into nxt a tile ago; the
    // scores of t + 1 and the exponentials of t are independent, so that the
    // matrix and the vector unit work side by side.
    auto step = [&](int t, Tile& cur, Tile& nxt, double (&s)[4], double (&s_nxt)[4]) {
        // The weights' reference m moves only when a score exceeds it by
        // LIMIT: float64 holds exp(LIMIT) times any count of keys, and a
        // common factor costs no relative precision.
        const double mx = fmax(fmax(s[0], s[1]), fmax(s[2], s[3]));
        if (__any(mx > m_run + LIMIT)) {
            const double m_new = fmax(m_run, xor_max(xor_max(mx, 16), 32));
            // (equal: also a query whose scores so far are all -inf, where the
            // difference is no number)
            const double alpha = m_new == m_run ? 1.0 : exp(m_run - m_new);
            m_run = m_new;
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 4; ++db) o[db] *= alpha;
        }
        // (a wavefront that has seen only scores of -inf: their weights are 0)
        const double m_sub = m_run == -INFINITY ? 0.0 : m_run;
        if (t + 1 < t1) scores(t + 1, nxt, s_nxt);
        double w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = exp(s[i] - m_sub);
            l_run += w[i];
        }
        if ((t + 1) * BKV > n_kv) {  // a row past the end weighs nothing, whatever it holds
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (t * BKV + 4 * i + g >= n_kv) cur.v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int db = 0; db < 4; ++db)
                o[db] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)cur.v[i][db], w[i], o[db], 0, 0, 0);
        load(min(t + 2, t1 - 1), cur);
    };
    if (t0 < t1) {
        Tile x, y;
        double sx[4], sy[4];
        load(t0, x);
        load(min(t0 + 1, t1 - 1), y);
        scores(t0, x, sx);
        for (int t = t0; t < t1; t += 2) {
            step(t, x, y, sx, sy);
            if (t + 1 < t1) step(t + 1, y, x, sy, sx);
        }
    }
    l_run = xor_sum(xor_sum(l_run, 16), 32);

    // The wavefronts' results (a wavefront without keys: m = -inf, l = 0)
    // against the common maximum, in wavefront order; wavefront w finishes
    // the rows r = w, w + NW, ...
    if (g == 0) {
        ml_lds[wave][0][c] = m_run;
        ml_lds[wave][1][c] = l_run;
    }
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 4; ++r) o_lds[wave][4 * db + r][lane] = o[db][r];
    __syncthreads();
    double m = ml_lds[0][0][c];
#pragma unroll
    for (int k = 1; k < NW; ++k) m = fmax(m, ml_lds[k][0][c]);
    double wt[NW], l = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        wt[k] = exp(ml_lds[k][0][c] - m);
        l = fma(ml_lds[k][1][c], wt[k], l);
    }
    const double inv = 1.0 / l;
    if (q0 + c >= p.nq) return;
    // Row r of lane group g holds head dimensions 16 r + 4 g + db.
    float* op = (float*)p.out + (int64_t)b * p.q_bstride + (int64_t)(q0 + c) * p.C + head_off + 4 * g;
    for (int r = wave; r < 4; r += NW) {
        f32x4 v;
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < NW; ++k) acc = fma(o_lds[k][4 * db + r][lane], wt[k], acc);
            v[db] = (float)(acc * inv);
        }
        *(f32x4*)(op + 16 * r) = v;
    }
}

}  // namespace

hipError_t launch_attention_f32(const AttnParams& p, hipStream_t stream) {
    const dim3 grid((p.nq + BQ - 1) / BQ, p.heads, p.batch);
    attn_f32_kernel<<<grid, 64 * NW, 0, stream>>>(p);
    return hipGetLastError();
}

}  // namespace pcpp
