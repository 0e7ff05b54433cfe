// Variable-length softmax attention on packed tokens: host entry points, the fp32 kernels (head_dim 64, 80, 128) and
// the scalar (one wave per query row) kernels for the head sizes that no matrix-core kernel covers.  The bf16
// matrix-core kernels live in attention_mfma.hip.
#include "common.h"
#include "launch.h"
#include "launch_plan.h"
#include "attention.h"
#include "mfma_tiles.h"

namespace {

__device__ __forceinline__ int find_seq(const int *cu, int n_seqs, int t) {
    int lo = 0, hi = n_seqs;  // largest b with cu[b] <= t (skips zero-length sequences)
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (cu[mid] <= t) lo = mid; else hi = mid;
    }
    return lo;
}

// grid (token, ceil(nq / 4)); wave = one query head.  Keys are visited 64 at a time: lanes first
// hold one key each (scores), then one or two output columns each (P V).
template <class T>
__global__ __launch_bounds__(256) void attn_fwd_scalar_kernel(const T *__restrict__ qkv, T *__restrict__ o,
                                                               float *__restrict__ lse, const int *__restrict__ cu,
                                                               int n_seqs, int n, int nq, int nkv, int hd, int causal,
                                                               float scale) {
    __shared__ float qs[4][128], ps[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x;
    const int h = blockIdx.y * 4 + wave;
    const bool active = h < nq;
    const int hh = active ? h : nq - 1;
    const int b = find_seq(cu, n_seqs, t);
    const int s0 = cu[b], s1 = causal ? t + 1 : cu[b + 1];
    const long ld = (long)(nq + 2 * nkv) * hd;
    const int g = hh / (nq / nkv);
    const T *qp = qkv + (long)t * ld + (long)hh * hd;
    const T *kb = qkv + (long)nq * hd + (long)g * hd;
    const T *vb = qkv + (long)(nq + nkv) * hd + (long)g * hd;
    for (int d = lane; d < hd; d += 64) qs[wave][d] = to_f32(qp[d]);
    __syncthreads();
    float m = -INFINITY, l = 0.f, acc0 = 0.f, acc1 = 0.f;
    for (int j0 = s0; j0 < s1; j0 += 64) {
        const int j = j0 + lane;
        float sc = -INFINITY;
        if (j < s1) {
            const T *kp = kb + (long)j * ld;
            float dot = 0.f;
            for (int d = 0; d < hd; ++d) dot += qs[wave][d] * to_f32(kp[d]);
            sc = dot * scale;
        }
        const float mnew = fmaxf(m, wave_max(sc));
        const float pj = j < s1 ? __expf(sc - mnew) : 0.f;
        const float corr = m == -INFINITY ? 0.f : __expf(m - mnew);
        l = l * corr + wave_sum(pj);
        acc0 *= corr;
        acc1 *= corr;
        m = mnew;
        ps[wave][lane] = pj;
        __syncthreads();
        const int cnt = s1 - j0 < 64 ? s1 - j0 : 64;
        for (int jj = 0; jj < cnt; ++jj) {
            const T *vp = vb + (long)(j0 + jj) * ld;
            const float w = ps[wave][jj];
            if (lane < hd) acc0 += w * to_f32(vp[lane]);
            if (lane + 64 < hd) acc1 += w * to_f32(vp[lane + 64]);
        }
        __syncthreads();
    }
    if (!active) return;
    T *op = o + (long)t * nq * hd + (long)h * hd;
    if (lane < hd) op[lane] = from_f32<T>(acc0 / l);
    if (lane + 64 < hd) op[lane + 64] = from_f32<T>(acc1 / l);
    if (lane == 0) lse[(long)h * n + t] = m + __logf(l);
}

// Backward, same decomposition.  dQ is produced directly; dK and dV are accumulated with fp32
// atomics into dkv[n, 2 * nkv * hd] (K heads then V heads), converted afterwards.
template <class T>
__global__ __launch_bounds__(256) void attn_bwd_scalar_kernel(const T *__restrict__ qkv, const T *__restrict__ o,
                                                               const float *__restrict__ lse, const T *__restrict__ d_o,
                                                               T *__restrict__ dqkv, float *__restrict__ dkv,
                                                               const int *__restrict__ cu, int n_seqs, int n, int nq,
                                                               int nkv, int hd, int causal, float scale) {
    __shared__ float qs[4][128], dos[4][128], ps[4][64], dss[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x;
    const int h = blockIdx.y * 4 + wave;
    const bool active = h < nq;
    const int hh = active ? h : nq - 1;
    const int b = find_seq(cu, n_seqs, t);
    const int s0 = cu[b], s1 = causal ? t + 1 : cu[b + 1];
    const long ld = (long)(nq + 2 * nkv) * hd;
    const long ldkv = (long)2 * nkv * hd;
    const int g = hh / (nq / nkv);
    const T *qp = qkv + (long)t * ld + (long)hh * hd;
    const T *kb = qkv + (long)nq * hd + (long)g * hd;
    const T *vb = qkv + (long)(nq + nkv) * hd + (long)g * hd;
    const T *dop = d_o + (long)t * nq * hd + (long)hh * hd;
    const T *op = o + (long)t * nq * hd + (long)hh * hd;
    float delta = 0.f;
    for (int d = lane; d < hd; d += 64) {
        qs[wave][d] = to_f32(qp[d]);
        const float dv = to_f32(dop[d]);
        dos[wave][d] = dv;
        delta += dv * to_f32(op[d]);
    }
    delta = wave_sum(delta);
    const float L = lse[(long)hh * n + t];
    __syncthreads();
    float dq0 = 0.f, dq1 = 0.f;
    for (int j0 = s0; j0 < s1; j0 += 64) {
        const int j = j0 + lane;
        float pj = 0.f, ds = 0.f;
        if (j < s1) {
            const T *kp = kb + (long)j * ld, *vp = vb + (long)j * ld;
            float dot = 0.f, dp = 0.f;
            for (int d = 0; d < hd; ++d) {
                dot += qs[wave][d] * to_f32(kp[d]);
                dp += dos[wave][d] * to_f32(vp[d]);
            }
            pj = __expf(dot * scale - L);
            ds = pj * (dp - delta) * scale;
        }
        ps[wave][lane] = pj;
        dss[wave][lane] = ds;
        __syncthreads();
        const int cnt = s1 - j0 < 64 ? s1 - j0 : 64;
        if (active)
            for (int jj = 0; jj < cnt; ++jj) {
                const long row = j0 + jj;
                const T *kp = kb + row * ld;
                const float w = ps[wave][jj], e = dss[wave][jj];
                float *dkp = dkv + row * ldkv + (long)g * hd;
                float *dvp = dkv + row * ldkv + (long)(nkv + g) * hd;
                if (lane < hd) {
                    dq0 += e * to_f32(kp[lane]);
                    unsafeAtomicAdd(dkp + lane, e * qs[wave][lane]);
                    unsafeAtomicAdd(dvp + lane, w * dos[wave][lane]);
                }
                if (lane + 64 < hd) {
                    dq1 += e * to_f32(kp[lane + 64]);
                    unsafeAtomicAdd(dkp + lane + 64, e * qs[wave][lane + 64]);
                    unsafeAtomicAdd(dvp + lane + 64, w * dos[wave][lane + 64]);
                }
            }
        __syncthreads();
    }
    if (!active) return;
    T *dqp = dqkv + (long)t * ld + (long)h * hd;
    if (lane < hd) dqp[lane] = from_f32<T>(dq0);
    if (lane + 64 < hd) dqp[lane + 64] = from_f32<T>(dq1);
}

// dqkv[t, nq*hd + c] = (T) dkv[t, c]
template <class T>
__global__ void dkv_convert_kernel(const float *__restrict__ dkv, T *__restrict__ dqkv, long total, int ckv, long ld,
                                   int qcols) {
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    long t = i / ckv;
    int c = i % ckv;
    dqkv[t * ld + qcols + c] = from_f32<T>(dkv[i]);
}

// ---------------------------------------------------------------- fp32 on the matrix cores
// v_mfma_f32_16x16x4_f32 (operand lane = row lane % 16, k lane / 16; accumulator register r of lane l = row
// 4 (l / 16) + r, column l % 16).  A workgroup of four waves owns 16 queries (forward, dQ) or 16 keys (dK / dV) of one
// head; its waves take every fourth 16-row block of the other side, without a barrier between blocks, and meet in LDS
// at the end.  Scores are computed as S^T = K Q^T for the query-owning kernels (as S = Q K^T for the key-owning one), so
// a lane holds four keys (queries) of its own column and the four accumulator registers are the B operand of the next
// product as they stand.  The fp32 sections are short (16 .. 128 tokens): the kernels are bound by latency, so every
// operand comes straight from global memory (L2) and nothing is staged.
constexpr int kF32Tile = kF32AttnTile;

// Operand fragments of 16 rows with the contraction over HD: component c of fragment f is element 16 f + 4 (lane / 16) + c.
template <int HD> struct RowFrag {
    float v[HD / 16][4];
    __device__ __forceinline__ void load(const float *row, int lane) {      // row: this lane's row (lane % 16)
#pragma unroll
        for (int f = 0; f < HD / 16; ++f) {
            const float4 t = *(const float4 *)(row + 16 * f + 4 * (lane >> 4));
            v[f][0] = t.x; v[f][1] = t.y; v[f][2] = t.z; v[f][3] = t.w;
        }
    }
};
template <int HD>
__device__ __forceinline__ f32x4 mfma_rows(const RowFrag<HD> &a, const RowFrag<HD> &b) {
    f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};      // two chains: half the dependent latency
#pragma unroll
    for (int f = 0; f < HD / 16; ++f)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[f][c], b.v[f][c], acc[c & 1], 0, 0, 0);
    return acc[0] + acc[1];
}
// 16 rows of X as the A operand of out^T[d][col] += sum over rows of X[row][d] w[row][col], w as a score accumulator holds
// it (row 4 (lane / 16) + r): component r of block f is X[row0 + 4 (lane / 16) + r][16 f + lane % 16].  Rows at or past
// row_end read as zeros (range check of the descriptor).
template <int HD> struct ColFrag {
    float v[HD / 16][4];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, long ld, int row0, int row_end, int col0, int lane) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = row0 + 4 * (lane >> 4) + r;
            const unsigned off = row < row_end ? (unsigned)((long)row * ld + col0 + (lane & 15)) * 4u : kOob;
#pragma unroll
            for (int f = 0; f < HD / 16; ++f) v[f][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, off, f * 64, 0));
        }
    }
};
template <int HD>
__device__ __forceinline__ void mfma_cols(f32x4 *acc, const ColFrag<HD> &x, const float *w) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int f = 0; f < HD / 16; ++f) acc[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[f][r], w[r], acc[f], 0, 0, 0);
}
// The same for a block on the causal diagonal, where some weights are zeros of masked pairs.  Zero times an infinite or
// NaN element would reach columns that never see its row, so a block that holds one adds up the visible pairs one by
// one: rows after the column's own token (BELOW = false, keys of a query) or before it (BELOW = true, queries of a key)
// are left out.
template <int HD, bool BELOW>
__device__ __forceinline__ void mfma_cols_diagonal(f32x4 *acc, const ColFrag<HD> &x, const float *w, const float *X, long ld, int row0,
                                                   int row_end, int col_token, int lane) {
    float z = 0.f;
#pragma unroll
    for (int f = 0; f < HD / 16; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) z += x.v[f][r] * 0.f;               // NaN if any element is not finite
    if (!__any(z != z)) {
        mfma_cols<HD>(acc, x, w);
        return;
    }
    for (int kk = 0; kk < kF32Tile; ++kk) {
        const float w0 = __shfl(w[0], (kk >> 2) * 16 + (lane & 15), 64), w1 = __shfl(w[1], (kk >> 2) * 16 + (lane & 15), 64);
        const float w2 = __shfl(w[2], (kk >> 2) * 16 + (lane & 15), 64), w3 = __shfl(w[3], (kk >> 2) * 16 + (lane & 15), 64);
        const float wk = (kk & 3) == 0 ? w0 : (kk & 3) == 1 ? w1 : (kk & 3) == 2 ? w2 : w3;
        const int row = row0 + kk;
        if (row >= row_end || (BELOW ? row < col_token : row > col_token)) continue;
#pragma unroll
        for (int f = 0; f < HD / 16; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[f][r] += wk * X[(long)row * ld + 16 * f + 4 * (lane >> 4) + r];
    }
}
__device__ __forceinline__ float cols_max(float v) { v = fmaxf(v, __shfl_xor(v, 16, 64)); return fmaxf(v, __shfl_xor(v, 32, 64)); }
__device__ __forceinline__ float cols_sum(float v) { v += __shfl_xor(v, 16, 64); return v + __shfl_xor(v, 32, 64); }

// grid: (n_seqs * ceil(max_seqlen / 16), nq)
template <int HD>
__global__ __launch_bounds__(256) void attn_fwd_f32_kernel(const float *__restrict__ qkv, float *__restrict__ o,
                                                            float *__restrict__ lse, const int *__restrict__ cu, int ntile_max,
                                                            int n, int nq, int nkv, int causal, float scale) {
    __shared__ float po[4][HD][kF32Tile + 1], pm[4][kF32Tile], pl[4][kF32Tile];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15;
    const int b = blockIdx.x / ntile_max, h = blockIdx.y, g = h / (nq / nkv);
    const int s0 = cu[b], s1 = cu[b + 1], q0 = s0 + (int)(blockIdx.x % ntile_max) * kF32Tile;
    if (q0 >= s1) return;
    const long ld = (long)(nq + 2 * nkv) * HD;
    const float *K = qkv + (long)(nq + g) * HD;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(qkv, (long)n * ld * 4);
    const int q = q0 + col;
    const int kend = causal && q0 + kF32Tile < s1 ? q0 + kF32Tile : s1;
    RowFrag<HD> qf;
    qf.load(qkv + (long)(q < s1 ? q : s1 - 1) * ld + (long)h * HD, lane);
    float m = -INFINITY, l = 0.f;
    f32x4 acc[HD / 16];
#pragma unroll
    for (int f = 0; f < HD / 16; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = s0 + wave * kF32Tile; k0 < kend; k0 += 4 * kF32Tile) {
        RowFrag<HD> kf;
        kf.load(K + (long)(k0 + col < s1 ? k0 + col : s1 - 1) * ld, lane);
        ColFrag<HD> vc;
        vc.load(rs, ld, k0, s1, (nq + nkv + g) * HD, lane);
        __builtin_amdgcn_sched_barrier(0);           // all requests of the block in front of its first product
        const f32x4 s = mfma_rows<HD>(kf, qf);
        float p[4], mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int key = k0 + 4 * (lane >> 4) + r;
            p[r] = key < kend && (!causal || key <= q) ? s[r] * scale : -INFINITY;
            mx = fmaxf(mx, p[r]);
        }
        const float mn = fmaxf(m, cols_max(mx));
        const float mu = mn == -INFINITY ? 0.f : mn, corr = __expf(m - mu);
        float sum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = __expf(p[r] - mu);
            sum += p[r];
        }
        l = l * corr + cols_sum(sum);
        m = mn;
#pragma unroll
        for (int f = 0; f < HD / 16; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[f][r] *= corr;
        if (causal && k0 + kF32Tile > q0) mfma_cols_diagonal<HD, false>(acc, vc, p, qkv + (long)(nq + nkv + g) * HD, ld, k0, s1, q, lane);
        else mfma_cols<HD>(acc, vc, p);
    }
#pragma unroll
    for (int f = 0; f < HD / 16; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) po[wave][16 * f + 4 * (lane >> 4) + r][col] = acc[f][r];
    if (lane < kF32Tile) {
        pm[wave][lane] = m;
        pl[wave][lane] = l;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kF32Tile * HD; i += 256) {
        const int c = i / HD, d = i % HD;
        if (q0 + c >= s1) continue;
        const float mm = fmaxf(fmaxf(pm[0][c], pm[1][c]), fmaxf(pm[2][c], pm[3][c]));   // finite: a query sees itself
        float ll = 0.f, oo = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = __expf(pm[w][c] - mm);
            ll += pl[w][c] * f;
            oo += po[w][d][c] * f;
        }
        o[(long)(q0 + c) * nq * HD + (long)h * HD + d] = oo / ll;
        if (d == 0) lse[(long)h * n + q0 + c] = mm + __logf(ll);
    }
}

// One launch for dQ (blockIdx.y < nq: 16 queries of a query head) and dK / dV (the rest: 16 keys of a key/value head,
// all query heads of its group, so that nothing is summed with atomics).  delta = rowsum(dO o O) is recomputed where it
// is needed.
template <int HD>
__global__ __launch_bounds__(256) void attn_bwd_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ o,
                                                            const float *__restrict__ lse, const float *__restrict__ d_o,
                                                            float *__restrict__ dqkv, const int *__restrict__ cu, int ntile_max,
                                                            int n, int nq, int nkv, int causal, float scale) {
    __shared__ float part[4][HD][kF32Tile + 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), col = lane & 15;
    const int b = blockIdx.x / ntile_max, grp = nq / nkv;
    const int s0 = cu[b], s1 = cu[b + 1], r0 = s0 + (int)(blockIdx.x % ntile_max) * kF32Tile;
    if (r0 >= s1) return;
    const long ld = (long)(nq + 2 * nkv) * HD, ldo = (long)nq * HD;
    const int own = r0 + col, ownc = own < s1 ? own : s1 - 1;       // this lane's query (dQ) or key (dK / dV)
    f32x4 acc[2][HD / 16];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int f = 0; f < HD / 16; ++f) acc[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto row_delta = [&](const RowFrag<HD> &df, const float *orow) __attribute__((always_inline)) {
        RowFrag<HD> of;
        of.load(orow, lane);
        float s = 0.f;
#pragma unroll
        for (int f = 0; f < HD / 16; ++f)
#pragma unroll
            for (int c = 0; c < 4; ++c) s += df.v[f][c] * of.v[f][c];
        return cols_sum(s);
    };
    // sums the four waves' partial outputs and writes 16 rows of HD columns
    auto reduce = [&](const f32x4 *a, float *dst, float mul) __attribute__((always_inline)) {
        __syncthreads();
#pragma unroll
        for (int f = 0; f < HD / 16; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave][16 * f + 4 * (lane >> 4) + r][col] = a[f][r];
        __syncthreads();
        for (int i = threadIdx.x; i < kF32Tile * HD; i += 256) {
            const int c = i / HD, d = i % HD;
            if (r0 + c < s1) dst[(long)(r0 + c) * ld + d] = (part[0][d][c] + part[1][d][c] + part[2][d][c] + part[3][d][c]) * mul;
        }
    };
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(qkv, (long)n * ld * 4), rd = make_rsrc(d_o, (long)n * ldo * 4);
    RowFrag<HD> f0, f1;
    if ((int)blockIdx.y < nq) {
        const int h = blockIdx.y, g = h / grp;
        const float *K = qkv + (long)(nq + g) * HD, *V = qkv + (long)(nq + nkv + g) * HD;
        f0.load(qkv + (long)ownc * ld + (long)h * HD, lane);
        f1.load(d_o + (long)ownc * ldo + (long)h * HD, lane);
        const float delta = row_delta(f1, o + (long)ownc * ldo + (long)h * HD), L = lse[(long)h * n + ownc];
        const int kend = causal && r0 + kF32Tile < s1 ? r0 + kF32Tile : s1;
        for (int k0 = s0 + wave * kF32Tile; k0 < kend; k0 += 4 * kF32Tile) {
            RowFrag<HD> kf, vf;
            const long kr = (long)(k0 + col < s1 ? k0 + col : s1 - 1) * ld;
            kf.load(K + kr, lane);
            vf.load(V + kr, lane);
            ColFrag<HD> kc;
            kc.load(rs, ld, k0, s1, (nq + g) * HD, lane);
            __builtin_amdgcn_sched_barrier(0);
            const f32x4 s = mfma_rows<HD>(kf, f0), dp = mfma_rows<HD>(vf, f1);
            float ds[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int key = k0 + 4 * (lane >> 4) + r;
                ds[r] = key < kend && (!causal || key <= own) ? __expf(s[r] * scale - L) * (dp[r] - delta) : 0.f;
            }
            if (causal && k0 + kF32Tile > r0) mfma_cols_diagonal<HD, false>(acc[0], kc, ds, K, ld, k0, s1, own, lane);
            else mfma_cols<HD>(acc[0], kc, ds);
        }
        reduce(acc[0], dqkv + (long)h * HD, scale);
        return;
    }
    const int g = (int)blockIdx.y - nq;
    f0.load(qkv + (long)ownc * ld + (long)(nq + g) * HD, lane);
    f1.load(qkv + (long)ownc * ld + (long)(nq + nkv + g) * HD, lane);
    for (int h = g * grp; h < (g + 1) * grp; ++h) {
        const float *Q = qkv + (long)h * HD, *dO = d_o + (long)h * HD;
        for (int q0 = (causal ? r0 : s0) + wave * kF32Tile; q0 < s1; q0 += 4 * kF32Tile) {
            RowFrag<HD> qf, df;
            const int qr = q0 + col < s1 ? q0 + col : s1 - 1;
            qf.load(Q + (long)qr * ld, lane);
            df.load(dO + (long)qr * ldo, lane);
            ColFrag<HD> qc, dc;
            qc.load(rs, ld, q0, s1, h * HD, lane);
            dc.load(rd, ldo, q0, s1, h * HD, lane);
            __builtin_amdgcn_sched_barrier(0);
            const float delta = row_delta(df, o + (long)qr * ldo + (long)h * HD), L = lse[(long)h * n + qr];
            const f32x4 s = mfma_rows<HD>(qf, f0), dp = mfma_rows<HD>(df, f1);
            float p[4], ds[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int qi = 4 * (lane >> 4) + r, qq = q0 + qi;
                const float Lr = __shfl(L, qi, 64), dr = __shfl(delta, qi, 64);
                const bool ok = qq < s1 && (!causal || own <= qq);
                p[r] = ok ? __expf(s[r] * scale - Lr) : 0.f;
                ds[r] = ok ? p[r] * (dp[r] - dr) : 0.f;
            }
            if (causal && q0 < r0 + kF32Tile) {
                mfma_cols_diagonal<HD, true>(acc[0], qc, ds, Q, ld, q0, s1, own, lane);
                mfma_cols_diagonal<HD, true>(acc[1], dc, p, dO, ldo, q0, s1, own, lane);
            } else {
                mfma_cols<HD>(acc[0], qc, ds);
                mfma_cols<HD>(acc[1], dc, p);
            }
        }
    }
    reduce(acc[0], dqkv + (long)(nq + g) * HD, scale);
    reduce(acc[1], dqkv + (long)(nq + nkv + g) * HD, 1.f);
}

bool f32_tiles_supported(int hd, int n, int n_seqs, int max_seqlen, int nq, int nkv, int heads, const void *qkv, const void *o) {
    return ms_f32_attention_tiles(hd, n, n_seqs, max_seqlen, nq, nkv, heads) && (((uintptr_t)qkv | (uintptr_t)o) & 15) == 0;
}

}  // namespace

static ms_status check_attn(const char *who, int dtype, int nq, int nkv, int hd, int n, int n_seqs, int max_seqlen,
                            const void *cu) {
    if (n < 0 || n_seqs < 0 || !cu) return ms_fail(MS_ERR_INVALID_ARG, "%s: bad batch", who);
    if (nq <= 0 || nkv <= 0 || nq % nkv) return ms_fail(MS_ERR_SHAPE, "%s: n_q_heads=%d must be a multiple of n_kv_heads=%d", who, nq, nkv);
    if (hd <= 0 || hd > 128) return ms_fail(MS_ERR_UNSUPPORTED, "%s: head_dim=%d above 128", who, hd);
    if (dtype != MS_BF16 && dtype != MS_F32) return ms_fail(MS_ERR_INVALID_ARG, "%s: bad dtype", who);
    if (max_seqlen < 0) return ms_fail(MS_ERR_INVALID_ARG, "%s: negative max_seqlen", who);
    return MS_OK;
}

extern "C" ms_status ms_k_attention_forward(int32_t dtype, int32_t causal, int32_t nq, int32_t nkv, int32_t hd,
                                            int32_t n, int32_t n_seqs, int32_t max_seqlen, const int32_t *cu,
                                            const void *qkv, void *o, float *lse, void *stream) {
    MS_TRY(check_attn("attention_forward", dtype, nq, nkv, hd, n, n_seqs, max_seqlen, cu));
    if (n == 0 || n_seqs == 0) return MS_OK;
    if (!qkv || !o || !lse) return ms_fail(MS_ERR_INVALID_ARG, "attention_forward: null pointer");
    hipStream_t s = (hipStream_t)stream;
    const float scale = 1.f / sqrtf((float)hd);
    ProfScope ps(2, 0.0, s);  // work (flops) depends on the sequence lengths: computed by the caller
    if (dtype == MS_BF16 && attn_mfma_forward_supported(hd))
        return attn_mfma_forward(causal, nq, nkv, hd, n, n_seqs, max_seqlen, cu, qkv, o, lse, s);
    if (dtype == MS_F32 && f32_tiles_supported(hd, n, n_seqs, max_seqlen, nq, nkv, nq, qkv, o)) {
        const int nt = ms_cdiv(max_seqlen, kF32Tile);
        const dim3 grid((unsigned)((long)n_seqs * nt), nq);
#define GO(HD) attn_fwd_f32_kernel<HD><<<grid, 256, 0, s>>>((const float *)qkv, (float *)o, lse, cu, nt, n, nq, nkv, causal, scale)
        if (hd == 64) GO(64); else if (hd == 80) GO(80); else GO(128);
#undef GO
        MS_LAUNCH_CHECK();
        return MS_OK;
    }
    dim3 grid(n, ms_cdiv(nq, 4));
    if (dtype == MS_BF16)
        attn_fwd_scalar_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t *)qkv, (bf16_t *)o, lse, cu, n_seqs, n, nq, nkv, hd, causal, scale);
    else
        attn_fwd_scalar_kernel<float><<<grid, 256, 0, s>>>((const float *)qkv, (float *)o, lse, cu, n_seqs, n, nq, nkv, hd, causal, scale);
    MS_LAUNCH_CHECK();
    return MS_OK;
}

extern "C" size_t ms_k_attention_backward_scratch_bytes(int32_t dtype, int32_t nq, int32_t nkv, int32_t hd, int32_t n) {
    if (nq <= 0 || nkv <= 0 || hd <= 0 || n < 0) return 0;
    if (dtype == MS_BF16 && attn_mfma_backward_supported(hd)) return attn_mfma_backward_scratch_bytes(nq, nkv, hd, n);
    return ms_align_up((size_t)n * 2 * nkv * hd * sizeof(float));
}

extern "C" ms_status ms_k_attention_backward(int32_t dtype, int32_t causal, int32_t nq, int32_t nkv, int32_t hd,
                                             int32_t n, int32_t n_seqs, int32_t max_seqlen, const int32_t *cu,
                                             const void *qkv, const void *o, const float *lse, const void *d_o,
                                             void *dqkv, void *scratch, void *stream) {
    MS_TRY(check_attn("attention_backward", dtype, nq, nkv, hd, n, n_seqs, max_seqlen, cu));
    if (n == 0 || n_seqs == 0) return MS_OK;
    if (!qkv || !o || !lse || !d_o || !dqkv || !scratch) return ms_fail(MS_ERR_INVALID_ARG, "attention_backward: null pointer");
    hipStream_t s = (hipStream_t)stream;
    const float scale = 1.f / sqrtf((float)hd);
    ProfScope ps(3, 0.0, s);
    if (dtype == MS_BF16 && attn_mfma_backward_supported(hd))
        return attn_mfma_backward(causal, nq, nkv, hd, n, n_seqs, max_seqlen, cu, qkv, o, lse, d_o, dqkv, scratch, s);
    if (dtype == MS_F32 && f32_tiles_supported(hd, n, n_seqs, max_seqlen, nq, nkv, nq + nkv, qkv, o) && (((uintptr_t)d_o) & 15) == 0) {
        const int nt = ms_cdiv(max_seqlen, kF32Tile);
        const dim3 grid((unsigned)((long)n_seqs * nt), nq + nkv);
#define GO(HD) attn_bwd_f32_kernel<HD><<<grid, 256, 0, s>>>((const float *)qkv, (const float *)o, lse, (const float *)d_o, (float *)dqkv, cu, nt, n, nq, nkv, causal, scale)
        if (hd == 64) GO(64); else if (hd == 80) GO(80); else GO(128);
#undef GO
        MS_LAUNCH_CHECK();
        return MS_OK;
    }
    float *dkv = (float *)scratch;
    const long total = (long)n * 2 * nkv * hd;
    MS_TRY(launch_fill_f32(dkv, total, 0.f, s));
    dim3 grid(n, ms_cdiv(nq, 4));
    const long ld = (long)(nq + 2 * nkv) * hd;
    if (dtype == MS_BF16) {
        attn_bwd_scalar_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t *)qkv, (const bf16_t *)o, lse, (const bf16_t *)d_o, (bf16_t *)dqkv, dkv, cu, n_seqs, n, nq, nkv, hd, causal, scale);
        MS_LAUNCH_CHECK();
        dkv_convert_kernel<bf16_t><<<ms_cdiv(total, 256), 256, 0, s>>>(dkv, (bf16_t *)dqkv, total, 2 * nkv * hd, ld, nq * hd);
    } else {
        attn_bwd_scalar_kernel<float><<<grid, 256, 0, s>>>((const float *)qkv, (const float *)o, lse, (const float *)d_o, (float *)dqkv, dkv, cu, n_seqs, n, nq, nkv, hd, causal, scale);
        MS_LAUNCH_CHECK();
        dkv_convert_kernel<float><<<ms_cdiv(total, 256), 256, 0, s>>>(dkv, (float *)dqkv, total, 2 * nkv * hd, ld, nq * hd);
    }
    MS_LAUNCH_CHECK();
    return MS_OK;
}
