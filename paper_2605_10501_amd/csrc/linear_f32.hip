// Linear layers of fp32 decoder sections with what stands around them: RMSNorm in front, rotary embedding (QKV) or SwiGLU
// (gate / up) behind.  The fp32 workload has a few hundred tokens and widths of 128 .. 688: a launch of any kind costs 2-8 us, most
// of it a few dependent memory latencies, so a layer's forward pass is five launches instead of nine.
//   * A workgroup computes 32 rows x two 16-column blocks, its four waves every fourth 16-deep slice of K each, with
//     v_mfma_f32_16x16x4_f32 on fragments straight from global memory (L2), three slices ahead; the waves' sums meet in LDS.
//   * The two column blocks are the ones the epilogue combines: elements i and i + head_dim / 2 of a head, or the gate and the
//     up column of an output column, so that no second kernel has to.
//   * The norm: a row's factor rstd is taken out of the product, y = rstd (x g) W^T.  Every workgroup sees whole rows of x on its
//     way through K, so it adds up their squares itself; the workgroups of the first columns also write the normed rows and rstd where
//     a backward pass will read them.
// One MI355X: c1 distillation step on 293 tokens, with the other launches saved in the same manner, 237 -> 200 us; one layer's forward
// pass (d 256) at 293 tokens 49.5 -> 38.4, at 8192 268 -> 253.  Up to d = 512: wider layers of a few thousand tokens are no longer bound by
// launches, and the squares and gains cost them up to 1.5 %.  Forward us, separate -> here, at 64 / 1000 / 12000 tokens: d 128 45 -> 32,
// 53 -> 43, 182 -> 173; d 384 52 -> 43, 110 -> 102, 821 -> 813; d 512 54 -> 45, 136 -> 128, 1288 -> 1277; d 640 63 -> 53, 212 -> 206,
// 1990 -> 2002; d 1024 85 -> 75, 414 -> 413, 4534 -> 4601.
#include "common.h"
#include "launch.h"
#include "launch_plan.h"
#include "mfma_tiles.h"

namespace {

typedef unsigned int u32x4 __attribute__((vector_size(16)));

struct NormLinear {
    const float *x, *g, *W;      // [M, K], [K], [N, K]
    int M, K, N, tiles_n;
    float eps;
    float *h, *rstd;             // normed rows [M, K] and row factors [M], both or none
    float *y;                    // rotary: [M, N]; SwiGLU: act [M, f]
    const int *pos;              // rotary: position of each row, table[position, hd / 2] of (cos, sin)
    const float2 *table;
    int hd, rotated;             // columns below `rotated` (queries, keys) are rotated
    float *up;                   // SwiGLU: pre-activations [M, 2 f], if a backward pass will read them
};

template <bool SWIGLU>
__global__ __launch_bounds__(256) void norm_linear_f32_kernel(NormLinear p) {
    __shared__ float part[4][32][33], squares[4][32], factor[32];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m0 = (int)(blockIdx.x / p.tiles_n) * 32, tn = (int)(blockIdx.x % p.tiles_n);
    const int f = p.N / 2, half = p.hd / 2, per_head = SWIGLU ? 1 : p.hd / 32;
    const int c0 = SWIGLU ? tn * 16 : tn / per_head * p.hd + tn % per_head * 16, c1 = c0 + (SWIGLU ? f : half);
    const int end0 = SWIGLU ? f : p.N;                       // columns of block 0 end here (a ragged last gate block)
    const __amdgpu_buffer_rsrc_t rx = make_rsrc(p.x, ms_matrix_extent(p.M, p.K, p.K) * 4), rw = make_rsrc(p.W, ms_matrix_extent(p.N, p.K, p.K) * 4),
                                 rg = make_rsrc(p.g, (long)p.K * 4);
    float a[4][2][4], b[4][2][4], g[4][4];
    auto load4 = [](__amdgpu_buffer_rsrc_t rs, unsigned off, float *v) __attribute__((always_inline)) {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = __uint_as_float(t[c]);
    };
    // slice s of this wave; rows, columns and k past the end arrive as zeros
    auto load = [&](int slot, int s) __attribute__((always_inline)) {
        const int k = (wave + 4 * s) * 16 + 4 * (lane >> 4);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int row = m0 + 16 * i + (lane & 15), col = (i ? c1 : c0) + (lane & 15);
            load4(rx, row < p.M && k < p.K ? (unsigned)((long)row * p.K + k) * 4u : kOob, a[slot][i]);
            load4(rw, col < (i ? p.N : end0) && k < p.K ? (unsigned)((long)col * p.K + k) * 4u : kOob, b[slot][i]);
        }
        load4(rg, k < p.K ? (unsigned)k * 4u : kOob, g[slot]);
    };
    const int slices = (p.K + 15) / 16, mine = slices > wave ? (slices - wave + 3) / 4 : 0;
    load(0, 0);
    load(1, 1);
    load(2, 2);
    // this thread's outputs: rows tid / 16 and 16 more, element tid % 16 of both column blocks
    const int q0 = tid >> 4, pc = tid & 15;
    const bool rotate = !SWIGLU && c0 < p.rotated;
    float2 cs[2] = {};
    if (rotate)
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (m0 + q0 + 16 * e < p.M) cs[e] = p.table[(long)p.pos[m0 + q0 + 16 * e] * half + tn % per_head * 16 + pc];
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float ss[2] = {0.f, 0.f};
    for (int s = 0; s < mine; s += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            load((u + 3) & 3, s + u + 3);
            __builtin_amdgcn_sched_barrier(0);        // the requests stay in front of the MFMAs
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    ss[i] = __builtin_fmaf(a[u][i][c], a[u][i][c], ss[i]);
                    const float xg = a[u][i][c] * g[u][c];
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xg, b[u][j][c], acc[i][j], 0, 0, 0);
                }
        }
    }
    // accumulator (i, j) register r: row 16 i + 4 (lane / 16) + r, column 16 j + lane % 16
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        ss[i] += __shfl_xor(ss[i], 16, 64);
        ss[i] += __shfl_xor(ss[i], 32, 64);
        if (lane < 16) squares[wave][16 * i + lane] = ss[i];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * (lane >> 4) + r][16 * j + (lane & 15)] = acc[i][j][r];
    }
    __syncthreads();
    if (tid < 32) factor[tid] = rsqrtf((squares[0][tid] + squares[1][tid] + squares[2][tid] + squares[3][tid]) / p.K + p.eps);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int q = q0 + 16 * e;
        const long row = m0 + q;
        const float lo = (part[0][q][pc] + part[1][q][pc] + part[2][q][pc] + part[3][q][pc]) * factor[q];
        const float hi = (part[0][q][16 + pc] + part[1][q][16 + pc] + part[2][q][16 + pc] + part[3][q][16 + pc]) * factor[q];
        if (row >= p.M || c0 + pc >= end0) continue;
        if constexpr (SWIGLU) {
            p.y[row * f + c0 + pc] = lo / (1.f + __expf(-lo)) * hi;
            if (p.up) {
                p.up[row * p.N + c0 + pc] = lo;
                p.up[row * p.N + c1 + pc] = hi;
            }
        } else {
            // (values are stored as they are: by (1, 0) an infinite one would turn its partner, half a head away, into NaN)
            p.y[row * p.N + c0 + pc] = rotate ? lo * cs[e].x - hi * cs[e].y : lo;
            p.y[row * p.N + c1 + pc] = rotate ? hi * cs[e].x + lo * cs[e].y : hi;
        }
    }
    if (tn == 0 && p.h) {
        const int vec = p.K / 4, rows = p.M - m0 < 32 ? p.M - m0 : 32;
        for (int i = tid; i < rows * vec; i += 256) {
            const int q = i / vec, k = i % vec * 4;
            const float4 x = *(const float4 *)(p.x + (long)(m0 + q) * p.K + k), w = *(const float4 *)(p.g + k);
            const float r = factor[q];
            *(float4 *)(p.h + (long)(m0 + q) * p.K + k) = make_float4(x.x * r * w.x, x.y * r * w.y, x.z * r * w.z, x.w * r * w.w);
        }
        if (tid < rows) p.rstd[m0 + tid] = factor[tid];
    }
}

constexpr int kMaxWidth = 512;
bool fits(const NormLinear &p, long tiles) {
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    return p.K <= kMaxWidth && p.K % 4 == 0 && al(p.x) && al(p.g) && al(p.W) && al(p.h) && ms_buffer_range_ok(p.M, p.K, p.K, 4) &&
           ms_buffer_range_ok(p.N, p.K, p.K, 4) && ms_launch_fits(tiles, 256);
}

}  // namespace

ms_status norm_qkv_rope_f32(int n, int d, int heads, int rotated_heads, int hd, float eps, const float *x, const float *g, const float *W,
                            const int *pos, const float *table, float *qkv, float *h, float *rstd, bool *done, hipStream_t s) {
    NormLinear p = {};
    p.x = x; p.g = g; p.W = W; p.M = n; p.K = d; p.N = heads * hd; p.tiles_n = p.N / 32; p.eps = eps;
    p.h = h; p.rstd = rstd; p.y = qkv; p.pos = pos; p.table = (const float2 *)table; p.hd = hd; p.rotated = rotated_heads * hd;
    const long tiles = (long)ms_cdiv(n, 32) * p.tiles_n;
    *done = hd % 32 == 0 && fits(p, tiles);
    if (!*done) return MS_OK;
    norm_linear_f32_kernel<false><<<(unsigned)tiles, 256, 0, s>>>(p);
    MS_LAUNCH_CHECK();
    return MS_OK;
}

ms_status norm_swiglu_f32(int n, int d, int f, float eps, const float *x, const float *g, const float *W, float *act, float *up, float *h,
                          float *rstd, bool *done, hipStream_t s) {
    NormLinear p = {};
    p.x = x; p.g = g; p.W = W; p.M = n; p.K = d; p.N = 2 * f; p.tiles_n = ms_cdiv(f, 16); p.eps = eps;
    p.h = h; p.rstd = rstd; p.y = act; p.up = up;
    const long tiles = (long)ms_cdiv(n, 32) * p.tiles_n;
    *done = fits(p, tiles);
    if (!*done) return MS_OK;
    norm_linear_f32_kernel<true><<<(unsigned)tiles, 256, 0, s>>>(p);
    MS_LAUNCH_CHECK();
    return MS_OK;
}
