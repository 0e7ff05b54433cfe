// Column reductions of a backward pass (norm gains and shifts, biases): where the partial rows of each go in the scratch, which are
// pending, and when they are added up.  No device code: this part also builds for the host alone (sanitizer runs); the
// kernels are in elementwise.hip.
#include "launch.h"

namespace {
constexpr int kPartialRows = 1024;   // partial rows of one reduction at most
}

extern "C" size_t ms_k_norm_backward_scratch_bytes(int32_t d) {
    return d > 0 ? 2 * ms_align_up((size_t)kPartialRows * d * sizeof(float)) : 0;
}

ms_status column_work_finish(ColumnWork *w, hipStream_t s) {
    ReduceJobs r;
    r.count = w->count;
    int blocks = 0;
    for (int k = 0; k < w->count; ++k) {
        r.job[k] = w->job[k];
        r.first[k] = blocks;
        blocks += ms_cdiv(w->job[k].c, 32);
    }
    w->count = 0;
    w->used = 0;
    return blocks ? launch_reduce_partials(r, blocks, s) : MS_OK;
}

namespace {
// Room for `np` partial rows of `c` columns each for the `k` outputs `out`, which become pending
ms_status take_rows(ColumnWork *w, int np, const int *c, float *const *out, int k, float **part, hipStream_t s) {
    size_t need = 0;
    bool again = w->count + k > ColumnWork::kJobs;
    for (int i = 0; i < k; ++i) {
        need += ms_align_up((size_t)np * c[i] * sizeof(float));
        for (int p = 0; p < w->count; ++p) again = again || (w->job[p].out < out[i] + c[i] && out[i] < w->job[p].out + w->job[p].c);
    }
    if (again || w->used + need > w->bytes) MS_TRY(column_work_finish(w, s));
    if (need > w->bytes) return ms_fail(MS_ERR_WORKSPACE, "column sums: scratch of %zu bytes for %zu", w->bytes, need);
    for (int i = 0; i < k; ++i) {
        part[i] = (float *)(w->scratch + w->used);
        w->used += ms_align_up((size_t)np * c[i] * sizeof(float));
        w->job[w->count++] = {part[i], out[i], np, c[i]};
    }
    return MS_OK;
}
}  // namespace

ms_status norm_backward_pending(int kind, int dtype, int x_fp32, int n, int d, const void *dy, const void *x, const void *g, const float *mean,
                                const float *rstd, const void *add, void *dx, float *dg, float *db, ColumnWork *w, hipStream_t s) {
    if (n == 0) return MS_OK;
    if (!dy || !x || !g || !rstd || !dx || !dg || !w->scratch || (kind == 1 && (!mean || !db)) || n < 0 || d <= 0)
        return ms_fail(MS_ERR_INVALID_ARG, "norm_backward: null pointer or bad size");
    const int V = dtype == MS_BF16 ? 8 : 4;
    if (d % V || d > ms_norm_backward_max_d(dtype))
        return ms_fail(MS_ERR_UNSUPPORTED, "norm_backward: d=%d must be a multiple of %d and at most %d", d, V,
                       ms_norm_backward_max_d(dtype));
    const int grid = n / 4 < 1 ? 1 : (n / 4 > kPartialRows ? kPartialRows : n / 4);   // one partial row per workgroup
    const int cols[2] = {d, d};
    float *const out[2] = {dg, db};
    float *part[2] = {nullptr, nullptr};
    MS_TRY(take_rows(w, grid, cols, out, kind == 1 ? 2 : 1, part, s));
    return launch_norm_backward(kind, dtype, x_fp32, n, d, dy, x, g, mean, rstd, add, dx, part[0], part[1], grid, s);
}

extern "C" ms_status ms_k_norm_backward(int32_t kind, int32_t dtype, int32_t x_fp32, int32_t n, int32_t d,
                                        const void *dy, const void *x, const void *g, const float *mean, const float *rstd,
                                        const void *add, void *dx, float *dg, float *db, void *scratch,
                                        void *stream) {
    ColumnWork w = {(char *)scratch, ms_k_norm_backward_scratch_bytes(d), 0, 0, {}};
    MS_TRY(norm_backward_pending(kind, dtype, x_fp32, n, d, dy, x, g, mean, rstd, add, dx, dg, db, &w, (hipStream_t)stream));
    return column_work_finish(&w, (hipStream_t)stream);
}

ms_status column_sums_pending(int dtype, int n, const ColSum *sums, int count, ColumnWork *w, hipStream_t s) {
    if (n == 0 || count == 0) return MS_OK;
    const int V = dtype == MS_BF16 ? 8 : 4;
    ColSums m;
    m.count = count;
    int c[4], blocks = 0;
    float *out[4];
    for (int k = 0; k < count; ++k) {
        if (!sums[k].x || !sums[k].out || !w->scratch || n < 0 || sums[k].c <= 0) return ms_fail(MS_ERR_INVALID_ARG, "colsum: null pointer or bad size");
        if (sums[k].c % V) return ms_fail(MS_ERR_UNSUPPORTED, "colsum: c=%d must be a multiple of %d", sums[k].c, V);
        m.x[k] = sums[k].x;
        m.c[k] = c[k] = sums[k].c;
        out[k] = sums[k].out;
        m.first[k] = blocks;
        blocks += ms_cdiv(c[k] / V, 64);
    }
    // one partial row per workgroup of four waves, about 16 rows a wave, as long as all workgroups fit on the chip at once
    const int most = 2048 / blocks < 32 ? 32 : 2048 / blocks > 256 ? 256 : 2048 / blocks;
    const int gy = n / 64 < 1 ? 1 : (n / 64 > most ? most : n / 64);
    for (int k = 1; k < count; ++k)
        for (int p = 0; p < k; ++p)
            if (out[p] < out[k] + c[k] && out[k] < out[p] + c[p]) {     // into the same row: one after the other
                for (int q = 0; q < count; ++q) MS_TRY(column_sums_pending(dtype, n, sums + q, 1, w, s));
                return MS_OK;
            }
    MS_TRY(take_rows(w, gy, c, out, count, m.part, s));
    return launch_column_sums(dtype, m, n, blocks, gy, s);
}

extern "C" ms_status ms_k_colsum(int32_t dtype, int32_t n, int32_t c, const void *x, float *out, void *scratch,
                                 void *stream) {
    if (n == 0) return MS_OK;
    if (!x || !out || !scratch || n < 0 || c <= 0) return ms_fail(MS_ERR_INVALID_ARG, "colsum: null pointer or bad size");
    const ColSum one = {x, out, c};
    ColumnWork w = {(char *)scratch, ms_k_norm_backward_scratch_bytes(c), 0, 0, {}};
    MS_TRY(column_sums_pending(dtype, n, &one, 1, &w, (hipStream_t)stream));
    return column_work_finish(&w, (hipStream_t)stream);
}
