// Internal launch helpers shared between the translation units of the library.
#pragma once
#include "common.h"

ms_status launch_fill_f32(float *p, long n, float v, hipStream_t s);
ms_status launch_convert_from_f32(int dtype, const float *src, void *dst, long n, hipStream_t s);
ms_status launch_convert_bf16_to_f32(const void *src, float *dst, long n, hipStream_t s);

// Student-logits GEMM whose epilogue consumes the logits instead of storing them (gemm.hip); mode 1: dz, mode 2:
// per-strip partial statistics [M][nparts][8] = (m_t, s_t, m_s, s_s, A, -, -, -) over 64-column strips.
bool gemm_kd_epilogue_supported(int M, int N, int K, const void *A, long lda, const void *B, long ldb, const float *zt,
                                long ldz, const void *dz, long lddz, int dz_fp32);
ms_status gemm_kd_epilogue(int mode, int M, int N, int K, const void *A, long lda, const void *B, long ldb, const float *zt,
                           long ldz, float *stats, float *part, int nparts, float inv_t, float coef, void *dz, long lddz,
                           int dz_fp32, hipStream_t s);

// The same (bf16 dz, rows of all [M, .] results ld apart, operands without padding) together with another chunk's teacher logits
// next_zt[M, Nt] = At[M, Kt] Bt[Nt, Kt]^T, which nothing here reads; in one launch where that is faster.
ms_status gemm_kd_and_teacher(int mode, int M, int N, int K, const void *A, const void *B, const float *zt, float *stats, float *part, int nparts,
                              float inv_t, float coef, void *dz, long ld, int Nt, int Kt, const void *At, const void *Bt, float *next_zt, hipStream_t s);

// Fused gate/up GEMM + SwiGLU (gemm.hip): act[M,F] = silu(A Wg^T) * (A Wu^T), W = [Wg | Wu] rows; gate_up (may be
// null) receives the rounded pre-activations [M, 2F].
bool gemm_swiglu_supported(int M, int F, int K, const void *A, long lda, const void *W, long ldw, const void *act, long ldact,
                           const void *gate_up, long ldgu);
ms_status gemm_swiglu(int M, int F, int K, const void *A, long lda, const void *W, long ldw, void *act, long ldact,
                      void *gate_up, long ldgu, hipStream_t s);

// fp32 decoder sections: RMSNorm + QKV + rotary embedding and RMSNorm + gate / up + SwiGLU in one launch each (linear_f32.hip; done =
// false: not for these sizes or pointers, nothing was launched).  h and rstd (normed rows and row factors) and up (pre-activations)
// are for a backward pass and may be null.
ms_status norm_qkv_rope_f32(int n, int d, int heads, int rotated_heads, int hd, float eps, const float *x, const float *g, const float *W,
                            const int *pos, const float *table, float *qkv, float *h, float *rstd, bool *done, hipStream_t s);
ms_status norm_swiglu_f32(int n, int d, int f, float eps, const float *x, const float *g, const float *W, float *act, float *up, float *h,
                          float *rstd, bool *done, hipStream_t s);
// Position of every token in its sequence and the (cos, sin) table of max_pos positions, one launch (elementwise.hip)
ms_status launch_rope_setup(int n, int n_seqs, const int32_t *cu, int32_t *pos, int max_pos, int hd, float base, float *table, hipStream_t s);
// Teacher and student logits of an fp32 chunk in one launch (gemm.hip): C_i [M, N] = A_i [M, K_i] B_i [N, K_i]^T, rows of C ldc apart
ms_status gemm_f32_two(int M, int N, const float *A0, const float *B0, float *C0, int K0, const float *A1, const float *B1, float *C1, int K1,
                       long ldc, hipStream_t s);

// Column reductions of a backward pass that nobody waits for (norm gains and shifts, biases): the kernels that produce their
// partial rows run when the data is there, one launch adds up what has gathered (column_work.cpp).  scratch holds the
// partial rows of everything pending; what does not fit, or adds to a row that is already pending, is preceded by a
// column_work_finish.
struct ColReduce { const float *part; float *out; int np, c; };        // out[c] += sum of np partial rows
struct ColumnWork {
    static constexpr int kJobs = 12;
    char *scratch;
    size_t bytes, used;
    int count;
    ColReduce job[kJobs];
};
struct ColSum { const void *x; float *out; int c; };                    // out[c] += column sums of x [n, c]
ms_status norm_backward_pending(int kind, int dtype, int x_fp32, int n, int d, const void *dy, const void *x, const void *g, const float *mean,
                                const float *rstd, const void *add, void *dx, float *dg, float *db, ColumnWork *w, hipStream_t s);
ms_status column_sums_pending(int dtype, int n, const ColSum *sums, int count, ColumnWork *w, hipStream_t s);
ms_status column_work_finish(ColumnWork *w, hipStream_t s);
// Their launches (elementwise.hip).  The norm backward writes one partial row for each of its `grid` workgroups (pg, pb), a column sum
// `rows` of them for each of up to four matrices of n rows (`blocks` blocks of columns in all).
struct ReduceJobs {
    int count, first[ColumnWork::kJobs + 1];      // first block of each job
    ColReduce job[ColumnWork::kJobs];
};
struct ColSums {
    int count, first[5];                          // first column block (64 vectors) of each matrix
    const void *x[4];
    float *part[4];
    int c[4];
};
ms_status launch_reduce_partials(const ReduceJobs &jobs, int blocks, hipStream_t s);
ms_status launch_norm_backward(int kind, int dtype, int x_fp32, int n, int d, const void *dy, const void *x, const void *g, const float *mean,
                               const float *rstd, const void *add, void *dx, float *pg, float *pb, int grid, hipStream_t s);
ms_status launch_column_sums(int dtype, const ColSums &m, int n, int blocks, int rows, hipStream_t s);

// KD-loss pieces (kd.hip)
ms_status kd_forward_backward(const ms_kd_config *kd, int n_tokens, const void *h_teacher, const void *h_student,
                              float *loss_dev, float *kl_tok_dev, void *d_h_student, void *d_w_student,
                              void *workspace, size_t workspace_bytes, hipStream_t s);
ms_status validate_kd(const ms_kd_config *kd, int n_tokens);

// Optional per-launch timing (api.cpp).  Usage: { ProfScope ps(cls, work, stream); kernel<<<...>>>(...); }
void prof_begin(int cls, double work, hipStream_t s, int *slot);
void prof_end(int slot, hipStream_t s);
struct ProfScope {
    int slot;
    hipStream_t s;
    ProfScope(int cls, double work, hipStream_t stream) : slot(-1), s(stream) { prof_begin(cls, work, stream, &slot); }
    ~ProfScope() { if (slot >= 0) prof_end(slot, s); }
};
