// GEMM kernels of the section path.
//
// bf16: C = alpha * A(m,k) B(n,k) on the CDNA4 matrix cores, all four operand layouts.
//   * gemm_bf16_pp_kernel: workgroup tile 256 x 256 x 64, K-contiguous operands, two wave groups that take turns;
//   * gemm_bf16_fast_kernel: workgroup tile 256 x 256 x 64 (8 waves, wave tile 128 x 64, one workgroup per CU) or
//     128 x 128 x 64 (4 waves, two per CU) for grids that fill the chip, and 128 x 256, 128 x 128, 64 x 128 and 64 x 64
//     tiles with a ring of three or four LDS stages for grids that do not (launch_plan.h);
//     v_mfma_f32_16x16x32_bf16 by default (v_mfma_f32_32x32x16_bf16 selectable for the first two);
//   * every operand tile goes global -> LDS directly (buffer_load ... lds), two (or more) LDS buffers per operand, one
//     barrier per K tile; a K-contiguous operand lands as [rows][64] with the 16-byte chunk index XOR-swizzled (applied on the
//     global side of the load; the swizzle makes every fragment read pattern free of LDS bank conflicts), a K-major operand (weight gradients, input gradients) lands as a row tile and is read
//     through the transposing LDS load (ds_read_b64_tr_b16), so no layout needs a transposed copy;
//   * fragments are double-buffered in registers, LDS reads of the next k-step interleaved with the MFMAs;
//   * epilogues (bias, bf16 / fp32 residual, fp32 or bf16 output, accumulate, fused SwiGLU, fused KD statistics / dz)
//     pass the accumulators through the idle LDS buffers so that each lane stores 4 consecutive columns, with
//     non-temporal global accesses; split-K uses fp32 atomics;
//   * workgroup ids are remapped so that each XCD works on a contiguous range of tiles, ordered in groups of M-tiles
//     x all N-tiles, and shares operand panels in its L2;
//   * gemm_bf16_kernel is the register-staged, bounds-checked fallback (K not a multiple of 64 with a K-contiguous
//     operand, matrices of 4 GB and more).
// fp32: v_mfma_f32_16x16x4_f32 on 32 x 32 tiles with K split over the waves of a workgroup.
#include <stdlib.h>

#include <atomic>

#include "common.h"
#include "launch.h"
#include "launch_plan.h"
#include "mfma_tiles.h"
#include <type_traits>
#include <utility>

namespace {

// gcc-style vectors: the return types of the buffer load builtins
typedef unsigned int u32x4 __attribute__((vector_size(16)));
typedef unsigned int u32x2 __attribute__((vector_size(8)));

struct GemmParams {
    const void *A, *B;
    void *C;
    const void *bias, *residual;
    long lda, ldb, ldc, ldr;
    int M, N, K;
    int tiles_m, tiles_n;
    int k_tiles_per_split;  // in units of 64
    float alpha;
    int c_fp32, accumulate, atomic, res_fp32, vec_epilogue;
    // KD epilogues (EPI != 0): the tile holds student logits zs; zt = teacher logits of the same chunk
    const float *kd_zt;      // [M, kd_ldz] fp32
    long kd_ldz;
    float *kd_stats;         // EPI_KD_DZ: [M][8] per-token statistics (lse_t at 6, lse_s at 7), read
    float *kd_part;          // EPI_KD_STATS: [M][kd_nparts][8] partial statistics per 64-column strip, written
    int kd_nparts;
    float kd_inv_t, kd_coef;
    // EPI_SWIGLU: B = [gate rows (sg_f) | up rows (sg_f)], N = sg_f output columns; C = silu(gate) * up
    // [M, ldc]; sg_gu (optional) also receives the rounded gate | up pre-activations [M, sg_ldgu]
    int sg_f;
    void *sg_gu;
    long sg_ldgu;
};

// EPI_SWIGLU_BWD: the tile holds da = dL/d(silu(gate) * up); sg_gu = the pre-activations [M, sg_ldgu], read; C = [dgate | dup] [M, ldc]
enum { EPI_NONE = 0, EPI_KD_DZ = 1, EPI_KD_STATS = 2, EPI_SWIGLU = 3, EPI_SWIGLU_BWD = 4 };

// Reductions over the four 16-lane groups of a wave, on the vector ALU (no LDS crossbar): lane l gets the result over lanes
// l % 16, l % 16 + 16, + 32 and + 48.  v_permlane16_swap of a register with itself leaves the even groups' values in one
// result and the odd groups' in the other, v_permlane32_swap the lower and the upper half's.
template <class F> __device__ __forceinline__ float across_groups(float v, F f) {
    const unsigned a = __builtin_bit_cast(unsigned, v);
    const auto q = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const unsigned b = __builtin_bit_cast(unsigned, f(__builtin_bit_cast(float, (unsigned)q[0]), __builtin_bit_cast(float, (unsigned)q[1])));
    const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return f(__builtin_bit_cast(float, (unsigned)h[0]), __builtin_bit_cast(float, (unsigned)h[1]));
}
// fmaxf of three values that no instruction has produced yet (loads) costs three more to quiet signalling NaNs; v_max3 does so itself
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Cache policy of the vector epilogues' global accesses (auxiliary operand of the buffer instructions): non-temporal.
// The output tile, the residual and the teacher logits stream through once, and the 4 MB L2 of an XCD is what
// keeps the operand panels that its 32 CUs share; left at the default policy the epilogue traffic evicts them
// (measured: fp32-output and fp32-residual GEMMs 7-8 % slower, the c2 step 2.5 %).  The operand loads keep the
// default: made non-temporal they lose that sharing (15 % slower).
constexpr int kStream = 2;

template <int BM, int BN, bool TA, bool TB>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmParams p) {
    constexpr int WTM = BM / 2, WTN = BN / 2, MI = WTM / 32, NI = WTN / 32;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    bf16_t *As = (bf16_t *)smem_raw;         // [2][BM*64]
    bf16_t *Bs = As + 2 * BM * BK;           // [2][BN*64]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // XCD-aware remap of the workgroup id, then grouped (8 tile rows) ordering
    int pid;
    {
        const int nb = gridDim.x, b = blockIdx.x;
        const int per = nb >> 3, rem = nb & 7, x = b & 7, q = b >> 3;
        pid = x * per + (x < rem ? x : rem) + q;
    }
    constexpr int GM = 8;
    const int group = pid / (GM * p.tiles_n);
    const int first_m = group * GM;
    const int gsize = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
    const int tm = first_m + (pid % (GM * p.tiles_n)) % gsize;
    const int tn = (pid % (GM * p.tiles_n)) / gsize;
    const int m0 = tm * BM, n0 = tn * BN;

    const int kt_begin = blockIdx.y * p.k_tiles_per_split;
    int kt_end = kt_begin + p.k_tiles_per_split;
    const int kt_total = (p.K + BK - 1) / BK;
    if (kt_end > kt_total) kt_end = kt_total;
    const int nk = kt_end - kt_begin;
    if (nk <= 0) return;
    const int k_end = p.K;

    const bf16_t *A = (const bf16_t *)p.A, *B = (const bf16_t *)p.B;
    Stager<BM, TA> sa;
    Stager<BN, TB> sb;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

    sa.load(A, p.lda, m0, p.M, kt_begin * BK, k_end, tid);
    sb.load(B, p.ldb, n0, p.N, kt_begin * BK, k_end, tid);
    sa.store(As, tid);
    sb.store(Bs, tid);
    __syncthreads();

    const int frow = lane & 31, fhalf = lane >> 5;
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) {
            sa.load(A, p.lda, m0, p.M, (kt_begin + kt + 1) * BK, k_end, tid);
            sb.load(B, p.ldb, n0, p.N, (kt_begin + kt + 1) * BK, k_end, tid);
        }
        // fragments of k-step kk+1 are fetched from LDS while the MFMAs of k-step kk run
        bf16x8 af[2][MI], bfr[2][NI];
        auto load_frags = [&](int kk, int slot) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
                af[slot][i] = *(const bf16x8 *)(As + cur * BM * BK + lds_off(wm * WTM + i * 32 + frow, kk * 2 + fhalf));
#pragma unroll
            for (int j = 0; j < NI; ++j)
                bfr[slot][j] = *(const bf16x8 *)(Bs + cur * BN * BK + lds_off(wn * WTN + j * 32 + frow, kk * 2 + fhalf));
        };
        load_frags(0, 0);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            if (kk + 1 < BK / 16) load_frags(kk + 1, (kk + 1) & 1);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk & 1][i], bfr[kk & 1][j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) {
            sa.store(As + (cur ^ 1) * BM * BK, tid);
            sb.store(Bs + (cur ^ 1) * BN * BK, tid);
        }
        __syncthreads();
    }

    // epilogue: acc[i][j][r] is C(row, col) with row = 8*(r/4) + 4*(lane/32) + r%4, col = lane%32
    const bf16_t *bias = (const bf16_t *)p.bias, *res = (const bf16_t *)p.residual;
    const float *res32 = (const float *)p.residual;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col = n0 + wn * WTN + j * 32 + frow;
            if (col >= p.N) continue;
            const float bv = bias ? (float)bias[col] : 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + wm * WTM + i * 32 + 8 * (r >> 2) + 4 * fhalf + (r & 3);
                if (row >= p.M) continue;
                float v = acc[i][j][r] * p.alpha + bv;
                if (res) v += p.res_fp32 ? res32[(long)row * p.ldr + col] : (float)res[(long)row * p.ldr + col];
                if (p.c_fp32) {
                    float *c = (float *)p.C + (long)row * p.ldc + col;
                    if (p.atomic) unsafeAtomicAdd(c, v);
                    else if (p.accumulate) *c += v;
                    else *c = v;
                } else {
                    ((bf16_t *)p.C)[(long)row * p.ldc + col] = (bf16_t)v;
                }
            }
        }
}

// ------------------------------------------------------------------ fast path
// Same tiling and MFMA loop, but
//   * an operand stored K-contiguous goes global -> LDS directly (buffer_load ... lds, 16 bytes per
//     lane, one instruction fills 8 tile rows = 1 KB): lane l of the instruction that fills rows
//     8G .. 8G+7 lands at row 8G + l/8, chunk position l%8, so it fetches the chunk that the LDS
//     swizzle assigns to that position.  No staging registers, no LDS store instructions; rows
//     past the end of the matrix read as zero through the buffer descriptor's range check;
//   * the epilogue addresses C (and the residual) through buffer descriptors as well, so rows
//     past M are dropped by the range check and columns past N by one select per column:
//     no per-element branches.
// Needs K % 64 == 0 when an operand is K-contiguous and every matrix below 4 GB.
// The same for an operand stored K-major: the tile is 64 k-rows x COLS columns, kept as COLS/64 sub-tiles
// [64][64]; instruction idx fills 8-row group idx % 8 of sub-tile idx / 8.  Rows past K fall outside the
// descriptor (zeros), so K needs no padding; columns past the matrix edge read the next row (never stored).
template <int COLS, int NWAVES>
struct RowTileStager {
    static constexpr int NI = COLS / 8 / NWAVES;
    unsigned base[NI];                     // byte offset of this lane's 16 bytes at k0 = 0, per instruction
    unsigned ldb;                          // bytes per k-row
    __device__ __forceinline__ void init(long ld, int col0, int wave, int lane) {
        ldb = (unsigned)(ld * 2);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int idx = wave * NI + i, sub = idx >> 3, g = idx & 7;
            const int r = g * 8 + (lane >> 3);
            const int c = (lane & 7) ^ swz_row(r);
            base[i] = (unsigned)r * ldb + (unsigned)(col0 + sub * 64 + c * 8) * 2;
        }
    }
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, bf16_t *tile, int k0, int wave, unsigned inv) const {
        const unsigned koff = (unsigned)k0 * ldb;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int idx = wave * NI + i;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(tile + (idx >> 3) * 4096 + (idx & 7) * 512), 16,
                                                     (base[i] + koff) | inv, 0, 0, 0);
        }
    }
};

// B tile of the fused gate/up + SwiGLU GEMM: tile row R = 64 * w + 32 * u + l holds weight row
// u * F + col0 + 32 * w + l (u = 0 gate, 1 up), so that the two 32-column blocks of wave column w are
// the gate and the up pre-activation of the same 32 output columns (same lane, same register).
template <int ROWS, int NWAVES>
struct GateUpStager {
    static constexpr int NI = ROWS / 8 / NWAVES;
    unsigned lanepart;                     // (lane >> 3) rows + swizzle-free part, in bytes
    unsigned ldb;                          // bytes per row
    int x, col0, f;
    __device__ __forceinline__ void init(long ld, int col0_, int f_, int lane) {
        ldb = (unsigned)(ld * 2);
        lanepart = (unsigned)(lane >> 3) * ldb;
        x = (lane & 7) ^ swz_row(lane >> 3);
        col0 = col0_;
        f = f_;
    }
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, bf16_t *tile, int k0, int wave, unsigned inv) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int g = wave * NI + i;                                   // 8-row group of the tile (scalar)
            const int wrow = ((g >> 2) & 1) * f + col0 + (g >> 3) * 32 + (g & 3) * 8;
            const unsigned voff = ((unsigned)wrow * ldb + lanepart + ((x ^ swz_row(8 * g)) << 4)) | inv;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(tile + g * 8 * BK), 16, voff, k0 * 2, 0, 0);
        }
    }
};

template <int ROWS, int NWAVES>
struct DmaStager {
    static constexpr int NI = ROWS / 8 / NWAVES;   // instructions per wave per tile
    unsigned rowoff;                       // byte offset of this lane's row within an 8-row group
    unsigned ld8;                          // bytes between 8-row groups
    int x;                                 // (lane & 7) ^ swz_row(lane >> 3): chunk swizzle without the group term swz_row(8 g)
    __device__ __forceinline__ void init(long ld, int row0, int lane) {
        rowoff = (unsigned)(((long)(row0 + (lane >> 3)) * ld) * 2);
        ld8 = (unsigned)(ld * 16);
        x = (lane & 7) ^ swz_row(lane >> 3);
    }
    // wave (scalar) fills 8-row groups wave*NI .. wave*NI + NI-1 of the tile
    // inv = 0, or kOob to fill the tile with zeros (OR-ing it in puts every lane out of range without a branch)
    __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, bf16_t *tile, int k0, int wave, unsigned inv) const {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int g = wave * NI + i;
            const unsigned voff = (rowoff + g * ld8 + ((x ^ swz_row(8 * g)) << 4)) | inv;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(tile + g * 8 * BK), 16, voff, k0 * 2, 0, 0);
        }
    }
};

// Scheduling pattern of one k-step: spread R LDS reads over the first MFMAs (R/M each, at least one),
// then the remaining MFMAs back to back.
template <int N>
__device__ __forceinline__ void sched_reads_then_mfma() {
    __builtin_amdgcn_sched_group_barrier(0x100, N, 0);   // N LDS reads
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
}
template <int R, int PER, int... I>
__device__ __forceinline__ void sched_pairs(std::integer_sequence<int, I...>) {
    (sched_reads_then_mfma<((I + 1) * PER <= R ? PER : R - I * PER)>(), ...);
}
// Scheduling pattern of one k-step with 16-row fragments: per row block, its NB MFMAs and then the reads that
// refill its A fragment (RA reads) and the next BPB of the NB B fragments (RB reads each).
// VM = number of direct-to-LDS loads issued in this k-step (0, or one tile's worth): spread evenly over the row blocks.
template <int NB, int RA, int RB, int VM, int... I>
__device__ __forceinline__ void sched_mfma_then_reads(std::integer_sequence<int, I...>) {
    constexpr int MB = sizeof...(I), PB = (VM + MB - 1) / MB;      // loads per row block
    constexpr int BPB = (NB + MB - 1) / MB;                        // B fragments per row block
    ((__builtin_amdgcn_sched_group_barrier(0x008, NB, 0),
      __builtin_amdgcn_sched_group_barrier(0x100, RA + RB * (I * BPB >= NB ? 0 : (NB - I * BPB < BPB ? NB - I * BPB : BPB)), 0),
      (I * PB < VM ? __builtin_amdgcn_sched_group_barrier(0x020, (VM - I * PB < PB ? VM - I * PB : PB), 0) : (void)0)), ...);
}
template <int R, int M>
__device__ __forceinline__ void interleave_reads_with_mfma() {
    constexpr int PER = R >= M ? (R + M - 1) / M : 1;     // reads in front of each of the first MFMAs
    constexpr int PAIRS = (R + PER - 1) / PER;
    static_assert(PAIRS <= M, "more read groups than MFMAs");
    sched_pairs<R, PER>(std::make_integer_sequence<int, PAIRS>{});
    if constexpr (M > PAIRS) __builtin_amdgcn_sched_group_barrier(0x008, M - PAIRS, 0);
}

// Addresses of the transposing reads of a K-major operand for v_mfma_f32_16x16x32_bf16: the 16 lanes of group g
// (= lane / 16) read k rows 8g .. 8g+7 of the k-step (two reads of four rows) for the 16 columns of a block.
// The LDS swizzle of those rows does not depend on the k-step, and the two 16-column halves of a 32-column
// block differ by one flipped chunk bit: four registers per operand, everything else is a constant offset.
struct TrFragAddr16 {
    int base[2][2];   // [16-column half of the 32-column block][first / second read], element offset within the tile
    __device__ __forceinline__ void init(int w32, int lane) {
        const int g = lane >> 4, r = lane & 15, q = r >> 2;
#pragma unroll
        for (int hf = 0; hf < 2; ++hf) {
            const int m = w32 * 32 + 16 * hf + 4 * (r & 3);
            const int sub = m >> 6, chunk = (m & 63) >> 3;
#pragma unroll
            for (int rd = 0; rd < 2; ++rd) {
                const int rl = 8 * g + q + 4 * rd;                       // row within the 32-row k-step
                const int sw = swz_row(rl);
                base[hf][rd] = sub * 4096 + rl * 64 + ((chunk ^ sw) << 3) + (m & 7);
            }
        }
    }
    // block16 = index of the wave's 16-column block; off = element offset of its 32-column block's sub-tile pair
    __device__ __forceinline__ bf16x8 frag(const bf16_t *tile, int kk, int block16, int off) const {
        return tr_frag(tile + base[block16 & 1][0] + kk * 2048 + off, tile + base[block16 & 1][1] + kk * 2048 + off);
    }
};

// Addresses of the 16-byte fragment reads of a K-contiguous operand for v_mfma_f32_16x16x32_bf16: lane = (row
// lane % 16 of the 16-row block, k-group lane / 16).  The LDS swizzle makes the chunk position depend on the
// parity of the block and on the k-step; four registers per operand cover all blocks with constant offsets.
struct KFragAddr16 {
    int base[2][2];   // [block parity][k-step], element offset within the tile of block 0 / 1
    __device__ __forceinline__ void init(int row0, int lane) {      // row0 = first tile row of the wave (multiple of 32)
        const int r = lane & 15, g = lane >> 4;
#pragma unroll
        for (int par = 0; par < 2; ++par)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) base[par][kk] = lds_off(row0 + par * 16 + r, kk * 4 + g) - par * 16 * BK;
    }
    __device__ __forceinline__ bf16x8 frag(const bf16_t *tile, int kk, int block16) const {
        return *(const bf16x8 *)(tile + base[block16 & 1][kk] + block16 * 16 * BK);
    }
};

// Epilogue of the fast kernels.  acc[i][j]: the wave's MI x NI accumulator blocks (16 x 16 with M16, else 32 x 32) of 64
// columns in all; the wave's 32-row block i starts at tile row row_base(i), its 32-column block j at tile column
// col_base(j); stg: 8 KB of LDS that belong to the wave (the operand buffers are idle by now).
template <int EPI, bool M16, bool TA, bool TB, int MI, int NI, class ACC, class RB, class CB>
__device__ __forceinline__ void gemm_epilogue(const GemmParams &p, ACC (&acc)[MI][NI], float *stg, int m0, int n0, int wn, int lane,
                                              RB row_base, CB col_base) {
    constexpr int FR = M16 ? 16 : 32, ACC_N = M16 ? 4 : 16, MI32 = MI * FR / 32, WTN = 64;
    static_assert(NI * FR == WTN, "staging assumes 64-column wave tiles");
    const int frow = lane & (FR - 1), fhalf = lane / FR;
    // ---- epilogue staging: the accumulators of the wave's 32-row block i go to LDS as [32 rows][64 columns]
    // fp32 (v = value transform), from where each lane reads 4 consecutive columns of a row.  The 16-column
    // group index (32x32 MFMA: column bit 5 only) is XOR-ed with row bits so that the lanes of one store
    // instruction, which hold the same columns of rows 4 apart, use different banks.
    auto stg_swz = [](int row) { return M16 ? ((row >> 2) & 3) << 4 : ((row >> 2) & 1) << 5; };
    // The lanes of a wave exchange data through the staging area, and the LDS executes a wave's accesses in
    // program order; what has to be kept is the program order itself: to the compiler a lane's reads and another
    // lane's writes are unrelated addresses that it may reorder.  wave_sync() is a compiler-level fence between the
    // two phases (no instruction).
    auto wave_sync = []() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto stage_block = [&](int i, auto v) __attribute__((always_inline)) {
        wave_sync();     // the reads of the previous block come first
        if constexpr (M16) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int row = h * 16 + 4 * fhalf + r;
                        stg[row * 64 + ((j * 16 + frow) ^ stg_swz(row))] = v(acc[2 * i + h][j][r]);
                    }
        } else {
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                    stg[row * 64 + ((j * 32 + frow) ^ stg_swz(row))] = v(acc[i][j][r]);
                }
        }
        wave_sync();     // every lane's values are in LDS before any lane reads
    };
    // ---- epilogue.  C and the residual are addressed through buffer descriptors: rows past M are
    // dropped (stores) or read as zero by the range check, columns past N by one select.
    // Byte offset of row r of the wave's block i: the lane's part (its row within the pass and its column) once, the rest, which is
    // the same in all lanes, on the scalar unit.  A product per row and lane on the vector ALU is a quarter-rate instruction; with the
    // packed conversions below it was 46 instead of 35 vector instructions for four rows of the dz epilogue, 42 instead of 32 for
    // SwiGLU's (distillation head of 8192 tokens, V = 151936 31.01 -> 30.84 ms, 1024 tokens, V = 32000 638 -> 635 us, others even).
    auto row_bytes = [&](int i, int r, long ld, int es) { return (unsigned)(m0 + row_base(i) + r) * (unsigned)ld * (unsigned)es; };
    // four values in the storage type, two conversions of two
    auto pack4 = [](const float *v) {
        typedef bf16_t pair_t __attribute__((ext_vector_type(2)));
        u32x2 w;
        w[0] = __builtin_bit_cast(unsigned, pair_t{(bf16_t)v[0], (bf16_t)v[1]});
        w[1] = __builtin_bit_cast(unsigned, pair_t{(bf16_t)v[2], (bf16_t)v[3]});
        return w;
    };
    const int esz = p.c_fp32 ? 4 : 2;
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(p.C, (long)p.M * p.ldc * esz);
    const int rsz = p.res_fp32 ? 4 : 2;
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.residual ? p.residual : p.C, p.residual ? (long)p.M * p.ldr * rsz : 0);
    const bf16_t *bias = (const bf16_t *)p.bias;
    if constexpr (EPI == EPI_SWIGLU) {
        // acc[i][0] = gate, acc[i][1] = up of output columns n0/2 + wn*32 + (0..31).  Both are rounded to
        // the storage type first (they are the values a separate activation kernel would read back), staged
        // through LDS as [32 rows][gate 32 | up 32], and each lane then owns 4 consecutive output columns.
        static_assert(!TA && !TB, "SwiGLU epilogue is built for the K-contiguous layout");
        const int prow = lane >> 3, pcol = (lane & 7) * 4;
        const int colg = n0 / 2 + wn * 32 + pcol;
        const bool cok = colg < p.N;
        const unsigned lane_c = (unsigned)((prow * p.ldc + colg) * 2), lane_g = (unsigned)((prow * p.sg_ldgu + colg) * 2);
        const __amdgpu_buffer_rsrc_t rg = make_rsrc(p.sg_gu ? p.sg_gu : p.C, p.sg_gu ? (long)p.M * p.sg_ldgu * 2 : 0);
#pragma unroll
        for (int i = 0; i < MI32; ++i) {
            stage_block(i, [&](float a) { return (float)(bf16_t)(a * p.alpha); });
#pragma unroll
            for (int ps = 0; ps < 4; ++ps) {
                const int row = ps * 8 + prow;
                const int flip = stg_swz(row);
                const float4 g4 = *(const float4 *)(stg + row * 64 + (pcol ^ flip));
                const float4 u4 = *(const float4 *)(stg + row * 64 + ((32 + pcol) ^ flip));
                const float gv[4] = {g4.x, g4.y, g4.z, g4.w}, uv[4] = {u4.x, u4.y, u4.z, u4.w};
                float a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)   // silu(g) u = g u / (1 + e^-g); hardware reciprocal (1 ulp) instead of the division sequence
                    a[e] = gv[e] * uv[e] * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * gv[e]));
                __builtin_amdgcn_raw_buffer_store_b64(pack4(a), rc, cok ? lane_c + row_bytes(i, ps * 8, p.ldc, 2) : kOob, 0, kStream);
                if (p.sg_gu) {
                    const unsigned go = cok ? lane_g + row_bytes(i, ps * 8, p.sg_ldgu, 2) : kOob;
                    __builtin_amdgcn_raw_buffer_store_b64(pack4(gv), rg, go, 0, kStream);
                    __builtin_amdgcn_raw_buffer_store_b64(pack4(uv), rg, cok ? go + (unsigned)p.sg_f * 2 : kOob, 0, kStream);
                }
            }
        }
        return;
    }
    // ---- vector epilogues.  Each wave passes its accumulators through LDS, 32 rows at a time, to turn the
    // MFMA layout (a lane owns one column) into rows: a lane then handles 4 consecutive columns of a row, so
    // global reads and writes are 8..16 bytes per lane and 128..256 contiguous bytes per row.  What the
    // epilogue reads from memory for a 32-row block (fp32/bf16 residual, C when accumulating, teacher logits)
    // is fetched one block ahead into registers: the loads of block i+1 are issued before the stores of
    // block i, so no pass waits for a store or for its own load's full latency.
    if (EPI != EPI_NONE || p.vec_epilogue) {
        const int prow = lane >> 4, pcol = (lane & 15) * 4;
        const int colg = n0 + col_base(pcol >> 5) + (pcol & 31);
        const bool cok = colg < p.N;
        // the prefetched stream: KD -> teacher logits (fp32); else residual (fp32 or bf16); else C (accumulate)
        // (SwiGLU backward -> gate and up, 4 bf16 each)
        const bool aux_res = EPI == EPI_NONE && p.residual != nullptr;
        const bool aux_c = EPI == EPI_NONE && !aux_res && p.accumulate && p.c_fp32;
        const bool has_aux = EPI != EPI_NONE || aux_res || aux_c;
        const bool aux4 = EPI != EPI_NONE || aux_c || p.res_fp32;                  // 4-byte elements
        const long aux_ld = EPI != EPI_NONE ? p.kd_ldz : (aux_res ? p.ldr : p.ldc);
        const __amdgpu_buffer_rsrc_t ra_ = EPI == EPI_SWIGLU_BWD ? make_rsrc(p.sg_gu, (long)p.M * p.sg_ldgu * 2)
                                           : EPI != EPI_NONE     ? make_rsrc(p.kd_zt, (long)p.M * p.kd_ldz * 4) : (aux_res ? rr : rc);
        const __amdgpu_buffer_rsrc_t rl = make_rsrc(EPI == EPI_KD_DZ ? (const void *)p.kd_stats : p.C, EPI == EPI_KD_DZ ? (long)p.M * 32 : 0);
        u32x4 aux[2][8];
        float2 lsev[2][8];                                                         // EPI_KD_DZ: (lse_t, lse_s) of the row
        const unsigned lane_c = (unsigned)((prow * p.ldc + colg) * esz), lane_aux = (unsigned)((prow * aux_ld + colg) * (aux4 ? 4 : 2));
        const unsigned lane_g = (unsigned)((prow * p.sg_ldgu + colg) * 2);
        auto prefetch = [&](int i, u32x4 *dst, float2 *ldst) {
#pragma unroll
            for (int ps = 0; ps < 8; ++ps) {
                if constexpr (EPI == EPI_SWIGLU_BWD) {
                    const unsigned go = cok ? lane_g + row_bytes(i, ps * 4, p.sg_ldgu, 2) : kOob;
                    const u32x2 g = __builtin_amdgcn_raw_buffer_load_b64(ra_, go, 0, kStream);
                    const u32x2 u = __builtin_amdgcn_raw_buffer_load_b64(ra_, cok ? go + (unsigned)p.sg_f * 2 : kOob, 0, kStream);
                    dst[ps][0] = g[0]; dst[ps][1] = g[1]; dst[ps][2] = u[0]; dst[ps][3] = u[1];
                    continue;
                }
                const unsigned off = cok ? lane_aux + row_bytes(i, ps * 4, aux_ld, aux4 ? 4 : 2) : kOob;
                if (aux4) dst[ps] = __builtin_amdgcn_raw_buffer_load_b128(ra_, off, 0, kStream);
                else {
                    const u32x2 q = __builtin_amdgcn_raw_buffer_load_b64(ra_, off, 0, kStream);
                    dst[ps][0] = q[0]; dst[ps][1] = q[1];
                }
                if constexpr (EPI == EPI_KD_DZ) ldst[ps] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rl, prow * 32 + 24 + row_bytes(i, ps * 4, 8, 4), 0, 0));
            }
        };
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if (EPI == EPI_NONE && bias && cok) {
            const uint2 b2 = *(const uint2 *)(bias + colg);
            bv[0] = (float)__builtin_bit_cast(bf16_t, (unsigned short)(b2.x & 0xffff));
            bv[1] = (float)__builtin_bit_cast(bf16_t, (unsigned short)(b2.x >> 16));
            bv[2] = (float)__builtin_bit_cast(bf16_t, (unsigned short)(b2.y & 0xffff));
            bv[3] = (float)__builtin_bit_cast(bf16_t, (unsigned short)(b2.y >> 16));
        }
        auto store4 = [&](const float *v, unsigned co) {
            if (p.c_fp32) {
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = __builtin_bit_cast(unsigned, v[e]);
                __builtin_amdgcn_raw_buffer_store_b128(w, rc, co, 0, kStream);
            } else {
                __builtin_amdgcn_raw_buffer_store_b64(pack4(v), rc, co, 0, kStream);
            }
        };
        const float it = p.kd_inv_t;
        const float it2 = it * 1.4426950408889634f;      // e^{z/T - m} = 2^{z it2 - m log2(e)}: one fused multiply-add feeds exp2
        // Statistics of the wave's 32-row block i: per row, over the wave's 64 columns, max and sum of exponentials of zt/T and
        // zs/T and the cross term sum e^{zt/T - m_t} (zt - zs)/T -> kd_part.  16 rows at a time both tiles go through LDS ([16][64]
        // fp32 each, 16-byte chunk c of row r at c ^ r: no bank conflicts on either side), from where lane l takes chunks l / 16 +
        // 4 k of row l % 16: a row is then 16 values in a lane and four lanes, and each of the five reductions costs two steps per
        // 16 rows.  With a row's four columns per lane as in the other epilogues it is four steps for every four rows, and their
        // moves, address arithmetic and branches were two thirds of this epilogue, which the vector ALU bounds.
        auto kd_statistics = [&](int i, const u32x4 *q) __attribute__((always_inline)) {
            const int r16 = lane & 15, grp = lane >> 4;
            const bool full = n0 + wn * WTN + WTN <= p.N;                          // wave-uniform
            float *stz = stg + 1024;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                wave_sync();
                if constexpr (M16) {
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int row = 4 * fhalf + r;
                            stg[row * 64 + ((j * 16 + frow) ^ (row << 2))] = acc[2 * i + h][j][r];
                        }
                } else {
#pragma unroll
                    for (int j = 0; j < NI; ++j)
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int row = 8 * (r >> 2) + 4 * fhalf + (r & 3);
                            stg[row * 64 + ((j * 32 + frow) ^ (row << 2))] = acc[i][j][8 * h + r];
                        }
                }
#pragma unroll
                for (int ps = 0; ps < 4; ++ps) {
                    const int row = ps * 4 + prow;
                    *(u32x4 *)(stz + row * 64 + (pcol ^ (row << 2))) = q[h * 4 + ps];
                }
                wave_sync();
                float zs[16], zt[16], d[16];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int at = r16 * 64 + (((4 * k + grp) ^ r16) << 2);
                    const float4 a = *(const float4 *)(stg + at), b = *(const float4 *)(stz + at);
                    zs[4 * k] = a.x; zs[4 * k + 1] = a.y; zs[4 * k + 2] = a.z; zs[4 * k + 3] = a.w;
                    zt[4 * k] = b.x; zt[4 * k + 1] = b.y; zt[4 * k + 2] = b.z; zt[4 * k + 3] = b.w;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) d[e] = zt[e] - zs[e];
                if (!full) {                                                       // columns past N take no part
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int c = (e & ~3) + grp;
                        const bool ok = n0 + col_base(c >> 3) + (c & 7) * 4 < p.N;
                        zs[e] = ok ? zs[e] : -INFINITY;
                        zt[e] = ok ? zt[e] : -INFINITY;
                        d[e] = ok ? d[e] : 0.f;
                    }
                }
                float mt = max3(zt[0], zt[1], zt[2]), ms = max3(zs[0], zs[1], zs[2]);
#pragma unroll
                for (int e = 3; e < 15; e += 2) {
                    mt = max3(mt, zt[e], zt[e + 1]);
                    ms = max3(ms, zs[e], zs[e + 1]);
                }
                auto larger = [](float a, float b) { return max3(a, b, b); };
                mt = across_groups(larger(mt, zt[15]), larger) * it;               // T > 0
                ms = across_groups(larger(ms, zs[15]), larger) * it;
                const float mt2 = mt == -INFINITY ? 0.f : mt * 1.4426950408889634f;
                const float ms2 = ms == -INFINITY ? 0.f : ms * 1.4426950408889634f;
                float st = 0.f, ss = 0.f, ac = 0.f;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float et = __builtin_amdgcn_exp2f(__builtin_fmaf(zt[e], it2, -mt2));
                    st += et;
                    ac = __builtin_fmaf(et, d[e], ac);
                    ss += __builtin_amdgcn_exp2f(__builtin_fmaf(zs[e], it2, -ms2));
                }
                auto sum = [](float a, float b) { return a + b; };
                st = across_groups(st, sum);
                ss = across_groups(ss, sum);
                ac = across_groups(ac * it, sum);
                const long rowg = m0 + row_base(i) + h * 16 + r16;
                if (grp == 0 && rowg < p.M && n0 + wn * WTN < p.N) {
                    float *o = p.kd_part + (rowg * p.kd_nparts + (n0 + wn * WTN) / 64) * 8;
                    *(float4 *)o = make_float4(mt, st, ms, ss);
                    o[4] = ac;
                }
            }
        };
        if (has_aux) prefetch(0, aux[0], lsev[0]);
#pragma unroll
        for (int i = 0; i < MI32; ++i) {
            if (has_aux && i + 1 < MI32) prefetch(i + 1, aux[(i + 1) & 1], lsev[(i + 1) & 1]);
            if constexpr (EPI == EPI_KD_STATS) {
                kd_statistics(i, aux[i & 1]);
                continue;
            }
            stage_block(i, [&](float a) { return EPI == EPI_KD_DZ ? a : a * p.alpha; });     // (the KD epilogues have alpha = 1)
#pragma unroll
            for (int ps = 0; ps < 8; ++ps) {
                const int row = ps * 4 + prow;
                const float4 t = *(const float4 *)(stg + row * 64 + (pcol ^ stg_swz(row)));
                const u32x4 q = aux[i & 1][ps];
                const unsigned co = cok ? lane_c + row_bytes(i, ps * 4, p.ldc, esz) : kOob;
                if constexpr (EPI == EPI_NONE) {
                    float v[4] = {t.x + bv[0], t.y + bv[1], t.z + bv[2], t.w + bv[3]};
                    if (aux_res || aux_c) {
                        if (aux4) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) v[e] += __uint_as_float(q[e]);
                        } else {
                            v[0] += (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[0] & 0xffff));
                            v[1] += (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[0] >> 16));
                            v[2] += (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[1] & 0xffff));
                            v[3] += (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[1] >> 16));
                        }
                    }
                    if (aux_res && p.accumulate && p.c_fp32) {        // both a residual and += : C is read in place
                        const u32x4 c4 = __builtin_amdgcn_raw_buffer_load_b128(rc, co, 0, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += __uint_as_float(c4[e]);
                    }
                    store4(v, co);
                } else if constexpr (EPI == EPI_SWIGLU_BWD) {
                    // da is rounded to the storage type first (it is what a separate activation kernel would read back)
                    const float da[4] = {(float)(bf16_t)t.x, (float)(bf16_t)t.y, (float)(bf16_t)t.z, (float)(bf16_t)t.w};
                    float dg[4], du[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float gg = (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[e >> 1] >> (16 * (e & 1))));
                        const float uu = (float)__builtin_bit_cast(bf16_t, (unsigned short)(q[2 + (e >> 1)] >> (16 * (e & 1))));
                        swiglu_derivative(da[e], gg, uu, &dg[e], &du[e]);
                    }
                    store4(dg, co);
                    store4(du, cok ? co + (unsigned)p.sg_f * 2 : kOob);
                } else {
                    // the tile holds student logits zs; q = teacher logits zt of the same elements
                    const float zs[4] = {t.x, t.y, t.z, t.w};
                    float zt[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) zt[e] = __uint_as_float(q[e]);
                    // dz = coef * (exp(zs/T - lse_s) - exp(zt/T - lse_t)) -> C (storage dtype)
                    const float lt2 = lsev[i & 1][ps].x * 1.4426950408889634f, ls2 = lsev[i & 1][ps].y * 1.4426950408889634f;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        v[e] = p.kd_coef * (__builtin_amdgcn_exp2f(__builtin_fmaf(zs[e], it2, -ls2)) -
                                            __builtin_amdgcn_exp2f(__builtin_fmaf(zt[e], it2, -lt2)));
                    store4(v, co);
                }
            }
        }
        return;
    }
    // scalar epilogue: split-K atomics and shapes whose rows are not 4-element aligned
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int col = n0 + (M16 ? col_base(j >> 1) + (j & 1) * 16 : col_base(j)) + frow;
        const bool cok = col < p.N;
        const float bv = (bias && cok) ? (float)bias[col] : 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int r = 0; r < ACC_N; ++r) {
                const int row = m0 + (M16 ? row_base(i >> 1) + (i & 1) * 16 : row_base(i)) + (M16 ? 4 * fhalf + r : 8 * (r >> 2) + 4 * fhalf + (r & 3));
                float v = acc[i][j][r] * p.alpha + bv;
                if (p.residual) {
                    const unsigned ro = cok ? (unsigned)(((long)row * p.ldr + col) * rsz) : kOob;
                    if (p.res_fp32) v += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rr, ro, 0, 0));
                    else v += (float)__builtin_bit_cast(bf16_t, __builtin_amdgcn_raw_buffer_load_b16(rr, ro, 0, 0));
                }
                const unsigned co = cok ? (unsigned)(((long)row * p.ldc + col) * esz) : kOob;
                if (p.c_fp32) {
                    if (p.atomic) {
                        if (cok && row < p.M) unsafeAtomicAdd((float *)p.C + (long)row * p.ldc + col, v);
                    } else {
                        if (p.accumulate) v += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rc, co, 0, 0));
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rc, co, 0, 0);
                    }
                } else {
                    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, (bf16_t)v), rc, co, 0, 0);
                }
            }
            // keep the scheduler from pulling every accumulator out of the AGPRs at once
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// M16 selects v_mfma_f32_16x16x32_bf16 (16-row fragments, two k-steps of 32 per K tile) instead of
// v_mfma_f32_32x32x16_bf16 (32-row fragments, four k-steps of 16): the same LDS traffic and the same number of
// accumulator registers, but on operands with realistic bit activity the chip sustains a higher clock on it.
// NST = LDS stages: two (a K tile is requested one tile time before its first use, which is what the big tile's LDS
// allows) or a deeper ring for grids that leave CUs with one workgroup, where a tile time is shorter than the latency
// of a load (see kTiles).
// The attribute only adds to what the launch bounds say for the two-stage 128 x 128 kernel with the dz epilogue: left to
// itself the compiler gives it 276 registers, which leave a CU with one workgroup, instead of 173 (dz at
// 3629 x 4480 x 1536: 70.9 us; 74.2 on v_mfma_f32_32x32x16, which needs fewer).
constexpr int fast_waves_per_simd(int bm, int waves, int epi, int nst) { return waves == 8 || (bm == 128 && nst == 2 && epi == EPI_KD_DZ) ? 2 : 1; }
template <int BM, int BN, int NST> struct FastLds {
    bf16_t *a[4], *b[4];
};
// The kernel's LDS: separate objects (not one carved array), because the compiler orders LDS reads against in-flight
// direct-to-LDS loads by alias analysis, and can only tell the buffer being filled from the buffer being read when
// they are distinct objects
#define MS_FAST_LDS(BM, BN, NST)                                                                                       \
    static_assert(NST >= 2 && NST <= 4, "ring of 2..4 stages");                                                        \
    __shared__ __align__(16) bf16_t As0[BM * BK], As1[BM * BK], As2[NST > 2 ? BM * BK : 8], As3[NST > 3 ? BM * BK : 8]; \
    __shared__ __align__(16) bf16_t Bs0[BN * BK], Bs1[BN * BK], Bs2[NST > 2 ? BN * BK : 8], Bs3[NST > 3 ? BN * BK : 8]; \
    const FastLds<BM, BN, NST> lds = {{As0, As1, As2, As3}, {Bs0, Bs1, Bs2, Bs3}}

// Workgroup b of the nb that compute one product (of one K split)
template <int BM, int BN, int WM, int WN, bool TA, bool TB, int EPI, bool M16, int NST>
__device__ __forceinline__ void gemm_fast_body(const GemmParams &p, const FastLds<BM, BN, NST> &lds, int b, int nb, int split) {
    constexpr int FR = M16 ? 16 : 32;                         // rows of an MFMA fragment / accumulator block
    constexpr int KSTEP = M16 ? 32 : 16, KS = BK / KSTEP;     // contraction depth of an MFMA, k-steps per K tile
    constexpr int WTM = BM / WM, WTN = BN / WN, MI = WTM / FR, NI = WTN / FR;
    constexpr int MI32 = WTM / 32, NI32 = WTN / 32;           // the epilogues work on 32-row blocks
    using acc_t = std::conditional_t<M16, f32x4, f32x16>;
    constexpr int ACC_N = M16 ? 4 : 16;
    bf16_t *const As0 = lds.a[0], *const As1 = lds.a[1], *const Bs0 = lds.b[0], *const Bs1 = lds.b[1];
    bf16_t *const Ast[4] = {lds.a[0], lds.a[1], lds.a[2], lds.a[3]}, *const Bst[4] = {lds.b[0], lds.b[1], lds.b[2], lds.b[3]};

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keep it in a scalar register
    const int wm = wave / WN, wn = wave % WN;
    int pid;
    {
        const int per = nb >> 3, rem = nb & 7, x = b & 7, q = b >> 3;
        pid = x * per + (x < rem ? x : rem) + q;
    }
    constexpr int GM = BM >= 256 ? 4 : 8;
    const int group = pid / (GM * p.tiles_n);
    const int first_m = group * GM;
    const int gsize = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
    const int tm = first_m + (pid % (GM * p.tiles_n)) % gsize;
    const int tn = (pid % (GM * p.tiles_n)) / gsize;
    const int m0 = tm * BM, n0 = tn * BN;

    const int kt_begin = split * p.k_tiles_per_split;
    int kt_end = kt_begin + p.k_tiles_per_split;
    const int kt_total = (p.K + BK - 1) / BK;
    if (kt_end > kt_total) kt_end = kt_total;
    const int nk = kt_end - kt_begin;
    if (nk <= 0) return;

    const bf16_t *A = (const bf16_t *)p.A, *B = (const bf16_t *)p.B;
    std::conditional_t<TA, RowTileStager<BM, WM * WN>, DmaStager<BM, WM * WN>> da;
    std::conditional_t<EPI == EPI_SWIGLU, GateUpStager<BN, WM * WN>,
                       std::conditional_t<TB, RowTileStager<BN, WM * WN>, DmaStager<BN, WM * WN>>> db;
    // descriptor ranges: rows x leading dimension of the matrix as stored ([M or N][K], or [K][M or N])
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(A, TA ? ((long)(p.K - 1) * p.lda + p.M) * 2 : ((long)(p.M - 1) * p.lda + p.K) * 2);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(B, TB ? ((long)(p.K - 1) * p.ldb + p.N) * 2
                                                      : ((long)((EPI == EPI_SWIGLU ? 2 * p.sg_f : p.N) - 1) * p.ldb + p.K) * 2);
    if constexpr (TA) da.init(p.lda, m0, wave, lane); else da.init(p.lda, m0, lane);
    if constexpr (EPI == EPI_SWIGLU) db.init(p.ldb, n0 / 2, p.sg_f, lane);   // tile tn covers output columns tn * BN/2 ..
    else if constexpr (TB) db.init(p.ldb, n0, wave, lane);
    else db.init(p.ldb, n0, lane);

    acc_t acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < ACC_N; ++r) acc[i][j][r] = 0.f;

    // Start moving K tile kt towards LDS; a tile past the end of this workgroup's K range arrives as zeros.
    // An operand stored K-major ([K][M]) is loaded as a "row tile" (64 k-rows x BM columns) and read back
    // through the transposing LDS load, so every layout goes global -> LDS without staging registers.
    auto fetch = [&](int kt, bf16_t *as, bf16_t *bs) {
        const bool valid = kt < nk;
        const unsigned inv = valid ? 0u : kOob;
        const int k0 = (kt_begin + kt) * BK;
        da.issue(ra, as, k0, wave, inv);
        db.issue(rb, bs, k0, wave, inv);
    };
    // lane -> (fragment row, k-group of 8 consecutive k): 32 rows x 2 groups, or 16 rows x 4 groups
    const int frow = lane & (FR - 1), fhalf = lane / FR;
    // 32-row block i (32-column block j) of this wave within the tile.  For a K-major operand the blocks
    // of a wave are spread one per 64-wide LDS sub-tile pair so that all of them share one LDS address
    // register (constant offsets); for a K-contiguous operand they are adjacent for the same reason.
    auto row_base = [&](int i) { return TA ? i * (32 * WM) + wm * 32 : wm * WTM + i * 32; };
    auto col_base = [&](int j) { return TB ? j * (32 * WN) + wn * 32 : wn * WTN + j * 32; };
    // the same for fragment blocks (16-row blocks are the halves of the 32-row blocks)
    auto frow_base = [&](int i) { return M16 ? row_base(i >> 1) + (i & 1) * 16 : row_base(i); };
    auto fcol_base = [&](int j) { return M16 ? col_base(j >> 1) + (j & 1) * 16 : col_base(j); };
    // Operand fragments are double-buffered in registers: the LDS reads of k-step kk+1 are issued between
    // the MFMAs of k-step kk.
    bf16x8 af[2][MI], bfr[2][NI];
    std::conditional_t<M16, TrFragAddr16, TrFragAddr> tra, trb, trb1;
    static_assert((WM == 2 || (WM == 4 && BM == 128 && M16)) && (WN >= 2 || M16), "K-major blocks are spread over sub-tile pairs");
    if constexpr (TA) tra.init(wm, lane);     // block i of the wave: columns i * 32 * WM + wm * 32 of the row tile
    if constexpr (TB) trb.init(wn, lane);
    if constexpr (TB && WN == 1) trb1.init(1, lane);   // one wave column: its two 32-column blocks are the halves of a sub-tile
    KFragAddr16 ka, kb;
    if constexpr (M16 && !TA) ka.init(wm * WTM, lane);
    if constexpr (M16 && !TB) kb.init(wn * WTN, lane);
    auto load_a = [&](const bf16_t *as, int kk, int slot, int i) {
        if constexpr (TA && M16) af[slot][i] = tra.frag(as, kk, i, (i >> 1) * (32 * WM / 64) * 4096);
        else if constexpr (TA) af[slot][i] = tra.frag(as, kk, i * (32 * WM / 64) * 4096);
        else if constexpr (M16) af[slot][i] = ka.frag(as, kk, i);
        else af[slot][i] = *(const bf16x8 *)(as + lds_off(frow_base(i) + frow, kk * (KSTEP / 8) + fhalf));
    };
    auto load_b = [&](const bf16_t *bs, int kk, int slot, int j) {
        if constexpr (TB && WN == 1) bfr[slot][j] = (j >> 1 ? trb1 : trb).frag(bs, kk, j, 0);
        else if constexpr (TB && M16) bfr[slot][j] = trb.frag(bs, kk, j, (j >> 1) * (32 * WN / 64) * 4096);
        else if constexpr (TB) bfr[slot][j] = trb.frag(bs, kk, j * (32 * WN / 64) * 4096);
        else if constexpr (M16) bfr[slot][j] = kb.frag(bs, kk, j);
        else bfr[slot][j] = *(const bf16x8 *)(bs + lds_off(fcol_base(j) + frow, kk * (KSTEP / 8) + fhalf));
    };
    auto load_frags = [&](const bf16_t *as, const bf16_t *bs, int kk, int slot) {
#pragma unroll
        for (int i = 0; i < MI; ++i) load_a(as, kk, slot, i);
#pragma unroll
        for (int j = 0; j < NI; ++j) load_b(bs, kk, slot, j);
    };
    auto mfma_step = [&](int slot) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if constexpr (M16) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[slot][i], bfr[slot][j], acc[i][j], 0, 0, 0);
                else acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[slot][i], bfr[slot][j], acc[i][j], 0, 0, 0);
            }
    };
    constexpr int LDS_READS = (TA ? 2 : 1) * MI + (TB ? 2 : 1) * NI, MFMAS = MI * NI;
    // One k-step: the MFMAs on fragment slot `cur`, with the reads of the next k-step's fragments (tile la / lb,
    // k-step lkk) between them.  With 32-row fragments all reads go in front (one per MFMA).  With 16-row
    // fragments there are twice as many fragment registers per k-step, so the A fragment of row block i is
    // read right after the MFMAs of row block i, into the registers those MFMAs have just released; only the
    // B fragments are held twice.
    auto step = [&](auto cur_c, auto fetch_c, const bf16_t *la, const bf16_t *lb, int lkk) __attribute__((always_inline)) {
        constexpr int cur = decltype(cur_c)::value;          // compile-time: the fragment arrays must stay registers
        constexpr int VM = decltype(fetch_c)::value ? (BM + BN) / 8 / (WM * WN) : 0;   // loads of a fetch issued just before
        if constexpr (M16) {
            constexpr int BPB = (NI + MI - 1) / MI;          // B fragments read behind each row block
            // (columns alternate in direction, so that neighbouring MFMAs differ in one operand: 0.3-0.5 % at the same power)
#pragma unroll
            for (int i = 0; i < MI; ++i) {
#pragma unroll
                for (int jj = 0; jj < NI; ++jj) {
                    const int j = (i & 1) ? NI - 1 - jj : jj;
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[cur][i], bfr[cur][j], acc[i][j], 0, 0, 0);
                }
                load_a(la, lkk, cur ^ 1, i);
#pragma unroll
                for (int j = i * BPB; j < NI && j < (i + 1) * BPB; ++j) load_b(lb, lkk, cur ^ 1, j);
            }
            sched_mfma_then_reads<NI, (TA ? 2 : 1), (TB ? 2 : 1), VM>(std::make_integer_sequence<int, MI>{});
        } else {
            load_frags(la, lb, lkk, cur ^ 1);
            mfma_step(cur);
            interleave_reads_with_mfma<LDS_READS, MFMAS>();
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // One K tile: steps 0..2 read the next step's fragments from the same tile; before the last step the
    // next tile has landed (own loads: vmcnt(0); the other waves': barrier) and everybody is done reading
    // this one, so its buffers are handed to the tile after next and the last step reads the first
    // fragments of the next tile.  One barrier per tile.
    auto tile = [&](const bf16_t *ca, const bf16_t *cb, const bf16_t *na, const bf16_t *nb, bf16_t *fa, bf16_t *fb,
                    int kt_fetch) __attribute__((always_inline)) {
        using S0 = std::integral_constant<int, 0>;
        using S1 = std::integral_constant<int, 1>;
        static_assert(KS == 2 || KS == 4, "k-steps per K tile");
        step(S0{}, S0{}, ca, cb, 1);
        if constexpr (KS == 4) {
            step(S1{}, S0{}, ca, cb, 2);
            step(S0{}, S0{}, ca, cb, 3);
        }
        if constexpr (NST == 2) {
            dma_publish_barrier();
        } else {
            // own loads of the next tile have landed; the NST - 2 younger tiles' loads stay in flight
            wait_vmcnt_lgkm0<(NST - 2) * ((BM + BN) / 8 / (WM * WN))>();
            lds_barrier();
        }
        fetch(kt_fetch, fa, fb);
        step(S1{}, S1{}, na, nb, 0);
    };

    if constexpr (NST == 2) {
        fetch(0, As0, Bs0);
        dma_publish_barrier();
        fetch(1, As1, Bs1);
    } else {
#pragma unroll
        for (int k = 0; k < NST; ++k) fetch(k, Ast[k], Bst[k]);
        wait_vmcnt_lgkm0<(NST - 1) * ((BM + BN) / 8 / (WM * WN))>();
        lds_barrier();
    }
    load_frags(As0, Bs0, 0, 0);
    // NST K tiles per trip so that each part names its LDS buffers statically; the tile count is
    // rounded up with tiles of zeros (a single loop exit keeps the accumulators in place)
    for (int kt = 0; kt < nk; kt += NST) {
#pragma unroll
        for (int k = 0; k < NST; ++k)
            tile(Ast[k], Bst[k], Ast[(k + 1) % NST], Bst[(k + 1) % NST], Ast[k], Bst[k], kt + k + NST);
    }
    dma_publish_barrier();   // the (all-zero) tiles still in flight must land before the epilogue reuses LDS

    // waves share the idle operand buffers, 8 KB each: WPA of them fit into one A buffer
    constexpr int WPA = BM / 64;
    const int sq = wave / WPA;
    float *stg = (float *)(sq == 0 ? As0 : sq == 1 ? As1 : sq == 2 ? Bs0 : Bs1) + (wave % WPA) * 2048;
    gemm_epilogue<EPI, M16, TA, TB>(p, acc, stg, m0, n0, wn, lane, row_base, col_base);
}

template <int BM, int BN, int WM, int WN, bool TA, bool TB, int EPI = EPI_NONE, bool M16 = false, int NST = 2>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(fast_waves_per_simd(BM, WM * WN, EPI, NST)))) void gemm_bf16_fast_kernel(GemmParams p) {
    MS_FAST_LDS(BM, BN, NST);
    gemm_fast_body<BM, BN, WM, WN, TA, TB, EPI, M16, NST>(p, lds, blockIdx.x, gridDim.x, blockIdx.y);
}

// Both products of a linear layer's backward pass, which share dy and nothing else, in one grid: the input gradient's
// workgroups (pd: dx = dy W, K-major B) and the weight gradient's (pw: dW += dy^T x, both K-major, `splits` parts of K).
// One product of a small micro-batch leaves CUs idle (100-250 workgroups) and any product has a last round; together they
// leave one.  The product with the longer workgroups comes first (see ms_choose_pair).  One MI355X, us, backward GEMMs of a
// layer apart -> together: c2 student at 2053 tokens 176 -> 146, encoder at 1031 tokens 175 -> 130; the fp32 form (five pairs in
// the c1 step) takes the step from 271 to 242.
// EPI = EPI_SWIGLU_BWD: x is the output of a SwiGLU; the input gradient goes through its derivative in the epilogue and leaves as
// [dgate | dup].  A kernel of its own read the 2 f pre-activations too, but also da, which the product had written (c5 student
// layer at 32768 tokens 532 us, 5.5 TB/s): 13.16 -> 13.09 ms, c2 student layer at 2053 tokens 438 -> 434 us; the epilogue's
// bursts are not behind MFMAs, which eats most of the bytes saved.
template <int BM, int BN, int WM, int WN, int NST, int EPI = EPI_NONE>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(fast_waves_per_simd(BM, WM * WN, EPI_NONE, NST)))) void gemm_bf16_pair_kernel(GemmParams pd, GemmParams pw, int nd, int nw, int wgrad_first) {
    MS_FAST_LDS(BM, BN, NST);
    const int b = blockIdx.x, total_w = gridDim.x - nd;
    if (wgrad_first ? b < total_w : b >= nd) {
        const int bw = wgrad_first ? b : b - nd;
        gemm_fast_body<BM, BN, WM, WN, true, true, EPI_NONE, true, NST>(pw, lds, bw % nw, nw, bw / nw);
    } else {
        gemm_fast_body<BM, BN, WM, WN, false, true, EPI, true, NST>(pd, lds, wgrad_first ? b - total_w : b, nd, 0);
    }
}

// The 256 x 256 tile with two wave groups that take turns on the matrix cores; K-contiguous operands only.
//   * Waves 0..3 and 4..7 (one of each per SIMD) run the same program half a phase apart: while one group issues the 16
//     MFMAs of a quarter of its wave tile (64 x 32, both k-steps), the other reads its next operand fragments from LDS
//     and requests the next half tile.  Two barriers per phase keep them in step; the one extra barrier that group 1
//     takes before the loop and group 0 after it is the offset.
//   * An operand tile is two halves of 128 rows with an LDS slot each and two stages: eight 16 KB slots.  Per K tile the
//     phases read A0 -> Bs -> A1 -> Bf of the next tile, where Bf / Bs are the B half used first / second; they swap roles
//     every tile, so that the quarters (A0 Bf)(A0 Bs)(A1 Bs)(A1 Bf) change one operand at a time.  Two of the eight
//     fragments of an A half are read in the phase before its own, so that every phase has six reads.  A phase requests
//     the half of tile t + 2 that goes into the slot whose last read was in the phase before: every half is requested at
//     least six phases (1.5 K tiles) before it is read, instead of one K tile in gemm_bf16_fast_kernel, and the wait
//     is for all but the 10 youngest loads of a wave, never for all of them.
//   * Same tile order, MFMA and order of K as the other tiles: bit-identical results.
// It is the 256 x 256 tile of K-contiguous operands for every shape and epilogue.  Against gemm_bf16_fast_kernel<256, 256> with
// operands that have left the caches, as they have when a step comes round to them again, it was faster on 108 of 110 shapes
// (M = 1500 .. 32768, 22 outputs; the other two within 0.6 %), us: 8192 x 8192 x 4096 with fp32 output 437 -> 391,
// 8192 x 1280 x 5120 135 -> 114, 4096 x 3072 x 2048 51.5 -> 44.5, 32768 x 4096 x 11008 2199 -> 2010, 32768 x 1536 x 1536
// 174 -> 170; the distillation head at 8192 tokens, V = 151936, H = 4096 / 2048 35.4 -> 32.8 ms.  On operands that stay in
// the 256 MB Infinity Cache the two are equal (8192^3 704 / 707) up to 4 % on a short K (32768 x 2048 x 1536 154 / 160).
// For K-major operands (twice the LDS reads) it was built too: 6-12 % slower warm, 2-8 % slower cold wherever the grid fills
// the chip (32768 x 8960 x 1536 736 -> 788), and in smaller grids behind the other tiles.
// B half g holds the rows 64 w + 32 g .. + 31 of every wave column w (a wave's 64 columns stay adjacent); for SwiGLU
// g = 0 gate rows, g = 1 up rows.
struct HalfStager {
    unsigned rowoff, ld2;
    int x;
    __device__ __forceinline__ void init(long ld, int row0, int lane) {
        rowoff = (unsigned)(((long)(row0 + (lane >> 3)) * ld) * 2);
        ld2 = (unsigned)(ld * 2);
        x = (lane & 7) ^ swz_row(lane >> 3);
    }
    // eight matrix rows from row0 + row into 8-row group lg of the half's slot (both wave-uniform)
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, bf16_t *slot, int row, int lg, int k0, unsigned inv) const {
        const unsigned voff = (rowoff + (unsigned)row * ld2 + ((x ^ swz_row(8 * lg)) << 4)) | inv;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(slot + lg * 8 * BK), 16, voff, k0 * 2, 0, 0);
    }
};
struct PpLds {
    bf16_t *a[2][2], *b[2][2];                          // [stage][half]
};
#define MS_PP_LDS                                                                                                     \
    constexpr int HS = 128 * BK; /* elements of a half tile */                                                        \
    __shared__ __align__(16) bf16_t A00[HS], A01[HS], A10[HS], A11[HS], B00[HS], B01[HS], B10[HS], B11[HS];           \
    const PpLds lds = {{{A00, A01}, {A10, A11}}, {{B00, B01}, {B10, B11}}}
// Workgroup b of the nb that compute one product (of one K split)
template <int EPI>
__device__ __forceinline__ void gemm_pp_body(const GemmParams &p, const PpLds &lds, int b, int nb, int split) {
    bf16_t *const A00 = lds.a[0][0], *const A01 = lds.a[0][1], *const A10 = lds.a[1][0], *const A11 = lds.a[1][1];
    bf16_t *const B00 = lds.b[0][0], *const B01 = lds.b[0][1], *const B10 = lds.b[1][0], *const B11 = lds.b[1][1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;            // wm = wave group
    int pid;
    {
        const int per = nb >> 3, rem = nb & 7, x = b & 7, q = b >> 3;
        pid = x * per + (x < rem ? x : rem) + q;
    }
    constexpr int GM = 4;
    const int group = pid / (GM * p.tiles_n);
    const int first_m = group * GM;
    const int gsize = (p.tiles_m - first_m) < GM ? (p.tiles_m - first_m) : GM;
    const int tm = first_m + (pid % (GM * p.tiles_n)) % gsize;
    const int tn = (pid % (GM * p.tiles_n)) / gsize;
    const int m0 = tm * 256, n0 = tn * 256;

    const int kt_begin = split * p.k_tiles_per_split;
    int kt_end = kt_begin + p.k_tiles_per_split;
    const int kt_total = (p.K + BK - 1) / BK;
    if (kt_end > kt_total) kt_end = kt_total;
    const int nk = kt_end - kt_begin;
    if (nk <= 0) return;

    const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.A, ((long)(p.M - 1) * p.lda + p.K) * 2);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.B, ((long)((EPI == EPI_SWIGLU ? 2 * p.sg_f : p.N) - 1) * p.ldb + p.K) * 2);
    HalfStager da, db;
    da.init(p.lda, m0, lane);
    db.init(p.ldb, EPI == EPI_SWIGLU ? n0 / 2 : n0, lane);
    // request half h of K tile kt (two loads per wave; a tile past the end arrives as zeros)
    auto fetch_a = [&](int kt, int h, bf16_t *slot) __attribute__((always_inline)) {
        const unsigned inv = kt < nk ? 0u : kOob;
        const int k0 = (kt_begin + kt) * BK;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int g = wave * 2 + i;
            da.load(ra, slot, h * 128 + g * 8, g, k0, inv);
        }
    };
    auto fetch_b = [&](int kt, int h, bf16_t *slot) __attribute__((always_inline)) {
        const unsigned inv = kt < nk ? 0u : kOob;
        const int k0 = (kt_begin + kt) * BK;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int g = wave * 2 + i;
            if constexpr (EPI == EPI_SWIGLU) db.load(rb, slot, h * p.sg_f + g * 8, g, k0, inv);
            else db.load(rb, slot, (g >> 2) * 64 + h * 32 + (g & 3) * 8, g, k0, inv);
        }
    };

    f32x4 acc[8][4];                                    // [16-row block: 4 h + b][16-column block: 2 g + c]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // A: [block][k-step] of the current half, its first two fragments apart (ax[half]); B: [half][block][k-step]
    bf16x8 af[4][2], ax[2][2], bfr[2][2][2];
    KFragAddr16 ka, kb;
    ka.init(wm * 64, lane);
    kb.init(wn * 32, lane);
    auto read_a_first = [&](auto half, const bf16_t *slot) __attribute__((always_inline)) {
        constexpr int h = decltype(half)::value;
        ax[h][0] = ka.frag(slot, 0, 0);
        ax[h][1] = ka.frag(slot, 0, 1);
    };
    auto read_a_rest = [&](const bf16_t *slot) __attribute__((always_inline)) {
        af[2][0] = ka.frag(slot, 0, 2);
        af[3][0] = ka.frag(slot, 0, 3);
#pragma unroll
        for (int b = 0; b < 4; ++b) af[b][1] = ka.frag(slot, 1, b);
    };
    auto read_b = [&](auto half, const bf16_t *slot) __attribute__((always_inline)) {
        constexpr int g = decltype(half)::value;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int c = 0; c < 2; ++c) bfr[g][c][kk] = kb.frag(slot, kk, c);
    };
    // End of a phase's first half: the half tile that the next phase reads has landed (own loads), this phase's reads are
    // done; then the quarter's MFMAs between two barriers.
    auto turn = [&](auto ah, auto bh) __attribute__((always_inline)) {
        constexpr int h = decltype(ah)::value, g = decltype(bh)::value;
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt_lgkm0<10>();
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    acc[4 * h + b][2 * g + c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk == 0 && b < 2 ? ax[h][b] : af[b][kk], bfr[g][c][kk], acc[4 * h + b][2 * g + c], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    // K tile kt in stage slots (a0, a1, f = its first B half F, s = its second B half); nb: the slot of the next tile's first
    // B half, which is half 1 - F
    auto tile = [&](int kt, auto F, bf16_t *a0, bf16_t *a1, bf16_t *f, bf16_t *s, const bf16_t *nb, const bf16_t *na) __attribute__((always_inline)) {
        constexpr int fh = decltype(F)::value;
        using FH = std::integral_constant<int, fh>;
        using SH = std::integral_constant<int, 1 - fh>;
        read_a_rest(a0);
        fetch_b(kt + 2, fh, f);
        turn(I0{}, FH{});
        read_b(SH{}, s);
        read_a_first(I1{}, a1);
        fetch_a(kt + 2, 0, a0);
        turn(I0{}, SH{});
        read_a_rest(a1);
        fetch_b(kt + 2, 1 - fh, s);
        turn(I1{}, SH{});
        // fragments of half F are still needed by this quarter; the next tile's first half goes to the other set
        read_b(SH{}, nb);
        read_a_first(I0{}, na);
        fetch_a(kt + 2, 1, a1);
        turn(I1{}, FH{});
    };
    // in the order in which the loop would have requested them
    fetch_b(0, 0, B00); fetch_a(0, 0, A00); fetch_b(0, 1, B01); fetch_a(0, 1, A01);
    fetch_b(1, 1, B11); fetch_a(1, 0, A10); fetch_b(1, 0, B10); fetch_a(1, 1, A11);
    wait_vmcnt_lgkm0<12>();
    lds_barrier();
    read_b(I0{}, B00);
    read_a_first(I0{}, A00);
    wait_vmcnt_lgkm0<10>();
    lds_barrier();
    if (wm == 1) lds_barrier();
    for (int kt = 0; kt < nk; kt += 2) {                // an odd count is rounded up with a tile of zeros
        tile(kt, I0{}, A00, A01, B00, B01, B11, A10);
        tile(kt + 1, I1{}, A10, A11, B11, B10, B00, A00);
    }
    if (wm == 0) lds_barrier();
    dma_publish_barrier();   // the (all-zero) half tiles still in flight must land before the epilogue reuses LDS
    auto row_base = [&](int i) { return (i >> 1) * 128 + wm * 64 + (i & 1) * 32; };
    auto col_base = [&](int j) { return wn * 64 + j * 32; };
    const int sq = wave >> 1;
    float *stg = (float *)(sq == 0 ? A00 : sq == 1 ? A01 : sq == 2 ? A10 : A11) + (wave & 1) * 2048;
    gemm_epilogue<EPI, true, false, false>(p, acc, stg, m0, n0, wn, lane, row_base, col_base);
}
template <int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_pp_kernel(GemmParams p) {
    MS_PP_LDS;
    gemm_pp_body<EPI>(p, lds, blockIdx.x, gridDim.x, blockIdx.y);
}

// A chunk's student logits with a KD epilogue (ps, EPI) and another chunk's teacher logits (pt) in one grid.  The student's
// epilogue reads the stored teacher logits, 256 KB per 256 x 256 tile; in a launch of its own all CUs come to it together
// and wait for HBM with idle matrix cores.  Here the two kinds of tiles take turns, a round of the chip each (`run`; the last rounds
// of both together), the kind with the longer workgroups first (`first`, 1: student): their
// times differ, so that one kind's epilogues come to run beside the other's main loops, and one last round is left instead of
// two (see ms_choose_two for what it gains).  The order is the one that ms_choose_two reckons with.  With runs of 256 also where a round is
// 512 workgroups, part of the longer ones waited for the shorter (64 x 128 tiles, 300 tokens, H = 4096 / 1536, chunks of 8192, loss
// only, V = 49152: 416 us, two launches 339).  In runs of 8 or 64 the two products' operand panels compete for the L2s from the start
// (256 x 256 tiles, 8192 tokens, V = 151936: 33.6 .. 34.0 ms; apart 32.98, in runs of 256 32.75).
struct TwoSlot { int student, index; };
__device__ __forceinline__ TwoSlot two_slot(int b, int nt, int ns, int run, int first) {
    const int both = (nt < ns ? nt : ns) / run * run;
    if (b < 2 * both) return {((b / run) & 1) ^ first, b / (2 * run) * run + b % run};
    const int r = b - 2 * both, more = (first ? ns : nt) - both;
    return r < more ? TwoSlot{first, both + r} : TwoSlot{first ^ 1, both + r - more};
}
template <int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_bf16_pp_two_kernel(GemmParams pt, GemmParams ps, int nt, int ns, int run, int first) {
    MS_PP_LDS;
    const TwoSlot t = two_slot(blockIdx.x, nt, ns, run, first);
    if (t.student) gemm_pp_body<EPI>(ps, lds, t.index, ns, 0);
    else gemm_pp_body<EPI_NONE>(pt, lds, t.index, nt, 0);
}
template <int BM, int BN, int WM, int WN, int NST, int EPI>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(fast_waves_per_simd(BM, WM * WN, EPI, NST)))) void gemm_bf16_two_kernel(GemmParams pt, GemmParams ps, int nt, int ns, int run, int first) {
    MS_FAST_LDS(BM, BN, NST);
    const TwoSlot t = two_slot(blockIdx.x, nt, ns, run, first);
    if (t.student) gemm_fast_body<BM, BN, WM, WN, false, false, EPI, true, NST>(ps, lds, t.index, ns, 0);
    else gemm_fast_body<BM, BN, WM, WN, false, false, EPI_NONE, true, NST>(pt, lds, t.index, nt, 0);
}

// ------------------------------------------------------------------ fp32
struct GemmF32Params {
    const float *A, *B;
    float *C;
    const float *bias, *residual;
    long lda, ldb, ldc, ldr;
    int M, N, K, tiles_n;
    float alpha;
    int accumulate;
    const float *sw_up;      // SwiGLU backward: pre-activations [M, 2 N]; the product is da and C = [dgate | dup]
};

// One operand's fragments for v_mfma_f32_16x16x4_f32: two 16-row blocks x 16 k.  Lane = (row lane % 16, k-group
// lane / 16); component c of a block's four values is k = k0 + 4 (lane / 16) + c, so four MFMAs (one per component)
// contract 16 k.  TRANS: the operand is stored [K][rows].  Rows and k past the end read as zero.  FAST: loads through a
// buffer descriptor whose range check returns the zeros, so that nothing but the MFMAs waits for a load.
template <bool TRANS, bool FAST> struct F32Frag {
    float v[2][4];
    __device__ __forceinline__ void load(const float *P, __amdgpu_buffer_rsrc_t rs, long ld, int row0, int rows, int k0, int K, int lane) {
        const int k = k0 + 4 * (lane >> 4);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int r = row0 + 16 * b + (lane & 15);
            if constexpr (FAST && !TRANS) {
                const unsigned off = r < rows && k < K ? (unsigned)((long)r * ld + k) * 4u : kOob;
                const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[b][c] = __uint_as_float(t[c]);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const bool ok = r < rows && k + c < K;
                    const long at = TRANS ? (long)(k + c) * ld + r : (long)r * ld + k + c;
                    if constexpr (FAST) v[b][c] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, ok ? (unsigned)at * 4u : kOob, 0, 0));
                    else v[b][c] = ok ? P[at] : 0.f;
                }
            }
        }
    }
};

// fp32 GEMM for the small matrices of the fp32 workload (a few hundred rows): latency is what it costs, not flops.  A
// workgroup computes a 32 x 32 tile; its four waves take every fourth 16-deep slice of K each (a quarter of the serial
// chain) and add up through LDS.  Fragments come straight from global memory (the operands are a few hundred KB and
// stay in L2), three slices ahead of the MFMAs that use them; what the epilogue reads is requested before the main loop.
// The 64 x 64 FMA kernel that this replaces took 1.3 us per 16 k (10..80 workgroups, a load latency and two barriers
// each): 47 us per launch on average in the c1 step, against 6.9 us now.
// FAST needs 16-byte aligned K-contiguous rows with K % 4 == 0 and operands below 4 GB; the other form covers the rest.
// (The first slices are requested before the loop, also where K = 0 leaves it nothing to do: the range is then empty.)
template <bool TA, bool TB, bool FAST>
__device__ __forceinline__ void gemm_f32_body(const GemmF32Params &p, float (&part)[4][32][33], int b_) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m0 = b_ / p.tiles_n * 32, n0 = b_ % p.tiles_n * 32;
    const int slices = (p.K + 15) / 16, mine = slices > wave ? (slices - wave + 3) / 4 : 0;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.A, FAST ? ms_matrix_extent(TA ? p.K : p.M, TA ? p.M : p.K, p.lda) * 4 : 0);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.B, FAST ? ms_matrix_extent(TB ? p.K : p.N, TB ? p.N : p.K, p.ldb) * 4 : 0);
    F32Frag<TA, FAST> a[4];
    F32Frag<TB, FAST> b[4];
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int slot, int s) __attribute__((always_inline)) {
        const int k0 = (wave + 4 * s) * 16;
        a[slot].load(p.A, ra, p.lda, m0, p.M, k0, p.K, lane);
        b[slot].load(p.B, rb, p.ldb, n0, p.N, k0, p.K, lane);
    };
    load(0, 0);
    load(1, 1);
    load(2, 2);
    // this thread's four output elements: rows threadIdx.x / 32 + 8 e, column threadIdx.x % 32
    const int rr = threadIdx.x >> 5, cc = threadIdx.x & 31, col = n0 + cc;
    float add[4] = {0.f, 0.f, 0.f, 0.f};
    if (p.bias && col < p.N) add[0] = add[1] = add[2] = add[3] = p.bias[col];
    float res[4] = {0.f, 0.f, 0.f, 0.f}, old[4] = {0.f, 0.f, 0.f, 0.f};
    auto inside = [&](int e) { return m0 + rr + 8 * e < p.M && col < p.N; };
    if (p.residual)
#pragma unroll
        for (int e = 0; e < 4; ++e) if (inside(e)) res[e] = p.residual[(long)(m0 + rr + 8 * e) * p.ldr + col];
    if (p.accumulate)
#pragma unroll
        for (int e = 0; e < 4; ++e) if (inside(e)) old[e] = p.C[(long)(m0 + rr + 8 * e) * p.ldc + col];
    if (p.sw_up)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (inside(e)) {
                res[e] = p.sw_up[(long)(m0 + rr + 8 * e) * 2 * p.N + col];            // gate
                old[e] = p.sw_up[(long)(m0 + rr + 8 * e) * 2 * p.N + p.N + col];      // up
            }
    for (int s = 0; s < mine; s += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            load((u + 3) & 3, s + u + 3);             // (slices past the end are zeros)
            __builtin_amdgcn_sched_barrier(0);        // the requests stay in front of the MFMAs
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u].v[i][c], b[u].v[j][c], acc[i][j], 0, 0, 0);
        }
    }
    // accumulator (i, j) register r: row 16 i + 4 (lane / 16) + r, column 16 j + lane % 16
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) part[wave][16 * i + 4 * (lane >> 4) + r][16 * j + (lane & 15)] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int q = rr + 8 * e;
        if (p.sw_up) {
            float dg, du;
            swiglu_derivative((part[0][q][cc] + part[1][q][cc] + part[2][q][cc] + part[3][q][cc]) * p.alpha, res[e], old[e], &dg, &du);
            if (inside(e)) {
                p.C[(long)(m0 + q) * p.ldc + col] = dg;
                p.C[(long)(m0 + q) * p.ldc + p.N + col] = du;
            }
            continue;
        }
        const float v = (part[0][q][cc] + part[1][q][cc] + part[2][q][cc] + part[3][q][cc]) * p.alpha + add[e] + res[e];
        if (inside(e)) p.C[(long)(m0 + q) * p.ldc + col] = p.accumulate ? old[e] + v : v;
    }
}
template <bool TA, bool TB, bool FAST>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32Params p) {
    __shared__ float part[4][32][33];
    gemm_f32_body<TA, TB, FAST>(p, part, (int)blockIdx.x);
}
// Both products of a linear layer's backward pass in one grid (see gemm_bf16_pair_kernel), the one with the longer workgroups, whose K is
// the token count or the layer's outputs, first.  With the weight gradient always behind, a few long workgroups were
// left over at large token counts (us, two launches / weight gradient last / this order: 688 x 256 at 4000 tokens 53.8 / 62.1 / 43.7,
// at 12000 139 / 179 / 114; 512 x 512 at 12000 159 / 203 / 137; over 11 layers x 64 .. 12000 tokens never slower than two).
template <bool WGRAD_FIRST>
__global__ __launch_bounds__(256) void gemm_f32_pair_kernel(GemmF32Params pd, GemmF32Params pw, int first) {
    __shared__ float part[4][32][33];
    const int b = (int)blockIdx.x;
    if ((b < first) != WGRAD_FIRST) gemm_f32_body<false, true, true>(pd, part, WGRAD_FIRST ? b - first : b);
    else gemm_f32_body<true, true, true>(pw, part, WGRAD_FIRST ? b : b - first);
}

// Two products with K-contiguous operands in one grid; the first n0 workgroups are the first one's.  Both load in the same way: where
// only one of them can be read 16 bytes at a time, it has a launch of its own (teacher and student logits of 2000 tokens, V = 8192, H = 1024
// / 512, student states 4 bytes off: head 4.36 ms together, 3.2 apart).
template <bool FAST>
__global__ __launch_bounds__(256) void gemm_f32_two_kernel(GemmF32Params p0, GemmF32Params p1, int n0) {
    __shared__ float part[4][32][33];
    const int b = (int)blockIdx.x;
    if (b < n0) gemm_f32_body<false, false, FAST>(p0, part, b);
    else gemm_f32_body<false, false, FAST>(p1, part, b - n0);
}

// Explicit instantiations: the host pass has been seen to reference the launch stubs of some of these
// without defining them when they are only instantiated implicitly from the launcher below.
#define MS_INST(BM, WN, TA, TB)                                                                          \
    template __global__ void gemm_bf16_fast_kernel<BM, BM, 2, WN, TA, TB, EPI_NONE, false>(GemmParams); \
    template __global__ void gemm_bf16_fast_kernel<BM, BM, 2, WN, TA, TB, EPI_NONE, true>(GemmParams)
template __global__ void gemm_bf16_fast_kernel<256, 256, 2, 4, false, false, EPI_NONE, false>(GemmParams);
MS_INST(256, 4, false, true); MS_INST(256, 4, true, false); MS_INST(256, 4, true, true);
MS_INST(128, 2, false, false); MS_INST(128, 2, false, true); MS_INST(128, 2, true, false); MS_INST(128, 2, true, true);
#undef MS_INST
template __global__ void gemm_bf16_pp_kernel<EPI_NONE>(GemmParams);
template __global__ void gemm_bf16_pp_kernel<EPI_SWIGLU>(GemmParams);
template __global__ void gemm_bf16_pp_kernel<EPI_KD_DZ>(GemmParams);
template __global__ void gemm_bf16_pp_kernel<EPI_KD_STATS>(GemmParams);
#define MS_INST_RING(BM, BN, WM, WN, NST, TA, TB) \
    template __global__ void gemm_bf16_fast_kernel<BM, BN, WM, WN, TA, TB, EPI_NONE, true, NST>(GemmParams)
#define MS_INST_RINGS(BM, BN, WM, WN, NST)                                                             \
    MS_INST_RING(BM, BN, WM, WN, NST, false, false); MS_INST_RING(BM, BN, WM, WN, NST, false, true);   \
    MS_INST_RING(BM, BN, WM, WN, NST, true, false); MS_INST_RING(BM, BN, WM, WN, NST, true, true);     \
    template __global__ void gemm_bf16_fast_kernel<BM, BN, WM, WN, false, false, EPI_KD_DZ, true, NST>(GemmParams);     \
    template __global__ void gemm_bf16_fast_kernel<BM, BN, WM, WN, false, false, EPI_KD_STATS, true, NST>(GemmParams);  \
    template __global__ void gemm_bf16_fast_kernel<BM, BN, WM, WN, false, false, EPI_SWIGLU, true, NST>(GemmParams)
MS_INST_RINGS(128, 128, 4, 2, 4); MS_INST_RINGS(128, 256, 2, 4, 3); MS_INST_RINGS(64, 128, 2, 2, 3); MS_INST_RINGS(64, 64, 2, 1, 4);
#undef MS_INST_RINGS
#define MS_INST_TWO(EPI)                                                                                              \
    template __global__ void gemm_bf16_pp_two_kernel<EPI>(GemmParams, GemmParams, int, int, int, int);                          \
    template __global__ void gemm_bf16_two_kernel<128, 128, 2, 2, 2, EPI>(GemmParams, GemmParams, int, int, int, int);          \
    template __global__ void gemm_bf16_two_kernel<128, 128, 4, 2, 4, EPI>(GemmParams, GemmParams, int, int, int, int);          \
    template __global__ void gemm_bf16_two_kernel<128, 256, 2, 4, 3, EPI>(GemmParams, GemmParams, int, int, int, int);          \
    template __global__ void gemm_bf16_two_kernel<64, 128, 2, 2, 3, EPI>(GemmParams, GemmParams, int, int, int, int);           \
    template __global__ void gemm_bf16_two_kernel<64, 64, 2, 1, 4, EPI>(GemmParams, GemmParams, int, int, int, int)
MS_INST_TWO(EPI_KD_DZ); MS_INST_TWO(EPI_KD_STATS);
#undef MS_INST_TWO
#define MS_INST_PAIR(BM, BN, WM, WN, NST)                                                                                    \
    template __global__ void gemm_bf16_pair_kernel<BM, BN, WM, WN, NST, EPI_NONE>(GemmParams, GemmParams, int, int, int);   \
    template __global__ void gemm_bf16_pair_kernel<BM, BN, WM, WN, NST, EPI_SWIGLU_BWD>(GemmParams, GemmParams, int, int, int)
MS_INST_PAIR(256, 256, 2, 4, 2); MS_INST_PAIR(128, 128, 2, 2, 2); MS_INST_PAIR(128, 128, 4, 2, 4); MS_INST_PAIR(128, 256, 2, 4, 3);
MS_INST_PAIR(64, 128, 2, 2, 3); MS_INST_PAIR(64, 64, 2, 1, 4);
#undef MS_INST_PAIR
#undef MS_INST_RING
#define MS_INST_EPI(EPI)                                                                                      \
    template __global__ void gemm_bf16_fast_kernel<256, 256, 2, 4, false, false, EPI, false>(GemmParams);    \
    template __global__ void gemm_bf16_fast_kernel<128, 128, 2, 2, false, false, EPI, false>(GemmParams);    \
    template __global__ void gemm_bf16_fast_kernel<128, 128, 2, 2, false, false, EPI, true>(GemmParams)
MS_INST_EPI(EPI_KD_DZ); MS_INST_EPI(EPI_KD_STATS); MS_INST_EPI(EPI_SWIGLU);
#undef MS_INST_EPI

// Kernel selection switches, for measurements and tests only: the environment gives the process-wide setting
// (MS_GEMM_TILE = a tile code of kTiles, or 256256, forces the fast kernels' tile, -1 disables them; MS_GEMM_MFMA16 = 0
// selects v_mfma_f32_32x32x16_bf16 and the two-stage tiles), ms_k_gemm_config overrides it at run time.  The overrides are atomics, so changing them
// from one thread while another launches is defined, but which setting a concurrent launch sees is not: production
// callers leave them alone (automatic choice by shape).
constexpr int kUnset = -1000;
std::atomic<int> g_tile_override{kUnset}, g_mfma16_override{kUnset};
int forced_tile() {
    static const int env = [] { const char *e = getenv("MS_GEMM_TILE"); return e ? atoi(e) : 0; }();
    const int o = g_tile_override.load(std::memory_order_relaxed);
    return o != kUnset ? o : env;
}
bool use_mfma16() {
    static const bool env = [] { const char *e = getenv("MS_GEMM_MFMA16"); return !e || atoi(e) != 0; }();
    const int o = g_mfma16_override.load(std::memory_order_relaxed);
    return o != kUnset ? o != 0 : env;
}

// The tile for an M x N output (N = rows of B) of kt K tiles whose epilogue moves out_bytes per element (ms_choose_tile)
int choose_tile(int M, int N, int kt, double out_bytes) { return ms_choose_tile(M, N, kt, out_bytes, forced_tile(), use_mfma16()); }

template <int BM, int BN, int WM, int WN, int NST, int EPI>
void launch_fast_tile(const GemmParams &p, int ta, int tb, dim3 grid, hipStream_t s) {
    constexpr int NT = 64 * WM * WN;
#define GO(TA, TB)                                                                                                  \
    do {                                                                                                            \
        if constexpr (NST > 2) gemm_bf16_fast_kernel<BM, BN, WM, WN, TA, TB, EPI, true, NST><<<grid, NT, 0, s>>>(p); \
        else if (!use_mfma16()) gemm_bf16_fast_kernel<BM, BN, WM, WN, TA, TB, EPI, false><<<grid, NT, 0, s>>>(p);    \
        else if constexpr (BM == 256 && !TA && !TB) gemm_bf16_pp_kernel<EPI><<<grid, NT, 0, s>>>(p);                \
        else gemm_bf16_fast_kernel<BM, BN, WM, WN, TA, TB, EPI, true><<<grid, NT, 0, s>>>(p);                        \
    } while (0)
    if constexpr (EPI != EPI_NONE) GO(false, false);
    else if (!ta && !tb) GO(false, false);
    else if (!ta && tb) GO(false, true);
    else if (ta && !tb) GO(true, false);
    else GO(true, true);
#undef GO
}

// p.tiles_m / tiles_n are set here; EPI_SWIGLU tiles cover bn / 2 output columns (gate and up rows of B)
template <int EPI>
ms_status launch_bf16_fast(GemmParams &p, int tile, int ta, int tb, int splits, double flops, hipStream_t s) {
    const MsTile &t = kTiles[tile];
    p.tiles_m = ms_cdiv(p.M, t.bm);
    p.tiles_n = ms_cdiv(p.N, EPI == EPI_SWIGLU ? t.bn / 2 : t.bn);
    dim3 grid(p.tiles_m * p.tiles_n, splits);
    ProfScope ps((ta || tb) ? 1 : 0, flops, s);
    switch (tile) {
        case T256: launch_fast_tile<256, 256, 2, 4, 2, EPI>(p, ta, tb, grid, s); break;
        case R128: launch_fast_tile<128, 128, 4, 2, 4, EPI>(p, ta, tb, grid, s); break;
        case R128x256: launch_fast_tile<128, 256, 2, 4, 3, EPI>(p, ta, tb, grid, s); break;
        case R64x128: launch_fast_tile<64, 128, 2, 2, 3, EPI>(p, ta, tb, grid, s); break;
        case R64: launch_fast_tile<64, 64, 2, 1, 4, EPI>(p, ta, tb, grid, s); break;
        default: launch_fast_tile<128, 128, 2, 2, 2, EPI>(p, ta, tb, grid, s); break;
    }
    MS_LAUNCH_CHECK();
    return MS_OK;
}

template <int BM, int BN>
ms_status launch_bf16(const GemmParams &p, int ta, int tb, int splits, hipStream_t s) {
    const size_t smem = (size_t)2 * (BM + BN) * BK * sizeof(bf16_t);
    dim3 grid(p.tiles_m * p.tiles_n, splits);
    ProfScope ps((ta || tb) ? 1 : 0, 2.0 * p.M * p.N * p.K, s);
#define GO(TA, TB)                                                                                        \
    do {                                                                                                  \
        static bool attr_set = false;                                                                     \
        if (!attr_set && smem > 48 * 1024) {                                                              \
            MS_CHECK_HIP(hipFuncSetAttribute((const void *)gemm_bf16_kernel<BM, BN, TA, TB>,              \
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));     \
            attr_set = true;                                                                              \
        }                                                                                                 \
        gemm_bf16_kernel<BM, BN, TA, TB><<<grid, 256, smem, s>>>(p);                                      \
    } while (0)
    if (!ta && !tb) GO(false, false);
    else if (!ta && tb) GO(false, true);
    else if (ta && !tb) GO(true, false);
    else GO(true, true);
#undef GO
    MS_LAUNCH_CHECK();
    return MS_OK;
}

// fp32: whether an operand (rows x K as the product sees it) can be read through a descriptor, 16 bytes at a time where it is
// K-contiguous
bool f32_fast(const void *q, long ld, bool trans, long rows, long K) {
    return (trans || (((uintptr_t)q & 15) == 0 && ld % 4 == 0 && K % 4 == 0)) && ms_buffer_range_ok(trans ? K : rows, trans ? rows : K, ld, 4);
}

// Checked arguments of a bf16 product, all but the split of K
struct Bf16Gemm {
    GemmParams p;
    bool fast;          // the direct-to-LDS kernels take it
    int kt;             // K tiles
    double out_bytes;   // what the epilogue moves per output element
};
ms_status prepare_bf16(int trans_a, int trans_b, int M, int N, int K, float alpha, const void *A, long lda, const void *B, long ldb,
                       void *C, long ldc, int c_fp32, int accumulate, const void *bias, const void *residual, long ldr,
                       int residual_fp32, Bf16Gemm *g) {
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    if (!al(A) || !al(B) || lda % 8 || ldb % 8 || (trans_a ? M % 8 : K % 8) || (trans_b ? N % 8 : K % 8))
        return ms_fail(MS_ERR_UNSUPPORTED,
                       "gemm(bf16): contiguous dimension of each operand must be a multiple of 8 and 16-byte aligned "
                       "(M=%d N=%d K=%d ta=%d tb=%d lda=%ld ldb=%ld)", M, N, K, trans_a, trans_b, (long)lda, (long)ldb);
    GemmParams &p = g->p;
    p = {};
    p.A = A; p.B = B; p.C = C; p.bias = bias; p.residual = residual;
    p.lda = lda; p.ldb = ldb; p.ldc = ldc; p.ldr = ldr; p.M = M; p.N = N; p.K = K; p.alpha = alpha;
    p.c_fp32 = c_fp32; p.accumulate = accumulate; p.res_fp32 = residual_fp32;
    // fast path (direct-to-LDS loads, descriptor-addressed epilogue) needs full K tiles for a K-contiguous
    // operand and 32-bit byte offsets
    const long lim = (1L << 32) - (1L << 20);
    const long rows_a = trans_a ? K : M, rows_b = trans_b ? K : N;
    g->fast = forced_tile() >= 0 && ((trans_a && trans_b) || K % BK == 0) && (rows_a + 256) * lda * 2 < lim &&
              (rows_b + 256) * ldb * 2 < lim && ((long)M + 256) * ldc * 4 < lim &&
              (!residual || ((long)M + 256) * ldr * 4 < lim);
    g->kt = ms_cdiv(K, BK) < 1 ? 1 : ms_cdiv(K, BK);
    g->out_bytes = (c_fp32 ? 4 : 2) + (residual ? (residual_fp32 ? 4 : 2) : 0) + (accumulate ? 4 : 0);
    return MS_OK;
}
// The last arguments, which depend on the number of K splits; returns how many there really are
int set_splits(Bf16Gemm &g, int splits) {
    GemmParams &p = g.p;
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    if (splits > g.kt) splits = g.kt;
    p.k_tiles_per_split = ms_cdiv(g.kt, splits);
    splits = ms_cdiv(g.kt, p.k_tiles_per_split);
    p.atomic = splits > 1;
    p.vec_epilogue = !p.atomic && p.N % 4 == 0 && p.ldc % 4 == 0 && al(p.C) && (!p.residual || (p.ldr % 4 == 0 && al(p.residual))) &&
                     (!p.bias || ((uintptr_t)p.bias & 7) == 0);
    return splits;
}

}  // namespace

extern "C" ms_status ms_k_gemm_config(int32_t tile, int32_t mfma16) {
    bool known = tile == -1 || tile == 0 || tile == kPingPong;
    for (const MsTile &t : kTiles) known = known || tile == t.code;
    if (!known || mfma16 < -1 || mfma16 > 1)
        return ms_fail(MS_ERR_INVALID_ARG, "gemm_config: tile must be -1, 0, 128, 256, 256256, 128128, 128256, 64128 or 64064 and mfma16 -1, 0 or 1");
    g_tile_override = tile == 0 ? kUnset : tile;
    g_mfma16_override = mfma16 < 0 ? kUnset : mfma16;
    return MS_OK;
}

extern "C" ms_status ms_k_gemm(int32_t dtype, int32_t trans_a, int32_t trans_b, int32_t M, int32_t N, int32_t K,
                               float alpha, const void *A, int64_t lda, const void *B, int64_t ldb, void *C,
                               int64_t ldc, int32_t c_fp32, int32_t accumulate, const void *bias,
                               const void *residual, int64_t ldr, int32_t residual_fp32, int32_t split_k,
                               void *stream) {
    if (M == 0 || N == 0) return MS_OK;
    if (!A || !B || !C || M < 0 || N < 0 || K < 0) return ms_fail(MS_ERR_INVALID_ARG, "gemm: null pointer or negative size");
    if (accumulate && !c_fp32 && dtype == MS_BF16) return ms_fail(MS_ERR_INVALID_ARG, "gemm: accumulate needs an fp32 C");
    hipStream_t s = (hipStream_t)stream;
    if (dtype == MS_F32) {
        GemmF32Params p = {};
        p.A = (const float *)A; p.B = (const float *)B; p.C = (float *)C;
        p.bias = (const float *)bias; p.residual = (const float *)residual;
        p.lda = lda; p.ldb = ldb; p.ldc = ldc; p.ldr = ldr; p.M = M; p.N = N; p.K = K; p.alpha = alpha; p.accumulate = accumulate;
        p.tiles_n = ms_cdiv(N, 32);
        const long tiles = (long)ms_cdiv(M, 32) * p.tiles_n;
        if (!ms_launch_fits(tiles, 256)) {   // more tiles than one launch takes: the two halves of C along its longer side
            const bool rows = ms_cdiv(M, 32) >= p.tiles_n;
            const int cut = (int)(((rows ? M : N) / 2L + 31) / 32 * 32);
            const long a = rows ? (trans_a ? cut : cut * lda) : 0, b = rows ? 0 : (trans_b ? cut : cut * ldb), c = rows ? cut * ldc : cut;
            const long r = rows ? cut * ldr : cut;
            MS_TRY(ms_k_gemm(dtype, trans_a, trans_b, rows ? cut : M, rows ? N : cut, K, alpha, A, lda, B, ldb, C, ldc, c_fp32, accumulate, bias,
                             residual, ldr, residual_fp32, split_k, stream));
            return ms_k_gemm(dtype, trans_a, trans_b, rows ? M - cut : M, rows ? N : N - cut, K, alpha, p.A + a, lda, p.B + b, ldb, p.C + c,
                             ldc, c_fp32, accumulate, bias && !rows ? p.bias + cut : bias, residual ? p.residual + r : nullptr, ldr,
                             residual_fp32, split_k, stream);
        }
        const unsigned grid = (unsigned)tiles;
#define GO(TA, TB)                                                                                     \
    do {                                                                                               \
        if (f32_fast(A, lda, TA, M, K) && f32_fast(B, ldb, TB, N, K)) gemm_f32_kernel<TA, TB, true><<<grid, 256, 0, s>>>(p);  \
        else gemm_f32_kernel<TA, TB, false><<<grid, 256, 0, s>>>(p);                                   \
    } while (0)
        if (!trans_a && !trans_b) GO(false, false);
        else if (!trans_a && trans_b) GO(false, true);
        else if (trans_a && !trans_b) GO(true, false);
        else GO(true, true);
#undef GO
        MS_LAUNCH_CHECK();
        return MS_OK;
    }
    Bf16Gemm g;
    MS_TRY(prepare_bf16(trans_a, trans_b, M, N, K, alpha, A, lda, B, ldb, C, ldc, c_fp32, accumulate, bias, residual, ldr, residual_fp32, &g));
    int tile = g.fast ? choose_tile(M, N, g.kt, g.out_bytes) : T128;
    int splits = split_k;
    if (splits <= 0) {  // automatic: only when accumulating into fp32 (weight gradients: small M x N, long K)
        splits = 1;
        if (accumulate && c_fp32 && g.fast) {
            const MsSplit c = ms_choose_split(M, N, g.kt, forced_tile(), use_mfma16());
            tile = c.tile;
            splits = c.splits;
        } else if (accumulate && c_fp32) {
            const int tiles = ms_cdiv(M, 128) * ms_cdiv(N, 128);
            while (tiles * splits < 512 && g.kt / (splits * 2) >= 8) splits *= 2;
        }
    }
    if (splits > 1 && !(accumulate && c_fp32)) return ms_fail(MS_ERR_INVALID_ARG, "gemm: split_k needs accumulate into fp32");
    splits = set_splits(g, splits);
    if (g.fast) return launch_bf16_fast<EPI_NONE>(g.p, tile, trans_a, trans_b, splits, 2.0 * M * N * K, s);
    g.p.tiles_m = ms_cdiv(M, 128); g.p.tiles_n = ms_cdiv(N, 128);
    return launch_bf16<128, 128>(g.p, trans_a, trans_b, splits, s);
}

// ------------------------------------------------------------------ backward pass of a linear layer
namespace {
// Input gradient d and weight gradient w of one layer in one grid, if that is estimated faster (done = false: it is not)
template <int EPI>
ms_status launch_pair(Bf16Gemm &d, Bf16Gemm &w, bool *done, hipStream_t s) {
    const int n = d.p.M, in = d.p.N, out = d.p.K;
    if (!d.fast || !w.fast || !use_mfma16()) return MS_OK;
    const MsPair c = ms_choose_pair(n, out, in, d.out_bytes, forced_tile());
    if (c.tile < 0) return MS_OK;
    set_splits(d, 1);
    const int splits = set_splits(w, c.splits);
    const MsTile &t = kTiles[c.tile];
    d.p.tiles_m = ms_cdiv(n, t.bm); w.p.tiles_m = ms_cdiv(out, t.bm);
    d.p.tiles_n = w.p.tiles_n = ms_cdiv(in, t.bn);
    const long nd = (long)d.p.tiles_m * d.p.tiles_n, nw = (long)w.p.tiles_m * w.p.tiles_n;
    if (!ms_launch_fits(nd + nw * splits, 512)) return MS_OK;
    *done = true;
    ProfScope ps(1, 4.0 * n * out * in, s);
    const unsigned grid = (unsigned)(nd + nw * splits);
#define GO(BM, BN, WM, WN, NST) gemm_bf16_pair_kernel<BM, BN, WM, WN, NST, EPI><<<grid, 64 * WM * WN, 0, s>>>(d.p, w.p, (int)nd, (int)nw, c.wgrad_first)
    switch (c.tile) {
        case T256: GO(256, 256, 2, 4, 2); break;
        case R128: GO(128, 128, 4, 2, 4); break;
        case R128x256: GO(128, 256, 2, 4, 3); break;
        case R64x128: GO(64, 128, 2, 2, 3); break;
        case R64: GO(64, 64, 2, 1, 4); break;
        default: GO(128, 128, 2, 2, 2); break;
    }
#undef GO
    MS_LAUNCH_CHECK();
    return MS_OK;
}
ms_status launch_pair_f32(int n, int out, int in, const float *dy, long ldy, const float *W, const float *x, float *dx, long ldx, int accumulate,
                          float *dW, const float *sw_up, bool *done, hipStream_t s) {
    const long nd = (long)ms_cdiv(n, 32) * ms_cdiv(in, 32), nw = (long)ms_cdiv(out, 32) * ms_cdiv(in, 32);
    // (dy rows that cannot be read 16 bytes at a time slow dx = dy W down, but not the weight gradient, which keeps its own launch then)
    if (!ms_launch_fits(nd + nw, 256) || !f32_fast(dy, ldy, false, n, out) || !f32_fast(W, in, true, in, out) || !f32_fast(dy, ldy, true, out, n) ||
        !f32_fast(x, in, true, in, n))
        return MS_OK;
    *done = true;
    GemmF32Params pd = {}, pw = {};
    pd.A = pw.A = dy; pd.lda = pw.lda = ldy;
    pd.B = W; pw.B = x; pd.ldb = pw.ldb = in;
    pd.C = dx; pd.ldc = ldx; pw.C = dW; pw.ldc = in;
    pd.M = n; pd.N = in; pd.K = out; pw.M = out; pw.N = in; pw.K = n;
    pd.tiles_n = pw.tiles_n = ms_cdiv(in, 32);
    pd.alpha = pw.alpha = 1.f; pd.accumulate = accumulate; pw.accumulate = 1;
    pd.sw_up = sw_up;
    if (n > out) gemm_f32_pair_kernel<true><<<(unsigned)(nd + nw), 256, 0, s>>>(pd, pw, (int)nw);
    else gemm_f32_pair_kernel<false><<<(unsigned)(nd + nw), 256, 0, s>>>(pd, pw, (int)nd);
    MS_LAUNCH_CHECK();
    return MS_OK;
}
}  // namespace

extern "C" ms_status ms_k_linear_backward(int32_t dtype, int32_t n, int32_t out, int32_t in, const void *dy, int64_t ldy, const void *W,
                                          const void *x, void *dx, int32_t dx_fp32, int32_t dx_accumulate, void *dW, void *stream) {
    auto one_by_one = [&]() {
        MS_TRY(ms_k_gemm(dtype, 0, 1, n, in, out, 1.f, dy, ldy, W, in, dx, in, dx_fp32, dx_accumulate, nullptr, nullptr, 0, 0, 1, stream));
        return ms_k_gemm(dtype, 1, 1, out, in, n, 1.f, dy, ldy, x, in, dW, in, 1, 1, nullptr, nullptr, 0, 0, 0, stream);
    };
    if (n <= 0 || out <= 0 || in <= 0 || !dy || !W || !x || !dx || !dW) return one_by_one();      // (which has the checks)
    hipStream_t s = (hipStream_t)stream;
    if (dtype == MS_F32) {
        bool done = false;
        MS_TRY(launch_pair_f32(n, out, in, (const float *)dy, ldy, (const float *)W, (const float *)x, (float *)dx, in, dx_accumulate, (float *)dW,
                               nullptr, &done, s));
        return done ? MS_OK : one_by_one();
    }
    if (dx_accumulate && !dx_fp32) return one_by_one();
    Bf16Gemm d, w;
    MS_TRY(prepare_bf16(0, 1, n, in, out, 1.f, dy, ldy, W, in, dx, in, dx_fp32, dx_accumulate, nullptr, nullptr, 0, 0, &d));
    MS_TRY(prepare_bf16(1, 1, out, in, n, 1.f, dy, ldy, x, in, dW, in, 1, 1, nullptr, nullptr, 0, 0, &w));
    bool done = false;
    MS_TRY(launch_pair<EPI_NONE>(d, w, &done, s));
    return done ? MS_OK : one_by_one();
}

// The down projection of a SwiGLU block backwards: dW += dy^T act and [dgate | dup] from da = dy W, which is not stored where the
// two products share a grid.
extern "C" ms_status ms_k_swiglu_linear_backward(int32_t dtype, int32_t n, int32_t out, int32_t f, const void *dy, const void *W, const void *act,
                                                 const void *gate_up, void *da, void *d_gate_up, void *dW, void *stream) {
    hipStream_t s = (hipStream_t)stream;
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    if (dtype == MS_BF16 && n > 0 && out > 0 && f > 0 && f % 4 == 0 && dy && W && act && gate_up && d_gate_up && dW && al(gate_up) && al(d_gate_up) && ((long)n + 256) * 2 * f * 2 < (1L << 32) - (1L << 20)) {
        Bf16Gemm d, w;
        MS_TRY(prepare_bf16(0, 1, n, f, out, 1.f, dy, out, W, f, d_gate_up, 2L * f, 0, 0, nullptr, nullptr, 0, 0, &d));
        MS_TRY(prepare_bf16(1, 1, out, f, n, 1.f, dy, out, act, f, dW, f, 1, 1, nullptr, nullptr, 0, 0, &w));
        d.p.sg_f = f;
        d.p.sg_gu = const_cast<void *>(gate_up);
        d.p.sg_ldgu = 2L * f;
        d.out_bytes = 8;
        bool done = false;
        MS_TRY(launch_pair<EPI_SWIGLU_BWD>(d, w, &done, s));
        if (done) return MS_OK;
    }
    if (dtype == MS_F32 && n > 0 && out > 0 && f > 0 && dy && W && act && gate_up && d_gate_up && dW) {
        bool done = false;
        MS_TRY(launch_pair_f32(n, out, f, (const float *)dy, out, (const float *)W, (const float *)act, (float *)d_gate_up, 2L * f, 0, (float *)dW,
                               (const float *)gate_up, &done, s));
        if (done) return MS_OK;
    }
    MS_TRY(ms_k_linear_backward(dtype, n, out, f, dy, out, W, act, da, 0, 0, dW, s));
    return ms_k_act_backward(0, dtype, n, f, da, gate_up, d_gate_up, s);
}

ms_status gemm_f32_two(int M, int N, const float *A0, const float *B0, float *C0, int K0, const float *A1, const float *B1, float *C1, int K1,
                       long ldc, hipStream_t s) {
    const long tiles = (long)ms_cdiv(M, 32) * ms_cdiv(N, 32);
    const bool fast = f32_fast(A0, K0, false, M, K0) && f32_fast(B0, K0, false, N, K0);
    if (!ms_launch_fits(2 * tiles, 256) || fast != (f32_fast(A1, K1, false, M, K1) && f32_fast(B1, K1, false, N, K1))) {
        MS_TRY(ms_k_gemm(MS_F32, 0, 0, M, N, K0, 1.f, A0, K0, B0, K0, C0, ldc, 1, 0, nullptr, nullptr, 0, 0, 1, s));
        return ms_k_gemm(MS_F32, 0, 0, M, N, K1, 1.f, A1, K1, B1, K1, C1, ldc, 1, 0, nullptr, nullptr, 0, 0, 1, s);
    }
    GemmF32Params p0 = {}, p1 = {};
    p0.A = A0; p0.B = B0; p0.C = C0; p0.lda = p0.ldb = p0.K = K0;
    p1.A = A1; p1.B = B1; p1.C = C1; p1.lda = p1.ldb = p1.K = K1;
    p0.ldc = p1.ldc = ldc; p0.M = p1.M = M; p0.N = p1.N = N; p0.tiles_n = p1.tiles_n = ms_cdiv(N, 32); p0.alpha = p1.alpha = 1.f;
    if (fast) gemm_f32_two_kernel<true><<<(unsigned)(2 * tiles), 256, 0, s>>>(p0, p1, (int)tiles);
    else gemm_f32_two_kernel<false><<<(unsigned)(2 * tiles), 256, 0, s>>>(p0, p1, (int)tiles);
    MS_LAUNCH_CHECK();
    return MS_OK;
}

// ------------------------------------------------------------------ student-logits GEMM with KD epilogues
// zs = A[M,K] B[N,K]^T is never stored: mode EPI_KD_STATS folds it (with the teacher logits zt of the same
// chunk) into per-strip partial statistics, mode EPI_KD_DZ turns it into dz.  bf16 fast path only.
bool gemm_kd_epilogue_supported(int M, int N, int K, const void *A, long lda, const void *B, long ldb, const float *zt,
                                long ldz, const void *dz, long lddz, int dz_fp32) {
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    const long lim = (1L << 32) - (1L << 20);
    const int forced = forced_tile();
    return forced >= 0 && M > 0 && N > 0 && K > 0 && K % BK == 0 && N % 4 == 0 && al(A) && al(B) && al(zt) && lda % 8 == 0 &&
           ldb % 8 == 0 && ldz % 4 == 0 && ((long)M + 256) * lda * 2 < lim && ((long)N + 256) * ldb * 2 < lim &&
           ((long)M + 256) * ldz * 4 < lim && (!dz || (al(dz) && lddz % 4 == 0 && ((long)M + 256) * lddz * (dz_fp32 ? 4 : 2) < lim));
}

static ms_status prepare_kd(int mode, int M, int N, int K, const void *A, long lda, const void *B, long ldb, const float *zt,
                            long ldz, float *stats, float *part, int nparts, float inv_t, float coef, void *dz, long lddz,
                            int dz_fp32, GemmParams *out) {
    if (!gemm_kd_epilogue_supported(M, N, K, A, lda, B, ldb, zt, ldz, mode == EPI_KD_DZ ? dz : nullptr, lddz, dz_fp32))
        return ms_fail(MS_ERR_UNSUPPORTED, "gemm_kd_epilogue: shape or alignment outside the fast path");
    if ((mode == EPI_KD_DZ && (!dz || !stats)) || (mode == EPI_KD_STATS && (!part || nparts < ms_cdiv(N, 64))) ||
        (mode != EPI_KD_DZ && mode != EPI_KD_STATS))
        return ms_fail(MS_ERR_INVALID_ARG, "gemm_kd_epilogue: bad mode or null buffer");
    GemmParams &p = *out;
    p = {};
    p.A = A; p.B = B; p.C = dz; p.lda = lda; p.ldb = ldb; p.ldc = lddz; p.M = M; p.N = N; p.K = K; p.alpha = 1.f;
    p.c_fp32 = dz_fp32;
    p.kd_zt = zt; p.kd_ldz = ldz; p.kd_stats = stats; p.kd_part = part; p.kd_nparts = nparts; p.kd_inv_t = inv_t; p.kd_coef = coef;
    p.k_tiles_per_split = ms_cdiv(K, BK);
    return MS_OK;
}

ms_status gemm_kd_epilogue(int mode, int M, int N, int K, const void *A, long lda, const void *B, long ldb, const float *zt,
                           long ldz, float *stats, float *part, int nparts, float inv_t, float coef, void *dz, long lddz,
                           int dz_fp32, hipStream_t s) {
    GemmParams p;
    MS_TRY(prepare_kd(mode, M, N, K, A, lda, B, ldb, zt, ldz, stats, part, nparts, inv_t, coef, dz, lddz, dz_fp32, &p));
    const int tile = choose_tile(M, N, p.k_tiles_per_split, kKdEpilogueBytes);
    if (mode == EPI_KD_DZ) return launch_bf16_fast<EPI_KD_DZ>(p, tile, 0, 0, 1, 2.0 * M * N * K, s);
    return launch_bf16_fast<EPI_KD_STATS>(p, tile, 0, 0, 1, 2.0 * M * N * K, s);
}

template <int EPI> static void launch_two(int tile, int first, GemmParams &pt, GemmParams &ps, hipStream_t s) {
    const MsTile &t = kTiles[tile];
    pt.tiles_m = ps.tiles_m = ms_cdiv(ps.M, t.bm);
    pt.tiles_n = ms_cdiv(pt.N, t.bn);
    ps.tiles_n = ms_cdiv(ps.N, t.bn);
    const int nt = pt.tiles_m * pt.tiles_n, ns = ps.tiles_m * ps.tiles_n, run = 256 * t.per_cu;
    if (tile == T256) {
        gemm_bf16_pp_two_kernel<EPI><<<nt + ns, 512, 0, s>>>(pt, ps, nt, ns, run, first);
        return;
    }
#define GO(BM, BN, WM, WN, NST) gemm_bf16_two_kernel<BM, BN, WM, WN, NST, EPI><<<nt + ns, 64 * WM * WN, 0, s>>>(pt, ps, nt, ns, run, first)
    switch (tile) {
        case R128: GO(128, 128, 4, 2, 4); break;
        case R128x256: GO(128, 256, 2, 4, 3); break;
        case R64x128: GO(64, 128, 2, 2, 3); break;
        case R64: GO(64, 64, 2, 1, 4); break;
        default: GO(128, 128, 2, 2, 2); break;
    }
#undef GO
}

ms_status gemm_kd_and_teacher(int mode, int M, int N, int K, const void *A, const void *B, const float *zt, float *stats, float *part, int nparts,
                              float inv_t, float coef, void *dz, long ld, int Nt, int Kt, const void *At, const void *Bt, float *next_zt, hipStream_t s) {
    GemmParams ps;
    MS_TRY(prepare_kd(mode, M, N, K, A, K, B, K, zt, ld, stats, part, nparts, inv_t, coef, dz, ld, 0, &ps));
    Bf16Gemm t;
    MS_TRY(prepare_bf16(0, 0, M, Nt, Kt, 1.f, At, Kt, Bt, Kt, next_zt, ld, 1, 0, nullptr, nullptr, 0, 0, &t));
    int first = 0;
    const int tile = t.fast && use_mfma16() ? ms_choose_two(M, N, ps.k_tiles_per_split, Nt, t.kt, forced_tile(), &first) : -1;
    if (tile >= 0 && ms_launch_fits(ms_tiles(kTiles[tile], M, N) + ms_tiles(kTiles[tile], M, Nt), 512)) {
        set_splits(t, 1);
        ProfScope prof(0, 2.0 * M * ((double)N * K + (double)Nt * Kt), s);
        if (mode == EPI_KD_DZ) launch_two<EPI_KD_DZ>(tile, first, t.p, ps, s);
        else launch_two<EPI_KD_STATS>(tile, first, t.p, ps, s);
        MS_LAUNCH_CHECK();
        return MS_OK;
    }
    MS_TRY(gemm_kd_epilogue(mode, M, N, K, A, K, B, K, zt, ld, stats, part, nparts, inv_t, coef, dz, ld, 0, s));
    return ms_k_gemm(MS_BF16, 0, 0, M, Nt, Kt, 1.f, At, Kt, Bt, Kt, next_zt, ld, 1, 0, nullptr, nullptr, 0, 0, 1, s);
}

// ------------------------------------------------------------------ fused gate/up GEMM + SwiGLU
// act[M, F] = silu(A W_gate^T) * (A W_up^T) with W = [gate rows | up rows] ([2F, K]); gate_up (optional,
// [M, 2F]) also receives the rounded pre-activations for the backward pass.  bf16 fast path only.
bool gemm_swiglu_supported(int M, int F, int K, const void *A, long lda, const void *W, long ldw, const void *act, long ldact,
                           const void *gate_up, long ldgu) {
    auto al = [](const void *q) { return ((uintptr_t)q & 15) == 0; };
    const long lim = (1L << 32) - (1L << 20);
    const int forced = forced_tile();
    return forced >= 0 && M > 0 && F > 0 && K > 0 && K % BK == 0 && F % 4 == 0 && al(A) && al(W) && al(act) && lda % 8 == 0 &&
           ldw % 8 == 0 && ldact % 4 == 0 && ((long)M + 256) * lda * 2 < lim && (2L * F + 256) * ldw * 2 < lim &&
           ((long)M + 256) * ldact * 2 < lim && (!gate_up || (al(gate_up) && ldgu % 4 == 0 && ((long)M + 256) * ldgu * 2 < lim));
}

ms_status gemm_swiglu(int M, int F, int K, const void *A, long lda, const void *W, long ldw, void *act, long ldact,
                      void *gate_up, long ldgu, hipStream_t s) {
    if (!gemm_swiglu_supported(M, F, K, A, lda, W, ldw, act, ldact, gate_up, ldgu))
        return ms_fail(MS_ERR_UNSUPPORTED, "gemm_swiglu: shape or alignment outside the fast path");
    GemmParams p = {};
    p.A = A; p.B = W; p.C = act; p.lda = lda; p.ldb = ldw; p.ldc = ldact; p.M = M; p.N = F; p.K = K; p.alpha = 1.f;
    p.sg_f = F; p.sg_gu = gate_up; p.sg_ldgu = ldgu;
    p.k_tiles_per_split = ms_cdiv(K, BK);
    return launch_bf16_fast<EPI_SWIGLU>(p, choose_tile(M, 2 * F, p.k_tiles_per_split, gate_up ? 3 : 1), 0, 0, 1, 4.0 * M * F * K, s);
}

extern "C" ms_status ms_k_gemm_swiglu(int32_t M, int32_t F, int32_t K, const void *A, int64_t lda, const void *W, int64_t ldw,
                                      void *act, int64_t ldact, void *gate_up, int64_t ldgu, void *stream) {
    if (!A || !W || !act) return ms_fail(MS_ERR_INVALID_ARG, "gemm_swiglu: null pointer");
    return gemm_swiglu(M, F, K, A, lda, W, ldw, act, ldact, gate_up, ldgu, (hipStream_t)stream);
}
