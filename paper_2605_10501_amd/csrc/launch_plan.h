// Host-side rules of the launches: operand ranges, launch limits, choice of kernels.  Plain C++ without HIP, so that the
// rules can be compiled and checked without a GPU.
#pragma once
#include <math.h>
#include <stddef.h>

// Elements from the first to the last one of a matrix stored as `outer` rows of `inner` elements, ld apart: the range of
// the buffer descriptor that its loads go through.  An empty matrix has none; without that case K = 0 with padded rows
// gives a negative number, which as an unsigned range covers the offset that stands for "out of range".
constexpr long ms_matrix_extent(long outer, long inner, long ld) {
    return outer > 0 && inner > 0 ? (outer - 1) * ld + inner : 0;
}
// Whether a kernel may load the matrix through a descriptor with 32-bit byte offsets (rows that go backwards may not)
constexpr long kBufferBytes = (1L << 32) - (1L << 20);
constexpr bool ms_buffer_range_ok(long outer, long inner, long ld, int es) {
    return (outer <= 1 || ld >= 0) && ms_matrix_extent(outer, inner, ld) * es < kBufferBytes;
}

// HIP refuses a launch of 2^32 threads or more along one dimension
constexpr long kLaunchThreads = 0xffffffffL;
constexpr bool ms_launch_fits(long workgroups, int threads) { return workgroups <= kLaunchThreads / threads; }

// fp32 attention on 16-row tiles: whether the batch can be addressed and launched (max_seqlen is an upper bound; heads =
// workgroups along y).  The scalar kernels, one workgroup per token, take the rest: a batch of very many short sequences
// under a large bound among them.
constexpr int kF32AttnTile = 16;
constexpr bool ms_f32_attention_tiles(int hd, long n, long n_seqs, long max_seqlen, int nq, int nkv, int heads) {
    return (hd == 64 || hd == 80 || hd == 128) && n * (nq + 2 * nkv) * hd * 4 < kBufferBytes && max_seqlen > 0 && heads <= 65535 &&
           ms_launch_fits(n_seqs * ((max_seqlen + kF32AttnTile - 1) / kF32AttnTile), 256);
}

// ------------------------------------------------------------------ workgroup tiles of the bf16 GEMMs
// 256 x 256 and 128 x 128 have two LDS stages; a K tile is then requested one tile time before its first use, which covers
// the latency of the load only when the CU is busy with a large tile (256) or a second workgroup (128).  The ring tiles
// keep two or three tiles in flight and are for grids that do not fill the chip with those: at one workgroup per CU the
// two-stage 128 x 128 kernel takes 0.61 us per K tile, the ring kernel of the same tile 0.36, and smaller tiles spread a
// small output over more CUs.
// Times are fits to sweeps on MI355X:
//   us_per_ktile: per 64-deep K tile with one workgroup per CU, few and all CUs busy (the L2s and the power budget are
//   shared), then with two per CU, few and all CUs with a second one;
//   us_round + us_out x bytes: prologue and epilogue of a round, the latter by what it reads and writes per output
//   element, for 256 x 256 elements;  us_call: once.
// `lin` (K-contiguous A) is fitted to what decides, the times of a shape's better tiles relative to each other, over 1278
// shapes (M = 128 .. 46000, N = 512 .. 22016, K = 512 .. 17920, K-contiguous and K-major B, bf16 / fp32 outputs, fp32
// residual, SwiGLU and KD epilogues; half of them choose as well for the other half).  Its 256 x 256 row is the two-stage kernel, which
// K-major B runs; K-contiguous products run the ping-pong kernel in that tile, which is up to 25 % faster.  `wgrad` (both operands K-major, +=
// into fp32) is a fit to such products of 300 .. 32768 tokens, in which the output has terms of its own.
struct MsTileTimes { double us_per_ktile[4], us_round, us_out, us_call; };
struct MsTile {
    int code, bm, bn, per_cu;
    MsTileTimes lin, wgrad;
};
enum { T256 = 0, T128 = 1, R128 = 2, R128x256 = 3, R64x128 = 4, R64 = 5, kNumTiles = 6 };
constexpr int kPingPong = 256256;       // another code of the 256 x 256 tile (whose K-contiguous form is the ping-pong kernel)
constexpr MsTile kTiles[kNumTiles] = {
    {256, 256, 256, 1, {{0.852, 1.483, 0, 0}, 1.58, 2.35, 0}, {{1.08, 1.48, 0, 0}, 3.5, 0, 0}},
    {128, 128, 128, 2, {{0.450, 0.618, 0.778, 0.949}, 0.10, 4.28, 3.03}, {{0.60, 0.70, 0.78, 0.97}, 1.8, 0, 0}},
    {128128, 128, 128, 1, {{0.289, 0.476, 0, 0}, 1.41, 2.43, 2.48}, {{0.36, 0.47, 0, 0}, 1.5, 0, 0}},
    {128256, 128, 256, 1, {{0.474, 0.813, 0, 0}, 2.33, 2.58, 1.74}, {{0.60, 0.80, 0, 0}, 2.5, 0, 0}},
    {64128, 64, 128, 2, {{0.236, 0.324, 0.554, 0.593}, 0.34, 3.74, 3.92}, {{0.33, 0.38, 0.54, 0.68}, 1.3, 0, 0}},
    {64064, 64, 64, 2, {{0.200, 0.235, 0.297, 0.365}, 0.91, 6.33, 3.47}, {{0.285, 0.32, 0.35, 0.41}, 1.2, 0, 0}}};
// What the KD epilogues cost in the same unit: 4 bytes of teacher logits, the exponentials, 2 bytes of dz or the statistics
constexpr double kKdEpilogueBytes = 8;

inline long ms_tiles(const MsTile &t, long M, long N) { return ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

// Estimated time (us) of a grid of `wgs` workgroups with kt K tiles each: full rounds of the chip, then the rest.
inline double ms_tile_time(const MsTile &t, const MsTileTimes &c, long wgs, int kt, double out_bytes) {
    const long slots = 256L * t.per_cu, full = wgs / slots, rest = wgs % slots;
    const double *u = c.us_per_ktile, fix = c.us_round + c.us_out * out_bytes * t.bm * t.bn / 65536.0;
    double est = c.us_call + full * (kt * u[2 * t.per_cu - 1] + fix);
    if (rest > 256) est += kt * (u[2] + (u[3] - u[2]) * (rest - 256) / 256) + fix;
    else if (rest > 0) est += kt * (u[0] + (u[1] - u[0]) * rest / 256) + fix;
    return est;
}

// The two-stage tile by occupancy: 256 x 256 runs about 1.25 times the rate of 128 x 128 where the grid fills whole rounds.
inline int ms_two_stage_tile(long M, long N) {
    const long a = ms_tiles(kTiles[T256], M, N), b = ms_tiles(kTiles[T128], M, N);
    const double ea = (double)a / ((a + 255) / 256 * 256), eb = (double)b / ((b + 511) / 512 * 512);
    return a >= 192 && 1.25 * ea > eb ? T256 : T128;
}
inline bool ms_tile_allowed(int i, int forced, bool mfma16) {
    return forced > 0 ? kTiles[i].code == (forced == kPingPong ? 256 : forced) : (mfma16 || i <= T128);
}

// The tile with the least estimated time, if that is clearly less than the time of the two-stage tile by occupancy.  Ties do
// not decide: without a margin, and with times that did not know the output, 128 x 256 displaced 256 x 256 and 128 x 128 on
// estimates 0.2-6 % apart and lost up to 18 % (2494 x 8192 x 1024 with fp32 output: 60.9 us instead of 51.3; 6500 x 8192 x
// 4096: 386.9 instead of 358.5).  Over the sweep the choice was 1.23 times as fast as the two-stage tile in the mean, never
// more than 4.5 % slower (3 shapes of 1278 by more than 2.5 %), and 0.4 % from the best tile; 256 x 256 was the two-stage kernel there
// for all operands.  With the ping-pong kernel the choice is the same, and 256 x 256 is now and then the better one: of 150 K-contiguous products
// (18 widths of 1024 .. 11008, 256 .. 32768 rows, bf16 output, operands out of the caches) 142 are within 2 % of the best tile, five 2-6 %
// behind, three 20 %, all of these one round of 256 x 256 (us: 1332 x 6144 x 4096 95, best 79; 1537 x 5120 x 5120 119, best 98).
// Every tile adds up K in the same order (one accumulator per element, ascending K), so the choice does not change
// results: the rows of a short micro-batch come out as they do in a long one.
constexpr double kTileMargin = 0.03;
inline int ms_choose_tile(long M, long N, int kt, double out_bytes, int forced, bool mfma16) {
    int best = -1;
    double best_us = 1e30;
    for (int i = 0; i < kNumTiles; ++i) {
        if (!ms_tile_allowed(i, forced, mfma16)) continue;
        const double us = ms_tile_time(kTiles[i], kTiles[i].lin, ms_tiles(kTiles[i], M, N), kt, out_bytes);
        if (us < best_us) { best_us = us; best = i; }
    }
    if (forced > 0) return best < 0 ? T128 : best;
    const int base = ms_two_stage_tile(M, N);
    const double base_us = ms_tile_time(kTiles[base], kTiles[base].lin, ms_tiles(kTiles[base], M, N), kt, out_bytes);
    return best_us < (1 - kTileMargin) * base_us ? best : base;
}

// Weight gradients (small M x N, long K, += into fp32): tile and number of K splits together, by the tiles' estimated time
// plus what the output costs: a read and a write of C without splits, one pass of fp32 atomics per split (1.6 TB/s) and the
// second round of prologues with them.  Above 200 K tiles the operands stream from HBM, where the smaller ring tiles lose
// 10-45 % (M = N = 1024, K = 32768: 221-285 us unsplit, 90-110 us for the tiles left in; 2048 x 1536, K = 14294: 129 us
// against 116) and 128 x 256 12 % (5632 x 1024, K = 14810: 221 us against 198 for 256 x 256 in two splits).
struct MsSplit { int tile, splits; double us; };
inline MsSplit ms_choose_split(long M, long N, int kt, int forced, bool mfma16) {
    MsSplit c = {T128, 1, 1e30};
    for (int i = 0; i < kNumTiles; ++i) {
        if (!ms_tile_allowed(i, forced, mfma16) || (forced <= 0 && kt > 200 && i > T128 && i != R128x256)) continue;
        const double stream = kt > 200 && i == R128x256 ? 1.12 : 1.0;
        for (int sp = 1; sp <= 8 && (sp == 1 || kt / sp >= 8); ++sp) {
            const double est = stream * ms_tile_time(kTiles[i], kTiles[i].wgrad, ms_tiles(kTiles[i], M, N) * sp, (kt + sp - 1) / sp, 0) +
                               (sp > 1 ? 2.5e-6 * M * N * sp + 4.0 : 1.6e-6 * M * N);
            if (est < c.us) c = {i, sp, est};
        }
    }
    return c;
}

// Both products of a linear layer's backward pass (dx [n, in] = dy W, dW [out, in] += dy^T x) as one grid of one tile: which
// tile, how many K splits of the weight gradient and which product comes first (the one with the longer workgroups); tile
// -1: one launch each.
// The times are a fit like kTiles' to such grids: 18 layers (out = 1024 .. 17920, in = 1024 .. 8960, KD chunks with an fp32 dx) x
// 18 token counts from 256 to 46173, operands out of the caches.  d, w: us per K tile of the input / weight gradient (as
// us_per_ktile), each with a part per round, us_out as in MsTileTimes; us_c: the weight gradient's read and write of C, in
// 1e-6 us per element (with splits atomics, as in ms_choose_split).  The best tile of a pair is 1.17 times as fast as two
// launches in the mean, the chosen one 1.15 times (two tiles' estimates may be close); pairs that are not estimated 3 % faster
// than two launches stay apart.  On 22 layers x 39 other token counts (64 .. 46173; 766 pairs) a layer's two products then take 0.85 of the time
// of two launches in the mean; 12 pairs lose more than 1 %, six of them 4-9 %: 600 .. 870 tokens with in >= 5120 (us, apart, together:
// 612 tokens, 1280 x 5120 32.9, 35.7; 861 tokens, 1536 x 8960 64.7, 68.1).  No margin tells those from pairs that gain.
// E.g. us, apart -> together: 2053 tokens, 5632 x 1024 87 -> 64; 1031 tokens, 1280 x 5120 50 -> 43; 32768 tokens, 1536 x 1536
// 285 -> 274; a KD chunk of 1024 tokens, 8192 x 1024 84 -> 67; 4096 tokens, 5632 x 1024 111, together 114: stays apart.
struct MsPairTimes { double d[4], us_round, us_out, us_call, w[4], us_round_w, us_c; };
constexpr MsPairTimes kPairTimes[kNumTiles] = {
    {{0.927, 1.331, 0, 0}, 5.80, 0.71, 0, {1.197, 1.532, 0, 0}, 1.56, 1.02},
    {{0.556, 0.560, 0.641, 0.840}, 3.70, 2.30, 0, {0.694, 0.695, 0.695, 0.949}, 5.36, 0.77},
    {{0.376, 0.428, 0, 0}, 2.76, 0.74, 0, {0.468, 0.572, 0, 0}, 3.26, 0.96},
    {{0.365, 0.717, 0, 0}, 5.44, 0.82, 0, {0.780, 0.888, 0, 0}, 2.53, 1.20},
    {{0.301, 0.301, 0.364, 0.365}, 3.13, 1.87, 0, {0.422, 0.604, 0.604, 0.709}, 2.10, 1.37},
    {{0.140, 0.182, 0.222, 0.222}, 3.28, 2.62, 1.27, {0.289, 0.371, 0.438, 0.438}, 3.00, 1.30}};
constexpr double kPairMargin = 0.03;
struct MsPair { int tile, splits, wgrad_first; double us; };
// us of a K tile while `wgs` workgroups are there
inline double ms_ktile_us(const double *u, int per_cu, long wgs) {
    if (per_cu == 1 || wgs <= 256) return u[0] + (u[1] - u[0]) * (wgs < 256 ? wgs : 256) / 256;
    return u[2] + (u[3] - u[2]) * ((wgs < 512 ? wgs : 512) - 256) / 256;
}
// When `slots` places are done with na workgroups of da us followed by nb of db us
inline double ms_two_kinds(long slots, long na, double da, long nb, double db) {
    const long full = na / slots, more = na % slots;          // `more` places have one more than `full` of the first kind
    const double late = (full + (more > 0)) * da, early = full * da;
    double best = 1e30;
    for (int g = 0; g < 2; ++g) {                             // the last one of the second kind runs in an early or a late place
        const double start = g ? late : early;
        for (long lo = 1, hi = nb; lo <= hi;) {               // the fewest rounds k there with room for nb in all
            const long k = (lo + hi) / 2;
            const double end = start + k * db + 1e-9;
            const long room = (end > early ? (long)((end - early) / db) : 0) * (slots - more) + (end > late ? (long)((end - late) / db) : 0) * more;
            if (room >= nb) { if (end < best) best = end; hi = k - 1; } else lo = k + 1;
        }
    }
    return best > late ? best : late;
}
inline MsPair ms_choose_pair(long n, long out, long in, double dx_bytes, int forced) {
    const int ktd = (int)((out + 63) / 64), ktw = (int)((n + 63) / 64);
    MsPair best = {-1, 1, 0, 1e30};
    for (int i = 0; i < kNumTiles; ++i) {
        if (!ms_tile_allowed(i, forced, true)) continue;
        const MsTile &t = kTiles[i];
        const MsPairTimes &c = kPairTimes[i];
        const long nd = ms_tiles(t, n, in), nw = ms_tiles(t, out, in), slots = 256L * t.per_cu;
        for (int sp = 1; sp <= 8 && (sp == 1 || ktw / sp >= 8); ++sp) {
            const long wgs = nd + nw * sp;
            const double dd = ktd * ms_ktile_us(c.d, t.per_cu, wgs) + c.us_round + c.us_out * dx_bytes * t.bm * t.bn / 65536.0;
            const double dw = (ktw + sp - 1) / sp * ms_ktile_us(c.w, t.per_cu, wgs) + c.us_round_w;
            const bool wf = dw > dd;
            const double us = c.us_call + (wf ? ms_two_kinds(slots, nw * sp, dw, nd, dd) : ms_two_kinds(slots, nd, dd, nw * sp, dw)) +
                              (sp > 1 ? 2.5e-6 * out * in * sp + 4.0 : c.us_c * 1e-6 * out * in);
            if (us < best.us) best = {i, sp, wf, us};
        }
    }
    if (forced > 0) return best;
    const MsTile &t = kTiles[ms_choose_tile(n, in, ktd, dx_bytes, 0, true)];
    const double apart = ms_tile_time(t, t.lin, ms_tiles(t, n, in), ktd, dx_bytes) + ms_choose_split(out, in, ktw, 0, true).us;
    if (best.us > (1 - kPairMargin) * apart) best.tile = -1;
    return best;
}

// The tile for a chunk's student logits [M, N] with a KD epilogue (kt K tiles) and another chunk's teacher logits [M, Nt] (ktt K tiles)
// as one grid, or -1 for one launch each; student_first: the student's workgroups are the longer ones and come first.  kTiles'
// times, with 0.87 for 256 x 256, which is the ping-pong kernel here (the fit is to the two-stage one), and 1.2 for 64 x 128, two of
// which share a CU: their estimate for such a grid is right, while those of the others, which decide against it, are
// 8-17 % too long.  Without the 1.2 they took grids of 640 workgroups, a round and a quarter, and lost to two launches of 128 x 128
// (H = 4096 / 2048, chunks of 8192, 257 .. 320 tokens, loss only, V = 40960: 290 tokens 8 % over two launches; with it 128 x 128 shared,
// 3 % under).  Whole heads of 16 .. 2600 tokens, H = 4096 / 2048, 4096 / 1536, 2048 / 1024, 1024 / 2048, chunks of 4096 / 8192, loss and
// gradients or loss only (384 of them): 0.89 of the time of two launches in the mean, the best tile 0.88; 4 by 1-3 % slower
// than two launches (800 tokens of H = 1024 / 2048 2.8 %, 900 of 4096 / 2048 1.3 %).  At several rounds of the chip the two are even.
constexpr double kPpFactor = 0.87, kShared64x128 = 1.2, kTwoMargin = 0.02;
inline int ms_choose_two(long M, long N, int kt, long Nt, int ktt, int forced, int *student_first = nullptr) {
    int best = -1, first = 0;
    double us = 1e30;
    for (int i = 0; i < kNumTiles; ++i) {
        if (!ms_tile_allowed(i, forced, true)) continue;
        const MsTile &t = kTiles[i];
        const MsTileTimes &c = t.lin;
        const long ns = ms_tiles(t, M, N), nt = ms_tiles(t, M, Nt), slots = 256L * t.per_cu;
        const double u = ms_ktile_us(c.us_per_ktile, t.per_cu, ns + nt), area = t.bm * t.bn / 65536.0, f = i == T256 ? kPpFactor : i == R64x128 ? kShared64x128 : 1.0;
        const double dt = f * (ktt * u + c.us_round + c.us_out * 4 * area), ds = f * (kt * u + c.us_round + c.us_out * kKdEpilogueBytes * area);
        const double est = c.us_call + (dt > ds ? ms_two_kinds(slots, nt, dt, ns, ds) : ms_two_kinds(slots, ns, ds, nt, dt));
        if (est < us) { us = est; best = i; first = ds > dt; }
    }
    if (student_first) *student_first = first;
    if (forced > 0) return best;
    auto apart = [&](long n, int k, double bytes) {
        const int i = ms_choose_tile(M, n, k, bytes, 0, true);
        return (i == T256 ? kPpFactor : 1.0) * ms_tile_time(kTiles[i], kTiles[i].lin, ms_tiles(kTiles[i], M, n), k, bytes);
    };
    return us < (1 - kTwoMargin) * (apart(N, kt, kKdEpilogueBytes) + apart(Nt, ktt, 4)) ? best : -1;
}

// ------------------------------------------------------------------ bf16 attention
// Workgroups of a (heads, sequences, tile levels) grid; the mapping is described at attn_slot (attention_mfma.hip).
constexpr int kAttnChunk = 8;
struct AttnGrid { int S, hpc, M; long blocks; };
constexpr AttnGrid attn_grid(int heads, int n_seqs, int nlevel_max) {
    const int low = heads & -heads, G = low < 8 ? low : 8;          // gcd(heads, 8)
    const int S = 8 / G, hpc = heads / G;
    const int M = ((nlevel_max + S - 1) / S + kAttnChunk - 1) / kAttnChunk * kAttnChunk;   // levels per stripe, whole chunks
    return {S, hpc, M, 8L * M * hpc * n_seqs};
}

// Expected 128-row tiles of a batch, all heads: each sequence's last one is half full in the mean.
inline double ms_attention_tiles(int heads, long n, long n_seqs) { return heads * (n + 64.0 * n_seqs) / 128; }

// Workgroups (of four waves) per CU in the forward and dQ kernels.  At head_dim 64 they fit three times; that gains 2-8 %
// where the grid fills the chip more than once, and 6-20 % where every sequence is a single tile.  Smaller grids of longer
// sequences are spread unevenly, three workgroups on one CU while another has one; causal tiles, whose walks differ, suffer
// longer from it.  Forward, us, three / two per CU: 16 heads bidirectional, 528 tiles 71.8 / 56.5, 656 tiles 70.6 / 87.6; 8
// causal heads, 656 tiles 54.5 / 42.6; 16 / 4 causal heads, 656 tiles 47.0 / 43.7, 1040 70.1 / 69.6, 1312 68.3 / 73.0; 32
// sequences of 64 17.2 / 20.9.
inline int ms_attention_waves(int hd, int heads, int causal, long n, long n_seqs, int max_seqlen) {
    return hd == 64 && (max_seqlen <= 128 || ms_attention_tiles(heads, n, n_seqs) >= (causal ? 1100 : 600)) ? 3 : 2;
}

// Backward pass under grouped-query attention on small batches.  A dK/dV workgroup walks the query tiles (32 rows) that see
// its 128 keys, a dQ workgroup the key tiles (64) of its 128 queries; where there are few walks, the launch waits for the
// longest one.  Its cost in steps of a dK/dV walk, fitted to 276 batches (head_dim 64, 80, 128, 6 .. 32 heads, equal and
// mixed lengths, 300 .. 8192 tokens): the longest walk and what a CU has to do in the mean, and what the parts of a walk
// cost by adding their 128 keys' sums with atomics.  Of a batch the host knows the token count, the number of sequences and
// a bound on their length; walks are taken to be half as long as that bound and half as the mean says.
//   parts: into how many parts of at least 8 query tiles a dK/dV walk is cut.  8 / 2 heads of 128, whole backward in us,
//     unsplit -> cut: one sequence of 620 tokens 66.2 -> 53.4, 2053 tokens in two 139 -> 103; four equal ones of 1024
//     stay unsplit (102.6; cut in three 125), and so do very many short ones.
//   two_way_dq: the keys of 64 queries are split over two wave pairs.  Such a workgroup has a CU to itself (128 KB of
//     LDS), also where it finds no tile of its own, so the grid has to be small, or small next to the walk that it halves:
//     2053 tokens in two 103 -> 85; 32 x 64 tokens 59.6 (with the split 76), 2048 tokens next to 500 single ones 504
//     (819).  Over the batches it loses nowhere more than 0.5 %.
// Without groups neither is done: there a sequence's gradients do not depend on what else is in the batch.  Under
// grouped-query attention they do: dK and dV are sums of atomics in any case, and the order in which dQ adds up its keys
// follows from this rule, that is from the batch.
struct AttnSplit { int parts; bool two_way_dq; };
inline AttnSplit ms_attention_split(int causal, int nq, int nkv, long n, long n_seqs, int max_seqlen) {
    AttnSplit a = {1, false};
    if (nq <= nkv || n <= 0 || n_seqs <= 0 || max_seqlen <= 0) return a;
    const double walks = ms_attention_tiles(nq, n, n_seqs);
    const double length = n_seqs > 1 ? 0.5 * max_seqlen + 0.5 * n / n_seqs : max_seqlen;
    const int longest = (max_seqlen + 31) / 32;
    const double mean = walks * (length / (causal ? 64 : 32) + 0.5) / 256;
    auto cost = [&](int p) { return hypot((longest + p - 1) / p, 1.5 * mean) + 9.0 * walks * p / 256; };
    const long blocks_kv = attn_grid(nq, (int)n_seqs, (max_seqlen + 127) / 128).blocks;
    double best = 0.92 * cost(1);                       // a cut has to be worth 8 %, the error of the fit
    for (int p = 2; longest / p >= 8 && ms_launch_fits(blocks_kv * p, 256); ++p)
        if (cost(p) < best) { best = cost(p); a.parts = p; }
    const int levels = (max_seqlen + 63) / 64;
    const long blocks_dq = attn_grid(nq, (int)n_seqs, levels).blocks;
    a.two_way_dq = walks < 290 && blocks_dq <= (levels * 40L > 512 ? levels * 40L : 512);
    return a;
}

// ------------------------------------------------------------------ AdamW
// Whether the fp32 state (weights, two moments, gradients: 16 bytes per parameter) is read and written non-temporally.  Above
// 80 MB the rest of a training step has pushed it out of the 256 MB Infinity Cache, and keeping it out of the caches is
// faster (three states in turn, us, non-temporal / default: 8 M parameters 47.9 / 54.3, 16 M 89 / 105, 40 M 227 / 258);
// below, a small model's state is still there (2 M 12.4 / 11.8, 4 M 25.1 / 21.0).
constexpr bool ms_adamw_streams(long n) { return 16 * n > 80L * 1000 * 1000; }
