// C entry points around the launch rules (csrc/launch_plan.h) for tests/test_launch_plan.py.
#include "launch_plan.h"

extern "C" long plan_matrix_extent(long outer, long inner, long ld) { return ms_matrix_extent(outer, inner, ld); }
extern "C" int plan_buffer_range_ok(long outer, long inner, long ld, int es) { return ms_buffer_range_ok(outer, inner, ld, es); }
extern "C" int plan_launch_fits(long wgs, int threads) { return ms_launch_fits(wgs, threads); }
extern "C" int plan_f32_attention_tiles(int hd, long n, long n_seqs, long max_seqlen, int nq, int nkv, int heads) {
    return ms_f32_attention_tiles(hd, n, n_seqs, max_seqlen, nq, nkv, heads);
}
extern "C" int plan_tile(long M, long N, int kt, double out_bytes) { return kTiles[ms_choose_tile(M, N, kt, out_bytes, 0, true)].code; }
extern "C" int plan_two_stage_tile(long M, long N) { return kTiles[ms_two_stage_tile(M, N)].code; }
extern "C" int plan_forced_tile(long M, long N, int forced, int mfma16) { return kTiles[ms_choose_tile(M, N, 16, 2, forced, mfma16 != 0)].code; }
extern "C" void plan_split(long M, long N, int kt, int *out) {
    const MsSplit c = ms_choose_split(M, N, kt, 0, true);
    out[0] = kTiles[c.tile].code;
    out[1] = c.splits;
}
extern "C" void plan_attention_split(int causal, int nq, int nkv, long n, long n_seqs, int max_seqlen, int *out) {
    const AttnSplit a = ms_attention_split(causal, nq, nkv, n, n_seqs, max_seqlen);
    out[0] = a.parts;
    out[1] = a.two_way_dq;
}
extern "C" long plan_attention_blocks(int heads, int n_seqs, int levels) { return attn_grid(heads, n_seqs, levels).blocks; }
extern "C" int plan_attention_waves(int hd, int heads, int causal, long n, long n_seqs, int max_seqlen) {
    return ms_attention_waves(hd, heads, causal, n, n_seqs, max_seqlen);
}
extern "C" int plan_adamw_streams(long n) { return ms_adamw_streams(n); }
