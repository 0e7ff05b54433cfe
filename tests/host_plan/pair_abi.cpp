// C entry points of the rules for the two products of a linear layer's backward pass (host code only).
#include "launch_plan.h"

extern "C" {
double pair_two_kinds(long slots, long na, double da, long nb, double db) { return ms_two_kinds(slots, na, da, nb, db); }
void pair_choose(long n, long out, long in, double dx_bytes, int forced, int *tile_splits_first) {
    const MsPair p = ms_choose_pair(n, out, in, dx_bytes, forced);
    tile_splits_first[0] = p.tile < 0 ? -1 : kTiles[p.tile].code;
    tile_splits_first[1] = p.splits;
    tile_splits_first[2] = p.wgrad_first;
}
}
extern "C" int two_choose(long m, long n, int kt, long nt, int ktt, int forced) {
    const int i = ms_choose_two(m, n, kt, nt, ktt, forced);
    return i < 0 ? -1 : kTiles[i].code;
}
extern "C" int two_student_first(long m, long n, int kt, long nt, int ktt) {
    int first = -1;
    ms_choose_two(m, n, kt, nt, ktt, 0, &first);
    return first;
}
