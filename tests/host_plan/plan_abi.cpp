// C entry points around the launch rules (csrc/launch_plan.h) for tests/test_launch_plan.py.
#include "launch_plan.h"

extern "C" long plan_matrix_extent(long outer, long inner, long ld) { return ms_matrix_extent(outer, inner, ld); }
extern "C" int plan_buffer_range_ok(long outer, long inner, long ld, int es) { return ms_buffer_range_ok(outer, inner, ld, es); }
