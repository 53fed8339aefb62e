// The forward beside the sort's passes for f32 rows of 4 elements per lane.
#include "hl_fwd_sort.h"

hl_sort_side_fn hl_fwd_sort_f32() { return eb_fwd_srt_passes<4, false>; }
