// The forward beside the sort's passes for bf16 rows of 8 elements per lane.
#include "hl_fwd_sort.h"

hl_sort_side_fn hl_fwd_sort_bf16() { return eb_fwd_srt_passes<8, true>; }
