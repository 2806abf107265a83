// Reorder-gather fused with the cost table for 32- and 256-column blocks (see fused.hip).  On the search's route for these the
// reordered weights and sensitivities are outputs: they are written on the way, so that a weight is read (6 bytes) and
// written (6 bytes) once, where gather and cost table one after the other read them twice.  Bound by HBM with few candidates, by
// vector issue with many.  Searches of two 8B-shaped layers, two passes -> one: 64 x 256 blocks, eight candidates 2560 -> 1919 us (gather and
// table 1760 -> 1120); 128 x 256, four 2040 -> 1828; 128 x 32, four 2270 -> 1971; 1024 x 1024, 256-column blocks 113 -> 106.
// The line: blocks of 512 columns, whose lane groups are a whole wave, and of 8 and 16, a lane or two, keep the two passes.  No instance
// of this kernel was built or measured for them: the octet sums of a row of 16384 elements (4 B per candidate and block column) would
// take 72 KiB of LDS at nine candidates in 8-column blocks, beside 96 KiB for the row.
#include "fused_core.hpp"

using namespace sbits;

int sbits_launch_fused_copies(int n, int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a)
{
    return n == 32 ? launch_fused_l<4>(K, z0, ctx, a) : launch_fused_l<32>(K, z0, ctx, a);
}
