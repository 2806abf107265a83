// Reorder-gather fused with the cost table for 32- and 256-column blocks (see fused.hip).  On the search's route for these the
// reordered weights and sensitivities are outputs: they are written on the way, so that a weight is read (6 bytes) and
// written (6 bytes) once, where gather and cost table one after the other read them twice.  Bound by HBM with few candidates, by
// vector issue with many.  Searches of two 8B-shaped layers, two passes -> one: 64 x 256 blocks, eight candidates 2560 -> 1919 us (gather and
// table 1760 -> 1120); 128 x 256, four 2040 -> 1828; 128 x 32, four 2270 -> 1971; 1024 x 1024, 256-column blocks 113 -> 106.
// The line: blocks of 8, 16 and 512 columns keep the two passes (their lane groups are no part of a row of 16 lanes, or more than half
// a wave).
#include "fused_core.hpp"

using namespace sbits;

int sbits_launch_fused_copies(int n, int K, bool z0, sbits_ctx *ctx, const FusedLaunch &a)
{
    return n == 32 ? launch_fused_l<4>(K, z0, ctx, a) : launch_fused_l<32>(K, z0, ctx, a);
}
