// How many workgroups the resident search takes.
#pragma once

#include <stdint.h>

namespace sbits {

// Workgroups of a search over N blocks on a device (or partition) of `cus` CUs: 2048 blocks each (four to a thread) up to 32
// workgroups, beyond that 4096, the most their registers hold (13 k blocks, 15 iterations: 181 us with 7 workgroups, 199
// with 4, 176 with 13; 27 k: 271 with 13, 300 with 7, 266 with 26; 107 k: 355 with 26, 457 with 64; below 4096 blocks one would
// do, 210 us for 4096, but two take 230 only).  At most half of the CUs, one of them takes one
// workgroup, so that two searches fit side by side: workgroups that have no place at the same time wait for each other in
// vain, and one of them does it all.  Larger tables live in memory then (4.2 M blocks: 3.6 ms; 4.9 ms with a launch per round).
// A single step over a table in memory is a pass or two over it and needs a third of the registers, so beyond 2 M blocks it
// takes a workgroup per 16384 blocks, up to twice as many (16.7 M blocks: 371 us, 533 with 128, 535 with a launch per round;
// 1 M: 76 and 72).
inline unsigned search_wgs(int64_t N, bool step, int cus)
{
    const int64_t g = N <= 32 * 2048 ? (N + 2047) / 2048 : (N + 4095) / 4096, half = cus / 2 < 1 ? 1 : cus / 2 < 128 ? cus / 2 : 128;
    int64_t most = half;
    if (step && N / 16384 > most) most = N / 16384 < 2 * half ? N / 16384 : 2 * half;
    return (unsigned)(g < most ? g : most);
}

}  // namespace sbits
