// drawn.hpp -- single small lattices swept with their random words drawn
// beforehand by the whole GPU (resident.hip).
//
// A lattice small enough for one workgroup's LDS runs on one CU, and its half
// sweeps are latency-bound there: each item's two Philox blocks are a chain of
// ten dependent rounds.  The words depend only on (seed, site, sweep), so a
// generator kernel spread over every CU draws them for a chunk of sweeps
// first (per 4-site group and half sweep: the four proposals scaled to q, and
// what the four acceptance words accept, a byte each), and the LDS-resident
// kernel loads them ahead instead of computing them.  Same words, same chain:
// results are identical to every other kernel's.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kernels.hpp"

namespace potts {

// the largest lattice (L % 16 == 0): a 4-site group of each colour per lane, two
// where there are more than 1024
constexpr uint32_t kDrawnMaxL = 96;
// sweeps drawn per generator launch
constexpr uint32_t kDrawnChunk = 1024;
// the resident kernel loads the words this many half sweeps ahead, up to
// kDrawnPad sweeps past the chunk's end (read and not used)
constexpr uint32_t kDrawnAhead = 16;
constexpr uint32_t kDrawnPad = kDrawnAhead;
// Whether a call of n sweeps draws its words in the resident kernel itself,
// which saves a launch.  Measured on MI355X (us per sweep, with the launch in
// brackets): L = 64 4.59 at n = 4 (4.7), 3.35 in 6 with the launch; L = 96 7.84 at
// n = 3 (6.8), 9.94 at 2 (10).
constexpr uint32_t kDrawnInline = 4;
inline bool drawn_inline(uint32_t L, int64_t n) { return n <= (L <= 64 ? (int64_t)kDrawnInline : 2); }

bool drawn_fits(uint32_t L, uint32_t q);
// bytes of the word buffer for chunks of up to kDrawnChunk sweeps
size_t drawn_words_bytes(uint32_t L);
// Draws the words of sweeps j.t0 .. j.t0 + j.nsweeps - 1 into words
// (j.nsweeps <= kDrawnChunk).
hipError_t launch_draw_words(const ResidentJob &j, uint32_t *words, hipStream_t stream);
// Runs sweeps j.t0 .. j.t0 + j.nsweeps - 1 of the single lattice j with the
// words launch_draw_words wrote for the same j; null: at most kDrawnInline
// sweeps, drawn by the kernel itself.  mirror: null, or host memory that takes
// the last sweep's record too.
hipError_t launch_resident_drawn(const ResidentJob &j, const uint32_t *words, unsigned long long *mirror,
                                 hipStream_t stream);

}  // namespace potts
