// edge.hpp -- plane rows whose L/2 sites are no multiple of the 16-byte item
// (L % 32 != 0): the last item of a row is partial.
//
// A row is stored in a pitch of whole items.  The sites past the row's end are
// updated like the others (with whatever neighbours the padding holds), but
// not counted; the wrap to the row's other end is put right in registers, so no
// ghost bytes are kept in memory:
//  - O == 1 (right neighbour): the side dword of a row's last item is its first
//    one; its byte 0 goes to the byte behind the last site.
//  - O == 0 (left neighbour): the side dword of the first item holds the row's
//    last site, in byte 3 or, when L/2 % 4 == 2, in byte 1: shifted up.
// The padding only ever holds values below q: it starts as zeros, and a site
// keeps its value or takes a proposal.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.hpp"
#include "sweep_row.hpp"

namespace potts {
namespace row {

// A lane's masks for its item at packed column col of rows of `half` sites.
struct Edge {
  uint32_t valid[4];  // bytes that are sites
  uint32_t behind[4]; // the byte behind the last site (none in a whole item)
  uint32_t shift;     // of the left side dword
  uint32_t missing;   // bytes that are no sites
};

__device__ __forceinline__ Edge edge_of(uint32_t col, uint32_t half) {
  Edge e;
  const uint32_t n = half - col < 16u ? half - col : 16u;
  e.missing = 16u - n;
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i) {
    const uint32_t in = n > 4u * i ? n - 4u * i : 0u;  // sites in this dword and the ones after it
    e.valid[i] = in >= 4u ? 0xFFFFFFFFu : (1u << (8u * in)) - 1u;
    e.behind[i] = n < 16u && n >= 4u * i && in < 4u ? 0xFFu << (8u * in) : 0u;
  }
  e.shift = col == 0 && (half & 2u) ? 16u : 0u;
  return e;
}

// packed column of the dword that holds the row's last site
__device__ __forceinline__ uint32_t last_dword(uint32_t half) { return (half - 1u) & ~3u; }

// passive row p with the wrapped byte behind its last site (O == 1)
__device__ __forceinline__ u32x4 with_wrap(const Edge &e, u32x4 p, uint32_t side) {
  const uint32_t first = perm(side, side, 0u);
  return u32x4{bfi(e.behind[0], first, p.x), bfi(e.behind[1], first, p.y), bfi(e.behind[2], first, p.z),
               bfi(e.behind[3], first, p.w)};
}

}  // namespace row
}  // namespace potts
