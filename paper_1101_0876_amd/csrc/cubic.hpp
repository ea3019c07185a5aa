// cubic.hpp -- launch parameters of the colour-split simple-cubic half sweep
// (cubic_packed.hip), used by the state code in cubic.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fold.hpp"

namespace potts {
namespace cube {

struct CubeThr {
  uint32_t v[6];  // thr[d-1], d = 1..6
};

struct CubeLaunch {
  uint8_t *planes;         // plane 0, then plane 1 (plane_bytes each)
  uint64_t plane_bytes;    // L^2 x plane_pitch(L)
  uint32_t L, q;
  uint32_t ipr;            // plane_pitch(L) / 16 items per row
  uint32_t rows;           // R: rows of one item's walk (even, divides L)
  uint32_t nitems;         // ipr * L * (L / R)
  uint32_t groups;         // workgroups of the half sweep (set_groups)
  uint32_t xcd_stride;     // groups / 8 when that is whole, else 0 (set_groups)
  uint32_t k0, k1;         // Philox key
  uint32_t t_lo, t_hi;     // sweep index
  CubeThr thr;
  uint32_t *parts;         // this sweep's totals, groups x (q + 1) words (fold.hpp): differing neighbours, populations
  RecordFold fold;         // the sweep before, folded by the colour-0 launch
};

void set_groups(CubeLaunch &l);
hipError_t launch_packed(const CubeLaunch &l, int colour, hipStream_t stream);
// Row-major cube (L^3 bytes) <-> the two colour planes.
hipError_t launch_pack(const uint8_t *cube, uint8_t *planes, uint32_t L, hipStream_t stream);
hipError_t launch_unpack(const uint8_t *planes, uint8_t *cube, uint32_t L, hipStream_t stream);

}  // namespace cube
}  // namespace potts
