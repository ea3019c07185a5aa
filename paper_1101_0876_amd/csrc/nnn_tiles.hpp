// nnn_tiles.hpp -- sweeps of the first-plus-second-neighbour lattice on LDS
// tiles with recomputed halos (nnn_tiles.hip), used by the state code in
// nnn.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fold.hpp"

namespace potts {
namespace nnn {

constexpr uint32_t kTileMaxSweeps = 4;

struct TileParams {
  const uint8_t *src;  // row-major L x L lattice, L % 12 == 0
  uint8_t *dst;        // the lattice after nsweeps sweeps (another buffer)
  uint32_t L, q;
  uint32_t k0, k1;     // Philox key = seed
  uint64_t t0;         // the launch's first sweep
  uint32_t nsweeps;    // sweeps of this launch, at most `sweeps`
  uint32_t sweeps;           // sweeps the halo is made for
  uint32_t tx, ty;           // tile interior: tx bytes (multiple of 12) x ty rows (multiple of 3)
  uint32_t hx, hy;           // halo: 12 bytes left and right, 3 rows above and below, per sweep
  uint32_t tiles_x, tiles_y; // ceil(L / tx), ceil(L / ty)
  uint32_t lift;             // a multiple of L, at least hx and hy
  uint32_t w_magic;          // ceil(2^32 / items per row)
  uint32_t narrow;           // the region wraps more than once
  uint32_t *parts;           // this launch's totals: tiles x (q + 2) words per sweep (e1, e2, populations)
  RecordFold fold;           // the launch before it
  uint64_t thr[81];          // as potts_nnn_table
};

// Sets the shape that a call of nsweeps sweeps takes least time with; false
// when there is none for p.L and p.q.
bool auto_tile_shape(TileParams &p, int64_t nsweeps);
hipError_t launch_tiles(const TileParams &p, hipStream_t stream);

}  // namespace nnn
}  // namespace potts
