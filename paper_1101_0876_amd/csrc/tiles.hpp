// tiles.hpp -- several sweeps per launch on LDS tiles with recomputed halos
// (tiles.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fold.hpp"
#include "kernels.hpp"

namespace potts {

constexpr uint32_t kTileMaxSweeps = 8;
constexpr uint32_t kTileMaxL = 65520;
constexpr size_t kTileMaxLds = 158u * 1024u;  // dynamic LDS of one tile (2 KB more are static)

// A launch's totals (fold.hpp): one part of q + 1 words per sweep and tile, or,
// past kTileMaxParts tiles, that many parts that tiles share (tile b adds to
// part b % kTileMaxParts).  Word 0 holds the differing neighbours of the
// colour-1 sites, word 1 + v the sites with value v.
constexpr uint32_t kTileMaxParts = 4096;
__host__ __device__ inline uint32_t tile_parts(uint32_t ntiles) { return ntiles < kTileMaxParts ? ntiles : kTileMaxParts; }

struct TileParams {
  const uint8_t *src;  // row-major L x L lattice
  uint8_t *dst;        // the lattice after nsweeps sweeps (another buffer)
  uint32_t L, q;
  uint32_t k0, k1;     // Philox key = seed
  Thresholds thr;
  uint64_t t0;         // sweep index of the launch's first sweep
  uint32_t nsweeps;    // sweeps of this launch, at most `sweeps`
  // the shape (set_tile_shape)
  uint32_t sweeps;           // sweeps the halo is made for
  uint32_t tx, ty;           // tile interior: tx bytes (multiple of 8) x ty rows (even)
  uint32_t hx, hy;           // halo bytes left and right, rows above and below
  uint32_t tiles_x, tiles_y; // ceil(L / tx), ceil(L / ty)
  uint32_t lift;             // a multiple of L, at least hx and hy
  uint32_t w_magic;          // ceil(2^32 / dwords per region row and plane)
  uint32_t narrow;           // the region wraps more than once
  uint32_t *parts;           // this launch's totals
  RecordFold fold;           // the launch before it, folded by extra workgroups
};

// Sets the shape fields for p.L and p.q; false when no launch of it exists.
bool set_tile_shape(TileParams &p, uint32_t tx, uint32_t ty, uint32_t sweeps);
// The shape that a call of nsweeps sweeps of an L x L lattice takes least time
// with, by a model of one launch (tiles.hip).
bool auto_tile_shape(TileParams &p, int64_t nsweeps);
hipError_t launch_tiles(const TileParams &p, hipStream_t stream);

}  // namespace potts
