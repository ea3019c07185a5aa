// tiles.hpp -- several sweeps per launch on LDS tiles with recomputed halos
// (tiles.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "fold.hpp"
#include "kernels.hpp"

namespace potts {

constexpr uint32_t kTileMaxSweeps = 8;
constexpr uint32_t kTileMaxL = 65520;
constexpr size_t kTileMaxLds = 155u * 1024u;  // dynamic LDS of one tile (its update's table, up to 5 KB, is static)

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
  const HbTable *heatbath;  // device: the heat bath's draw table; null: Metropolis
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
  uint64_t total;            // many lattices per launch (TileRun): sweeps of the whole run
};

// Sets the shape fields for p.L and p.q; false when no launch of it exists.
bool set_tile_shape(TileParams &p, uint32_t tx, uint32_t ty, uint32_t sweeps);
// The shape that a call of nsweeps sweeps of an L x L lattice takes least time
// with, by a model of one launch (tiles.hip).
bool auto_tile_shape(TileParams &p, int64_t nsweeps);
hipError_t launch_tiles(const TileParams &p, hipStream_t stream);

// Many lattices per launch: launch `turn` runs sweeps turn * sweeps .. of every
// job that has them left (TileParams::total), from src to dst on even turns and
// back on odd ones, into the halves of parts in turn, and folds the turn
// before.  A workgroup finds its job and tile (or kTileFold | fold workgroup)
// in a table.
struct TileRef {
  uint32_t job, tile;
};
constexpr uint32_t kTileFold = 0x80000000u;

struct TileTable {
  const TileParams *jobs;
  const TileRef *refs;
  uint32_t turn;
};

// One group of such jobs (one comparison class and table form): `refs` holds
// the tiles' entries, then (from ntiles) the folds'.
struct TileRun {
  uint32_t qc = 0;      // comparison class: q <= 16, <= 64, <= 128, <= 256
  bool wide = false;
  std::vector<TileParams> jobs;
  std::vector<TileRef> refs;
  uint32_t ntiles = 0, turns = 0;
  size_t parts_words = 0;  // totals of all jobs
  uint32_t ni = 0, waves = 0;
  size_t lds = 0;
};

// What the routes of small lattices take, in microseconds, so that a batch or an
// iteration of the serving loop goes the faster way (tiles.hip: the figures).
struct SweepJob {
  uint32_t L, q;
  uint64_t sweeps, cap;  // cap: slots of its record ring
};
float tile_run_us(const std::vector<SweepJob> &jobs);  // one TileRun; 0: it has no shape
float resident_us(const std::vector<SweepJob> &jobs);  // one launch of the LDS-resident kernel
float strip_us(const std::vector<SweepJob> &jobs);     // a launch per colour and sweep
// With as many jobs, the LDS-resident launch has a workgroup on every CU, and no
// halo to recompute: tiles are not considered (256 jobs of L = 64 / 128 / 256, 100
// sweeps, q = 9: 0.30 / 0.77 / 2.60 ms resident, 0.74 / 1.47 / 4.58 on tiles).
constexpr size_t kTileJobs = 256;
// Tiles are taken when their estimate is this much below the other route's,
// which covers the errors of both.
constexpr float kTileMargin = 0.9f;

// Adds a lattice of L % 4 == 0 to the run: nsweeps sweeps from t0, lattice in
// `spins`, `other` a buffer of its size, records to ring.
void add_tile_job(TileRun &r, uint8_t *spins, uint8_t *other, uint32_t L, uint32_t q, uint64_t seed,
                  const uint32_t thr[4], uint64_t t0, uint64_t nsweeps, unsigned long long *ring, uint64_t cap);
// Picks the run's tile shape, lays out its table and counts its totals.
bool plan_tile_run(TileRun &r);
// parts: device memory for parts_words words
void place_tile_run(TileRun &r, uint32_t *parts);
// the jobs whose lattice ends in `other` (an odd number of turns)
bool tile_job_odd(const TileParams &p);
// All turns of the run, from the run's jobs and refs copied to the device.
hipError_t launch_tile_run(const TileRun &r, const TileParams *jobs, const TileRef *refs, hipStream_t stream);

}  // namespace potts
