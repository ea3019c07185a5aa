// fold.hpp -- record totals that workgroups store without atomics, and their
// sum into the record ring by extra workgroups of a later launch.
//
// A launch's workgroups all end at about the same time; adding their totals to
// one record (one or two cache lines) with 64-bit atomics then serializes
// them: 1024 workgroups of the cubic kernel took 19 us a half sweep that way,
// against 9 us of work.  Each workgroup stores its totals as a part of its own
// instead, and the fold runs beside the next sweep's work.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace potts {

// The parts of one or more finished sweeps: sweep s, part b, word w at
// ((s * nparts + b) * n + w).
struct RecordFold {
  uint32_t *parts;
  uint32_t nparts;
  uint32_t n;                // words of a record
  uint32_t comp;             // the first comp words hold differing neighbours: bonds - their sum goes to the ring
  bool shared;               // parts that several workgroups add to: cleared once read
  uint32_t nsweeps;          // 0: nothing to fold
  uint64_t t0;               // the first sweep; record of t0 + s to ring slot (t0 + s) % cap
  unsigned long long *ring;
  uint64_t cap;              // a power of two, at least nsweeps
  uint64_t bonds;
  unsigned long long *mirror;  // host memory: the last sweep's record once more, or null
};

// Words of one sweep that a workgroup of the fold sums: 8 lanes side by side (4
// where a record is that short), the parts over the other lanes.  (A
// workgroup for all words took 40 us for 256 parts at q = 200, longer than the
// launch it ran beside.)
constexpr uint32_t kFoldWords = 8;

__host__ __device__ inline uint32_t fold_width(uint32_t n) { return n <= 4 ? 4u : kFoldWords; }

__host__ __device__ inline uint32_t fold_groups(const RecordFold &f) {
  return f.nsweeps * ((f.n + fold_width(f.n) - 1u) / fold_width(f.n));
}

// Workgroup g of the fold; acc: kFoldWords words of LDS; blockDim.x a multiple
// of kFoldWords.
__device__ __forceinline__ void fold_part(const RecordFold &f, uint32_t g, unsigned long long *acc) {
  const uint32_t n = f.n, width = fold_width(n), per = (n + width - 1u) / width;
  const uint32_t lane = threadIdx.x & (width - 1u), row = threadIdx.x / width, rows = blockDim.x / width;
  const uint32_t s = g / per, w = (g - s * per) * width + lane;
  if (threadIdx.x < kFoldWords) acc[threadIdx.x] = 0;
  __syncthreads();
  if (w < n) {
    uint32_t *at = f.parts + (size_t)s * f.nparts * n + w;
    unsigned long long sum = 0;
    // sixteen reads in flight: the parts come from other XCDs' workgroups
#pragma unroll 16
    for (uint32_t b = row; b < f.nparts; b += rows) sum += at[(size_t)b * n];
    if (f.shared)
      for (uint32_t b = row; b < f.nparts; b += rows) at[(size_t)b * n] = 0;
    if (sum) atomicAdd(&acc[lane], sum);
  }
  __syncthreads();
  if (row == 0 && w < n) {
    const unsigned long long total = w < f.comp ? f.bonds - acc[lane] : acc[lane];
    f.ring[((f.t0 + s) & (f.cap - 1)) * (uint64_t)n + w] = total;
    if (f.mirror && s + 1 == f.nsweeps) f.mirror[w] = total;
  }
}

// The fold as a launch of its own, after the last sweep of a call.
hipError_t launch_record_fold(const RecordFold &f, hipStream_t stream);

}  // namespace potts
