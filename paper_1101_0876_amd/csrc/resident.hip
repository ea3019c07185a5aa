// resident.hip -- LDS-resident multi-sweep kernel for small lattices
// (L % 16 == 0, L*L <= 64 KiB).
//
// One workgroup owns one lattice: it copies the lattice into LDS once, runs
// all requested sweeps there (colour 0, barrier, colour 1, barrier, records),
// and writes the lattice back at the end.  Every sweep's record {e_sat,
// hist[q]} is reduced inside the workgroup and stored directly in its ring
// slot, so one launch replaces 2 x nsweeps launches of the streaming kernel.
// A launch may hold many jobs (one per workgroup), which is how batches of
// small lattices run.
//
// Work item: 8 bytes of one row (4 active sites), updated by the shared
// 4-site row routine (sweep_row.hpp); 512 lanes, so a 64 x 64 lattice gives
// every lane one item per half sweep and each SIMD two waves to overlap.
// Items are ordered so that all rows of one parity come first: a wave then
// usually sees a single byte parity and the parity branch is uniform.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.hpp"
#include "drawn.hpp"
#include "kernels.hpp"
#include "sweep_row.hpp"

namespace potts {
namespace {

using namespace row;

// A single lattice runs 8-byte items on 512 lanes (latency first: a 64 x 64
// lattice gives each lane one item per half sweep and each SIMD two waves);
// a batch runs 16-byte items on 256 lanes per lattice (fewer instructions per
// site, many workgroups per CU).
constexpr int kMaxWaves = 8;

__device__ __forceinline__ u32x4 lds16(const uint8_t *lat, uint32_t off) {
  return *reinterpret_cast<const u32x4 *>(lat + off);
}
__device__ __forceinline__ uint32_t lds4(const uint8_t *lat, uint32_t off) {
  return *reinterpret_cast<const uint32_t *>(lat + off);
}

__device__ __forceinline__ uint2 lds8(const uint8_t *lat, uint32_t off) {
  return *reinterpret_cast<const uint2 *>(lat + off);
}

// One 8-byte row item of the LDS lattice (row y, byte column col): 4 active
// sites.  Returns the differing-neighbour count of its new spins (colour 1).
template <int COLOUR, int O, int CMP, bool PRIV, bool WIDE>
__device__ __forceinline__ uint32_t item_update(uint8_t *lat, const ResidentJob &j, uint32_t y,
                                                uint32_t col, const PhiloxHead &h,
                                                const uint8_t *table, uint8_t *hist,
                                                uint32_t lane_off) {
  const uint32_t L = j.L;
  const uint32_t ro = y * L;
  const uint32_t ru = (y == 0 ? L - 1 : y - 1) * L;
  const uint32_t rd = (y + 1 == L ? 0 : y + 1) * L;
  const uint2 cur = lds8(lat, ro + col);
  const uint2 up = lds8(lat, ru + col);
  const uint2 dn = lds8(lat, rd + col);
  const uint32_t side = O == 0 ? lds4(lat, ro + (col == 0 ? L - 4 : col - 4))
                               : lds4(lat, ro + (col + 8 == L ? 0u : col + 8));
  const Row4 r = update4<COLOUR, O, CMP, WIDE>(
      perm(cur.y, cur.x, kSel<O>), perm(cur.y, cur.x, kSel<O ^ 1>), perm(up.y, up.x, kSel<O>),
      perm(dn.y, dn.x, kSel<O>), side, y * (L >> 2) + (col >> 2), h, j.q, table);
  *reinterpret_cast<uint2 *>(lat + ro + col) = make_uint2(r.out_x, r.out_y);
  if (COLOUR == 1) {
    // every site is final after colour 1: count all 8 bytes
    if (PRIV)
      count_active_private(hist, lane_off, r.out_x, r.out_y);
    else
      count_active_shared(reinterpret_cast<uint32_t *>(hist), r.out_x, r.out_y);
    return __popc(r.nz & 0xF0F0F0F0u);
  }
  return 0;
}

template <int COLOUR, int CMP, bool PRIV, bool WIDE, int BLOCK>
__device__ __forceinline__ uint32_t half_sweep8(uint8_t *lat, const ResidentJob &j, uint64_t t,
                                               const uint8_t *table, uint8_t *hist, uint32_t lane_off) {
  const PhiloxHead h = philox_head((uint32_t)t, (uint32_t)(t >> 32), (uint32_t)COLOUR, j.k0, j.k1);
  const uint32_t L = j.L;
  const uint32_t cpr = L >> 3;                  // 8-byte items per row
  const uint32_t per_parity = (L >> 1) * cpr;   // items in the rows of one parity
  uint32_t nz = 0;
  for (uint32_t i = threadIdx.x; i < 2 * per_parity; i += BLOCK) {
    const uint32_t par = i >= per_parity;
    const uint32_t k = i - par * per_parity;
    const uint32_t rr = k / cpr;
    const uint32_t y = 2 * rr + par;
    const uint32_t col = (k - rr * cpr) * 8u;
    if (((COLOUR + y) & 1u) == 0)
      nz += item_update<COLOUR, 0, CMP, PRIV, WIDE>(lat, j, y, col, h, table, hist, lane_off);
    else
      nz += item_update<COLOUR, 1, CMP, PRIV, WIDE>(lat, j, y, col, h, table, hist, lane_off);
  }
  return nz;
}


// One 16-byte row item of the LDS lattice (row y, byte column col): 8 active
// sites (batches: many lattices per launch, throughput first).
template <int COLOUR, int O, int CMP, bool PRIV, bool WIDE>
__device__ __forceinline__ uint32_t item_update16(uint8_t *lat, const ResidentJob &j, uint32_t y,
                                                uint32_t col, const PhiloxHead &h,
                                                const uint8_t *table, uint8_t *hist,
                                                uint32_t lane_off) {
  const uint32_t L = j.L;
  const uint32_t ro = y * L;
  const uint32_t ru = (y == 0 ? L - 1 : y - 1) * L;
  const uint32_t rd = (y + 1 == L ? 0 : y + 1) * L;
  const u32x4 cur = lds16(lat, ro + col);
  const u32x4 up = lds16(lat, ru + col);
  const u32x4 dn = lds16(lat, rd + col);
  const uint32_t side = O == 0 ? lds4(lat, ro + (col == 0 ? L - 4 : col - 4))
                               : lds4(lat, ro + (col + 16 == L ? 0u : col + 16));
  const Row8 r = update8<COLOUR, O, CMP, WIDE>(
      perm(cur.y, cur.x, kSel<O>), perm(cur.w, cur.z, kSel<O>),
      perm(cur.y, cur.x, kSel<O ^ 1>), perm(cur.w, cur.z, kSel<O ^ 1>),
      perm(up.y, up.x, kSel<O>), perm(up.w, up.z, kSel<O>),
      perm(dn.y, dn.x, kSel<O>), perm(dn.w, dn.z, kSel<O>), side,
      y * (L >> 2) + (col >> 2), h, j.q, table);
  *reinterpret_cast<u32x4 *>(lat + ro + col) = r.out;
  if (COLOUR == 1) {
    if (PRIV)
      count_row_private(hist, lane_off, r.out);
    else
      count_row_shared(reinterpret_cast<uint32_t *>(hist), r.out);
    return __popc(r.nz_lo & 0xF0F0F0F0u) + __popc(r.nz_hi & 0xF0F0F0F0u);
  }
  return 0;
}

template <int COLOUR, int CMP, bool PRIV, bool WIDE, int BLOCK>
__device__ __forceinline__ uint32_t half_sweep16(uint8_t *lat, const ResidentJob &j, uint64_t t,
                                               const uint8_t *table, uint8_t *hist, uint32_t lane_off) {
  const PhiloxHead h = philox_head((uint32_t)t, (uint32_t)(t >> 32), (uint32_t)COLOUR, j.k0, j.k1);
  const uint32_t L = j.L;
  const uint32_t cpr = L >> 4;                  // 16-byte items per row
  const uint32_t per_parity = (L >> 1) * cpr;   // items in the rows of one parity
  uint32_t nz = 0;
  for (uint32_t i = threadIdx.x; i < 2 * per_parity; i += BLOCK) {
    const uint32_t par = i >= per_parity;
    const uint32_t k = i - par * per_parity;
    const uint32_t rr = k / cpr;
    const uint32_t y = 2 * rr + par;
    const uint32_t col = (k - rr * cpr) * 16u;
    if (((COLOUR + y) & 1u) == 0)
      nz += item_update16<COLOUR, 0, CMP, PRIV, WIDE>(lat, j, y, col, h, table, hist, lane_off);
    else
      nz += item_update16<COLOUR, 1, CMP, PRIV, WIDE>(lat, j, y, col, h, table, hist, lane_off);
  }
  return nz;
}


template <int CMP, bool PRIV, bool WIDE, bool NARROW>
__global__ __launch_bounds__(NARROW ? 512 : 256) void resident_kernel(ResidentLaunch p) {
  constexpr int kBlock = NARROW ? 512 : 256;
  constexpr int kWaves = kBlock / 64;
  // table, counters and totals in static LDS (addresses fold into the LDS
  // instructions' offsets); the lattice in dynamic LDS
  __shared__ __align__(16) uint32_t table_words[512];
  constexpr uint32_t kHistWords = PRIV ? 64u * (CMP == 0 ? 16u : kPrivateHistMaxQ) : 256u;
  __shared__ __align__(16) uint32_t hist[kHistWords];  // PRIV: q x 64 lane columns; else q bins
  __shared__ uint32_t partial[256 + kMaxWaves];        // q totals, then kWaves bond sums
  extern __shared__ __align__(16) uint32_t lds[];
  const ResidentJob j = p.jobs ? p.jobs[blockIdx.x] : p.single;
  const uint32_t L = j.L, q = j.q, nbytes = L * L;
  uint8_t *lat = reinterpret_cast<uint8_t *>(lds);
  uint8_t *table = reinterpret_cast<uint8_t *>(table_words);
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint32_t lane_off = lane * 4u;

  fill_accept_table<WIDE>(table, j.thr);
  for (uint32_t off = threadIdx.x * 16u; off < nbytes; off += kBlock * 16u)
    *reinterpret_cast<u32x4 *>(lat + off) = *reinterpret_cast<const u32x4 *>(j.spins + off);
  __syncthreads();

  const uint32_t nh = PRIV ? 64 * q : q;
  for (uint32_t s = 0; s < j.nsweeps; ++s) {
    const uint64_t t = j.t0 + s;
    for (uint32_t i = threadIdx.x; i < nh; i += kBlock) hist[i] = 0;
    uint8_t *hb = reinterpret_cast<uint8_t *>(hist);
    if (NARROW)
      half_sweep8<0, CMP, PRIV, WIDE, kBlock>(lat, j, t, table, hb, lane_off);
    else
      half_sweep16<0, CMP, PRIV, WIDE, kBlock>(lat, j, t, table, hb, lane_off);
    __syncthreads();
    const uint32_t nz = NARROW ? half_sweep8<1, CMP, PRIV, WIDE, kBlock>(lat, j, t, table, hb, lane_off)
                               : half_sweep16<1, CMP, PRIV, WIDE, kBlock>(lat, j, t, table, hb, lane_off);
    const uint32_t nz_w = wave_sum(nz);
    __syncthreads();
    if (PRIV) {
      for (uint32_t v = wave; v < q; v += kWaves) {
        const uint32_t c = wave_sum(hist[v * 64u + lane]);
        if (lane == 0) partial[v] = c;
      }
    } else {
      for (uint32_t v = threadIdx.x; v < q; v += kBlock) partial[v] = hist[v];
    }
    if (lane == 0) partial[q + wave] = nz_w;
    __syncthreads();
    unsigned long long *rec = j.ring + (t & (j.cap - 1)) * (uint64_t)(q + 1);
    for (uint32_t v = threadIdx.x; v < q; v += kBlock) rec[1 + v] = partial[v];
    if (threadIdx.x == 0) {
      uint32_t nzt = 0;
      for (int w = 0; w < kWaves; ++w) nzt += partial[q + w];
      // each colour-1 site has 4 bonds; e_sat = 4 * (N/2) - differing neighbours
      rec[0] = (unsigned long long)(2u * nbytes - nzt);
    }
  }

  __syncthreads();
  for (uint32_t off = threadIdx.x * 16u; off < nbytes; off += kBlock * 16u)
    *reinterpret_cast<u32x4 *>(j.spins + off) = *reinterpret_cast<const u32x4 *>(lat + off);
}

// ---- pre-drawn words (drawn.hpp) ---------------------------------------------

// A site's acceptance word against all thresholds at once.  d = (differing
// neighbours of the proposal) - (of the current value): accepted when d <= 0 or
// word < thr[d - 1].  MONO (thr does not rise with d, as exp(-beta d)): the
// largest accepted d, kept as the byte 0x70 - 16 d; else the bits of the d = 1
// .. 4 that are accepted at bits 4 .. 7 of the byte (0 .. 3: d = -3 .. 0).
template <bool MONO>
__device__ __forceinline__ uint32_t accept_level(uint32_t w, const Thresholds &thr) {
  uint32_t n = 0;
#pragma unroll
  for (int d = 0; d < 4; ++d) n = MONO ? n + (w < thr.v[d]) : n | (w < thr.v[d] ? 16u << d : 0u);
  return MONO ? 0x70u - 16u * n : n | 15u;
}

// Words of one 4-site group (a dword of a plane): packed proposals and levels.
template <bool MONO>
__device__ __forceinline__ uint2 group_words(const Words &b0, const Words &b1, uint32_t q, const Thresholds &thr) {
  return make_uint2(
      pack4(scale_to_q(b0.w0, q), scale_to_q(b0.w2, q), scale_to_q(b1.w0, q), scale_to_q(b1.w2, q)),
      pack4(accept_level<MONO>(b0.w1, thr), accept_level<MONO>(b0.w3, thr), accept_level<MONO>(b1.w1, thr),
            accept_level<MONO>(b1.w3, thr)));
}

// One thread per (8 bytes of the row-major lattice, half sweep of the chunk):
// half sweep hs is colour hs & 1 of sweep t0 + hs / 2.
template <bool MONO>
__global__ __launch_bounds__(256) void draw_words_kernel(ResidentJob j, uint32_t ngroups, uint2 *words) {
  const uint32_t hs = blockIdx.y;
  const uint32_t g = blockIdx.x * 256u + threadIdx.x;
  if (g >= ngroups) return;
  const uint64_t t = j.t0 + (hs >> 1);
  const PhiloxHead h = philox_head((uint32_t)t, (uint32_t)(t >> 32), hs & 1u, j.k0, j.k1);
  Words b0, b1;
  philox_tail2(h.a0 ^ (2u * g), h.a0 ^ (2u * g + 1u), h, b0, b1);
  words[(size_t)hs * ngroups + g] = group_words<MONO>(b0, b1, j.q, j.thr);
}

// Per byte, 16 x the number of the four neighbours that differ from v, plus c.
template <int CMP>
__device__ __forceinline__ uint32_t differing(uint32_t v, uint32_t u, uint32_t d, uint32_t l, uint32_t r, uint32_t c) {
  auto f = [](uint32_t x) {
    if (CMP == 0) return (x + 0x0F0F0F0Fu) & 0x10101010u;
    if (CMP == 1) return ((x + 0x7F7F7F7Fu) >> 3) & 0x10101010u;
    return ((((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) >> 3) & 0x10101010u;
  };
  return (f(v ^ l) + f(v ^ r) + c) + f(v ^ u) + f(v ^ d);
}

// The four sites of one dword: s, words w (proposals, levels), the neighbour
// dwords; returns the new dword, adds 16 x its differing neighbours to nz.
template <int COLOUR, int CMP, bool MONO>
__device__ __forceinline__ uint32_t drawn_sites(uint32_t s, uint2 w, uint32_t u, uint32_t d, uint32_t l, uint32_t r,
                                                uint32_t &nz) {
  const uint32_t ps = differing<CMP>(s, u, d, l, r, 0u);
  uint32_t rej, pk;  // bit 7 of the bytes refused
  if (MONO) {
    // byte-wise: level byte a = 16 (7 - level + differing(k)); refused when a -
    // ps >= 0x80, which needs a >= 0x80; bit 7 set beforehand keeps every
    // byte's difference above 0
    const uint32_t a = differing<CMP>(w.x, u, d, l, r, w.y);
    pk = a - w.y;
    rej = a & ((a | 0x80808080u) - ps);  // bit 7; the others are masked below
  } else {
    pk = differing<CMP>(w.x, u, d, l, r, 0u);
    const uint32_t gap = ((pk + 0x40404040u) - ps) >> 4;  // d + 4 per byte
    rej = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint32_t bits = byte_of(w.y, b) << 1 | 1u;  // bit d + 4: accepted
      rej |= (~(bits >> (byte_of(gap, b) & 15u)) & 1u) << (8 * b + 7);
    }
  }
  // one v_and_or_b32, which takes one constant from a scalar register
  uint32_t first = 0x03020100u;
  asm("" : "+v"(first));
  const uint32_t sel = ((rej >> 5) & 0x04040404u) | first;
  if (COLOUR == 1) nz = __builtin_amdgcn_sad_u8(perm(ps, pk, sel), 0u, nz);
  return perm(s, w.x, sel);
}

// sweeps between two reductions of the counters
constexpr uint32_t kDrawnGroup = 8;
static_assert(kDrawnAhead == 2 * kDrawnGroup, "a group of sweeps is one pass of the unrolled loop");

// counter words of one sweep: 64 lane columns of differing neighbours, then 64
// per value (PRIV; q <= 16: room for 16 values, so that a set's place is a
// constant and folds into the instructions), or q shared bins
__host__ __device__ inline uint32_t drawn_set_words(uint32_t q, bool priv) {
  return 64u + (priv ? 64u * 16u : (q + 3u) & ~3u);
}

// One lattice on one CU, its words drawn before (drawn.hpp) or, for short calls
// (INLINE), by the lanes themselves, at half the launches.  A lane owns 16 bytes
// of a row: two dwords of each colour plane, in registers; the planes in LDS
// serve the neighbours.  A half sweep of L = 64 issues about 60 instructions on
// each of four waves, one per SIMD, and waits for three LDS reads, one write
// and a barrier.  What else was on that path, and is not any more: the
// acceptance table in LDS (the levels compare in registers), re-splitting the
// row's bytes by colour, the counting, which the next half sweep does while
// its reads are in flight, and the reduction into a record, done for eight
// sweeps at once.  The words of the next eight sweeps load into registers
// meanwhile: sixteen half sweeps ahead, since one takes less than a fifth of
// the time of an access to memory.
template <int CMP, bool PRIV, bool MONO, bool INLINE, int D>
__global__ __launch_bounds__(1024) void drawn_kernel(ResidentJob j, const uint2 *words,
                                                      unsigned long long *mirror) {
  struct Group {
    uint32_t v[D];
  };
  struct GroupWords {
    uint2 v[D];
  };
  extern __shared__ __align__(16) uint32_t lds[];
  const uint32_t L = j.L, q = j.q, n = L * L / (8u * D), W = L >> 3;  // items; dwords per row and plane
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t has = threadIdx.x < n;
  const uint32_t me = has ? threadIdx.x : 0u;  // lanes past the last item repeat the first, uncounted
  const uint32_t i = D * me, y = i / W;
  const uint32_t set = drawn_set_words(q, PRIV);
  uint32_t *planes[2] = {lds + kDrawnGroup * set, lds + kDrawnGroup * set + D * n};
  const uint32_t up = y == 0 ? i + (L - 1u) * W : i - W, dn = y + 1u == L ? i - (L - 1u) * W : i + W;
  const uint32_t left = i == y * W ? i + W - 1u : i - 1u, right = i + D == (y + 1u) * W ? i + D - W : i + D;
  const bool odd = y & 1u;
  // colour c, row y: O = (c + y) & 1, the passive dword beside the item and the
  // bytes of {neighbour dword, own dword} that make the second neighbours
  const uint32_t side[2] = {odd ? right : left, odd ? left : right};
  const uint32_t pick[2] = {odd ? 0x04030201u : 0x02010007u, odd ? 0x02010007u : 0x04030201u};

  GroupWords w[INLINE ? 1 : kDrawnAhead];
  const GroupWords *from = reinterpret_cast<const GroupWords *>(words) + me;
  if (!INLINE) {
#pragma unroll
    for (uint32_t h = 0; h < kDrawnAhead; ++h) w[h] = from[(size_t)h * n];
  }
  // even bytes of an even row are colour 0, of an odd row colour 1
  Group own[2];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint2 row = reinterpret_cast<const uint2 *>(j.spins)[i + k];
    const uint32_t even = perm(row.y, row.x, kSel<0>), od = perm(row.y, row.x, kSel<1>);
    own[0].v[k] = odd ? od : even;
    own[1].v[k] = odd ? even : od;
  }
  const uint32_t sets = min(j.nsweeps, kDrawnGroup);
  for (uint32_t k = threadIdx.x; k < sets * set / 4u; k += blockDim.x)
    reinterpret_cast<u32x4 *>(lds)[k] = u32x4{0, 0, 0, 0};
  auto group_at = [](uint32_t *plane, uint32_t at) -> Group & { return *reinterpret_cast<Group *>(plane + at); };
  group_at(planes[0], i) = own[0];
  group_at(planes[1], i) = own[1];

  // the group's values into the populations of counter set b
  const uint32_t lane_off = lane * 4u;
  auto count = [&](const Group &g, uint32_t b) {
    uint8_t *pops = reinterpret_cast<uint8_t *>(lds) + 4u * (b * set + 64u);
#pragma unroll
    for (uint32_t k = 0; k < 4 * D; ++k) {
      const uint32_t v = g.v[k >> 2];
      const uint32_t at = PRIV ? perm(v, lane_off, 0x0C0C0000u | ((4u + (k & 3u)) << 8)) : 4u * byte_of(v, k & 3u);
      atomicAdd(reinterpret_cast<uint32_t *>(pops + at), has);
    }
  };
  // half sweep of colour C, counter set b; `counts`: the values of the half
  // sweep before are counted (into b for colour 1, the set before for 0)
  uint32_t nz = 0;
  auto half = [&](auto colour, const GroupWords &hw, uint32_t b, bool counts) {
    constexpr int C = decltype(colour)::value;
    uint32_t *pas = planes[1 - C];
    const Group u = group_at(pas, up), d = group_at(pas, dn);
    const uint32_t sd = pas[side[C]];
    if (counts) {
      count(own[1 - C], C ? b : b - 1u);
      if (C == 0) atomicAdd(&lds[(b - 1u) * set + lane], nz * has);
    }
    const Group p = own[1 - C];
    const bool O = (C == 1) != odd;
    nz = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const uint32_t next = k + 1 < D ? p.v[(k + 1) % D] : sd, prev = k > 0 ? p.v[(k + D - 1) % D] : sd;
      const uint32_t x = perm(D == 1 ? sd : O ? next : prev, p.v[k], pick[C]);
      own[C].v[k] = drawn_sites<C, CMP, MONO>(own[C].v[k], hw.v[k], u.v[k], d.v[k], p.v[k], x, nz);
    }
    group_at(planes[C], i) = own[C];
    __syncthreads();
  };
  // the records of sweeps s0 .. s0 + m - 1 from the counter sets, which are
  // cleared; four lanes per 64-lane column.  On a ring of fewer slots only the
  // last `cap` of them are stored: two sweeps of the group that share a slot are
  // written by different lanes, in no order.
  auto records = [&](uint32_t s0, uint32_t m) {
    const uint32_t skip = j.cap < m ? m - (uint32_t)j.cap : 0u;
    count(own[1], m - 1u);
    atomicAdd(&lds[(m - 1u) * set + lane], nz * has);
    __syncthreads();
    const uint32_t n1 = q + 1u, per = PRIV ? n1 : 1u, columns = 4u * m * per;
    for (uint32_t c4 = threadIdx.x; c4 < columns; c4 += blockDim.x) {
      const uint32_t c = c4 >> 2, s = PRIV ? c / n1 : c, v = c - s * per;
      u32x4 *col = reinterpret_cast<u32x4 *>(lds + s * set + 64u * v) + 4u * (c4 & 3u);
      const u32x4 t = col[0] + col[1] + col[2] + col[3];
      for (int k = 0; k < 4; ++k) col[k] = u32x4{0, 0, 0, 0};
      uint32_t sum = t.x + t.y + t.z + t.w;
      sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
      sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
      unsigned long long *rec = j.ring + ((j.t0 + s0 + s) & (j.cap - 1)) * (uint64_t)n1;
      // each colour-1 site has 4 bonds; e_sat = 4 * (N/2) - differing neighbours
      const uint32_t total = v == 0 ? 2u * L * L - (sum >> 4) : sum;
      if ((c4 & 3u) == 0 && s >= skip) rec[v] = total;
      if ((c4 & 3u) == 0 && mirror && s0 + s + 1 == j.nsweeps) mirror[v] = total;
    }
    if (!PRIV)
      for (uint32_t c = threadIdx.x; c < m * q; c += blockDim.x) {
        const uint32_t s = c / q, v = c - s * q;
        uint32_t *bin = lds + s * set + 64u + v;
        if (s >= skip) j.ring[((j.t0 + s0 + s) & (j.cap - 1)) * (uint64_t)n1 + 1u + v] = *bin;
        if (mirror && s0 + s + 1 == j.nsweeps) mirror[1u + v] = *bin;
        *bin = 0;
      }
  };
  constexpr std::integral_constant<int, 0> k0{};
  constexpr std::integral_constant<int, 1> k1{};
  __syncthreads();
  if (INLINE) {
    auto draw = [&](uint32_t s, uint32_t colour) {
      const uint64_t t = j.t0 + s;
      const PhiloxHead h = philox_head((uint32_t)t, (uint32_t)(t >> 32), colour, j.k0, j.k1);
      GroupWords r;
#pragma unroll
      for (int k = 0; k < D; ++k) {
        Words b0, b1;
        philox_tail2(h.a0 ^ (2u * (i + k)), h.a0 ^ (2u * (i + k) + 1u), h, b0, b1);
        r.v[k] = group_words<MONO>(b0, b1, q, j.thr);
      }
      return r;
    };
    for (uint32_t s = 0; s < j.nsweeps; ++s) {  // at most kDrawnGroup
      half(k0, draw(s, 0u), s, s > 0);
      half(k1, draw(s, 1u), s, true);
    }
    records(0, j.nsweeps);
  } else {
    const uint32_t groups = j.nsweeps / kDrawnGroup, rest = j.nsweeps % kDrawnGroup;
    for (uint32_t g = 0; g < groups; ++g) {
      from += (size_t)kDrawnAhead * n;  // the next group's (the last reads the padding)
#pragma unroll
      for (uint32_t s = 0; s < kDrawnGroup; ++s) {
        half(k0, w[2 * s], s, s > 0);
        w[2 * s] = from[(size_t)(2 * s) * n];
        half(k1, w[2 * s + 1], s, true);
        w[2 * s + 1] = from[(size_t)(2 * s + 1) * n];
      }
      records(g * kDrawnGroup, kDrawnGroup);
    }
#pragma unroll
    for (uint32_t s = 0; s < kDrawnGroup - 1; ++s) {
      if (s >= rest) break;
      half(k0, w[2 * s], s, s > 0);
      half(k1, w[2 * s + 1], s, true);
    }
    if (rest) records(groups * kDrawnGroup, rest);
  }
  if (has)
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const uint32_t even = odd ? own[1].v[k] : own[0].v[k], od = odd ? own[0].v[k] : own[1].v[k];
      reinterpret_cast<uint2 *>(j.spins)[i + k] = make_uint2(perm(od, even, 0x05010400u), perm(od, even, 0x07030602u));
    }
}

template <int CMP, bool PRIV, bool WIDE>
hipError_t launch_t(const ResidentLaunch &p, unsigned n, size_t lds, hipStream_t stream) {
  if (p.jobs)
    hipLaunchKernelGGL((resident_kernel<CMP, PRIV, WIDE, false>), dim3(n), dim3(256), lds, stream, p);
  else
    hipLaunchKernelGGL((resident_kernel<CMP, PRIV, WIDE, true>), dim3(n), dim3(512), lds, stream, p);
  return hipGetLastError();
}

template <bool WIDE>
hipError_t launch_w(const ResidentLaunch &p, unsigned n, uint32_t q, size_t lds, hipStream_t stream) {
  if (q <= 16) return launch_t<0, true, WIDE>(p, n, lds, stream);
  if (q <= kPrivateHistMaxQ) return launch_t<1, true, WIDE>(p, n, lds, stream);
  if (q <= 128) return launch_t<1, false, WIDE>(p, n, lds, stream);
  return launch_t<2, false, WIDE>(p, n, lds, stream);
}

}  // namespace

// dynamic LDS: the lattice (the rest is static, at most 19 KB)
size_t resident_lds_bytes(uint32_t L, uint32_t q) {
  (void)q;
  return (size_t)L * L;
}

bool resident_fits(uint32_t L, uint32_t q) {
  return L % 16 == 0 && (uint64_t)L * L <= 65536 && q >= 2 && q <= 256;
}

bool drawn_fits(uint32_t L, uint32_t q) { return resident_fits(L, q) && L <= kDrawnMaxL; }

size_t drawn_words_bytes(uint32_t L) {
  // per 4-site group and half sweep: the packed proposals and levels
  return (size_t)2u * (kDrawnChunk + kDrawnPad) * (L * L >> 3) * 8u;
}

static bool falls(const Thresholds &t) { return t.v[0] >= t.v[1] && t.v[1] >= t.v[2] && t.v[2] >= t.v[3]; }

hipError_t launch_draw_words(const ResidentJob &j, uint32_t *words, hipStream_t stream) {
  if (j.nsweeps == 0) return hipSuccess;
  if (!drawn_fits(j.L, j.q) || j.nsweeps > kDrawnChunk) return hipErrorInvalidValue;
  const uint32_t n = j.L * j.L >> 3;
  const dim3 grid((n + 255) / 256, 2u * j.nsweeps);
  if (falls(j.thr))
    hipLaunchKernelGGL(draw_words_kernel<true>, grid, dim3(256), 0, stream, j, n, reinterpret_cast<uint2 *>(words));
  else
    hipLaunchKernelGGL(draw_words_kernel<false>, grid, dim3(256), 0, stream, j, n, reinterpret_cast<uint2 *>(words));
  return hipGetLastError();
}

template <int CMP, bool PRIV, bool MONO>
static hipError_t launch_d(const ResidentJob &j, const uint32_t *words, unsigned long long *mirror, hipStream_t stream) {
  const int D = j.L * j.L <= 8192u ? 1 : 2;
  const uint32_t items = (j.L * j.L >> 3) / D, block = (items + 63u) & ~63u;
  const size_t lds = 4u * ((size_t)kDrawnGroup * drawn_set_words(j.q, PRIV) + 2u * D * items);
  const uint2 *w = reinterpret_cast<const uint2 *>(words);
  auto kernel = drawn_kernel<CMP, PRIV, MONO, false, 1>;
  if (D == 1 && !w) kernel = drawn_kernel<CMP, PRIV, MONO, true, 1>;
  if (D == 2) kernel = w ? drawn_kernel<CMP, PRIV, MONO, false, 2> : drawn_kernel<CMP, PRIV, MONO, true, 2>;
  if (lds > 48u * 1024u) {
    const hipError_t e =
        hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(1), dim3(block), lds, stream, j, w, mirror);
  return hipGetLastError();
}

template <bool MONO>
static hipError_t launch_dm(const ResidentJob &j, const uint32_t *words, unsigned long long *mirror, hipStream_t stream) {
  if (j.q <= 16) return launch_d<0, true, MONO>(j, words, mirror, stream);
  if (j.q <= 128) return launch_d<1, false, MONO>(j, words, mirror, stream);
  return launch_d<2, false, MONO>(j, words, mirror, stream);
}

hipError_t launch_resident_drawn(const ResidentJob &j, const uint32_t *words, unsigned long long *mirror,
                                 hipStream_t stream) {
  if (j.nsweeps == 0) return hipSuccess;
  if (!drawn_fits(j.L, j.q) || j.nsweeps > (words ? kDrawnChunk : kDrawnInline)) return hipErrorInvalidValue;
  return falls(j.thr) ? launch_dm<true>(j, words, mirror, stream) : launch_dm<false>(j, words, mirror, stream);
}

hipError_t launch_resident(const ResidentLaunch &p, unsigned njobs, uint32_t max_L, uint32_t max_q,
                           bool wide, hipStream_t stream) {
  if (njobs == 0) return hipSuccess;
  const size_t lds = resident_lds_bytes(max_L, max_q);
  return wide ? launch_w<true>(p, njobs, max_q, lds, stream)
              : launch_w<false>(p, njobs, max_q, lds, stream);
}

}  // namespace potts
