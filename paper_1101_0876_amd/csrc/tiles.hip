// tiles.hip -- several Metropolis or heat-bath sweeps per launch on LDS tiles whose halos
// are recomputed (temporal blocking), for lattices of any L % 4 == 0 whose
// half sweep is too short to hide a kernel boundary.
//
// A workgroup owns a tile of ty rows x tx bytes of the row-major lattice.  It
// copies the tile and a halo around it (hy = 2S rows above and below, hx >= 2S
// bytes left and right, S sweeps per launch) from `src` into LDS, runs up to
// S sweeps there, and writes the tile's interior to `dst` (a second buffer:
// other workgroups still read their halos from `src`).  Because every site's
// random words are a function of (seed, site, sweep) alone (Sec. 3.2's
// independent streams, here counter-based), a workgroup can recompute its
// neighbours' updates exactly: a site is exact after k half sweeps if it lies
// at least k sites inside the copied region.  After s sweeps (2s half sweeps)
// everything at distance >= 2s is exact, which covers the interior and, for
// the energy, its neighbours; half sweep h leaves the rows alone that nothing
// exact reads any more (h + 1 at either end).  Rows and columns wrap, however
// often: a region wider than a small lattice holds copies of its sites, which
// evolve alike.  The last tile of a row or column of tiles may be cut short
// (L need not be a multiple of tx or ty); it copies and updates a whole
// region, but counts and writes only the sites that are its own.
//
// What bounds it: half sweeps of a tile are short (hundreds of sites on each
// SIMD), so latency first (the chain of Philox rounds, LDS reads, the table
// lookup and the barrier, about a microsecond), then VALU issue.  Hence:
//  - Work item: 8 row bytes, 4 sites of each colour, one dword of each colour
//    plane.  The planes are kept apart in LDS, so an update reads five dwords
//    and writes one and no bytes are shuffled.
//  - The rows of one parity are stored together, so that the items of a wave
//    are consecutive dwords of every row they read (no bank conflicts) and a
//    wave sees one byte offset O: no divergent branch, no per-item addresses.
//  - The words of a half sweep do not depend on the spins: with up to two
//    items per lane the next half sweep's are drawn while this one's reads are
//    in flight, the two Philox blocks in step (a dependent instruction of one
//    wave issues 8 cycles after the last, an independent one after 4), and an
//    item has no branch.
//  - Records: populations and differing neighbours of every sweep of the launch go to
//    counters of their own and are reduced once, at its end, so a sweep has
//    two barriers and no reduction; the workgroup stores its totals, and extra
//    workgroups of the next launch (a small kernel after the last one) add
//    them into the record ring, so the sum costs no launch of its own.
// Measured on MI355X (q = 6, 200 sweeps a call): L = 256 1.6 us per sweep (one
// workgroup with the lattice in LDS: 21.9), L = 1000 3.2 (the chunk kernel:
// 29.8), L = 1024 3.2 (16-byte items of row-major rows in LDS, the words drawn
// at their use, totals and a fold launch per launch: 6.3), L = 2048 7.0.  Of a
// launch of eight sweeps at L = 256, 17 us in an earlier form, the copy in
// took 2.0 us, the sixteen half sweeps 0.6 each, the totals 2.0 and the gap to
// the next launch 2.6; reading the lattice before anything else, 16-byte clears and
// four lanes per column of counters brought it to 13.4.
// The heat bath (heatbath_draw.hpp) differs in an item's words and update; an
// update repeated with the same words draws the same value.  Its chain from
// table to table is longer and it issues twice the operations: L = 256 2.5 us per
// sweep (one launch per half sweep: 19), L = 1000 4.7 (31), L = 2048 13 (21).
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "device.hpp"
#include "heatbath_draw.hpp"
#include "kernels.hpp"
#include "sweep_row.hpp"
#include "tiles.hpp"

namespace potts {
namespace {

using namespace row;

constexpr uint32_t kMaxBlock = 1024;

// Counters of a launch's sweeps in dynamic LDS: 64 lane columns of differing
// neighbours per sweep, then the populations, hist_set words per sweep: 64
// lane columns per value (PRIV), or q shared bins; q <= 16 has them in static
// LDS, with room for 16 values so that the sweep index fits in a value's high
// nibble.
struct Counters {
  uint32_t hist_set, words;
};

__host__ __device__ inline Counters counters_of(uint32_t q, uint32_t nsweeps, bool priv) {
  const uint32_t set = q <= 16 ? 0u : priv ? 64u * q : (q + 3u) & ~3u;
  return Counters{set, (set + 64u) * nsweeps};
}

// A lane's item: dword i of both planes, in row r of the region.  The lanes
// past the last item of a row parity repeat its first one, as halo, maybe in
// another wave and so after it: harmless, since an update repeated with the
// same words changes nothing (a value taken is proposed to itself, a value
// refused is refused again).
struct Item {
  uint32_t i, r;
  uint32_t iu;      // the dword above it in the other plane; the one below is W further
  uint32_t c0, c1;  // Philox chunks of its two 4-byte halves
  uint32_t mask;    // the bytes whose sites the tile owns (0: halo)
  bool valid;
};

struct Region {
  uint32_t y0, x0;    // the tile's first row and byte
  uint32_t W, R;      // dwords per row and plane, rows
  uint32_t H, groups; // items of one row parity, and groups of 64 of them
  uint32_t own_x, own_y;
};

// v mod L, v < 3 L unless the region is wider than the lattice (p.narrow)
__device__ __forceinline__ uint32_t wrap(uint32_t v, const TileParams &p) {
  if (p.narrow) return v % p.L;
  v = v < p.L ? v : v - p.L;
  return v < p.L ? v : v - p.L;
}

// Item `lane` of group g of the rows of parity par.
__device__ __forceinline__ Item item_of(const TileParams &p, const Region &a, uint32_t par, uint32_t g, uint32_t lane) {
  const uint32_t j = g * 64u + lane;
  Item it;
  it.valid = j < a.H;
  const uint32_t jj = it.valid ? j : 0u;
  const uint32_t rr = __umulhi(jj, p.w_magic), k = jj - rr * a.W;
  it.i = par * a.H + jj;
  it.r = 2u * rr + par;
  // rows r - 1 and r + 1 are of the other parity; the region's first and last
  // row, whose sites are spoiled anyway, take the rows one further in
  const uint32_t up = par ? it.i - a.H : it.i + a.H - a.W;
  it.iu = it.r == 0 ? up + a.W : it.r + 1u == a.R ? up - a.W : up;
  const uint32_t rw = p.L >> 2;
  const uint32_t gy = wrap(a.y0 + it.r + p.lift - p.hy, p);
  const uint32_t gc = wrap(a.x0 + 8u * k + p.lift - p.hx, p) >> 2;
  it.c0 = gy * rw + gc;
  it.c1 = gy * rw + (gc + 1u == rw ? 0u : gc + 1u);
  // interior rows hy .. hy + own_y - 1, bytes hx .. hx + own_x - 1 (a cut tile
  // may end in the middle of an item)
  const uint32_t bx = 8u * k;
  const bool in = it.valid && it.r >= p.hy && it.r < p.hy + a.own_y && bx >= p.hx && bx < p.hx + a.own_x;
  it.mask = !in ? 0u : bx + 4u < p.hx + a.own_x ? 0xFFFFFFFFu : 0x0000FFFFu;
  return it;
}

// The words of an item's four sites: proposals and acceptance words, or (HB) the
// heat bath's words in a0 .. a3.
struct Drawn {
  uint32_t k, a0, a1, a2, a3;
};

template <bool HB>
__device__ __forceinline__ Drawn draw_words(const Item &it, const PhiloxHead &h, uint32_t q) {
  Words b0, b1;
  philox_tail2(h.a0 ^ it.c0, h.a0 ^ it.c1, h, b0, b1);
  if (HB) return Drawn{0u, b0.w0, b0.w2, b1.w0, b1.w2};
  return Drawn{pack4(scale_to_q(b0.w0, q), scale_to_q(b0.w2, q), scale_to_q(b1.w0, q), scale_to_q(b1.w2, q)), b0.w1,
               b0.w3, b1.w1, b1.w3};
}

struct Ctx {
  uint32_t *act, *pas;  // planes of the active and the other colour
  const uint8_t *table;
  uint32_t *hist;       // this sweep's populations (q <= 16: all sweeps')
  uint32_t *nz;         // this sweep's differing neighbours, this lane's column
  uint32_t lane_off, set_nibbles;
  uint32_t W;
};

// One item of a half sweep with its words w, and the draw of the next half
// sweep's words (AHEAD; head h) while its loads are in flight.  No branch: halo
// items count nothing by adding 0.
template <int COLOUR, int PAR, int CMP, bool PRIV, bool WIDE, bool AHEAD, bool HB>
__device__ __forceinline__ void tile_item(const Ctx &x, const Item &it, Drawn &w, const PhiloxHead &h, uint32_t q) {
  constexpr int O = COLOUR ^ PAR;
  const uint32_t s = HB ? 0u : x.act[it.i];
  const uint32_t p = x.pas[it.i];
  const uint32_t u = x.pas[it.iu];
  const uint32_t d = x.pas[it.iu + x.W];
  const uint32_t side = O == 0 ? x.pas[(int)it.i - 1] : x.pas[it.i + 1];
  const Drawn now = w;
  if (AHEAD) w = draw_words<HB>(it, h, q);
  Site4 o;
  if (HB) {
    const uint32_t over = O == 0 ? alignbyte(p, side, 3) : alignbyte(side, p, 1);
    const uint32_t lf = O == 0 ? over : p, rt = O == 0 ? p : over;
    o.ns = draw4<CMP, WIDE>(u, d, lf, rt, now.a0, now.a1, now.a2, now.a3, x.table);
    o.nz = COLOUR == 1 ? diff_pattern<CMP>(o.ns, u, d, lf, rt) : 0u;
  } else {
    o = update_sites4<COLOUR, O, CMP, WIDE>(s, p, u, d, side, now.k, now.a0, now.a1, now.a2, now.a3, x.table);
  }
  x.act[it.i] = o.ns;
  const uint32_t one = it.mask & 1u, two = (it.mask >> 16) & 1u;
  if (PRIV && CMP == 0) {
    // counter (sweep, value, lane) at byte sweep << 12 | value << 8 | lane << 2
    const uint32_t v = o.ns | x.set_nibbles;
    uint8_t *hb = reinterpret_cast<uint8_t *>(x.hist);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0400u)), one);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0500u)), one);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0600u)), two);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0700u)), two);
  } else {
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b) {
      const uint32_t v = byte_of(o.ns, b);
      atomicAdd(&x.hist[PRIV ? v * 64u + (x.lane_off >> 2) : v], b < 2 ? one : two);
    }
  }
  if (COLOUR == 1) atomicAdd(x.nz, (uint32_t)__popc(o.nz & it.mask & 0xF0F0F0F0u));
}

template <int CMP, bool PRIV>
constexpr uint32_t kStaticHist = PRIV && CMP == 0 ? 64u * 16u * kTileMaxSweeps : 1u;

// bytes of the acceptance table, or of the heat bath's draw table (HB)
template <bool WIDE, bool HB>
constexpr uint32_t kTableBytes = !HB ? 2048u : WIDE ? HbTable::kBytes : HbTable::kCut64;

// NI 1: one item per lane, the even rows' items on the first waves, the odd
// rows' on the others.  NI 2, 4, 6: NI / 2 items of each parity per lane, all
// on the same wave.  The items' addresses, chunks and masks stay in
// registers.
template <int CMP, bool PRIV, bool WIDE, int NI, bool HB>
__device__ __forceinline__ void tile_body(const TileParams &p, uint32_t tile, uint32_t *table_words, uint32_t *hist16,
                                          uint32_t *lds) {
  const uint32_t ntiles = p.tiles_x * p.tiles_y;
  uint8_t *table = reinterpret_cast<uint8_t *>(table_words);
  const uint32_t L = p.L, q = p.q;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const uint32_t tyi = tile / p.tiles_x, txi = tile - tyi * p.tiles_x;
  Region a;
  a.y0 = tyi * p.ty;
  a.x0 = txi * p.tx;
  a.W = (p.tx + 2u * p.hx) >> 3;
  a.R = p.ty + 2u * p.hy;
  a.H = (a.R >> 1) * a.W;
  a.groups = (a.H + 63u) >> 6;
  a.own_x = min(p.tx, L - a.x0);
  a.own_y = min(p.ty, L - a.y0);
  const Counters cn = counters_of(q, p.nsweeps, PRIV);
  uint32_t *nzc = lds;                       // differing neighbours
  uint32_t *bins = lds + 64u * p.nsweeps;    // populations, q > 16
  uint32_t *plane0 = lds + cn.words + 4u;    // a dword on either side is read, and not used
  uint32_t *plane1 = plane0 + 2u * a.H;

  const uint32_t *src = reinterpret_cast<const uint32_t *>(p.src);
  // even bytes of an even row are colour 0, of an odd row colour 1
  auto put_item = [&](const Item &it, uint32_t d0, uint32_t d1) {
    if (!it.valid) return;
    const uint32_t even = perm(d1, d0, kSel<0>), odd = perm(d1, d0, kSel<1>);
    plane0[it.i] = it.r & 1u ? odd : even;
    plane1[it.i] = it.r & 1u ? even : odd;
  };
  // item n of this lane: row parity and group
  constexpr int kHalf = NI > 1 ? NI / 2 : 1;
  const uint32_t par1 = wave >= a.groups;  // NI 1
  auto par_of = [&](int n) { return NI == 1 ? par1 : (uint32_t)(n >= kHalf); };
  auto group_of = [&](int n) { return NI == 1 ? wave - par1 * a.groups : wave + (uint32_t)(n % kHalf) * waves; };
  Item item[NI];
  uint32_t raw[2 * NI];
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    item[n] = item_of(p, a, par_of(n), group_of(n), lane);
    raw[2 * n] = src[item[n].c0];
    raw[2 * n + 1] = src[item[n].c1];
  }
  // while the lattice is on its way
  if (HB) {
    const u32x4 *from = reinterpret_cast<const u32x4 *>(p.heatbath->bytes);
    for (uint32_t i = threadIdx.x; i < kTableBytes<WIDE, HB> / 16u; i += blockDim.x)
      reinterpret_cast<u32x4 *>(table)[i] = from[i];
  } else {
    fill_accept_table<WIDE>(table, p.thr);
  }
  u32x4 *clear = reinterpret_cast<u32x4 *>(lds);
  for (uint32_t i = threadIdx.x; i < cn.words / 4u; i += blockDim.x) clear[i] = u32x4{0, 0, 0, 0};
  if (PRIV && CMP == 0) {
    clear = reinterpret_cast<u32x4 *>(hist16);
    for (uint32_t i = threadIdx.x; i < 256u * p.nsweeps; i += blockDim.x) clear[i] = u32x4{0, 0, 0, 0};
  }
#pragma unroll
  for (int n = 0; n < NI; ++n) put_item(item[n], raw[2 * n], raw[2 * n + 1]);
  if (threadIdx.x < 4) plane0[(int)threadIdx.x - 4] = plane1[2u * a.H + threadIdx.x] = 0;

  Ctx x;
  x.table = table;
  x.lane_off = lane * 4u;
  x.W = a.W;
  auto head = [&](uint32_t hs) {
    const uint64_t t = p.t0 + (hs >> 1);
    return philox_head((uint32_t)t, (uint32_t)(t >> 32), (hs & 1u) + (HB ? 4u : 0u), p.k0, p.k1);
  };
  // the half sweeps that update anything of item n's group: rows hs + 1 ..
  // R - 2 - hs
  constexpr bool kAhead = NI == 1 || NI == 2;
  Drawn w[NI];
  uint32_t reach[NI];
  const PhiloxHead first = head(0);
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    if (kAhead) w[n] = draw_words<HB>(item[n], first, q);
    const uint32_t lo = group_of(n) * 64u / a.W, hi = min(group_of(n) * 64u + 63u, a.H - 1u) / a.W;
    const uint32_t rlo = 2u * lo + par_of(n), rhi = 2u * hi + par_of(n);
    reach[n] = group_of(n) >= a.groups ? 0u : min(rhi, a.R - 1u - rlo);
  }
  auto half_sweep = [&](auto colour, uint32_t hs) {
    constexpr int C = decltype(colour)::value;
    x.act = C ? plane1 : plane0;
    x.pas = C ? plane0 : plane1;
    const PhiloxHead h = head(kAhead ? hs + 1u : hs);
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      if (hs >= reach[n]) continue;
      if (!kAhead) w[n] = draw_words<HB>(item[n], h, q);
      if (par_of(n) == 0)
        tile_item<C, 0, CMP, PRIV, WIDE, kAhead, HB>(x, item[n], w[n], h, q);
      else
        tile_item<C, 1, CMP, PRIV, WIDE, kAhead, HB>(x, item[n], w[n], h, q);
    }
    __syncthreads();
  };
  __syncthreads();
  for (uint32_t s = 0; s < p.nsweeps; ++s) {
    x.hist = PRIV && CMP == 0 ? hist16 : bins + s * cn.hist_set;
    x.set_nibbles = s * 0x10101010u;
    x.nz = nzc + s * 64u + lane;
    half_sweep(std::integral_constant<int, 0>{}, 2u * s);
    half_sweep(std::integral_constant<int, 1>{}, 2u * s + 1u);
  }

  // the interior to dst
  uint32_t *dst = reinterpret_cast<uint32_t *>(p.dst);
  auto store_item = [&](const Item &it) {
    if (!it.mask) return;
    const uint32_t v0 = plane0[it.i], v1 = plane1[it.i];
    const uint32_t even = it.r & 1u ? v1 : v0, odd = it.r & 1u ? v0 : v1;
    dst[it.c0] = perm(odd, even, 0x05010400u);
    if (it.mask >> 16) dst[it.c1] = perm(odd, even, 0x07030602u);
  };
#pragma unroll
  for (int n = 0; n < NI; ++n) store_item(item[n]);
  // the tile's totals of each sweep
  const uint32_t n1 = q + 1u;
  const uint32_t nparts = tile_parts(ntiles), mine = tile % nparts;
  auto put = [&](uint32_t s, uint32_t word, uint32_t sum) {
    uint32_t *at = p.parts + ((size_t)s * nparts + mine) * n1 + word;
    if (nparts == ntiles)
      *at = sum;
    else
      atomicAdd(at, sum);
  };
  // four lanes per 64-lane column: 16 words each, in four 16-byte reads
  const uint32_t per = PRIV ? n1 : 1u, columns = 4u * p.nsweeps * per;
  for (uint32_t c4 = threadIdx.x; c4 < columns; c4 += blockDim.x) {
    const uint32_t c = c4 >> 2, s = PRIV ? c / n1 : c, v = c - s * per;
    const uint32_t *pops = PRIV && CMP == 0 ? hist16 + 1024u * s : bins + s * cn.hist_set;
    const u32x4 *col = reinterpret_cast<const u32x4 *>(v == 0 ? nzc + s * 64u : pops + (v - 1u) * 64u) + 4u * (c4 & 3u);
    const u32x4 t = col[0] + col[1] + col[2] + col[3];
    uint32_t sum = t.x + t.y + t.z + t.w;
    sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    if ((c4 & 3u) == 0) put(s, v, sum);
  }
  if (!PRIV)
    for (uint32_t c = threadIdx.x; c < p.nsweeps * q; c += blockDim.x) {
      const uint32_t s = c / q, v = c - s * q;
      put(s, 1u + v, bins[s * cn.hist_set + v]);
    }
}

#define POTTS_TILE_LDS                                                                  \
  __shared__ __align__(16) uint32_t table_words[kTableBytes<WIDE, HB> / 4u];              \
  /* q <= 16: populations in static LDS, whose address folds into the instructions' */   \
  /* offsets */                                                                          \
  __shared__ __align__(16) uint32_t hist16[kStaticHist<CMP, PRIV>];                      \
  extern __shared__ __align__(16) uint32_t lds[]

template <int CMP, bool PRIV, bool WIDE, int NI, bool HB>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void tile_kernel(TileParams p) {
  POTTS_TILE_LDS;
  const uint32_t ntiles = p.tiles_x * p.tiles_y;
  if (blockIdx.x >= ntiles)
    fold_part(p.fold, blockIdx.x - ntiles, reinterpret_cast<unsigned long long *>(lds));
  else
    tile_body<CMP, PRIV, WIDE, NI, HB>(p, blockIdx.x, table_words, hist16, lds);
}

// The same for many lattices (TileTable).
template <int CMP, bool PRIV, bool WIDE, int NI>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void tile_jobs_kernel(TileTable t) {
  constexpr bool HB = false;
  POTTS_TILE_LDS;
  const TileRef ref = t.refs[blockIdx.x];
  TileParams p = t.jobs[ref.job];
  const uint64_t before = (uint64_t)t.turn * p.sweeps;  // sweeps of the turns before
  const size_t words = (size_t)p.sweeps * tile_parts(p.tiles_x * p.tiles_y) * (p.q + 1u);
  if (ref.tile & kTileFold) {
    RecordFold f = p.fold;
    if (before == 0 || before - p.sweeps >= p.total) return;
    f.t0 = p.t0 + before - p.sweeps;
    f.nsweeps = (uint32_t)min((uint64_t)p.sweeps, p.total - (before - p.sweeps));
    f.parts = p.parts + ((t.turn & 1u) ? 0u : words);
    const uint32_t g = ref.tile & ~kTileFold;
    if (g < fold_groups(f)) fold_part(f, g, reinterpret_cast<unsigned long long *>(lds));
    return;
  }
  if (before >= p.total) return;
  p.nsweeps = (uint32_t)min((uint64_t)p.sweeps, p.total - before);
  p.t0 += before;
  if (t.turn & 1u) {
    const uint8_t *from = p.dst;
    p.dst = const_cast<uint8_t *>(p.src);
    p.src = from;
    p.parts += words;
  }
  tile_body<CMP, PRIV, WIDE, NI, HB>(p, ref.tile, table_words, hist16, lds);
}
#undef POTTS_TILE_LDS

// dynamic LDS of a workgroup
size_t lds_bytes(const TileParams &p, bool priv) {
  const size_t words = counters_of(p.q, p.sweeps, priv).words + 8u + 2u * (size_t)(p.ty + 2u * p.hy) * ((p.tx + 2u * p.hx) >> 3);
  const size_t acc = kFoldWords * 8;  // the fold's sums
  return words * 4 < acc ? acc : words * 4;
}

// lane-private counters up to kPrivateHistMaxQ values, where they fit
bool private_counters(const TileParams &p) {
  return p.q <= 16 || (p.q <= kPrivateHistMaxQ && lds_bytes(p, true) <= kTileMaxLds);
}

// Items per lane (NI) and waves of a workgroup: one item where the region's
// groups of 64 fit 16 waves, else as many of each row parity as they need, up
// to three (0: more).
struct Lanes {
  uint32_t ni, waves;
};

Lanes lanes_of(uint32_t tx, uint32_t ty, uint32_t hx, uint32_t hy) {
  const uint32_t H = ((ty + 2u * hy) >> 1) * ((tx + 2u * hx) >> 3);
  const uint32_t groups = (H + 63u) >> 6;  // per row parity
  constexpr uint32_t kMaxWaves = kMaxBlock / 64u;
  if (2u * groups <= kMaxWaves) return Lanes{1u, 2u * groups};
  for (uint32_t n = 1; n <= 3; ++n)
    if (groups <= n * kMaxWaves) return Lanes{2u * n, (groups + n - 1u) / n};
  return Lanes{0u, kMaxWaves};
}

template <int CMP, bool PRIV, bool WIDE, bool HB>
hipError_t launch_n(const TileParams &p, hipStream_t stream) {
  const Lanes n = lanes_of(p.tx, p.ty, p.hx, p.hy);
  const size_t lds = lds_bytes(p, PRIV);
  const dim3 grid(p.tiles_x * p.tiles_y + fold_groups(p.fold)), block(64u * n.waves);
  auto go = [&](auto kernel) {
    hipError_t e = hipSuccess;
    if (lds > 48u * 1024u)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, p);
    return hipGetLastError();
  };
  switch (n.ni) {
    case 1: return go(tile_kernel<CMP, PRIV, WIDE, 1, HB>);
    case 2: return go(tile_kernel<CMP, PRIV, WIDE, 2, HB>);
    case 4: return go(tile_kernel<CMP, PRIV, WIDE, 4, HB>);
    case 6: return go(tile_kernel<CMP, PRIV, WIDE, 6, HB>);
    default: return hipErrorInvalidValue;  // tile_fits has refused it
  }
}

template <bool WIDE, bool HB>
hipError_t launch_w(const TileParams &p, hipStream_t stream) {
  if (p.q <= 16) return launch_n<0, true, WIDE, HB>(p, stream);
  if (private_counters(p)) return launch_n<1, true, WIDE, HB>(p, stream);
  if (p.q <= 128) return launch_n<1, false, WIDE, HB>(p, stream);
  return launch_n<2, false, WIDE, HB>(p, stream);
}

}  // namespace

uint32_t tile_halo_x(uint32_t sweeps) { return (2u * sweeps + 7u) & ~7u; }

bool tile_fits(const TileParams &p) {
  if (p.L < 4 || p.L % 4 || p.L > kTileMaxL || p.q < 2 || p.q > 256) return false;
  if (p.tx < 8 || p.tx % 8 || p.ty < 2 || p.ty % 2 || p.sweeps < 1 || p.sweeps > kTileMaxSweeps) return false;
  if (p.hy != 2u * p.sweeps || p.hx != tile_halo_x(p.sweeps)) return false;
  if (!lanes_of(p.tx, p.ty, p.hx, p.hy).ni) return false;
  if (p.tiles_x != (p.L + p.tx - 1) / p.tx || p.tiles_y != (p.L + p.ty - 1) / p.ty) return false;
  return lds_bytes(p, private_counters(p)) <= kTileMaxLds - (p.q <= 16 ? 4u * kStaticHist<0, true> : 0u);
}

bool set_tile_shape(TileParams &p, uint32_t tx, uint32_t ty, uint32_t sweeps) {
  p.tx = tx;
  p.ty = ty;
  p.sweeps = sweeps;
  p.hx = tile_halo_x(sweeps);
  p.hy = 2u * sweeps;
  p.tiles_x = tx ? (p.L + tx - 1) / tx : 0;
  p.tiles_y = ty ? (p.L + ty - 1) / ty : 0;
  p.lift = p.L ? (2u * kTileMaxSweeps + p.L - 1) / p.L * p.L : 0;  // a multiple of L, at least hx and hy
  if (!tile_fits(p)) return false;
  const uint32_t W = (tx + 2u * p.hx) / 8u;
  p.w_magic = (uint32_t)(((1ull << 32) + W - 1) / W);  // exact for the few thousand items of a region
  p.narrow = p.tx + p.hx > p.L || p.ty + p.hy > p.L || p.lift > p.L;
  return true;
}

// Time of one launch in microseconds, measured on MI355X (q = 6) over 5400
// shapes of L = 100 .. 4096 and fitted: a launch, the copies and the totals,
// then per half sweep 0.47 us of latency or the issue time of the n items that
// a SIMD holds (rows that are not updated any more, S / R of them on average,
// left out); more tiles than the GPU's 256 CUs take turns.  The shapes it picks
// took 1 % longer than the best measured ones on average, 6 % at most.  The heat
// bath's constants are fitted likewise to 66 shapes of L = 256 .. 2048.  0: no
// launch of this shape exists.
static float tile_launch_us(const TileParams &p, uint32_t tx, uint32_t ty, uint32_t sweeps) {
  const uint32_t R = ty + 4u * sweeps;
  const Lanes lanes = lanes_of(tx, ty, tile_halo_x(sweeps), 2u * sweeps);
  if (!lanes.ni) return 0;
  const bool hb = p.heatbath != nullptr;
  const float n = (float)(lanes.ni * ((lanes.waves + 3u) / 4u));
  const float issue = (hb ? 0.3f : 0.2f) + (hb ? 0.45f : 0.2f) * n * (1.0f - (float)sweeps / (float)R);
  const float least = hb ? 0.6f : 0.47f;
  const float turns = (float)((((p.L + tx - 1) / tx) * ((p.L + ty - 1) / ty) + 255u) / 256u);
  return ((hb ? 5.0f : 3.5f) + 0.4f * n + 2.0f * (float)sweeps * (issue > least ? issue : least)) *
         (turns > 1.0f ? 0.95f * turns : 1.0f);
}

// The shape out of tiles with these sides; false: none of them fits.
static bool best_tile_shape(TileParams &p, int64_t nsweeps, const uint32_t *sides, uint32_t nsides) {
  const int64_t n = nsweeps > 64 ? 64 : nsweeps < 1 ? 1 : nsweeps;  // long calls: per sweep
  float best = 0;
  uint32_t btx = 0, bty = 0, bs = 0;
  for (uint32_t s = 1; s <= kTileMaxSweeps && (int64_t)s <= n; ++s) {
    const float launches = nsweeps > 64 ? 64.0f / (float)s : (float)((n + s - 1) / s);
    for (uint32_t i = 0; i < nsides; ++i)
      for (uint32_t j = 0; j < nsides; ++j) {
        const uint32_t tx = sides[i], ty = sides[j];
        if (tx > 2u * ty || ty > 2u * tx) continue;
        const float us = launches * tile_launch_us(p, tx, ty, s);
        if (us > 0 && (bs == 0 || us < best)) {
          best = us;
          btx = tx;
          bty = ty;
          bs = s;
        }
      }
  }
  return bs != 0 && set_tile_shape(p, btx, bty, bs);
}

bool auto_tile_shape(TileParams &p, int64_t nsweeps) {
  // sides of 16 .. 256 that cut L into 1 .. 32 equal parts (rounded up to 8)
  uint32_t sides[40], nsides = 0;
  for (uint32_t k = 1; k <= 32; ++k) {
    uint32_t t = ((p.L + k - 1) / k + 7u) & ~7u;
    t = t < 16u ? 16u : t;
    if (t <= 256u && (nsides == 0 || sides[nsides - 1] != t)) sides[nsides++] = t;
  }
  if (nsides && best_tile_shape(p, nsweeps, sides, nsides)) return true;
  // from L = 6672 the parts are too large for a workgroup (above 8192 there are
  // none): tiles of these sides, the last ones cut
  static const uint32_t fixed[] = {256, 224, 192, 160, 128};
  return best_tile_shape(p, nsweeps, fixed, 5);
}

// ---- many lattices per launch -------------------------------------------------

void add_tile_job(TileRun &r, uint8_t *spins, uint8_t *other, uint32_t L, uint32_t q, uint64_t seed,
                  const uint32_t thr[4], uint64_t t0, uint64_t nsweeps, unsigned long long *ring, uint64_t cap) {
  TileParams p{};
  p.src = spins;
  p.dst = other;
  p.L = L;
  p.q = q;
  p.k0 = (uint32_t)seed;
  p.k1 = (uint32_t)(seed >> 32);
  for (int i = 0; i < 4; ++i) p.thr.v[i] = thr[i];
  p.t0 = t0;
  p.total = nsweeps;
  p.fold.n = q + 1u;
  p.fold.comp = 1;
  p.fold.ring = ring;
  p.fold.cap = cap;
  p.fold.bonds = 2ull * L * L;
  r.jobs.push_back(p);
}

bool tile_job_odd(const TileParams &p) { return ((p.total + p.sweeps - 1) / p.sweeps) & 1u; }

// Time of one turn over `tiles` tiles of side x side (tile_launch_us; beyond
// one tile per CU their issue times add up, a little overlapped).
static float tile_turn_us(uint32_t side, uint32_t sweeps, uint64_t tiles) {
  const uint32_t R = side + 4u * sweeps;
  const Lanes lanes = lanes_of(side, side, tile_halo_x(sweeps), 2u * sweeps);
  if (lanes.ni != 1 && lanes.ni != 2) return 0;
  const float n = (float)(lanes.ni * ((lanes.waves + 3u) / 4u));
  const float issue = 0.2f + 0.2f * n * (1.0f - (float)sweeps / (float)R);
  const float half = issue > 0.47f ? issue : 0.47f, turns = (float)tiles / 256.0f;
  const float shared = 0.85f * issue * turns;
  return 3.5f + 0.4f * n + 2.0f * (float)sweeps * (turns > 1.0f && shared > half ? shared : half);
}

// The run's shape: sides of its tiles and sweeps a turn; side 0: none.
struct RunShape {
  uint32_t side, sweeps;
};

static RunShape run_shape(const std::vector<SweepJob> &jobs) {
  uint64_t most = 0;
  std::vector<std::pair<uint32_t, uint64_t>> sizes;  // L, jobs of it
  for (const SweepJob &p : jobs) {
    most = p.sweeps > most ? p.sweeps : most;
    size_t i = 0;
    while (i < sizes.size() && sizes[i].first != p.L) ++i;
    if (i == sizes.size()) sizes.push_back({p.L, 0});
    ++sizes[i].second;
  }
  static const uint32_t sides[] = {16, 24, 32, 48, 64, 80, 96};
  float best = 0;
  RunShape shape{0, 0};
  for (uint32_t t : sides) {
    uint64_t tiles = 0;
    for (const auto &z : sizes) tiles += z.second * ((z.first + t - 1) / t) * ((z.first + t - 1) / t);
    for (uint32_t s = 1; s <= kTileMaxSweeps && s <= most; ++s) {
      const float us = tile_turn_us(t, s, tiles) * (float)((most + s - 1) / s);
      if (us > 0 && (best == 0 || us < best)) {
        best = us;
        shape = RunShape{t, s};
      }
    }
  }
  return shape;
}

// Sweeps a turn of one job: at most the shape's, the ring's slots, and so few
// that the lattice ends where it began where that can be had: a copy back costs
// 3.5 us a job (64 jobs of L = 16: one turn of one sweep 0.30 ms, two turns of two
// 0.09).  The turns that it adds cost about what the copies do (us a run of 100
// sweeps, the longest turns and a copy in brackets: 1 job of L = 256 277 (269), 16 of
// 128 315 (334), 16 of 256 437 (439), 64 of 192 721 (846), 96 of 128 705 (699)).
static uint32_t job_sweeps(uint64_t total, uint64_t cap, uint32_t sweeps) {
  const uint32_t most = sweeps < cap ? sweeps : (uint32_t)cap;
  for (uint32_t per = most; per >= 1; --per)
    if (((total + per - 1) / per) % 2 == 0) return per;
  return most;
}

// Measured on MI355X over 1100 batches of 1 .. 4096 jobs of L = 16 .. 2048, q = 3 ..
// 200, 1 .. 100 sweeps, and 60 mixed ones: by these estimates none of them takes a
// route that is slower than its other one by more than 5 %.
//
// Tiles: a turn is the launch and the slowest CU.  Of a workgroup's time all but
// the launch repeats for the tiles that a CU gets beyond those it holds at once
// (16 waves), unless their issue times add up to more.  The folds of all sweeps add
// 0.4 ns a wave of each fold workgroup, of which a job has (q + 1) / 8 a sweep:
// 512 jobs of L = 64 take 1.3 ms at q = 9 and 8.5 at q = 200.
float tile_run_us(const std::vector<SweepJob> &jobs) {
  const RunShape shape = run_shape(jobs);
  if (!shape.side) return 0;
  const Lanes lanes = lanes_of(shape.side, shape.side, tile_halo_x(shape.sweeps), 2u * shape.sweeps);
  uint64_t turns = 0, odd = 0, tiles = 0;  // tiles: of all turns
  uint32_t per_most = 1, q = 0;
  float folds = 0;
  for (const SweepJob &p : jobs) {
    const uint32_t per = job_sweeps(p.sweeps, p.cap, shape.sweeps);
    const uint64_t n = (p.sweeps + per - 1) / per, side = (p.L + shape.side - 1) / shape.side;
    turns = n > turns ? n : turns;
    odd += n & 1u;
    tiles += side * side * n;
    per_most = per > per_most ? per : per_most;
    q = p.q > q ? p.q : q;
    folds += (float)p.sweeps * (float)((p.q + fold_width(p.q + 1u)) / fold_width(p.q + 1u));
  }
  const float s = (float)per_most, k = (float)((tiles + turns * 256u - 1u) / (turns * 256u));
  const float n = (float)(lanes.ni * ((lanes.waves + 3u) / 4u)), held = lanes.waves > 8u ? 1.0f : 16.0f / (float)lanes.waves;
  const float issue = 0.2f + 0.2f * n * (1.0f - s / ((float)shape.side + 4.0f * s));
  const float one = 3.5f + 0.4f * n + 2.0f * s * (issue > 0.47f ? issue : 0.47f);
  const float waits = 2.0f + k / held * (one - 2.0f), issues = 2.0f + k * (2.0f * s * issue + 0.3f * n);
  float turn = one > waits ? one : waits;
  turn = turn > issues ? turn : issues;
  return 20.0f + 3.5f * (float)odd + (float)turns * (turn + (q <= 16u ? 2.0f : 4.0f)) + 4e-4f * (float)lanes.waves * folds;
}

// Every job's workgroup runs its sweeps alone (1.5 us for each round of its 256
// lanes over the items, and the record), or shares its CU with others.
float resident_us(const std::vector<SweepJob> &jobs) {
  float chain = 0, load = 0;
  for (const SweepJob &p : jobs) {
    const float n = (float)p.sweeps, rounds = (float)((p.L * p.L + 4095u) / 4096u);
    const float one = 0.7f + 1.52f * rounds + (p.q > 16u && p.q <= kPrivateHistMaxQ ? 0.03f * (float)p.q : 0.0f);
    chain = n * one > chain ? n * one : chain;
    load += n * (1.4f * rounds > 0.8f ? 1.4f * rounds : 0.8f);
  }
  return chain > load / 256.0f ? chain : load / 256.0f;
}

// Two launches a sweep, however few the sites, and 0.66 ps a site.
float strip_us(const std::vector<SweepJob> &jobs) {
  uint64_t most = 0;
  uint32_t L = 0;
  float sites = 0;
  for (const SweepJob &p : jobs) {
    most = p.sweeps > most ? p.sweeps : most;
    L = p.L > L ? p.L : L;
    sites += (float)p.sweeps * (float)p.L * (float)p.L;
  }
  return (float)most * (15.0f + 3.5f * (float)L / 1024.0f) + 0.66e-6f * sites;
}

bool plan_tile_run(TileRun &r) {
  std::vector<SweepJob> all;
  for (const TileParams &p : r.jobs) all.push_back(SweepJob{p.L, p.q, p.total, p.fold.cap});
  const RunShape shape = run_shape(all);
  const uint32_t side = shape.side, sweeps = shape.sweeps;
  if (!side) return false;
  const Lanes lanes = lanes_of(side, side, tile_halo_x(sweeps), 2u * sweeps);
  r.ni = lanes.ni;
  r.waves = lanes.waves;
  r.refs.clear();
  r.parts_words = 0;
  r.turns = 0;
  r.lds = 0;
  r.ntiles = 0;
  std::vector<TileRef> folds;
  for (size_t j = 0; j < r.jobs.size(); ++j) {
    TileParams &p = r.jobs[j];
    const uint32_t per = job_sweeps(p.total, p.fold.cap, sweeps);
    if (!set_tile_shape(p, side, side, per)) return false;
    const uint32_t tiles = p.tiles_x * p.tiles_y, turns = (uint32_t)((p.total + per - 1) / per);
    if (tiles > kTileMaxParts) return false;
    for (uint32_t t = 0; t < tiles; ++t) r.refs.push_back(TileRef{(uint32_t)j, t});
    p.fold.nparts = tiles;
    p.fold.nsweeps = per;
    for (uint32_t g = 0; g < fold_groups(p.fold); ++g) folds.push_back(TileRef{(uint32_t)j, kTileFold | g});
    r.parts_words += 2u * (size_t)per * tiles * (p.q + 1u);
    r.turns = turns > r.turns ? turns : r.turns;
    const size_t lds = lds_bytes(p, r.qc == 0);
    r.lds = lds > r.lds ? lds : r.lds;
  }
  r.ntiles = (uint32_t)r.refs.size();
  r.refs.insert(r.refs.end(), folds.begin(), folds.end());
  return true;
}

void place_tile_run(TileRun &r, uint32_t *parts) {
  for (TileParams &p : r.jobs) {
    p.parts = parts;
    parts += 2u * (size_t)p.sweeps * p.fold.nparts * (p.q + 1u);
  }
}

template <int CMP, bool PRIV, bool WIDE>
static hipError_t launch_run_n(const TileRun &r, const TileParams *jobs, const TileRef *refs, hipStream_t stream) {
  auto kernel = r.ni == 1 ? tile_jobs_kernel<CMP, PRIV, WIDE, 1> : tile_jobs_kernel<CMP, PRIV, WIDE, 2>;
  hipError_t e = hipSuccess;
  if (r.lds > 48u * 1024u)
    e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)r.lds);
  const unsigned nfold = (unsigned)(r.refs.size() - r.ntiles);
  for (uint32_t turn = 0; turn <= r.turns && e == hipSuccess; ++turn) {
    // the last launch only folds
    const bool last = turn == r.turns;
    hipLaunchKernelGGL(kernel, dim3(last ? nfold : r.ntiles + (turn ? nfold : 0u)), dim3(64u * r.waves), r.lds, stream,
                       TileTable{jobs, last ? refs + r.ntiles : refs, turn});
    e = hipGetLastError();
  }
  return e;
}

template <bool WIDE>
static hipError_t launch_run_w(const TileRun &r, const TileParams *jobs, const TileRef *refs, hipStream_t stream) {
  if (r.qc == 0) return launch_run_n<0, true, WIDE>(r, jobs, refs, stream);
  if (r.qc <= 2) return launch_run_n<1, false, WIDE>(r, jobs, refs, stream);
  return launch_run_n<2, false, WIDE>(r, jobs, refs, stream);
}

hipError_t launch_tile_run(const TileRun &r, const TileParams *jobs, const TileRef *refs, hipStream_t stream) {
  if (r.ntiles == 0 || r.turns == 0) return hipSuccess;
  if ((r.ni != 1 && r.ni != 2) || r.waves == 0 || r.waves > kMaxBlock / 64u) return hipErrorInvalidValue;
  return r.wide ? launch_run_w<true>(r, jobs, refs, stream) : launch_run_w<false>(r, jobs, refs, stream);
}

hipError_t launch_tiles(const TileParams &p, hipStream_t stream) {
  if (p.nsweeps == 0) return hipSuccess;
  if (!tile_fits(p) || p.nsweeps > p.sweeps || p.lift < p.hx || p.lift < p.hy || p.lift % p.L || !p.src || !p.dst ||
      !p.parts || (p.fold.nsweeps && (!p.fold.parts || p.fold.n != p.q + 1u)))
    return hipErrorInvalidValue;
  const bool wide = !p.thr.v[0] || !p.thr.v[1] || !p.thr.v[2] || !p.thr.v[3];
  if (p.heatbath) return wide ? launch_w<true, true>(p, stream) : launch_w<false, true>(p, stream);
  return wide ? launch_w<true, false>(p, stream) : launch_w<false, false>(p, stream);
}

}  // namespace potts
