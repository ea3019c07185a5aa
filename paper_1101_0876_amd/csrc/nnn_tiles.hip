// nnn_tiles.hip -- whole sweeps (nine colour passes each, contract in nnn.hip)
// of the first-plus-second-neighbour lattice on LDS tiles whose halos are
// recomputed, as tiles.hip does for the nearest-neighbour lattice.
//
// How far a sweep reaches: a site of colour c = 3 (y mod 3) + (x mod 3) depends
// on neighbours of lower colours updated before it in the same sweep, and so
// on.  Such a chain of falling colours goes up at most 3 rows (row classes 2,
// 1, 0, then the row above's old values) and down at most 2; left at most 9
// sites (nine colours, one column each) and right at most 5.  A halo of 3 rows
// and 12 bytes per sweep covers it and keeps rows and bytes aligned with the
// classes.
//
// LDS: every row of the region as three runs of W dwords, one per column class
// x mod 3 (dword k: the sites x = 12 k + class + 3 j, j = 0..3).  An item, one
// dword of one class, then has each of its eight neighbour views in one dword
// of the same index, or of two shifted by a byte across the row's next or
// previous dword (class 0's left and class 2's right neighbours): no byte
// gathering, where row-major rows in LDS take 27 v_perm an item.
//
// What bounds it: VALU issue (about 42 operations a site, 17 of them the
// random words, against 60 of the row-class kernel in nnn.hip) on large
// lattices, on small ones the chain of each of the nine passes (half a
// microsecond) and the launch.  The words of the next pass are drawn while this
// one's reads are in flight; records as in tiles.hip.  Measured on MI355X (q =
// 9, us per sweep; three row-class launches and a fold launch in brackets): L = 60
// 6.1 (20.0), 504 6.6 (19.5), 1020 8.0 (22.5), 2040 14.3 (27.4), 4092 36 (56),
// 6000 76 (79), 8184 158 (135).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "device.hpp"
#include "nnn_tiles.hpp"
#include "sweep_row.hpp"

namespace potts {
namespace nnn {
namespace {

using namespace row;

constexpr uint32_t kMaxBlock = 1024;
constexpr size_t kMaxLds = 158u * 1024u;

struct Item {
  uint32_t i;     // its dword of class 0 in the first of its three rows
  uint32_t seg;   // Philox segment of its first six bytes in that row
  uint32_t own;   // all bits set: the tile's own site, 0: halo
  uint32_t gy, gx;
  bool valid;
};

struct Region {
  uint32_t y0, x0, W, R, H, groups, own_x, own_y;
};

__device__ __forceinline__ uint32_t wrap(uint32_t v, const TileParams &p) {
  if (p.narrow) return v % p.L;
  v = v < p.L ? v : v - p.L;
  return v < p.L ? v : v - p.L;
}

// Item `lane` of group g: 12 bytes of three rows (one of each class).  Lanes
// past the last item repeat the first one as halo (an update repeated with the
// same words changes nothing).
__device__ __forceinline__ Item item_of(const TileParams &p, const Region &a, uint32_t g, uint32_t lane) {
  const uint32_t j = g * 64u + lane;
  Item it;
  it.valid = j < a.H;
  const uint32_t jj = it.valid ? j : 0u;
  const uint32_t rr = __umulhi(jj, p.w_magic), k = jj - rr * a.W;
  it.i = rr * 9u * a.W + k;
  it.gy = wrap(a.y0 + 3u * rr + p.lift - p.hy, p);
  it.gx = wrap(a.x0 + 12u * k + p.lift - p.hx, p);
  it.seg = it.gy * (p.L / 6u) + it.gx / 6u;
  const bool in = it.valid && 3u * rr >= p.hy && 3u * rr < p.hy + a.own_y && 12u * k >= p.hx && 12u * k < p.hx + a.own_x;
  it.own = in ? 0xFFFFFFFFu : 0u;
  return it;
}

struct Drawn {
  uint32_t k, a0, a1, a2, a3;
};

__device__ __forceinline__ Drawn draw(uint32_t seg, const PhiloxHead &h, uint32_t q) {
  Words b0, b1;
  philox_tail2(h.a0 ^ seg, h.a0 ^ (seg + 1u), h, b0, b1);
  return Drawn{pack4(scale_to_q(b0.w0, q), scale_to_q(b0.w2, q), scale_to_q(b1.w0, q), scale_to_q(b1.w2, q)), b0.w1,
               b0.w3, b1.w1, b1.w3};
}

struct Ctx {
  uint32_t *lds;         // the region
  const uint8_t *table;  // acceptance entries, 16 per number of nearest drops
  uint32_t *hist;        // populations of this sweep (q <= 16: of all)
  uint32_t *bonds;       // this sweep's {e1, e2} columns, this lane's
  uint32_t lane_off, set_nibbles, W;
};

// left, centre and right views of the item's sites of class CX in the row at i
template <int CX>
__device__ __forceinline__ void views(const uint32_t *r, uint32_t W, uint32_t &l, uint32_t &c, uint32_t &t) {
  if (CX == 0) {
    c = r[0];
    t = r[W];
    l = alignbyte(r[2u * W], r[(int)(2u * W) - 1], 3);
  } else if (CX == 1) {
    l = r[0];
    c = r[W];
    t = r[2u * W];
  } else {
    l = r[W];
    c = r[2u * W];
    t = alignbyte(r[1], r[0], 1);
  }
}

// Per byte, the proposal's "differs" flags above and the current value's
// "equal" flags below: popcount of byte j = drop + 4 of its site.
__device__ __forceinline__ uint32_t count_flags(uint32_t k, uint32_t s) {
  return __builtin_amdgcn_bitop3_b32(0xF0F0F0F0u, k, ~(s >> 4), 0xCA);
}

// Pass (cy, CX) of one item with its words w; the next pass's are drawn while
// its reads are in flight (AHEAD: head h, segment seg).
template <int CX, int CMP, bool PRIV, bool WIDE, bool AHEAD>
__device__ __forceinline__ void pass_item(const Ctx &x, uint32_t cy, const Item &it, Drawn &w, const PhiloxHead &h,
                                          uint32_t seg, uint32_t q) {
  uint32_t *rc = x.lds + it.i + cy * 3u * x.W;
  uint32_t l, s, r, ul, U, ur, dl, D, dr;
  views<CX>(rc, x.W, l, s, r);
  views<CX>(rc - 3u * x.W, x.W, ul, U, ur);
  views<CX>(rc + 3u * x.W, x.W, dl, D, dr);
  const Drawn now = w;
  if (AHEAD) w = draw(seg, h, q);
  const uint32_t s1 = diff_pattern<CMP>(s, l, r, U, D), k1 = diff_pattern<CMP>(now.k, l, r, U, D);
  const uint32_t s2 = diff_pattern<CMP>(s, ul, ur, dl, dr), k2 = diff_pattern<CMP>(now.k, ul, ur, dl, dr);
  const uint32_t c1 = count_flags(k1, s1), c2 = count_flags(k2, s2);
  auto entry = [&](uint32_t j) {
    const uint32_t m = 0xFFu << (8u * j);
    return ((uint32_t)__popc(c1 & m) * 16u + (uint32_t)__popc(c2 & m)) * (WIDE ? 8u : 4u);
  };
  uint32_t acc = 0;  // 0xFF in every byte whose proposal is taken
  const uint32_t zero = 0, ones = 0xFFFFFFFFu;
  if (!WIDE) {
    const uint32_t t0 = *reinterpret_cast<const uint32_t *>(x.table + entry(0));
    const uint32_t t1 = *reinterpret_cast<const uint32_t *>(x.table + entry(1));
    const uint32_t t2 = *reinterpret_cast<const uint32_t *>(x.table + entry(2));
    const uint32_t t3 = *reinterpret_cast<const uint32_t *>(x.table + entry(3));
    accept_byte<0>(acc, now.a0, t0, zero, ones);
    accept_byte<1>(acc, now.a1, t1, zero, ones);
    accept_byte<2>(acc, now.a2, t2, zero, ones);
    accept_byte<3>(acc, now.a3, t3, zero, ones);
  } else {
    const uint32_t a[4] = {now.a0, now.a1, now.a2, now.a3};
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j)
      if ((uint64_t)a[j] < *reinterpret_cast<const uint64_t *>(x.table + entry(j))) acc |= 0xFFu << (8u * j);
  }
  const uint32_t ns = bfi(acc, now.k, s);
  rc[CX * x.W] = ns;
  // A bond is counted when its later-coloured end is updated, from that end's
  // final value: left where CX >= 1, right where it is 2, the row above where
  // cy >= 1, the row below where it is 2 (flags at bits 7..4: left, right, up,
  // down / up-left, up-right, down-left, down-right).
  const uint32_t up = cy >= 1u ? 1u : 0u, dn = cy == 2u ? 1u : 0u;
  const uint32_t m1 = ((CX >= 1 ? 0x80u : 0u) | (CX == 2 ? 0x40u : 0u) | up * 0x20u | dn * 0x10u) * 0x01010101u;
  const uint32_t m2 = (up * 0xC0u | dn * 0x30u) * 0x01010101u;
  const uint32_t e1 = __popc(m1 & it.own & ~bfi(acc, k1, s1)), e2 = __popc(m2 & it.own & ~bfi(acc, k2, s2));
  atomicAdd(x.bonds, e1);
  atomicAdd(x.bonds + 64, e2);
  const uint32_t one = it.own & 1u;
  if (PRIV) {  // counter (sweep, value, lane) at byte sweep << 12 | value << 8 | lane << 2
    const uint32_t v = ns | x.set_nibbles;
    uint8_t *hb = reinterpret_cast<uint8_t *>(x.hist);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0400u)), one);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0500u)), one);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0600u)), one);
    atomicAdd(reinterpret_cast<uint32_t *>(hb + perm(v, x.lane_off, 0x0C0C0700u)), one);
  } else {
#pragma unroll
    for (uint32_t b = 0; b < 4; ++b) atomicAdd(&x.hist[byte_of(ns, b)], one);
  }
}

// words of the counters in dynamic LDS: 2 x 64 bond columns per sweep, then,
// for q > 16, q shared bins per sweep
__host__ __device__ inline uint32_t counter_words(uint32_t q, uint32_t nsweeps) {
  return nsweeps * (128u + (q <= 16 ? 0u : (q + 3u) & ~3u));
}

// PRIV: q <= 16, populations in static LDS columns; NI items per lane.
template <int CMP, bool PRIV, bool WIDE, int NI>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void nnn_tile_kernel(TileParams p) {
  __shared__ __align__(16) uint64_t table_words[WIDE ? 9 * 16 : 9 * 8];
  __shared__ __align__(16) uint32_t hist16[PRIV ? 1024u * kTileMaxSweeps : 1u];
  extern __shared__ __align__(16) uint32_t lds[];
  const uint32_t ntiles = p.tiles_x * p.tiles_y;
  if (blockIdx.x >= ntiles) {
    fold_part(p.fold, blockIdx.x - ntiles, reinterpret_cast<unsigned long long *>(lds));
    return;
  }
  const uint32_t L = p.L, q = p.q;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
  const uint32_t tyi = blockIdx.x / p.tiles_x, txi = blockIdx.x - tyi * p.tiles_x;
  Region a;
  a.y0 = tyi * p.ty;
  a.x0 = txi * p.tx;
  a.W = (p.tx + 2u * p.hx) / 12u;
  a.R = p.ty + 2u * p.hy;
  a.H = (a.R / 3u) * a.W;
  a.groups = (a.H + 63u) >> 6;
  a.own_x = min(p.tx, L - a.x0);
  a.own_y = min(p.ty, L - a.y0);
  const uint32_t ncount = counter_words(q, p.nsweeps);
  // a row and a dword on either side are read, and spoil what the halo covers
  const uint32_t pad = (3u * a.W + 7u) & ~3u, cells = 3u * a.W * a.R;
  uint32_t *region = lds + ncount + pad;

  Item item[NI];
  uint32_t raw[9 * NI];
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    item[n] = item_of(p, a, wave + (uint32_t)n * waves, lane);
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) {
      const uint32_t *at = reinterpret_cast<const uint32_t *>(p.src + (size_t)(item[n].gy + c) * L + item[n].gx);
#pragma unroll
      for (uint32_t d = 0; d < 3; ++d) raw[9 * n + 3 * c + d] = at[d];
    }
  }
  // while the lattice is on its way
  for (uint32_t i = threadIdx.x; i < 81; i += blockDim.x) {
    const uint32_t to = i / 9u * 16u + i % 9u;
    if (WIDE)
      table_words[to] = p.thr[i];
    else
      reinterpret_cast<uint32_t *>(table_words)[to] = (uint32_t)(p.thr[i] - 1u);  // accept iff word <= entry
  }
  for (uint32_t i = threadIdx.x; i < ncount + pad; i += blockDim.x) lds[i] = 0;
  for (uint32_t i = threadIdx.x; i < pad; i += blockDim.x) region[cells + i] = 0;
  if (PRIV) {
    u32x4 *clear = reinterpret_cast<u32x4 *>(hist16);
    for (uint32_t i = threadIdx.x; i < 256u * p.nsweeps; i += blockDim.x) clear[i] = u32x4{0, 0, 0, 0};
  }
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    if (!item[n].valid) continue;
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) {
      const uint32_t d0 = raw[9 * n + 3 * c], d1 = raw[9 * n + 3 * c + 1], d2 = raw[9 * n + 3 * c + 2];
      uint32_t *to = region + item[n].i + c * 3u * a.W;
      // class j: bytes j, j + 3, j + 6, j + 9
      to[0] = perm(d2, perm(d1, d0, 0x0C060300u), 0x05020100u);
      to[a.W] = perm(d2, perm(d1, d0, 0x0C070401u), 0x06020100u);
      to[2u * a.W] = perm(d2, perm(d1, d0, 0x0C0C0502u), 0x07040100u);
    }
  }

  Ctx x;
  x.lds = region;
  x.table = reinterpret_cast<const uint8_t *>(table_words);
  x.lane_off = lane * 4u;
  x.W = a.W;
  constexpr bool kAhead = NI <= 2;
  // pass n of the launch: colour n % 9 of sweep n / 9
  auto head = [&](uint32_t s, uint32_t colour) {
    const uint64_t t = p.t0 + s;
    return philox_head((uint32_t)t, (uint32_t)(t >> 32), 16u + colour, p.k0, p.k1);
  };
  const uint32_t row_segs = L / 6u;
  Drawn w[NI];
  if (kAhead) {
    const PhiloxHead h = head(0, 0);
#pragma unroll
    for (int n = 0; n < NI; ++n) w[n] = draw(item[n].seg, h, q);
  }
  auto pass = [&](auto cx, uint32_t s, uint32_t cy) {
    constexpr int CX = decltype(cx)::value;
    const uint32_t colour = 3u * cy + CX, next = colour + 1u;
    const PhiloxHead h = !kAhead ? head(s, colour) : next < 9u ? head(s, next) : head(s + 1u, 0);
    // the next pass's row of the item (its words are drawn a pass ahead)
    const uint32_t row = kAhead ? (CX < 2 ? cy : cy < 2u ? cy + 1u : 0u) : cy;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      if (wave + (uint32_t)n * waves >= a.groups) continue;
      const uint32_t seg = item[n].seg + row * row_segs;
      if (!kAhead) w[n] = draw(seg, h, q);
      pass_item<CX, CMP, PRIV, WIDE, kAhead>(x, cy, item[n], w[n], h, seg, q);
    }
    __syncthreads();
  };
  __syncthreads();
  for (uint32_t s = 0; s < p.nsweeps; ++s) {
    x.hist = PRIV ? hist16 : lds + 128u * p.nsweeps + s * ((q + 3u) & ~3u);
    x.set_nibbles = s * 0x10101010u;
    x.bonds = lds + 128u * s + lane;
    for (uint32_t cy = 0; cy < 3; ++cy) {
      pass(std::integral_constant<int, 0>{}, s, cy);
      pass(std::integral_constant<int, 1>{}, s, cy);
      pass(std::integral_constant<int, 2>{}, s, cy);
    }
  }

#pragma unroll
  for (int n = 0; n < NI; ++n) {
    if (!item[n].own) continue;
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) {
      const uint32_t *from = region + item[n].i + c * 3u * a.W;
      const uint32_t c0 = from[0], c1 = from[a.W], c2 = from[2u * a.W];
      uint32_t *to = reinterpret_cast<uint32_t *>(p.dst + (size_t)(item[n].gy + c) * L + item[n].gx);
      to[0] = perm(c2, perm(c1, c0, 0x010C0400u), 0x03040100u);
      to[1] = perm(c2, perm(c1, c0, 0x06020C05u), 0x03020500u);
      to[2] = perm(c2, perm(c1, c0, 0x0C07030Cu), 0x07020106u);
    }
  }
  // the tile's totals of each sweep: four lanes per 64-lane column
  const uint32_t n2 = q + 2u, per = PRIV ? n2 : 2u;
  for (uint32_t c4 = threadIdx.x; c4 < 4u * p.nsweeps * per; c4 += blockDim.x) {
    const uint32_t c = c4 >> 2, s = c / per, v = c - s * per;
    const uint32_t *at = v < 2u ? lds + 128u * s + 64u * v : hist16 + 1024u * s + (v - 2u) * 64u;
    const u32x4 *col = reinterpret_cast<const u32x4 *>(at) + 4u * (c4 & 3u);
    const u32x4 t = col[0] + col[1] + col[2] + col[3];
    uint32_t sum = t.x + t.y + t.z + t.w;
    sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    sum += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)sum, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    if ((c4 & 3u) == 0) p.parts[((size_t)s * ntiles + blockIdx.x) * n2 + v] = sum;
  }
  if (!PRIV)
    for (uint32_t c = threadIdx.x; c < p.nsweeps * q; c += blockDim.x) {
      const uint32_t s = c / q, v = c - s * q;
      p.parts[((size_t)s * ntiles + blockIdx.x) * n2 + 2u + v] = lds[128u * p.nsweeps + s * ((q + 3u) & ~3u) + v];
    }
}

uint32_t items_of(uint32_t tx, uint32_t ty, uint32_t sweeps) {
  return (ty / 3u + 2u * sweeps) * (tx / 12u + 2u * sweeps);
}

// Items per lane and waves of a workgroup (0 items: too many).
uint32_t lanes_of(uint32_t items, uint32_t *waves) {
  const uint32_t groups = (items + 63u) >> 6;
  for (uint32_t n = 1; n <= 3; ++n)
    if (groups <= n * (kMaxBlock / 64u)) {
      *waves = (groups + n - 1u) / n;
      return n;
    }
  return 0;
}

size_t lds_bytes(const TileParams &p) {
  const uint32_t W = p.tx / 12u + 2u * p.sweeps, R = p.ty + 6u * p.sweeps;
  const size_t words = counter_words(p.q, p.sweeps) + 2u * (size_t)((3u * W + 7u) & ~3u) + 3u * (size_t)W * R;
  return words * 4 < kFoldWords * 8 ? kFoldWords * 8 : words * 4;
}

size_t static_lds(uint32_t q) { return q <= 16 ? 4096u * kTileMaxSweeps + 1152u : 1152u; }

bool set_shape(TileParams &p, uint32_t tx, uint32_t ty, uint32_t sweeps) {
  p.tx = tx;
  p.ty = ty;
  p.sweeps = sweeps;
  p.hx = 12u * sweeps;
  p.hy = 3u * sweeps;
  p.tiles_x = (p.L + tx - 1) / tx;
  p.tiles_y = (p.L + ty - 1) / ty;
  p.lift = (12u * kTileMaxSweeps + p.L - 1) / p.L * p.L;
  const uint32_t W = (tx + 2u * p.hx) / 12u;
  p.w_magic = (uint32_t)(((1ull << 32) + W - 1) / W);  // exact for the few thousand items of a region
  p.narrow = tx + p.hx > p.L || ty + p.hy > p.L || p.lift > p.L;
  uint32_t waves;
  return lanes_of(items_of(tx, ty, sweeps), &waves) != 0 && lds_bytes(p) + static_lds(p.q) <= kMaxLds;
}

// Time of one launch in microseconds, as in tiles.hip measured on MI355X (q =
// 9, 3900 shapes of L = 60 .. 6000) and fitted: the launch and the copies, then
// per pass 0.5 us of latency or the issue time of the n items that a SIMD
// holds; tiles narrower than 1.5 times their height up to 10 % more.  The shapes
// it picks took 3 % longer than the best measured ones on average, 8 % at most.
float launch_us(uint32_t L, uint32_t tx, uint32_t ty, uint32_t sweeps) {
  uint32_t waves = 0;
  const uint32_t ni = lanes_of(items_of(tx, ty, sweeps), &waves);
  if (!ni) return 0;
  const float n = (float)(ni * ((waves + 3u) / 4u));
  const float issue = 0.1f + 0.3f * n, wide = (float)tx / (1.5f * (float)ty);
  const float turns = (float)((((L + tx - 1) / tx) * ((L + ty - 1) / ty) + 255u) / 256u);
  return (4.0f + n + 9.0f * (float)sweeps * (issue > 0.5f ? issue : 0.5f)) * turns *
         (wide < 1.0f ? 1.1f - 0.1f * wide : 1.0f);
}

template <int CMP, bool PRIV, bool WIDE>
hipError_t launch_n(const TileParams &p, hipStream_t stream) {
  uint32_t waves = 0;
  const uint32_t ni = lanes_of(items_of(p.tx, p.ty, p.sweeps), &waves);
  const size_t lds = lds_bytes(p);
  const dim3 grid(p.tiles_x * p.tiles_y + fold_groups(p.fold)), block(64u * waves);
  auto go = [&](auto kernel) {
    hipError_t e = hipSuccess;
    if (lds > 48u * 1024u)
      e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, p);
    return hipGetLastError();
  };
  if (ni == 1) return go(nnn_tile_kernel<CMP, PRIV, WIDE, 1>);
  if (ni == 2) return go(nnn_tile_kernel<CMP, PRIV, WIDE, 2>);
  return ni == 3 ? go(nnn_tile_kernel<CMP, PRIV, WIDE, 3>) : hipErrorInvalidValue;
}

template <bool WIDE>
hipError_t launch_w(const TileParams &p, hipStream_t stream) {
  if (p.q <= 16) return launch_n<0, true, WIDE>(p, stream);
  if (p.q <= 128) return launch_n<1, false, WIDE>(p, stream);
  return launch_n<2, false, WIDE>(p, stream);
}

}  // namespace

bool auto_tile_shape(TileParams &p, int64_t nsweeps) {
  if (p.L < 12 || p.L % 12 || p.q < 2 || p.q > 256) return false;
  // sides that cut L into 1 .. 32 equal parts, tx in twelves, ty in threes
  uint32_t side[2][40], n[2] = {0, 0};
  for (int d = 0; d < 2; ++d) {
    const uint32_t unit = d ? 3u : 12u, least = d ? 9u : 12u;
    for (uint32_t k = 1; k <= 32; ++k) {
      uint32_t t = ((p.L + k - 1) / k + unit - 1u) / unit * unit;
      t = t < least ? least : t;
      if (t <= (d ? 288u : 432u) && (n[d] == 0 || side[d][n[d] - 1] != t)) side[d][n[d]++] = t;
    }
    if (n[d] == 0)
      for (uint32_t t = 288; t >= 144; t -= 24) side[d][n[d]++] = t;
  }
  const int64_t m = nsweeps > 64 ? 64 : nsweeps < 1 ? 1 : nsweeps;  // long calls: per sweep
  float best = 0;
  TileParams found = p;
  for (uint32_t s = 1; s <= kTileMaxSweeps && (int64_t)s <= m; ++s) {
    const float launches = nsweeps > 64 ? 64.0f / (float)s : (float)((m + s - 1) / s);
    for (uint32_t i = 0; i < n[0]; ++i)
      for (uint32_t j = 0; j < n[1]; ++j) {
        const uint32_t tx = side[0][i], ty = side[1][j];
        if (tx > 3u * ty || ty > 3u * tx) continue;
        const float us = launches * launch_us(p.L, tx, ty, s);
        if (us > 0 && (best == 0 || us < best) && set_shape(p, tx, ty, s)) {
          best = us;
          found = p;
        }
      }
  }
  p = found;
  return best > 0;
}

hipError_t launch_tiles(const TileParams &p, hipStream_t stream) {
  if (p.nsweeps == 0) return hipSuccess;
  if (p.nsweeps > p.sweeps || p.sweeps > kTileMaxSweeps || !p.src || !p.dst || !p.parts || p.hx != 12u * p.sweeps ||
      p.hy != 3u * p.sweeps || p.lift % p.L || p.lift < p.hx || (p.fold.nsweeps && !p.fold.parts))
    return hipErrorInvalidValue;
  bool wide = false;  // some entry is 0
  for (int i = 0; i < 81; ++i) wide = wide || p.thr[i] == 0;
  return wide ? launch_w<true>(p, stream) : launch_w<false>(p, stream);
}

}  // namespace nnn
}  // namespace potts
