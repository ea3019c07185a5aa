// heatbath_packed.hip -- heat-bath half sweeps of a single lattice on its
// colour-split copy (the planes packed.hip sweeps; Sec. 7 names the heat bath
// as the other single-spin-flip update).
//
// The new value of a site does not depend on its current value, so a colour-c
// half sweep reads only plane c^1 (the neighbours) and writes plane c: N bytes
// per half sweep.  A work item is 16 packed bytes (16 sites of colour c) of R
// rows, walked downwards as in packed.hip, each passive row loaded once; the
// operands of two rows are read before either is stored, and L % 32 != 0 has
// partial items (edge.hpp).  VALU issue bounds it (about 66 operations a site).
// Measured on MI355X (q = 6, us per sweep): L = 8192 113 (117 with a row's
// operands read after the store before it, on walks of four rows), 6144 70 (80),
// L = 5000 59.5 (147 with one 4-byte chunk per thread).
//
// The draw (contract: value v weighs D[n_max - n(v)], D[0] = 2^32, D[d] =
// thr[d-1]; the distinct neighbour values in order of first appearance among
// (up, down, left, right), then the others ascending; r = floor(w Z / 2^32)
// picks the first value whose cumulative weight exceeds r):
//   * which neighbour values are equal (six flags, four sites at a time with
//     byte-wise arithmetic) indexes a 64-entry table built on the host;
//   * the cumulative weights of the ranked neighbour values c_i are turned
//     into cuts on the word itself: r < c_i exactly when w < ceil(c_i 2^32 /
//     Z), so four 32-bit compares and byte selects pick among the neighbour
//     values;
//   * past them (r >= S, the neighbour values' total), the run of other
//     values, each of weight w0 = D[n_max], is indexed by j = floor((r - S) /
//     w0) (an FP32 estimate from above and one integer check), and the j-th
//     value held by no neighbour comes from a bit mask of the neighbour values
//     (q <= 16) or from the sorted neighbour values.
#include <hip/hip_runtime.h>

#include <string.h>

#include <algorithm>

#include "device.hpp"
#include "edge.hpp"
#include "heatbath_draw.hpp"
#include "kernels.hpp"
#include "sweep_row.hpp"

namespace potts {
namespace {

constexpr int kBlock = 256;
constexpr int kWaves = kBlock / 64;

using namespace row;

struct HbCarry {
  u32x4 u;  // passive row y-1
  u32x4 p;  // passive row y
};

// Operands of one item row: the passive row below at d_off, the passive dword
// beside the item at side_off (left of it when O == 0, right of it when O == 1).
struct HbIn {
  u32x4 dn;
  uint32_t side;
};

__device__ __forceinline__ HbIn hb_load(__amdgpu_buffer_rsrc_t rs, uint32_t d_off, uint32_t side_off) {
  return HbIn{load16(rs, d_off), load4(rs, side_off)};
}

// One item row: the 16 active sites at a_off (written).  ctr: Philox chunk of
// the item's first byte (a multiple of 8 unless RAG), h: the half sweep's
// Philox head.  RAG: partial items (edge.hpp).
template <int COLOUR, int O, int CMP, bool PRIV, bool WIDE, bool RAG>
__device__ __forceinline__ void hb_row(const PhiloxHead &h, __amdgpu_buffer_rsrc_t rs, const uint8_t *tab,
                                       uint8_t *hist, uint32_t lane_off, const Edge &edge, const HbIn &in,
                                       uint32_t a_off, uint32_t ctr, HbCarry &cy, uint32_t &nz) {
  const u32x4 dn = in.dn;
  const uint32_t side = RAG && O == 0 ? in.side << edge.shift : in.side;
  const u32x4 pp = RAG && O == 1 ? with_wrap(edge, cy.p, side) : cy.p;
  const uint32_t P[4] = {pp.x, pp.y, pp.z, pp.w};
  const uint32_t U[4] = {cy.u.x, cy.u.y, cy.u.z, cy.u.w};
  const uint32_t D[4] = {dn.x, dn.y, dn.z, dn.w};
  uint32_t out[4];
  const uint32_t x0 = h.a0 ^ ctr;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    // the other horizontal neighbour: the passive byte one site over
    const uint32_t x = O == 0 ? alignbyte(P[g], g == 0 ? side : P[g - 1], 3)
                              : alignbyte(g == 3 ? side : P[g + 1], P[g], 1);
    const uint32_t lf = O == 0 ? x : P[g];
    const uint32_t rt = O == 0 ? P[g] : x;
    // packed bytes 4g, 4g+1 use block 2g (words 0, 2), 4g+2, 4g+3 block 2g+1
    const Words b0 = philox_tail(RAG ? h.a0 ^ (ctr + (uint32_t)(2 * g)) : x0 ^ (uint32_t)(2 * g), h);
    const Words b1 = philox_tail(RAG ? h.a0 ^ (ctr + (uint32_t)(2 * g + 1)) : x0 ^ (uint32_t)(2 * g + 1), h);
    out[g] = draw4<CMP, WIDE>(U[g], D[g], lf, rt, b0.w0, b0.w2, b1.w0, b1.w2, tab);
    if (COLOUR == 1) {
      const uint32_t differs = diff_pattern<CMP>(out[g], U[g], D[g], lf, rt) & 0xF0F0F0F0u;
      nz += __popc(RAG ? differs & edge.valid[g] : differs);
    }
    if (RAG) out[g] &= edge.valid[g];  // bytes that are no sites stay 0, and are counted as that
  }
  u32x4 o;
  o.x = out[0];
  o.y = out[1];
  o.z = out[2];
  o.w = out[3];
  store16(rs, a_off, o);
  if (PRIV) {
    count_active_private(hist, lane_off, out[0], out[1]);
    count_active_private(hist, lane_off, out[2], out[3]);
  } else {
    count_active_shared(reinterpret_cast<uint32_t *>(hist), out[0], out[1]);
    count_active_shared(reinterpret_cast<uint32_t *>(hist), out[2], out[3]);
  }
  cy.u = cy.p;
  cy.p = dn;
}

// The compiler's register choice (about 92 VGPRs, 5 waves per SIMD) measured
// faster than 6 or 8 waves per SIMD forced (1.81 against 1.91 and 1.94 ps per
// site update at L = 8192, q = 9: the forced forms spill inside the loop).
template <int COLOUR, int CMP, bool PRIV, bool WIDE, bool RAG>
__global__ __launch_bounds__(kBlock) void hb_packed_kernel(HbLaunch launch) {
  __shared__ __align__(16) uint8_t tab[HbTable::kBytes];
  constexpr uint32_t kHistWords = PRIV ? 64u * (CMP == 0 ? 16u : kPrivateHistMaxQ) : 256u;
  __shared__ __align__(16) uint32_t hist[kHistWords];
  __shared__ uint32_t partial[256];
  __shared__ unsigned long long esum;
  __shared__ uint32_t no_sites;  // counted bytes that are no sites (RAG)
  const StripParams &p = launch.p;
  const uint32_t bid = COLOUR == 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const uint32_t first = bid * kBlock + threadIdx.x;
  const uint32_t stride = gridDim.x * kBlock;
  const uint64_t t = p.t0 + launch.sweep;
  const PhiloxHead h = philox_head((uint32_t)t, (uint32_t)(t >> 32), (uint32_t)COLOUR + 4u, p.k0, p.k1);
  const uint32_t q = p.q;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave = threadIdx.x >> 6;

  {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(launch.table);
    u32x4 *dst = reinterpret_cast<u32x4 *>(tab);
    const uint32_t n = (WIDE ? HbTable::kBytes : HbTable::kCut64) / 16;
    for (uint32_t i = threadIdx.x; i < n; i += kBlock) dst[i] = src[i];
  }
  const uint32_t nh = PRIV ? 64 * q : q;
  for (uint32_t i = threadIdx.x; i < nh; i += kBlock) hist[i] = 0;
  if (threadIdx.x == 0) {
    esum = 0;
    no_sites = 0;
  }
  if (p.stripes) {
    __shared__ unsigned long long fold_acc[COLOUR == 0 ? 257 : 1];
    if (COLOUR == 0 && bid == 0 && launch.sweep > 0) fold_stripes<kBlock>(p, t - 1, fold_acc);
  } else if (COLOUR == 1 && bid == 0) {
    unsigned long long *rec_next = p.ring + ((t + 1) & (p.cap - 1)) * (uint64_t)(q + 1);
    for (uint32_t i = threadIdx.x; i < q + 1; i += kBlock) rec_next[i] = 0;
  }
  __syncthreads();

  const __amdgpu_buffer_rsrc_t rs = lattice_rsrc(p.spins);
  uint8_t *hist_bytes = reinterpret_cast<uint8_t *>(hist);
  const uint32_t lane_off = lane * 4u;
  const uint32_t L = p.L;
  const uint32_t half = L >> 1;                     // sites per plane row
  const uint32_t pitch = RAG ? p.ipr * 16u : half;  // bytes per plane row
  const uint32_t plane = pitch * L;
  const uint32_t a_base = COLOUR == 0 ? 0u : plane;
  const uint32_t p_base = COLOUR == 0 ? plane : 0u;
  const uint32_t rows = p.rows;
  uint32_t nz = 0, sites = 0, missing = 0;

  for (uint32_t item = first; item < p.nitems; item += stride) {
    const uint32_t rb = p.item_shift >= 0 ? item >> p.item_shift
                                          : (uint32_t)__umul64hi((uint64_t)item, p.item_magic);
    const uint32_t xi = item - rb * p.ipr;
    const uint32_t col = xi * 16u;
    const uint32_t left_col = col == 0 ? (RAG ? last_dword(half) : half - 4u) : col - 4u;
    const uint32_t right_col = col + 16u == pitch ? 0u : col + 16u;
    Edge edge{};
    if (RAG) edge = edge_of(col, half);
    const uint32_t r0 = rb * rows;
    const uint32_t rp = r0 == 0 ? L - 1 : r0 - 1;
    HbCarry cy;
    cy.u = load16(rs, p_base + rp * pitch + col);
    cy.p = load16(rs, p_base + r0 * pitch + col);
    uint32_t ctr = r0 * p.row_words + (col >> 1);
    // row parity 0: O = COLOUR
    const uint32_t side0 = COLOUR == 0 ? left_col : right_col, side1 = COLOUR == 0 ? right_col : left_col;
    for (uint32_t k = 0; k < rows; k += 2) {
      const uint32_t y = r0 + k;
      const uint32_t yd = k + 2 == rows ? (r0 + rows == L ? 0u : r0 + rows) : y + 2;
      // both rows' operands before either row's store, which would hold them back
      const HbIn in0 = hb_load(rs, p_base + (y + 1) * pitch + col, p_base + y * pitch + side0);
      const HbIn in1 = hb_load(rs, p_base + yd * pitch + col, p_base + (y + 1) * pitch + side1);
      hb_row<COLOUR, COLOUR, CMP, PRIV, WIDE, RAG>(h, rs, tab, hist_bytes, lane_off, edge, in0,
                                                   a_base + y * pitch + col, ctr, cy, nz);
      ctr += p.row_words;
      hb_row<COLOUR, COLOUR ^ 1, CMP, PRIV, WIDE, RAG>(h, rs, tab, hist_bytes, lane_off, edge, in1,
                                                       a_base + (y + 1) * pitch + col, ctr, cy, nz);
      ctr += p.row_words;
    }
    sites += (RAG ? 16u - edge.missing : 16u) * rows;
    missing += edge.missing * rows;
  }

  if (COLOUR == 1) {
    const uint32_t e = wave_sum(4u * sites - nz);
    if (lane == 0 && e) atomicAdd(&esum, (unsigned long long)e);
  }
  if (RAG) {
    const uint32_t m = wave_sum(missing);
    if (lane == 0 && m) atomicAdd(&no_sites, m);
  }
  __syncthreads();
  if (PRIV) {
    for (uint32_t v = wave; v < q; v += kWaves) {
      const uint32_t s = wave_sum(hist[v * 64u + lane]);
      if (lane == 0) partial[v] = s;
    }
    __syncthreads();
  }
  unsigned long long *rec = p.ring + (t & (p.cap - 1)) * (uint64_t)(q + 1);
  unsigned long long *dst =
      p.stripes ? p.stripes + ((t & 1) * p.nstripes + (bid & (p.nstripes - 1))) * (uint64_t)stripe_words(q) : rec;
  for (uint32_t v = threadIdx.x; v < q; v += kBlock) {
    uint32_t s = PRIV ? partial[v] : hist[v];
    if (RAG && v == 0) s -= no_sites;
    if (s) atomicAdd(&dst[1 + v], (unsigned long long)s);
  }
  if (COLOUR == 1 && threadIdx.x == 0 && esum) atomicAdd(&dst[0], esum);
}

template <int COLOUR, bool WIDE, bool RAG>
hipError_t launch_w(const HbLaunch &l, unsigned grid, uint32_t q, hipStream_t stream) {
  if (q <= 16)
    hipLaunchKernelGGL((hb_packed_kernel<COLOUR, 0, true, WIDE, RAG>), dim3(grid), dim3(kBlock), 0, stream, l);
  else if (q <= kPrivateHistMaxQ)
    hipLaunchKernelGGL((hb_packed_kernel<COLOUR, 1, true, WIDE, RAG>), dim3(grid), dim3(kBlock), 0, stream, l);
  else if (q <= 128)
    hipLaunchKernelGGL((hb_packed_kernel<COLOUR, 1, false, WIDE, RAG>), dim3(grid), dim3(kBlock), 0, stream, l);
  else
    hipLaunchKernelGGL((hb_packed_kernel<COLOUR, 2, false, WIDE, RAG>), dim3(grid), dim3(kBlock), 0, stream, l);
  return hipGetLastError();
}

}  // namespace

bool build_heatbath_table(const uint32_t thr[4], uint32_t q, HbTable *t) {
  memset(t->bytes, 0, sizeof(t->bytes));
  const bool wide = !thr[0] || !thr[1] || !thr[2] || !thr[3];
  uint32_t *cut = reinterpret_cast<uint32_t *>(t->bytes + HbTable::kCut);
  uint32_t *zs = reinterpret_cast<uint32_t *>(t->bytes + HbTable::kZs);
  uint32_t *wi = reinterpret_cast<uint32_t *>(t->bytes + HbTable::kWi);
  uint64_t *cut64 = reinterpret_cast<uint64_t *>(t->bytes + HbTable::kCut64);
  auto weight = [&](uint32_t gap) -> uint64_t { return gap == 0 ? (1ull << 32) : (uint64_t)thr[gap - 1]; };
  for (uint32_t pat = 0; pat < 64; ++pat) {
    const uint32_t eab = !(pat & 32u), eac = !(pat & 16u), ead = !(pat & 8u);
    const uint32_t ebc = !(pat & 4u), ebd = !(pat & 2u), ecd = !(pat & 1u);
    const uint32_t na = 1 + eab + eac + ead, nb = 1 + eab + ebc + ebd;
    const uint32_t nc = 1 + eac + ebc + ecd, nd = 1 + ead + ebd + ecd;
    const uint32_t nmax = std::max(std::max(na, nb), std::max(nc, nd));
    // b, c, d count where they appear first
    const bool fb = !eab, fc = !eac && !ebc, fd = !ead && !ebd && !ecd;
    const uint64_t wa = weight(nmax - na);
    const uint64_t wb = fb ? weight(nmax - nb) : 0;
    const uint64_t wc = fc ? weight(nmax - nc) : 0;
    const uint64_t wd = fd ? weight(nmax - nd) : 0;
    const uint32_t m = 1 + fb + fc + fd;
    const uint64_t w0 = nmax >= 1 && nmax <= 4 ? (uint64_t)thr[nmax - 1] : 0;
    const uint64_t S = wa + wb + wc + wd;
    uint64_t Z = S + (q > m ? (uint64_t)(q - m) * w0 : 0);
    if (Z == 0) Z = 1;  // a pattern no four values show (equality is transitive)
    const uint64_t c[4] = {wa, wa + wb, wa + wb + wc, S};
    for (int i = 0; i < 4; ++i) {
      // r = floor(w Z / 2^32) < c  <=>  w < ceil(c 2^32 / Z)
      const unsigned __int128 num = ((unsigned __int128)c[i] << 32) + (Z - 1);
      uint64_t T = (uint64_t)(num / Z);
      if (T > (1ull << 32)) T = 1ull << 32;
      cut64[pat * 4 + i] = T;
      cut[pat * 4 + i] = T == 0 ? 0u : (uint32_t)(T - 1);
    }
    zs[pat * 4 + 0] = (uint32_t)Z;
    zs[pat * 4 + 1] = (uint32_t)(Z >> 32);
    zs[pat * 4 + 2] = (uint32_t)S;
    zs[pat * 4 + 3] = (uint32_t)(S >> 32);
    // 1/w0 rounded up by 2^-19 relative, so the kernel's FP32 estimate of
    // floor(X / w0) is never below it
    const float inv = w0 ? (float)((1.0 + 0x1p-19) / (double)w0) : 0.0f;
    uint32_t inv_bits;
    memcpy(&inv_bits, &inv, 4);
    wi[pat * 4 + 0] = (uint32_t)w0;
    wi[pat * 4 + 1] = inv_bits;
  }
  return wide;
}

hipError_t launch_heatbath_packed(const HbLaunch &l, int colour, unsigned grid, bool wide, hipStream_t stream) {
  if (grid == 0) return hipSuccess;
  const uint32_t q = l.p.q;
  if (l.p.L % 32) {
    if (l.p.ipr * 16u != plane_pitch(l.p.L)) return hipErrorInvalidValue;
    if (colour == 0)
      return wide ? launch_w<0, true, true>(l, grid, q, stream) : launch_w<0, false, true>(l, grid, q, stream);
    return wide ? launch_w<1, true, true>(l, grid, q, stream) : launch_w<1, false, true>(l, grid, q, stream);
  }
  if (colour == 0)
    return wide ? launch_w<0, true, false>(l, grid, q, stream) : launch_w<0, false, false>(l, grid, q, stream);
  return wide ? launch_w<1, true, false>(l, grid, q, stream) : launch_w<1, false, false>(l, grid, q, stream);
}

}  // namespace potts
