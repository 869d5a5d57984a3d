// Relaxation step of the multi-phase SPH mesh generator (Ji, Fu, Hu & Adams, arXiv 1906.07925)
// on MI355X / gfx950.  The C ABI is declared in include/mpsph.h.
//
// A context holds one or more independent domains of the same dimension (a batch).  Domains
// occupy contiguous ranges of every particle array and of the global cell index space, so one
// launch of each kernel serves all of them; kernels read their domain's parameters from a device
// table.  The step counter lives on the device, so a captured step can be replayed.
//
// Data layout (HBM, structure of arrays, n particles over all domains):
//   state  (order of the previous step): key u32 (domain cell base + packed cell), off float4 (cell
//          offsets, arrival number), ct u32 (type | colour << 2), id u32 (index at load), cell u32
//          (search cell)
//   work   (this step's search order): key u32, pos float4 (offsets, h), fix float4 (fixed-point
//          coordinates, h), jaux u32 (colour | type << 30), id u32
//   per step: acc float4 (a, e = rho_t nu_coeff r_c |a|), search table u32[cells+1]; rho, sum|term|,
//             a~, v, nearest distance only in debug mode
// Positions are an integer cell coordinate per axis (packed in the key: x fastest and at
// sub-cell resolution, 3D rows numbered in tiles by row_index) plus a float offset in [0, 1) in
// cell units.  The pair passes read neighbours as 32-bit fixed-point coordinates of the same positions
// (multiples of 2^-27 cells as a rule), so a separation is an exact integer difference, rounded once.
// The order of the particles and the table of the pair scan belong to a search grid of their own,
// whose rows follow the cut-off (search_rows_rule).  Lengths inside the kernels are
// in cell units; accelerations and velocities are the domain values divided by the cell size
// (time is unchanged; the EOS constant is scaled by cs^(d-2) to make this exact).
//
// Launch sequence of one step (all on the context stream, no host synchronisation):
//   cell_scan, cell_place   search table and order from the counts that the load and the integrator
//                   keep (cells.hip)
//   reorder_field   gather the state in search order, evaluate the target field (Eq. 1-2, 16)
//   pass_density_force  density (Eq. 17), pressure + surface tension (Eq. 18-19, 23-25),
//                   projection (Eq. 30-31), first time step (Eq. 29, block minima); like the
//                   viscous pass, a lane group per particle walks its candidates through a row
//                   table in LDS (scan_group_table in pair_scan.h)
//   pass_viscous_integrate  mid-point velocity (Eq. 26), viscosity (Eq. 21-22), viscous
//                   acceleration (Eq. 20), second time step (Eq. 29), velocity (Eq. 27), drift
//                   (Eq. 28), feature projection and re-tagging (Eq. 32)
//   finalize        FP64 reduction of the per-block partials in a fixed order (small grids: at the end
//                   of pass_viscous_integrate)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "mpsph.h"
#include "mpsph_device.h"
#include "adjoint.h"
#include "cells.h"
#include "pair_scan.h"

using namespace mpsph;

namespace {

// ------------------------------------------------------------------------------------------
// Kernels
// ------------------------------------------------------------------------------------------

// Counts a particle into its new search cell and returns its arrival number there as the bits of a
// float (kept in the offset's fourth word).
// The atomics make the viscous pass of 2M particles 22 us longer, with or without the answer;
// taking the arrival numbers in cell_place instead costs 34 us more there.
__device__ __forceinline__ float count_arrival(uint32_t *counts, uint32_t key) {
  return __uint_as_float(atomicAdd(&counts[key], 1u));
}

// Domain units -> (cell, offset) in FP64 (identical inputs give identical keys), validation.
// Internal particles [i0, i1) of one dimension group.
template <int D>
__global__ __launch_bounds__(kBlock) void load_kernel(const DomDev *__restrict__ doms, int ndom, int i0, int i1,
                                                      const float *__restrict__ pos, const int32_t *__restrict__ colour,
                                                      const int32_t *__restrict__ type, uint32_t *__restrict__ key,
                                                      float4 *__restrict__ off, uint32_t *__restrict__ ct,
                                                      uint32_t *__restrict__ id, uint32_t *__restrict__ cell,
                                                      uint32_t *__restrict__ counts, int *__restrict__ bad) {
  const int i = i0 + blockIdx.x * kBlock + threadIdx.x;
  if (i >= i1) return;
  const DomDev &dd = doms[domain_of(doms, ndom, i)];
  const int local = i - dd.off;
  const int u = dd.uoff + local;
  const float *x = pos + dd.xoff + (int64_t)local * D;
  int c[3] = {0, 0, 0};
  float o[3] = {0.f, 0.f, 0.f};
  bool ok = true;
  for (int a = 0; a < D; ++a) {
    double X = ((double)x[a] - dd.lo[a]) * dd.inv_cs;
    if (!(X >= 0.0 && X <= dd.xhi[a])) ok = false;
    if (dd.g.geometry == 0 && X >= dd.xhi[a]) X -= dd.xhi[a];   // periodic: hi is lo
    double f = floor(X);
    float fo = (float)(X - f);
    if (fo >= 1.0f) {
      fo = 0.0f;
      f += 1.0;
    }
    if (!(f >= 0.0 && f <= (double)dd.g.gmax)) ok = false;
    c[a] = ok ? (int)f : 0;
    o[a] = ok ? fo : 0.f;
  }
  const int col = colour[u];
  const int t = type ? type[u] : 0;
  if (col < 0 || col >= (1 << 16) || t < 0 || t > 3) ok = false;
  if (!ok) atomicOr(bad, 1);
  key[i] = dd.cellbase + pack_key<D>(c, o, dd.g);
  const uint32_t sc = dd.sbase + search_key<D>(c, o, dd.g);
  cell[i] = sc;
  off[i] = make_float4(o[0], o[1], D == 3 ? o[2] : 0.f, count_arrival(counts, sc));
  ct[i] = (uint32_t)(t & 3) | ((uint32_t)col << 2);
  id[i] = (uint32_t)u;
}

// Waves per SIMD the pair kernels are compiled for (their register budget: 64 VGPRs and 96 SGPRs
// at 8 waves); 0 leaves it to the compiler, which otherwise settles at 7 waves.  Measured on the
// 2M-particle graded cube: 8 waves make both pair passes 12-13 % faster.
#ifndef MPSPH_PAIR_WAVES
#define MPSPH_PAIR_WAVES 8
#endif
#if MPSPH_PAIR_WAVES > 0
#define MPSPH_PAIR_OCCUPANCY __attribute__((amdgpu_waves_per_eu(MPSPH_PAIR_WAVES, MPSPH_PAIR_WAVES)))
#else
#define MPSPH_PAIR_OCCUPANCY
#endif

// Gather the state in search order, evaluate the size field (h = tau s, Eq. 16) and write the working
// arrays; sorted indices [i0, i1) of one dimension group.  Slot i names one of its search cell's
// particles, whose place in the cell is its rank by index among the cell's slots (a cell's particles
// are all candidates of one another, so the ranking is small against the pair passes whatever the
// occupancy).  The first nreset threads also reset the time-step slots.
#define MPSPH_GATHER_PARAMS                                                                                            \
  const DomDev *__restrict__ doms, int ndom, int i0, int i1, int nreset, const uint32_t *__restrict__ slots,           \
      const uint32_t *__restrict__ cstart, const uint32_t *__restrict__ cell, const uint32_t *__restrict__ skey,       \
      const float4 *__restrict__ soff, const uint32_t *__restrict__ sct, const uint32_t *__restrict__ sid,             \
      uint32_t *__restrict__ wkey, float4 *__restrict__ wpos, float4 *__restrict__ wfix, uint32_t *__restrict__ wjaux, \
      uint32_t *__restrict__ wid, uint32_t *__restrict__ perm, uint32_t *__restrict__ dtslots
#define MPSPH_GATHER_ARGS \
  doms, ndom, i0, i1, nreset, slots, cstart, cell, skey, soff, sct, sid, wkey, wpos, wfix, wjaux, wid, perm, dtslots
template <int D>
__device__ __forceinline__ void reorder_block(int blk, MPSPH_GATHER_PARAMS) {
  const int t = blk * kBlock + threadIdx.x;
  if (t < nreset) dtslots[t * kDtStride] = kInfBits;
  const int i = i0 + t;
  if (i >= i1) return;
  const uint32_t s = slots[i];
  const uint32_t sc = cell[s];
  const uint32_t a = cstart[sc], b = cstart[sc + 1u];
  uint32_t at = a;
  if (b - a > 1u)
    for (uint32_t q = a; q < b; ++q) at += slots[q] < s ? 1u : 0u;
  const DomDev &dd = doms[domain_of(doms, ndom, i)];
  const uint32_t key = skey[s];
  const float4 o4 = soff[s];
  const uint32_t ct = sct[s];
  int c[3];
  unpack_key<D>(key - dd.cellbase, dd.g, c);
  const float o[3] = {o4.x, o4.y, o4.z};
  const float h = dd.sp.tau * field_spacing<D>(dd.f, c, o);
  perm[at] = s;
  wkey[at] = key;
  wpos[at] = make_float4(o4.x, o4.y, o4.z, h);
  wfix[at] = make_float4(fixed_bits(c[0], o[0], dd.g), fixed_bits(c[1], o[1], dd.g),
                         D == 3 ? fixed_bits(c[2], o[2], dd.g) : 0.f, h);
  wjaux[at] = pack_aux(ct & 3u, ct >> 2);
  wid[at] = sid[s];
}

template <int D>
__global__ __launch_bounds__(kBlock) void reorder_field(MPSPH_GATHER_PARAMS) {
  reorder_block<D>(blockIdx.x, MPSPH_GATHER_ARGS);
}

// Both dimension groups: the 2D particles [i0, im) in the first nblk2 blocks, the 3D ones after them.
__global__ __launch_bounds__(kBlock) void reorder_field_mixed(int im, int nblk2, MPSPH_GATHER_PARAMS) {
  if ((int)blockIdx.x < nblk2) {
    i1 = im;
    reorder_block<2>(blockIdx.x, MPSPH_GATHER_ARGS);
  } else {
    i0 = im;
    nreset = 0;
    reorder_block<3>((int)blockIdx.x - nblk2, MPSPH_GATHER_ARGS);
  }
}

// Pass 1: density (Eq. 17, self term included, radius kappa h_i) and
//   a_i = -sum_j (1 + beta_ij) (P_i + P_j) dW(r_ij, h_ij)/dr e_ij   (Eq. 18, 23; gamma = 2, Eq. 19)
// with e_ij = r_ij / |r_ij|, r_ij = r_i - r_j, beta_ij = sigma for different colours (Eq. 24),
// P = p0 / rho_t^2, h_ij = (h_i + h_j)/2, over j with r_ij < kappa h_ij that particle i feels.
// Writes acc = (a after the force mapping of Eq. 30-31, e_i) with e_i = rho_t nu_coeff r_c |a_i|,
// the viscosity of Eq. 21-22 per unit of dt1/2, and the first time-step candidate (Eq. 29).
// L lanes per particle (group) sum its pairs; the block's first 256/L threads then finish one
// particle each (the epilogue) and the first wave combines the block's metric partials.
// LDS-staged density pass (3D; pair-kernel variant MPSPH_PAIRS_TILE): the targets of a block share one
// copy of their neighbours in LDS.  The union of the targets' candidate rows (y, z) and, per row,
// of their x-runs is formed with LDS atomics; every union row's particles (offsets and h, flags)
// are copied into LDS once; the targets' row tables then index that copy.  A block whose union
// has more than kTileRows rows or MPSPH_TILE_CAP particles reads its neighbours from global memory.
// Staged particles per block.  Measured on the 2M-particle graded cube (2^6 cells, 8 lanes):
// 768 particles (39 KB of LDS per block with the row table, 4 waves per SIMD) 1.82 ms per density
// pass (1536, 54 KB and 3 waves, took 1.8 times as long), against 0.91 ms for the pass that reads its neighbours
// through the caches at 8 waves per SIMD.
#ifndef MPSPH_TILE_CAP
#define MPSPH_TILE_CAP 768
#endif
constexpr int kTileRows = kBlock;
struct TileLds {
  int y0, y1, z0, z1;
  int ux0[kTileRows], ux1[kTileRows];        // union x-run of each search row (x sub-cells)
  uint32_t ra[kTileRows];                    // global index of the first staged particle of a row
  uint32_t roff[kTileRows + 1];              // LDS index of a row's first particle; roff[rows] = total
  float4 pos[MPSPH_TILE_CAP];
  uint32_t aux[MPSPH_TILE_CAP];
};
struct TileRemap {
  const TileLds *T;
  int w;   // rows per z of the union
  __device__ __forceinline__ uint32_t operator()(int cy, int cz, uint32_t a) const {
    const int r = (cz - T->z0) * w + (cy - T->y0);
    return T->roff[r] + (a - T->ra[r]);
  }
};

// Exclusive prefix sum over the block's threads; *total receives the sum (every thread).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *total) {
  __shared__ uint32_t wsum[kBlock / kWave];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  if (lane == kWave - 1) wsum[w] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kBlock / kWave; ++k) {
    if (k < w) base += wsum[k];
    tot += wsum[k];
  }
  __syncthreads();
  *total = tot;
  return base + incl - v;
}

// Stages the neighbours of the block's targets (3D, no periodic wrap); the rows and x-runs are
// those of scan_group_table.  Called by every thread of the block; returns the same value in
// every thread (false: the union does not fit).
template <int L>
__device__ bool stage_tile(TileLds *T, bool active, int sub, const OwnRow &own, float rs, const GridDev &g,
                           uint32_t sbase, const uint32_t *__restrict__ cstart, const float4 *__restrict__ wfix,
                           const uint32_t *__restrict__ wjaux) {
  rs = fminf(fmaxf(rs, 0.f), 2.f * (float)g.gmax + 2.f) * g.rowinv;
  const float rs2 = rs * rs;
  const int gmaxr = (1 << g.skr) - 1;
  int y0 = 0, y1 = -1, z0 = 0, z1 = -1;
  if (active) {
    z0 = max(0, own.rz + (int)floorf(own.oz - rs));
    z1 = min(gmaxr, own.rz + (int)floorf(own.oz + rs));
    y0 = max(0, own.ry + (int)floorf(own.oy - rs));
    y1 = min(gmaxr, own.ry + (int)floorf(own.oy + rs));
  }
  if (threadIdx.x == 0) {
    T->y0 = INT_MAX;
    T->y1 = -1;
    T->z0 = INT_MAX;
    T->z1 = -1;
  }
  __syncthreads();
  if (active && sub == 0) {
    atomicMin(&T->y0, y0);
    atomicMax(&T->y1, y1);
    atomicMin(&T->z0, z0);
    atomicMax(&T->z1, z1);
  }
  __syncthreads();
  const int W = T->y1 - T->y0 + 1, H = T->z1 - T->z0 + 1;
  const int nr = T->y1 >= 0 ? W * H : 0;
  if (nr > kTileRows) return false;
  for (int r = threadIdx.x; r < nr; r += kBlock) {
    T->ux0[r] = INT_MAX;
    T->ux1[r] = -1;
  }
  __syncthreads();
  const int xi = own.cx << g.xb, xlast = ((g.gmax + 1) << g.xb) - 1;
  const float oxs = own.ox * g.fx;
  if (active) {
    const int ny = y1 - y0 + 1, nrows = ny * (z1 - z0 + 1);
    for (int q = sub; q < nrows; q += L) {
      const int cz = z0 + q / ny, cy = y0 + q % ny;
      const float lz = (float)(cz - own.rz) - own.oz, hz = lz + 1.f;
      const float ez = lz > 0.f ? lz : (hz < 0.f ? -hz : 0.f);
      const float ly = (float)(cy - own.ry) - own.oy, hy = ly + 1.f;
      const float ey = ly > 0.f ? ly : (hy < 0.f ? -hy : 0.f);
      const float d2 = ey * ey + ez * ez;
      if (d2 < rs2) {
        const float wx = fast_sqrt(fmaxf(rs2 - d2, 0.f)) * g.rfx;
        const int x0 = max(0, xi + (int)floorf(oxs - wx));
        const int x1 = min(xlast, xi + (int)floorf(oxs + wx));
        const int r = (cz - T->z0) * W + (cy - T->y0);
        atomicMin(&T->ux0[r], x0);
        atomicMax(&T->ux1[r], x1);
      }
    }
  }
  __syncthreads();
  // global range of each union row (one thread per row), LDS offsets by a prefix sum
  uint32_t a = 0u, cnt = 0u;
  const int r = threadIdx.x;
  if (r < nr && T->ux1[r] >= 0) {
    const int cy = T->y0 + r % W, cz = T->z0 + r / W;
    const int x0 = T->ux0[r], x1 = T->ux1[r];
    const uint32_t kb = sbase + ((uint32_t)x0 | (search_row(cy, cz, g) << (g.k + g.xb)));
    a = cstart[kb];
    const uint32_t b = min(cstart[kb + (uint32_t)(x1 - x0) + 1u], (uint32_t)g.n);
    cnt = b > a ? b - a : 0u;
  }
  uint32_t total;
  const uint32_t off = block_exclusive_scan(cnt, &total);
  if (r < nr) {
    T->ra[r] = a;
    T->roff[r] = off;
  }
  if (threadIdx.x == 0) T->roff[nr] = total;
  __syncthreads();
  if (total > (uint32_t)MPSPH_TILE_CAP) return false;
  for (uint32_t s = threadIdx.x; s < total; s += kBlock) {
    // the row holding staged slot s: the last row whose offset is <= s (never an empty row)
    int lo = 0, hi = nr - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (T->roff[mid] <= s) lo = mid;
      else hi = mid - 1;
    }
    const uint32_t j = T->ra[lo] + (s - T->roff[lo]);
    T->pos[s] = wfix[j];
    T->aux[s] = wjaux[j];
  }
  __syncthreads();
  return true;
}

// One logical block lb of the pass (blocks of a domain are consecutive; doms is the table the
// block numbers refer to); rowtab is the block's LDS row table, tile the LDS copy of the
// neighbours of the TILE variant (unused otherwise).  With PIPE the scan issues the neighbour
// loads of a lane's next slot before the arithmetic of the current one (same arithmetic, same
// order: the results do not depend on it).  The default passes take it; the persistent and staged
// variants keep the one-round body.  K2: kappa = 2 (the paper's) in every domain of the launch; the sums
// are the same bit for bit, without the tests that a shorter cut-off needs.  The pass is bound by
// the vector instructions and neighbour loads of its pair loop: with this and the wave-uniform loop of
// the scan, 1018 -> 976 us on the 2^21-particle cube; whole steps 695 -> 675 us (relaxed 2^20-particle
// cube), 125 -> 116 us (annulus of 2^18 particles), 69 us instead of 74 (seeded ball of 20000).
// The issue of vector instructions is the bound: the kernel in u = 1 - q/2 alone and the nearest distance
// by its bits (4 instructions of some 57 per candidate) took 976 to 956 us and 329 to 319 us on the cubes;
// waiting for fewer loads in the scan changed nothing.
#define MPSPH_PASS1_PARAMS                                                                                   \
  const DomDev *__restrict__ doms, int ndom, const int64_t *__restrict__ stepctr,                            \
      const uint32_t *__restrict__ wkey, const float4 *__restrict__ wpos, const float4 *__restrict__ wfix,    \
      const uint32_t *__restrict__ wjaux, const uint32_t *__restrict__ cstart, float4 *__restrict__ acc, float *__restrict__ rho_out,           \
      float *__restrict__ nn_out, float *__restrict__ aabs_out, uint32_t *__restrict__ dtslots,             \
      const double *__restrict__ metrics, double *__restrict__ partials
#define MPSPH_PASS1_ARGS \
  doms, ndom, stepctr, wkey, wpos, wfix, wjaux, cstart, acc, rho_out, nn_out, aabs_out, dtslots, metrics, partials
// WIDE: a wide domain (GridDev::wide).
template <int D, int L, bool PER, bool DBG, bool TILE, bool PIPE, bool K2, bool WIDE = false>
__device__ __forceinline__ void density_force_block(int lb, uint2 *rowtab, TileLds *tile, MPSPH_PASS1_PARAMS) {
  static_assert(!(TILE && WIDE), "the staged variant copies fixed-point coordinates");
  const int d = domain_of_block(doms, ndom, lb);
  const GridDev g = doms[d].g;
  const StepDev sp = doms[d].sp;
  const uint32_t cellbase = doms[d].cellbase;
  const int local = (lb - doms[d].blk0) * kBlock + threadIdx.x;
  const int li = local / L, sub = local % L;
  const int i = doms[d].off + li;
  const bool active = li < doms[d].n;
  const float sigma = sigma_of(sp, (float)*stepctr, metrics[(size_t)d * 32 + kAutoT0]);
  // the group's sums (wsum, a, nearest distance, counts), valid in lane 0 of each group
  float gw = 0.f, gx = 0.f, gy = 0.f, gz = 0.f, gA = 0.f, gn = INFINITY;
  uint32_t gp = 0u, gi = 0u, gc = 0u;
  bool staged = false;
  uint32_t self_t = 0u;
  int tw = 0;
  if constexpr (TILE) {
    static_assert(D == 3 && !PER, "the staged variant covers 3D regions without periodic wrap");
    OwnRow own{0, 0, 0, 0.f, 0.f, 0.f};
    float rst = 0.f;
    if (active) {
      int cs[3] = {0, 0, 0};
      unpack_key<D>(wkey[i] - cellbase, g, cs);
      const float4 p4 = wfix[i];
      own = own_row<D>(cs, fixed_of(p4), g);
      rst = fminf(sp.search_fac * p4.w, sp.kappa * 0.5f * (p4.w + sp.hmax)) * 1.0001f;
    }
    staged = stage_tile<L>(tile, active, sub, own, rst, g, doms[d].sbase, cstart, wfix, wjaux);
    if (staged) {
      tw = tile->y1 - tile->y0 + 1;
      if (active) {
        const int r = (own.rz - tile->z0) * tw + (own.ry - tile->y0);
        self_t = tile->roff[r] + ((uint32_t)i - tile->ra[r]);
      }
    }
  }
  if (active) {
    const PairPos<D, PER, WIDE> pos(g, cellbase, i, wkey, wfix);
    const uint32_t ai = wjaux[i];
    const int ti = aux_type(ai);
    const float hi = pos.h;
    // P = p0 / rho_t^2 = p0 tau^-2d h^2d and -dW/dr / r = 5 alpha 2^(d+2) (h_i + h_j)^-(d+2) (1 - q/2)^3
    // for the pair's h_ij: the pair sum takes h^2d and (h_i + h_j)^-(d+2), and the factors
    // common to every pair are applied once to the group's total.  Separations are in units of
    // pos.unit cells, the distance is converted to cells
    const float Phi = powd<D>(hi * hi);
    const float fscale = sp.p0c * powd<D>(sp.inv_tau * sp.inv_tau) * (5.f * sp.alpha) * (D == 3 ? 32.f : 16.f) * pos.unit;
    const float mhh = -0.5f * fast_rcp(hi);
    const float rci = sp.kappa * hi;
    const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
    const float kh = 0.5f * sp.kappa;
    const float unit = pos.unit;
    const float opb = 1.f + sigma;
    float wsum = 0.f, ax = 0.f, ay = 0.f, az = 0.f, A = 0.f;
    uint32_t npair = 0, nifc = 0, nn = kInfBits;
    const BufRes raux = buf_res(wjaux, 4, (uint32_t)g.n);
    using NbPos = typename PairPos<D, PER, WIDE>::Nb;
    const auto pair = [&](const NbPos &nj, const uint32_t aj) {
      const float4 pj = nj.p;
      float dx, dy, dz = 0.f;
      pos.sep(nj, dx, dy, dz);
      float r2 = dx * dx + dy * dy;
      if constexpr (D == 3) r2 += dz * dz;
      const float r = fast_sqrt(r2) * unit;
      const float hs = hi + pj.w;                   // 2 h_ij
      const bool inter = r < (K2 ? hs : kh * hs);   // kappa h_ij
      // the counts in every lane, so that the branch below is taken only for the force
      const bool diff = colour_differs(aj, ai);
      const bool feel = inter && type_at_least(aj, ti);
      nifc += (inter && diff) ? 1u : 0u;
      npair += feel ? 1u : 0u;
      // an empty statement that reads and writes both counts keeps their additions here, beside
      // the compares, where each becomes one add-with-carry of the compare's lane mask instead
      // of a select and an add after the branch
      asm volatile("" : "+v"(npair), "+v"(nifc));
      // (1 - q/2)^4 (1 + 2q) = u^4 (5 - 4u) with u = 1 - q/2
      const float u0 = fmaf(mhh, r, 1.f);
      if constexpr (K2) {
        // the kernel's support ends at the cut-off: its factor clamped to [0, 1] (an output modifier)
        // is zero beyond, without a test
        const float u = __builtin_amdgcn_fmed3f(u0, 0.f, 1.f), u2 = u * u;
        wsum = fmaf(u2 * u2, fmaf(-4.f, u, 5.f), wsum);
      } else {
        const float u2 = u0 * u0;
        if (r < rci) wsum = fmaf(u2 * u2, fmaf(-4.f, u0, 5.f), wsum);
      }
      // the nearest distance counts for normal particles, which feel every type; the debug export
      // has it for all
      // (as bits, in whose order non-negative floats are: one instruction, fminf takes three)
      if constexpr (DBG) {
        if (inter) nn = min(nn, __float_as_uint(r));
      }
      // coincident particles (two particles clamped into one corner) need no test: their separation
      // is zero and the force factor finite
      if (!feel) return;
      if constexpr (!DBG) nn = min(nn, __float_as_uint(r));
      const float hj2 = pj.w * pj.w;
      // (P_i + P_j) (-dW/dr / r) over the common factor fscale (>= 0)
      const float s = (diff ? opb : 1.f) * powd_add<D>(hj2, Phi) * kernel_slope_factor<D>(r, fast_rcp(hs));
      ax = fmaf(s, dx, ax);
      ay = fmaf(s, dy, ay);
      az = fmaf(s, dz, az);
      if constexpr (DBG) A = fmaf(s, r, A);        // sum of |pair terms| (debug export only)
    };
    struct Nb {
      NbPos p;
      uint32_t a;
    };
    const auto body = pair_body<PIPE>([&](uint32_t j) { return Nb{pos.fetch(j), buf_u32(raux, j)}; },
                                      [&](const Nb &nb) { pair(nb.p, nb.a); });
    const uint32_t sbase = doms[d].sbase;
    uint32_t ncand;
    if constexpr (TILE) {
      if (staged) {
        // slots index the LDS copy
        const auto tbody = [&](uint32_t j) { pair(NbPos{tile->pos[j]}, tile->aux[j]); };
        ncand = scan_group_table<D, L, row_table_rows<L>(), PER>(self_t, sub, rowtab + threadIdx.x / L,
                                                                 row_table_stride<L>(), pos.row, rs, g, sbase, cstart, tbody,
                                                                 TileRemap{tile, tw});
      } else {
        ncand = scan_group_table<D, L, row_table_rows<L>(), PER>(
            (uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row, rs, g, sbase, cstart, body);
      }
    } else {
      ncand = scan_group_table<D, L, row_table_rows<L>(), PER>(
          (uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row, rs, g, sbase, cstart, body);
    }
    gw = group_sum<L>(wsum);
    gx = fscale * group_sum<L>(ax);
    gy = fscale * group_sum<L>(ay);
    if constexpr (D == 3) gz = fscale * group_sum<L>(az);
    if constexpr (DBG) gA = fscale * (float)(1u << g.fb) * group_sum<L>(A);
    gn = group_min<L>(__uint_as_float(nn));
    gp = group_sum_u<L>(npair);
    gi = group_sum_u<L>(nifc);
    gc = ncand;
  }
  // Per-particle epilogue at one thread per particle: the groups' sums pass through the row
  // table's LDS to the block's first P threads, so that the epilogue does not run in every wave
  // with one lane in L busy.
  constexpr int P = kBlock / L;                  // particles per block
  constexpr int kEp = DBG ? 9 : 8;               // values per particle
  float *ep = reinterpret_cast<float *>(rowtab);
  __syncthreads();                               // every wave is done with the row table
  if (active && sub == 0) {
    const int p = threadIdx.x / L;
    ep[0 * P + p] = gw;
    ep[1 * P + p] = gx;
    ep[2 * P + p] = gy;
    ep[3 * P + p] = gz;
    ep[4 * P + p] = gn;
    ep[5 * P + p] = __uint_as_float(gp);
    ep[6 * P + p] = __uint_as_float(gi);
    ep[7 * P + p] = __uint_as_float(gc);
    if constexpr (DBG) ep[8 * P + p] = gA;
  }
  __syncthreads();
  double red[14];                                // the metrics' partials, interface flag, time-step candidate
#pragma unroll
  for (int s = 0; s < 14; ++s) red[s] = 0.0;
  red[P_ELRMIN] = INFINITY;
  red[13] = INFINITY;
  const int lp = (lb - doms[d].blk0) * P + (int)threadIdx.x;   // the thread's particle of the domain
  if (threadIdx.x < P && lp < doms[d].n) {
    const int ip = doms[d].off + lp;
    const int p = threadIdx.x;
    int ci[3];
    unpack_key<D>(wkey[ip] - cellbase, g, ci);
    const float4 pi = wpos[ip];
    const float oi[3] = {pi.x, pi.y, pi.z};
    const int ti = aux_type(wjaux[ip]);
    const float hi = pi.w, ihi = fast_rcp(hi), si = hi * sp.inv_tau, rci = sp.kappa * hi;
    const float wsum = ep[0 * P + p], nn = ep[4 * P + p];
    const uint32_t npair = __float_as_uint(ep[5 * P + p]), nifc = __float_as_uint(ep[6 * P + p]);
    const uint32_t ncand = __float_as_uint(ep[7 * P + p]);
    const float ihd = D == 3 ? ihi * ihi * ihi : ihi * ihi;
    const float rho = sp.alpha * ihd * (1.f + wsum);
    float a[3] = {ep[1 * P + p], ep[2 * P + p], ep[3 * P + p]};
    project_feature<D>(g, ti, ci, oi, a);
    const float am2 = a[0] * a[0] + a[1] * a[1] + (D == 3 ? a[2] * a[2] : 0.f);
    // the hardware square roots below (about 1 ulp) are well inside the step's FP32 error
    const float am = fast_sqrt(am2);
    const float ehat = sp.nu_coeff * rci * am / powd<D>(si);  // rho_t nu_coeff r_c |a|
    acc[ip] = make_float4(a[0], a[1], D == 3 ? a[2] : 0.f, ehat);
    if (rho_out) rho_out[ip] = rho;
    if (nn_out) nn_out[ip] = nn;
    if constexpr (DBG) {
      if (aabs_out) aabs_out[ip] = ep[8 * P + p];
    }
    if (ti != 3 && am2 > 0.f) red[13] = (double)(sp.c_acc * fast_sqrt(rci * fast_rsq(am2)));
    const bool fin = isfinite(am2) && isfinite(rho);
    if (ti == 0) {
      const double e = (double)(rho * powd<D>(si)) - 1.0;   // rho / rho_t - 1
      red[P_E2] = e * e;
      red[P_EMAX] = fabs(e);
      red[P_NNORM] = 1.0;
      if (nn < INFINITY) {
        const double elr = (double)nn / (double)si;
        red[P_ELR] = elr;
        red[P_ELR2] = elr * elr;
        red[P_ELRMIN] = elr;
        red[P_ELRMAX] = elr;
        red[P_NELR] = 1.0;
      }
    }
    red[P_PAIRS] = (double)npair;
    red[P_IFC] = (double)nifc;
    red[P_CAND] = (double)ncand;
    red[P_NONFIN1] = fin ? 0.0 : 1.0;
    red[12] = nifc > 0 ? 1.0 : 0.0;
  }
  // block results through LDS (after the epilogue's values when both fit in the row table)
  constexpr size_t kEpBytes = (size_t)kEp * P * sizeof(float), kRedBytes = (size_t)(P + 1) * 14 * sizeof(double);
  constexpr size_t kTableBytes = (size_t)row_table_rows<L>() * row_table_stride<L>() * sizeof(uint2);
  constexpr bool kApart = kEpBytes + kRedBytes <= kTableBytes;
  static_assert(kRedBytes <= kTableBytes && kEpBytes <= kTableBytes, "the epilogue and the reduction fit in the row table");
  double *rb = reinterpret_cast<double *>(reinterpret_cast<char *>(rowtab) + (kApart ? (kEpBytes + 15) / 16 * 16 : 0));
  constexpr uint32_t kMinSlots = (1u << P_ELRMIN) | (1u << 13), kMaxSlots = (1u << P_EMAX) | (1u << P_ELRMAX);
  double *out = partials + (size_t)lb * kNumPartials;
  block_reduce_lds<14, P, !kApart>(red, threadIdx.x < P ? (int)threadIdx.x : -1, kMinSlots, kMaxSlots, rb,
                                   [&](int s, double x) {
    if (s < 12) out[s] = x;
    else if (s == 12) out[P_IFCP] = x;
    else if (x < INFINITY) atomic_min_pos(&dtslots[d * kDtWords + (lb & (kDtSlots - 1)) * kDtStride], (float)x);   // one atomic per block
  });
}

// The pass over the logical blocks b0 + [0, gridDim.x) (of one dimension group, of wide domains or of narrow ones).  In
// 3D the wide pass holds one round of loads: with a second one it spilled 7 to 21 registers.
template <int D, int L, bool PER, bool DBG, bool K2, bool WIDE>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_density_force(int b0, MPSPH_PASS1_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  density_force_block<D, L, PER, DBG, false, !WIDE || D == 2, K2, WIDE>(b0 + xcd_block(blockIdx.x, gridDim.x), rowtab, nullptr,
                                                                        MPSPH_PASS1_ARGS);
}

// The staged copy limits a CU to 4 blocks (4 waves per SIMD), which the register budget follows.
template <int L, bool DBG>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void pass_density_force_tile(
    int b0, MPSPH_PASS1_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  __shared__ TileLds tile;
  density_force_block<3, L, false, DBG, true, false, false>(b0 + xcd_block(blockIdx.x, gridDim.x), rowtab, &tile, MPSPH_PASS1_ARGS);
}


// Box type from the number of faces a particle lies on.
// Mirror image through the lower wall (X = c + o < 0  ->  -X), in (cell, offset) form.
__device__ __forceinline__ void mirror_low(int &c, float &o) {
  int cn = -c - 1;
  float on = 1.f - o;
  if (on >= 1.f) {
    on = 0.f;
    cn += 1;
  }
  c = cn;
  o = on;
}

// Mirror image through the upper wall W = wc + wo (X = c + o > W  ->  2 W - X).
__device__ __forceinline__ void mirror_high(int &c, float &o, int wc, float wo) {
  const float x = wo - ((float)(c - wc) + (o - wo));
  const float fl = floorf(x);
  c = wc + (int)fl;
  o = x - fl;
  if (o >= 1.f) {
    o = 0.f;
    c += 1;
  }
}

__device__ __forceinline__ int type_from_faces(int nf, int d) {
  return nf <= 0 ? 0 : (nf == 1 ? 1 : (nf == 2 ? (d == 3 ? 2 : 3) : 3));
}

// Combines partials of one slot: sums, or min / max for the slots that hold extrema.  All three are formed
// and one is selected: as branches, which diverge over the slots of a wave, the step's end took 8 us.
struct SlotOp {
  bool mx, mn;
  __device__ __forceinline__ explicit SlotOp(int s) : mx(s == P_EMAX || s == P_ELRMAX), mn(s == P_ELRMIN) {}
  __device__ __forceinline__ double identity() const { return mn ? INFINITY : 0.0; }
  __device__ __forceinline__ double operator()(double a, double b) const {
    const double sum = a + b, hi = fmax(a, b), lo = fmin(a, b);
    return mx ? hi : (mn ? lo : sum);
  }
};

// End of a domain's step by one thread, after the slots 0..15 of its metrics block md are known (red): 16: dt1,
// 17: dt2, 18..20: running totals of pairs, candidates and steps (tot: their old values), then the
// automatic t0.  stepctr (may be null) is the context's step counter, advanced with its first domain.
__device__ __forceinline__ void close_domain_step(const StepDev &sp, float d1, const double *tot, double *md,
                                                  const double *red, int64_t *stepctr) {
  md[16] = (double)d1;
  md[17] = (double)(d1 * sp.dt2_factor);
  // running totals since the last load (exact integers below 2^53)
  md[18] = tot[0] + red[P_PAIRS];
  md[19] = tot[1] + red[P_CAND];
  md[20] = tot[2] + 1.0;
  // automatic t0 (reading of the paper's "topology static for some iterations"): the
  // interface-pair count and the number of particles with an interface pair stay within
  // t0_tol of a reference for t0_window steps; otherwise the reference restarts here
  if (sp.auto_t0 && !(md[kAutoT0] > 0.0)) {
    const double t = tot[2];  // index of this step since the load
    const double I = red[P_IFC] * 0.5, P = red[P_IFCP];
    const double tol = (double)sp.t0_tol;
    if (t == 0.0 || fabs(I - md[kAutoT0 + 1]) > tol * md[kAutoT0 + 1] ||
        fabs(P - md[kAutoT0 + 2]) > tol * md[kAutoT0 + 2]) {
      md[kAutoT0 + 1] = I;
      md[kAutoT0 + 2] = P;
      md[kAutoT0 + 3] = t;
    } else if (t - md[kAutoT0 + 3] >= (double)sp.t0_window) {
      md[kAutoT0] = t + 1.0;
    }
  }
  if (stepctr) *stepctr += 1;
}

// The step's end: the block partials of each domain reduced to its metrics block, its step closed.
// Contexts whose domains all have at most kFusedBlocks pair-kernel blocks close it inside the viscous
// pass: the last block of a domain to finish reduces the domain's partials.  The others launch
// finalize after it, one block per reduction row; the last row of a domain reduces the domain's rows.
// (The viscous pass of larger grids gains nothing from closing the step: every block waits about
// 2 us for its counter, 5 % of a block's life in each round of blocks.)  All sums run in a fixed
// order, so the result does not depend on which block does them.
struct StepEnd {
  int d0;             // first domain of the launch (doms, metrics and dtslots start there)
  uint32_t *domdone;  // finished blocks (or rows) per domain, zero between steps
  double *metrics;
  int64_t *stepctr;
};

// What another block of the same launch may have written: read at agent scope (past this XCD's L2).
__device__ __forceinline__ double agent_load(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether the calling block is the last of `total` to get here.  The first wave's agent-scope stores
// before the call are complete when the counter moves.  lds: one word.
__device__ __forceinline__ bool last_to_finish(uint32_t *counter, uint32_t total, uint32_t *lds) {
  if (threadIdx.x < kWave) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0) *lds = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  const bool last = *lds == total - 1u;
  if (last) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (threadIdx.x == 0) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return last;
}

// Rows [0, n) of kNumPartials slots combined in a fixed order; the result of slot s in the threads with
// threadIdx.x mod kNumPartials = s.  red: kBlock / kWave * kNumPartials doubles of LDS.
// SAME: rows that other blocks of the same launch wrote.
template <bool SAME>
__device__ __forceinline__ double combine_rows(const double *rows, int n, double *red) {
  static_assert(kNumPartials == 16, "slot and row of a lane");
  const int s = threadIdx.x & (kNumPartials - 1), r0 = threadIdx.x / kNumPartials;
  constexpr int kAhead = 8;      // rows in flight per thread
  const SlotOp op(s);
  double acc = op.identity();
#pragma unroll 1
  for (int r = r0; r < n; r += kAhead * (kBlock / kNumPartials)) {
    double v[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int rr = r + q * (kBlock / kNumPartials);
      const double *p = &rows[(size_t)min(rr, n - 1) * kNumPartials + s];
      const double x = SAME ? agent_load(p) : *p;
      v[q] = rr < n ? x : op.identity();
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) acc = op(acc, v[q]);
  }
  acc = op(acc, __shfl_xor(acc, 16, kWave));
  acc = op(acc, __shfl_xor(acc, 32, kWave));
  if ((threadIdx.x & (kWave - 1)) < kNumPartials) red[threadIdx.x / kWave * kNumPartials + s] = acc;
  __syncthreads();
  acc = red[s];
#pragma unroll
  for (int w = 1; w < kBlock / kWave; ++w) acc = op(acc, red[w * kNumPartials + s]);
  return acc;
}

// Closes the domain's step from its `total` partial rows (called by every thread of one block).
// red: kEndDoubles doubles of LDS, not in use by any wave.
constexpr int kEndDoubles = (kBlock / kWave + 1) * kNumPartials + 1;
template <bool SAME>
__device__ __forceinline__ void reduce_domain(const StepEnd &fin, const DomDev &dd, int d, const double *rows, int total,
                                              const uint32_t *dtslots, double *red) {
  double *md = fin.metrics + (size_t)d * 32;
  // loads that the sums do not depend on first
  const float d1 = read_dt1(dtslots + d * kDtWords);
  const double tot[3] = {md[18], md[19], md[20]};
  const double x = combine_rows<SAME>(rows, total, red);
  double *out = red + kBlock / kWave * kNumPartials;
  if (threadIdx.x < kNumPartials) {
    md[threadIdx.x] = x;
    out[threadIdx.x] = x;
  }
  __syncthreads();
  if (threadIdx.x == 0) close_domain_step(dd.sp, d1, tot, md, out, fin.d0 + d == 0 ? fin.stepctr : nullptr);
}

// One of the `total` partial rows of domain d (at rows) is stored, by agent-scope stores of the first
// wave; the last one to get here closes the domain's step.  Called by every thread of the block.
__device__ __forceinline__ void close_step(const StepEnd &fin, const DomDev &dd, int d, const double *rows, int total,
                                           const uint32_t *dtslots, double *red) {
  if (!last_to_finish(fin.domdone + fin.d0 + d, (uint32_t)total, reinterpret_cast<uint32_t *>(red + kEndDoubles - 1))) return;
  reduce_domain<true>(fin, dd, d, rows, total, dtslots, red);
}

// Pass 2: viscous acceleration (Eq. 20 with rho = rho_t, Eq. 22)
//   a~_i = sum_j [2 eta_i eta_j / (eta_i + eta_j)] (1/rho_t,i^2 + 1/rho_t,j^2) dW(r_ij,h_ij)/dr v~_ij / r_ij
// over the same pairs as pass 1, with the mid-point velocity v~ = a dt1 / 2 (Eq. 26 after the
// velocity reset) and eta = rho_t nu_coeff r_c |v~| (Eq. 21-22) formed from pass 1's output.
// Then per particle: projection, v = v~ + a~ dt2 / 2 (Eq. 27), drift r += v dt2 (Eq. 28),
// feature projection / re-tagging (Eq. 32); the new state is written in this step's order.
// With v~ = a dt1/2 the three criteria of Eq. 29 are increasing functions of r_c/|a| and give
// dt2 = dt1 min(1, 2 min(c_vel, c_visc / nu_coeff) / c_acc^2) (sp.dt2_factor).
#define MPSPH_PASS2_PARAMS                                                                                    \
  const DomDev *__restrict__ doms, int ndom, const uint32_t *__restrict__ wkey, const float4 *__restrict__ wpos, \
      const float4 *__restrict__ wfix, const uint32_t *__restrict__ wjaux, const uint32_t *__restrict__ wid,      \
      const uint32_t *__restrict__ cstart,                                                                       \
      const float4 *__restrict__ acc, const uint32_t *__restrict__ dtslots, uint32_t *__restrict__ skey,         \
      float4 *__restrict__ soff, uint32_t *__restrict__ sct, uint32_t *__restrict__ sid, uint32_t *__restrict__ cell, \
      uint32_t *__restrict__ counts,                                                                             \
      float4 *__restrict__ at_out, float4 *__restrict__ v_out,                                                    \
      double *__restrict__ partials, StepEnd fin
#define MPSPH_PASS2_ARGS \
  doms, ndom, wkey, wpos, wfix, wjaux, wid, cstart, acc, dtslots, skey, soff, sct, sid, cell, counts, at_out, v_out, partials, \
      fin
// One logical block lb of the pass; PIPE and WIDE as for density_force_block, END: the pass closes the step.
template <int D, int L, bool PER, bool PIPE, bool END = false, bool K2 = false, bool WIDE = false>
__device__ __forceinline__ void viscous_integrate_block(int lb, uint2 *rowtab, MPSPH_PASS2_PARAMS) {
  const int d = domain_of_block(doms, ndom, lb);
  const GridDev g = doms[d].g;
  const StepDev sp = doms[d].sp;
  const uint32_t cellbase = doms[d].cellbase;
  const int local = (lb - doms[d].blk0) * kBlock + threadIdx.x;
  const int li = local / L, sub = local % L;
  const int i = doms[d].off + li;
  float gbx = 0.f, gby = 0.f, gbz = 0.f;   // the group's pair sums, valid in lane 0 of each group
  // dt1 is published in LDS and read again after the pair sum, so that no copy of it stays live
  // across the pair loop
  __shared__ float sdt1;
  const float dt1 = read_dt1(dtslots + d * kDtWords);
  if (threadIdx.x == 0) sdt1 = dt1;
  __syncthreads();
  if (li < doms[d].n) {
    float bx = 0.f, by = 0.f, bz = 0.f;
    {
      // the pair sum; the particle's own data is scoped to it (the epilogue reads it again)
      const PairPos<D, PER, WIDE> pos(g, cellbase, i, wkey, wfix);
      const int ti = aux_type(wjaux[i]);
      const float hi = pos.h;
      // 1 / rho_t^2 = tau^-2d h^2d, v = (dt1/2) a, eta = (dt1/2) e and dW/dr / r =
      // -5 alpha 2^(d+2) (h_i + h_j)^-(d+2) (1 - q/2)^3 for the pair's h_ij: the pair sum takes h^2d,
      // a, e and (h_i + h_j)^-(d+2), and the factors common to every pair are applied once to the
      // group's total
      const float invi = powd<D>(hi * hi);
      const float4 acci = acc[i];
      const float ei = (0.5f * dt1) * acci.w;
      const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
      const float kh = 0.5f * sp.kappa;
      const float unit = pos.unit;
      // with eta_i = 0 every harmonic-mean viscosity of particle i vanishes: nothing to sum
      if (ei > 0.f) {
        const BufRes raux = buf_res(wjaux, 4, (uint32_t)g.n), racc = buf_res(acc, 16, (uint32_t)g.n);
        struct Nb {
          typename PairPos<D, PER, WIDE>::Nb p;
          float4 acc;
          uint32_t a;
        };
        // a normal particle feels every type: only feature particles load their neighbours' flags
        const auto fetch = [&](uint32_t j) {
          return Nb{pos.fetch(j), buf_f4(racc, j), ti > 0 ? buf_u32(raux, j) : 0xFFFFFFFFu};
        };
        const auto use = [&](const Nb &nb) {
          const float4 pj = nb.p.p, accj = nb.acc;
          float dx, dy, dz = 0.f;
          pos.sep(nb.p, dx, dy, dz);
          float r2 = dx * dx + dy * dy;
          if constexpr (D == 3) r2 += dz * dz;
          const float r = fast_sqrt(r2) * unit;
          const float hs = hi + pj.w;   // 2 h_ij
          // the particle itself and coincident particles have r = 0 exactly
          if (!(r > 0.f && r < (K2 ? hs : kh * hs) && type_at_least(nb.a, ti))) return;
          // e_j / (e_i + e_j): half the harmonic mean e_i e_j / (e_i + e_j) over e_i, which
          // multiplies the sum once; e_i > 0 here and e_j >= 0, so the sum is positive
          const float eh = accj.w * fast_rcp(acci.w + accj.w);
          const float hj2 = pj.w * pj.w;
          const float s = eh * powd_add<D>(hj2, invi) * kernel_slope_factor<D>(r, fast_rcp(hs));
          bx = fmaf(s, acci.x - accj.x, bx);
          by = fmaf(s, acci.y - accj.y, by);
          if constexpr (D == 3) bz = fmaf(s, acci.z - accj.z, bz);
        };
        scan_group_table<D, L, row_table_rows<L>(), PER, false>((uint32_t)i, sub, rowtab + threadIdx.x / L,
                                                                 row_table_stride<L>(), pos.row, rs, g, doms[d].sbase,
                                                                 cstart, pair_body<PIPE>(fetch, use));
        // the factor e_i of every pair term
        bx *= acci.w;
        by *= acci.w;
        bz *= acci.w;
      }
    }
    gbx = group_sum<L>(bx);
    gby = group_sum<L>(by);
    if constexpr (D == 3) gbz = group_sum<L>(bz);
  }
  // Per-particle epilogue at one thread per particle: the groups' sums pass through the row
  // table's LDS to the block's first P threads, so that the epilogue does not run in every wave
  // with one lane in L busy.
  constexpr int P = kBlock / L;                  // particles per block
  float *ep = reinterpret_cast<float *>(rowtab);
  __syncthreads();                               // every wave is done with the row table
  if (li < doms[d].n && sub == 0) {
    const int p = threadIdx.x / L;
    ep[0 * P + p] = gbx;
    ep[1 * P + p] = gby;
    ep[2 * P + p] = gbz;
  }
  __syncthreads();
  double part[3] = {0.0, 0.0, 0.0};
  const int lp = (lb - doms[d].blk0) * P + (int)threadIdx.x;   // the thread's particle of the domain
  if (threadIdx.x < P && lp < doms[d].n) {
    {
      const int io = doms[d].off + lp;
      const int p = threadIdx.x;
      const float hdt = 0.5f * sdt1;
      const float dt2 = sdt1 * sp.dt2_factor;
      // the factors left out of the pair sum: 2 of the harmonic mean, -5 alpha 2^(d+2), tau^-2d and
      // (dt1/2)^2
      const float vscale = (-2.f * 5.f * sp.alpha * (D == 3 ? 32.f : 16.f)) * powd<D>(sp.inv_tau * sp.inv_tau) * hdt * hdt;
      int ci[3];
      unpack_key<D>(wkey[io] - cellbase, g, ci);
      const float4 pe = wpos[io];
      const float oi[3] = {pe.x, pe.y, pe.z};
      const uint32_t ai = wjaux[io];
      int ti = aux_type(ai);
      const float4 acce = acc[io];
      const float vix = hdt * acce.x, viy = hdt * acce.y, viz = hdt * acce.z;
      float b[3] = {vscale * ep[0 * P + p], vscale * ep[1 * P + p], D == 3 ? vscale * ep[2 * P + p] : 0.f};
      project_feature<D>(g, ti, ci, oi, b);
      float v[3] = {vix + 0.5f * b[0] * dt2, viy + 0.5f * b[1] * dt2, viz + 0.5f * b[2] * dt2};
      if (ti == 3) v[0] = v[1] = v[2] = 0.f;
      float dr[3] = {v[0] * dt2, v[1] * dt2, v[2] * dt2};
      float ke = 0.f;
#pragma unroll
      for (int a = 0; a < D; ++a) ke += 0.5f * v[a] * v[a];
      const bool fin = isfinite(b[0]) && isfinite(b[1]) && isfinite(b[2]) && isfinite(dr[0]) && isfinite(dr[1]) &&
                       isfinite(dr[2]);
      // drift in (cell, offset) form with carry
      int c[3] = {ci[0], ci[1], D == 3 ? ci[2] : 0};
      float o[3] = {oi[0], oi[1], D == 3 ? oi[2] : 0.f};
      if (ti != 3 && fin) {
#pragma unroll
        for (int a = 0; a < D; ++a) {
          const float x = o[a] + dr[a];
          const float fl = floorf(x);
          c[a] += (int)fl;
          o[a] = x - fl;
          if (o[a] >= 1.f) {
            o[a] = 0.f;
            c[a] += 1;
          }
        }
        if (PER && g.geometry == 0) {
          // periodic box: wrap into [0, P)
#pragma unroll
          for (int a = 0; a < D; ++a) c[a] = ((c[a] % (g.gmax + 1)) + (g.gmax + 1)) % (g.gmax + 1);
        } else if (g.geometry == 1 && g.seeded) {
          // box with seeded features: a coordinate that left the box is mirrored at the wall it
          // crossed; types never change
#pragma unroll
          for (int a = 0; a < D; ++a) {
            if (c[a] < 0) {
              mirror_low(c[a], o[a]);
              if (c[a] > g.whi_c[a] || (c[a] == g.whi_c[a] && o[a] > g.whi_o[a])) {
                c[a] = g.whi_c[a];
                o[a] = g.whi_o[a];
              }
            } else if (c[a] > g.whi_c[a] || (c[a] == g.whi_c[a] && o[a] > g.whi_o[a])) {
              mirror_high(c[a], o[a], g.whi_c[a], g.whi_o[a]);
              if (c[a] < 0) {
                c[a] = 0;
                o[a] = 0.f;
              }
            }
          }
        } else if (g.geometry == 1) {
          // box: closest-point projection is a clamp to the walls; type from the faces touched
          int nf = 0;
#pragma unroll
          for (int a = 0; a < D; ++a) {
            if (c[a] < 0) {
              c[a] = 0;
              o[a] = 0.f;
            }
            if (c[a] > g.whi_c[a] || (c[a] == g.whi_c[a] && o[a] > g.whi_o[a])) {
              c[a] = g.whi_c[a];
              o[a] = g.whi_o[a];
            }
            if ((c[a] == 0 && o[a] == 0.f) || (c[a] == g.whi_c[a] && o[a] == g.whi_o[a])) ++nf;
          }
          ti = max(ti, type_from_faces(nf, D));
        } else if (g.geometry == 4) {
          // level set on the background mesh: r <- r - phi N (Eq. 32) for feature particles
          // and for normal particles that left the positive phase (re-tagged as surface)
          float gr[3];
          const float phi = mesh_interp<D>(g.phi, g.gn, g.ginv, c, o, gr);
          if (ti != 0 || phi < 0.f) {
            const float gn2 = gr[0] * gr[0] + gr[1] * gr[1] + (D == 3 ? gr[2] * gr[2] : 0.f);
            if (gn2 > 0.f) {
              // seeded features: a normal particle is mirrored through the zero level instead
              const float sc = (g.seeded && ti == 0 ? 2.f : 1.f) * phi * fast_rsq(gn2);
#pragma unroll
              for (int a = 0; a < D; ++a) {
                const float x = o[a] - sc * gr[a];
                const float fl = floorf(x);
                c[a] += (int)fl;
                o[a] = x - fl;
                if (o[a] >= 1.f) {
                  o[a] = 0.f;
                  c[a] += 1;
                }
              }
            }
            if (!g.seeded) ti = max(ti, 1);
          }
        } else {
          // annulus / ball: radial projection onto the nearest boundary circle / sphere
          float rel[3], r2 = 0.f;
#pragma unroll
          for (int a = 0; a < D; ++a) {
            rel[a] = (float)(c[a] - g.gc_c[a]) + (o[a] - g.gc_o[a]);
            r2 += rel[a] * rel[a];
          }
          const float rr = sqrtf(r2);
          const float phi = g.geometry == 2 ? fminf(rr - g.r_in, g.r_out - rr) : g.r_out - rr;
          if ((ti != 0 || phi < 0.f) && rr > 0.f) {
            float rb = g.r_out;
            if (g.geometry == 2 && (rr - g.r_in) < (g.r_out - rr)) rb = g.r_in;
            // seeded features: a normal particle is mirrored through the circle / sphere it crossed
            if (g.seeded && ti == 0) rb = rr > g.r_out ? 2.f * g.r_out - rr : 2.f * g.r_in - rr;
            const float sc = rb / rr;
#pragma unroll
            for (int a = 0; a < D; ++a) {
              // new coordinate relative to the origin of cell c[a]: centre + rel * rb / |rel|
              const float x = (float)(g.gc_c[a] - c[a]) + g.gc_o[a] + rel[a] * sc;
              const float fl = floorf(x);
              c[a] += (int)fl;
              o[a] = x - fl;
              if (o[a] >= 1.f) {
                o[a] = 0.f;
                c[a] += 1;
              }
            }
            if (!g.seeded) ti = max(ti, 1);
          }
        }
      }
      // keys must stay inside the grid whatever the arithmetic above produced
#pragma unroll
      for (int a = 0; a < D; ++a) {
        if (!(o[a] >= 0.f && o[a] < 1.f)) o[a] = 0.f;
        if (c[a] < 0) {
          c[a] = 0;
          o[a] = 0.f;
        }
        if (c[a] > g.gmax) {
          c[a] = g.gmax;
          o[a] = 0.f;
        }
      }
      skey[io] = cellbase + pack_key<D>(c, o, g);
      const uint32_t sc = doms[d].sbase + search_key<D>(c, o, g);
      cell[io] = sc;
      soff[io] = make_float4(o[0], o[1], D == 3 ? o[2] : 0.f, count_arrival(counts, sc));
      sct[io] = (uint32_t)ti | (aux_colour(ai) << 2);
      sid[io] = wid[io];
      if (at_out) at_out[io] = make_float4(b[0], b[1], b[2], 0.f);
      if (v_out) v_out[io] = make_float4(v[0], v[1], v[2], 0.f);
      part[0] = (double)ke;
      part[1] = fin ? 0.0 : 1.0;
      part[2] = ti != 0 ? 1.0 : 0.0;
    }
  }
  // block sums through LDS, after the epilogue's values
  constexpr size_t kEpBytes = (size_t)3 * P * sizeof(float), kRedBytes = (size_t)(P + 1) * 3 * sizeof(double);
  constexpr size_t kEndBytes = (size_t)kEndDoubles * sizeof(double);
  static_assert((kEpBytes + 15) / 16 * 16 + (kRedBytes > kEndBytes ? kRedBytes : kEndBytes) <=
                    (size_t)row_table_rows<L>() * row_table_stride<L>() * sizeof(uint2),
                "the epilogue and the reductions fit in the row table");
  double *rb = reinterpret_cast<double *>(reinterpret_cast<char *>(rowtab) + (kEpBytes + 15) / 16 * 16);
  double *out = partials + (size_t)lb * kNumPartials + P_KE;
  block_reduce_lds<3, P, false>(part, threadIdx.x < P ? (int)threadIdx.x : -1, 0u, 0u, rb,
                                [&](int s, double x) {
    if constexpr (END) agent_store(&out[s], x);
    else out[s] = x;
  });
  if constexpr (END) {
    __syncthreads();   // the first wave is done with the reduction's LDS
    close_step(fin, doms[d], d, partials + (size_t)doms[d].blk0 * kNumPartials, doms[d].nblk, dtslots, rb);
  }
}

template <int D, int L, bool PER, bool END, bool K2, bool WIDE>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_viscous_integrate(int b0, MPSPH_PASS2_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  viscous_integrate_block<D, L, PER, !WIDE || D == 2, END, K2, WIDE>(b0 + xcd_block(blockIdx.x, gridDim.x), rowtab,
                                                                     MPSPH_PASS2_ARGS);
}

// Row-table entries of a launch that serves 2D blocks at L lanes and 3D blocks at L3.
template <int L, int L3>
constexpr int mixed_table() {
  constexpr int a = row_table_rows<L>() * row_table_stride<L>(), b = row_table_rows<L3>() * row_table_stride<L3>();
  return a > b ? a : b;
}

// Both dimension groups of a batch in one launch: the longer 3D blocks first, the nb2 blocks of the 2D
// domains in the last wave of blocks that those leave partly empty, and one launch less.  Batch of 12
// domains of both dimensions, 359,000 particles, 4 steps with load and metrics: 1208 us with a launch per
// dimension, 1115 this way.
template <bool PER, bool K2>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_density_force_mixed(int nb2, MPSPH_PASS1_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[mixed_table<MPSPH_LANES, MPSPH_LANES_3D>()];
  const int b = blockIdx.x, nb3 = (int)gridDim.x - nb2;
  if (b < nb3)
    density_force_block<3, MPSPH_LANES_3D, PER, false, false, true, K2>(nb2 + xcd_block(b, nb3), rowtab, nullptr, MPSPH_PASS1_ARGS);
  else
    density_force_block<2, MPSPH_LANES, PER, false, false, true, K2>(xcd_block(b - nb3, nb2), rowtab, nullptr, MPSPH_PASS1_ARGS);
}

template <bool PER, bool END, bool K2>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_viscous_integrate_mixed(int nb2, MPSPH_PASS2_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[mixed_table<MPSPH_LANES, MPSPH_LANES_3D>()];
  const int b = blockIdx.x, nb3 = (int)gridDim.x - nb2;
  if (b < nb3)
    viscous_integrate_block<3, MPSPH_LANES_3D, PER, true, END, K2>(nb2 + xcd_block(b, nb3), rowtab, MPSPH_PASS2_ARGS);
  else
    viscous_integrate_block<2, MPSPH_LANES, PER, true, END, K2>(xcd_block(b - nb3, nb2), rowtab, MPSPH_PASS2_ARGS);
}

// Persistent launches of the two pair passes: a fixed grid serves the logical blocks
// b0 + [0, nb) from a work queue in device memory, either of one dimension group (DM = 2 or 3) or
// of both in one launch (DM = 5: blocks below nb2 are 2D, the others 3D).  The blocks
// are split into 8 contiguous ranges, one per XCD; a workgroup (XCD blockIdx.x mod 8 under the
// round-robin dispatch) takes the next block of its own range and then of the others.  q[0..7]
// count the blocks taken from each range, q[8] the workgroups that finished; the last one resets
// the queue, so the launch needs no memset and can be captured in a graph.
__device__ __forceinline__ int queue_next(uint32_t *q, int nb) {
  const int x = blockIdx.x & 7, per = nb >> 3, rem = nb & 7;
  for (int k = 0; k < 8; ++k) {
    const int r = (x + k) & 7;
    const int start = r * per + (r < rem ? r : rem), len = per + (r < rem ? 1 : 0);
    const uint32_t t = atomicAdd(&q[r], 1u);
    if ((int)t < len) return start + (int)t;
  }
  return nb;
}
__device__ __forceinline__ void queue_done(uint32_t *q) {
  __threadfence();
  if (atomicAdd(&q[8], 1u) == gridDim.x - 1u) {
    for (int k = 0; k < 9; ++k) q[k] = 0u;
    __threadfence();
  }
}

template <int DM, int L, int L3, bool PER, bool DBG>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_density_force_queue(int b0, int nb2, int nb,
                                                                                        uint32_t *queue,
                                                                                        MPSPH_PASS1_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[mixed_table<L, L3>()];
  __shared__ int sitem;
  for (;;) {
    __syncthreads();   // the previous block's LDS (row table, reductions) is no longer read
    if (threadIdx.x == 0) sitem = queue_next(queue, nb);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(sitem);   // the same in every lane
    if (it >= nb) break;
    if constexpr (DM == 5) {
      if (it < nb2) density_force_block<2, L, PER, DBG, false, false, false>(b0 + it, rowtab, nullptr, MPSPH_PASS1_ARGS);
      else density_force_block<3, L3, PER, DBG, false, false, false>(b0 + it, rowtab, nullptr, MPSPH_PASS1_ARGS);
    } else {
      density_force_block<DM, DM == 3 ? L3 : L, PER, DBG, false, false, false>(b0 + it, rowtab, nullptr, MPSPH_PASS1_ARGS);
    }
  }
  if (threadIdx.x == 0) queue_done(queue);
}

template <int DM, int L, int L3, bool PER>
__global__ __launch_bounds__(kBlock) MPSPH_PAIR_OCCUPANCY void pass_viscous_integrate_queue(int b0, int nb2, int nb,
                                                                                            uint32_t *queue,
                                                                                            MPSPH_PASS2_PARAMS) {
  __shared__ __align__(16) uint2 rowtab[mixed_table<L, L3>()];
  __shared__ int sitem;
  for (;;) {
    __syncthreads();   // the previous block's LDS (row table, reductions) is no longer read
    if (threadIdx.x == 0) sitem = queue_next(queue, nb);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(sitem);   // the same in every lane
    if (it >= nb) break;
    if constexpr (DM == 5) {
      if (it < nb2) viscous_integrate_block<2, L, PER, false>(b0 + it, rowtab, MPSPH_PASS2_ARGS);
      else viscous_integrate_block<3, L3, PER, false>(b0 + it, rowtab, MPSPH_PASS2_ARGS);
    } else {
      viscous_integrate_block<DM, DM == 3 ? L3 : L, PER, false>(b0 + it, rowtab, MPSPH_PASS2_ARGS);
    }
  }
  if (threadIdx.x == 0) queue_done(queue);
}


// Debug: ordered geometric neighbour pairs (i, j != i, r_ij < kappa h_ij, no type mask) of the
// last step's start-of-step state, enumerated with the same candidate scan and predicate as the
// pair passes (two lanes per particle).  Pairs go to (out_i, out_j) as load indices while the
// running count stays below cap; *count receives the total.
template <int D, bool PER, bool WIDE>
__global__ __launch_bounds__(kBlock) void dump_pairs(const DomDev *__restrict__ doms, int ndom, int i0, int i1,
                                                     const uint32_t *__restrict__ wkey, const float4 *__restrict__ wfix,
                                                     const uint32_t *__restrict__ wid,
                                                     const uint32_t *__restrict__ cstart, unsigned long long cap,
                                                     uint32_t *__restrict__ out_i, uint32_t *__restrict__ out_j,
                                                     unsigned long long *__restrict__ count) {
  constexpr int L = 2;   // lanes per particle, as in the pair passes
  const int t = blockIdx.x * kBlock + threadIdx.x;
  const int i = i0 + t / L, sub = t % L;
  if (i >= i1) return;   // both lanes of a particle leave together
  const DomDev &dd = doms[domain_of(doms, ndom, i)];
  const GridDev &g = dd.g;
  if ((g.wide != 0) != WIDE) return;
  const StepDev &sp = dd.sp;
  const PairPos<D, PER, WIDE> pos(g, dd.cellbase, i, wkey, wfix);
  const float hi = pos.h;
  const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
  const float kh = 0.5f * sp.kappa;
  const uint32_t idi = wid[i];
  __shared__ uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  scan_group_table<D, L, row_table_rows<L>(), PER>((uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(),
                                                   pos.row, rs, g, dd.sbase, cstart, [&](uint32_t j) {
    const auto nj = pos.fetch(j);
    float dx, dy, dz = 0.f;
    pos.sep(nj, dx, dy, dz);
    float r2 = dx * dx + dy * dy;
    if constexpr (D == 3) r2 += dz * dz;
    if (!(fast_sqrt(r2) * pos.unit < kh * (hi + nj.p.w))) return;
    const unsigned long long k = atomicAdd(count, 1ull);
    if (k < cap) {
      out_i[k] = idi;
      out_j[k] = wid[j];
    }
  });
}

// The step's end as a launch of its own: block r reduces the pair-kernel block partials of reduction
// row r (groups[r]: domain, first and last block partial, none of another domain), the last row of a
// domain to finish the domain's rows.
__global__ __launch_bounds__(kBlock) void finalize(const DomDev *__restrict__ doms, const int4 *__restrict__ groups,
                                                   const double *__restrict__ partials, double *__restrict__ rows,
                                                   const uint32_t *__restrict__ dtslots, StepEnd fin) {
  __shared__ double red[kEndDoubles];
  const int4 gr = groups[blockIdx.x];
  const DomDev &dd = doms[gr.x];
  const double *first = partials + (size_t)gr.y * kNumPartials;
  if (dd.nrow == 1) {
    reduce_domain<false>(fin, dd, gr.x, first, gr.z - gr.y, dtslots, red);
    return;
  }
  const double x = combine_rows<false>(first, gr.z - gr.y, red);
  if (threadIdx.x < kNumPartials) agent_store(&rows[(size_t)blockIdx.x * kNumPartials + threadIdx.x], x);
  __syncthreads();
  close_step(fin, dd, gr.x, rows + (size_t)dd.row0 * kNumPartials, dd.nrow, dtslots, red);
}

// Positions back to domain units (FP64) in the load order; state indices [i0, i1).
template <int D>
__global__ __launch_bounds__(kBlock) void store_kernel(const DomDev *__restrict__ doms, int ndom, int i0, int i1,
                                                       const uint32_t *__restrict__ skey, const float4 *__restrict__ soff,
                                                       const uint32_t *__restrict__ sct, const uint32_t *__restrict__ sid,
                                                       float *__restrict__ pos, int32_t *__restrict__ type) {
  const int i = i0 + blockIdx.x * kBlock + threadIdx.x;
  if (i >= i1) return;
  const DomDev &dd = doms[domain_of(doms, ndom, i)];
  int c[3];
  unpack_key<D>(skey[i] - dd.cellbase, dd.g, c);
  const float4 o = soff[i];
  const float oo[3] = {o.x, o.y, o.z};
  const uint32_t id = sid[i];
  if (pos) {
    float *x = pos + dd.xoff + (int64_t)((int)id - dd.uoff) * D;
    for (int a = 0; a < D; ++a) x[a] = (float)(dd.lo[a] + ((double)c[a] + (double)oo[a]) * dd.cs);
  }
  if (type) type[id] = (int32_t)(sct[i] & 3u);
}

// Scatter one per-particle quantity of the last step to load order, converted to domain units;
// sorted indices [i0, i1).  vscale[d] multiplies vector quantities (dt1 / 2 of the domain for
// v~; NULL: 1).
template <int D>
__global__ __launch_bounds__(kBlock) void dump_kernel(const DomDev *__restrict__ doms, int ndom, int i0, int i1,
                                                      int which, const uint32_t *__restrict__ wkey,
                                                      const float4 *__restrict__ wpos, const uint32_t *__restrict__ wid,
                                                      const float *__restrict__ sc, const float4 *__restrict__ vec,
                                                      const float *__restrict__ vscale, float *__restrict__ out) {
  const int i = i0 + blockIdx.x * kBlock + threadIdx.x;
  if (i >= i1) return;
  const int d = domain_of(doms, ndom, i);
  const DomDev &dd = doms[d];
  const uint32_t id = wid[i];
  float *ov = out + dd.xoff + (int64_t)((int)id - dd.uoff) * D;  // row of a vector quantity
  const float4 p = wpos[i];
  const double csd = dd.cs;
  switch (which) {
    case MPSPH_F_RHO:
      out[id] = (float)((double)sc[i] / pow(csd, D));
      break;
    case MPSPH_F_RHO_T: {
      const double s = (double)p.w / dd.sp.tau * csd;
      out[id] = (float)pow(s, -D);
      break;
    }
    case MPSPH_F_H:
      out[id] = (float)((double)p.w * csd);
      break;
    case MPSPH_F_NN:
    case MPSPH_F_A_ABS:
      out[id] = (float)((double)sc[i] * csd);
      break;
    case MPSPH_F_X0: {
      int c[3];
      unpack_key<D>(wkey[i] - dd.cellbase, dd.g, c);
      const float oo[3] = {p.x, p.y, p.z};
      for (int a = 0; a < D; ++a) ov[a] = (float)(dd.lo[a] + ((double)c[a] + (double)oo[a]) * csd);
      break;
    }
    default: {  // vector quantities in cell units per time: scale by cs (and vscale)
      const float4 v = vec[i];
      const float vv[3] = {v.x, v.y, v.z};
      const float f = vscale ? vscale[d] : 1.f;
      for (int a = 0; a < D; ++a) ov[a] = (float)((double)(vv[a] * f) * csd);
    }
  }
}

// ------------------------------------------------------------------------------------------
// Host side
// ------------------------------------------------------------------------------------------

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

struct Derived {
  int dim, k, gmax;
  int xe;                  // x sub-cells per cell in the cell key: 2^xe
  int rb, xb;              // search grid: rows of 2^rb cells, 2^xb x sub-cells per cell
  int fb;                  // bits of the fixed-point coordinates' fraction
  bool wide;               // separations may leave the range of those coordinates (GridDev::wide)
  double L, cs, inv_cs, lo[3], xhi[3];
  double smin, smax, lip;  // spacing bounds (domain units), Lipschitz constant of s
  double search_fac;
};

const char *kErr[] = {"ok", "invalid argument", "out of memory", "device error", "bad context state",
                      "non-finite values", "unsupported configuration",
                      "the problem needs more workspace than the static scratch array holds"};

bool valid_params(const mpsph_params *p) {
  if (!p) return false;
  if (p->dim != 2 && p->dim != 3) return false;
  if (p->geometry < MPSPH_PERIODIC || p->geometry > MPSPH_LEVELSET) return false;
  if (p->geometry == MPSPH_PERIODIC)  // periodic: a cube (a square in 2D), every side one period
    for (int a = 1; a < p->dim; ++a)
      if (p->hi[a] - p->lo[a] != p->hi[0] - p->lo[0]) return false;
  if (p->geometry == MPSPH_LEVELSET || p->field == MPSPH_GRID) {
    int64_t nodes = 1;
    for (int a = 0; a < p->dim; ++a) {
      if (p->grid_n[a] < 2 || p->grid_n[a] > (1 << 14)) return false;
      nodes *= p->grid_n[a];
    }
    if (nodes > ((int64_t)1 << 27)) return false;
    if (p->geometry == MPSPH_LEVELSET && !p->grid_phi) return false;
    if (p->field == MPSPH_GRID) {
      if (!p->grid_s) return false;
      for (int64_t k = 0; k < nodes; ++k)
        if (!(p->grid_s[k] > 0) || !std::isfinite(p->grid_s[k])) return false;
    }
  }
  if (p->geometry == MPSPH_ANNULUS && p->dim != 2) return false;
  for (int a = 0; a < p->dim; ++a)
    if (!(p->hi[a] > p->lo[a]) || !std::isfinite(p->lo[a]) || !std::isfinite(p->hi[a])) return false;
  if (p->field < MPSPH_UNIFORM || p->field > MPSPH_GRID) return false;
  if (p->field == MPSPH_RBF_EXP && (p->n_rbf < 0 || p->n_rbf > 64 || (p->n_rbf > 0 && (!p->rbf_centre || !p->rbf_coeff)) ||
                                    !(p->rbf_width > 0)))
    return false;
  // the kernel's support is 2h: a cut-off beyond it would only add zero terms, and the pair
  // kernels evaluate the kernel's polynomial without clamping it to its support
  if (!(p->tau > 0) || !(p->kappa > 0 && p->kappa <= 2) || !(p->p0 > 0) || !(p->sigma0 >= 0)) return false;
  if (p->t0 < -2 || (p->t0 >= 0 && p->t1 < p->t0)) return false;
  if (!(p->nu_coeff >= 0) || !(p->c_acc > 0) || !(p->c_vel > 0) || !(p->c_visc > 0)) return false;
  if ((p->geometry == MPSPH_ANNULUS || p->geometry == MPSPH_BALL) && !(p->r_out > 0)) return false;
  if (p->geometry == MPSPH_ANNULUS && !(p->r_in > 0 && p->r_in < p->r_out)) return false;
  if (p->cell_log2 != -1 && (p->cell_log2 < 1 || p->cell_log2 > 12)) return false;
  return true;
}

double box_dist_range(const mpsph_params *p, const double *c, double *dmax) {
  double dmin2 = 0.0, dmax2 = 0.0;
  for (int a = 0; a < p->dim; ++a) {
    double lo = p->lo[a] - c[a], hi = p->hi[a] - c[a];
    double near = (lo > 0) ? lo : (hi < 0 ? -hi : 0.0);
    double far = std::max(std::fabs(lo), std::fabs(hi));
    dmin2 += near * near;
    dmax2 += far * far;
  }
  *dmax = std::sqrt(dmax2);
  return std::sqrt(dmin2);
}

// Multilinear interpolation on the background mesh (host, FP64), optional gradient.
double host_mesh(const mpsph_params *p, const double *nodes, const double *x, double *grad = nullptr) {
  const int d = p->dim;
  int base[3] = {0, 0, 0};
  double f[3] = {0, 0, 0}, inv[3] = {1, 1, 1};
  for (int a = 0; a < d; ++a) {
    inv[a] = (double)(p->grid_n[a] - 1) / (p->hi[a] - p->lo[a]);
    const double u = (x[a] - p->lo[a]) * inv[a];
    const int i = std::min(std::max((int)std::floor(u), 0), p->grid_n[a] - 2);
    base[a] = i;
    f[a] = u - i;
  }
  double val = 0.0, g[3] = {0, 0, 0};
  for (int cn = 0; cn < (1 << d); ++cn) {
    size_t idx = 0, stride = 1;
    double w = 1.0, dw[3] = {1, 1, 1};
    for (int a = 0; a < d; ++a) {
      const int bit = (cn >> a) & 1;
      idx += (size_t)(base[a] + bit) * stride;
      stride *= (size_t)p->grid_n[a];
      const double wa = bit ? f[a] : 1.0 - f[a];
      for (int b = 0; b < d; ++b) dw[b] *= b == a ? (bit ? inv[a] : -inv[a]) : wa;
      w *= wa;
    }
    val += w * nodes[idx];
    for (int b = 0; b < d; ++b) g[b] += dw[b] * nodes[idx];
  }
  if (grad)
    for (int a = 0; a < 3; ++a) grad[a] = a < d ? g[a] : 0.0;
  return val;
}

// Spacing of the field in domain units at a point (host, FP64), with scale s0.
double host_spacing(const mpsph_params *p, double s0, const double *x) {
  if (p->field == MPSPH_GRID) return s0 * host_mesh(p, p->grid_s, x);
  auto dist = [&](const double *c) {
    double s = 0;
    for (int a = 0; a < p->dim; ++a) s += (x[a] - c[a]) * (x[a] - c[a]);
    return std::sqrt(s);
  };
  switch (p->field) {
    case MPSPH_UNIFORM:
      return s0;
    case MPSPH_RADIAL_LINEAR:
      return s0 * (1.0 + p->fa * (dist(p->fcentre) - p->fb));
    case MPSPH_SPHERE_DISTANCE:
      return s0 * (1.0 + p->fa * std::fabs(dist(p->fcentre) - p->fb));
    default: {
      double e = 0;
      for (int k = 0; k < p->n_rbf; ++k) {
        double r = dist(p->rbf_centre + k * p->dim);
        e += p->rbf_coeff[k] * std::exp(-r * r / (2 * p->rbf_width * p->rbf_width));
      }
      return s0 * std::exp(e);
    }
  }
}

bool inside_region(const mpsph_params *p, const double *x) {
  if (p->geometry == MPSPH_BOX || p->geometry == MPSPH_PERIODIC) return true;
  if (p->geometry == MPSPH_LEVELSET) return host_mesh(p, p->grid_phi, x) > 0.0;
  double r = 0;
  for (int a = 0; a < p->dim; ++a) r += (x[a] - p->centre[a]) * (x[a] - p->centre[a]);
  r = std::sqrt(r);
  if (p->geometry == MPSPH_ANNULUS) return r >= p->r_in && r <= p->r_out;
  return r <= p->r_out;
}

// Gauss-Legendre nodes on [0,1] (8 points).
void gauss8(double *xg, double *wg) {
  static const double t[4] = {0.1834346424956498, 0.5255324099163290, 0.7966664774136267, 0.9602898564975363};
  static const double w[4] = {0.3626837833783620, 0.3137066458778873, 0.2223810344533745, 0.1012285362903763};
  for (int i = 0; i < 4; ++i) {
    xg[3 - i] = 0.5 * (1 - t[i]);
    xg[4 + i] = 0.5 * (1 + t[i]);
    wg[3 - i] = 0.5 * w[i];
    wg[4 + i] = 0.5 * w[i];
  }
}

// Integral of s^-d over the region for s0 = 1: composite 8-point Gauss-Legendre in Cartesian
// panels (box) or polar / spherical coordinates (annulus, ball).
double field_integral_unit(const mpsph_params *p) {
  double xg[8], wg[8];
  gauss8(xg, wg);
  const int d = p->dim;
  const double pi = 3.14159265358979323846;
  double total = 0.0;
  if (p->geometry == MPSPH_LEVELSET) {
    // midpoint rule over sub-cells of the bounding box with the indicator of the positive phase
    const int M = d == 2 ? 1024 : 160;
    double h[3] = {0, 0, 0}, vol = 1.0;
    for (int a = 0; a < d; ++a) {
      h[a] = (p->hi[a] - p->lo[a]) / M;
      vol *= h[a];
    }
    const int64_t cells = d == 2 ? (int64_t)M * M : (int64_t)M * M * M;
    for (int64_t cidx = 0; cidx < cells; ++cidx) {
      double x[3];
      int64_t r = cidx;
      for (int a = 0; a < d; ++a) {
        x[a] = p->lo[a] + ((double)(r % M) + 0.5) * h[a];
        r /= M;
      }
      if (!(host_mesh(p, p->grid_phi, x) > 0.0)) continue;
      total += std::pow(host_spacing(p, 1.0, x), -d);
    }
    return total * vol;
  }
  const bool boxlike = p->geometry == MPSPH_BOX || p->geometry == MPSPH_PERIODIC;
  if (p->field == MPSPH_UNIFORM) {  // s = 1: the measure of the region
    if (boxlike) {
      double v = 1.0;
      for (int a = 0; a < d; ++a) v *= p->hi[a] - p->lo[a];
      return v;
    }
    if (p->geometry == MPSPH_ANNULUS) return pi * (p->r_out * p->r_out - p->r_in * p->r_in);
    return d == 2 ? pi * p->r_out * p->r_out : 4.0 / 3.0 * pi * p->r_out * p->r_out * p->r_out;
  }
  if (boxlike) {
    const int M = d == 2 ? 256 : (p->field == MPSPH_GRID ? 24 : 48);
    const int np = M * 8;
    std::vector<double> node[3], wt[3];
    for (int a = 0; a < d; ++a) {
      double h = (p->hi[a] - p->lo[a]) / M;
      for (int m = 0; m < M; ++m)
        for (int q = 0; q < 8; ++q) {
          node[a].push_back(p->lo[a] + (m + xg[q]) * h);
          wt[a].push_back(wg[q] * h);
        }
    }
    double x[3];
    if (d == 2) {
      for (int i = 0; i < np; ++i)
        for (int j = 0; j < np; ++j) {
          x[0] = node[0][i];
          x[1] = node[1][j];
          total += wt[0][i] * wt[1][j] * std::pow(host_spacing(p, 1.0, x), -d);
        }
    } else {
      for (int i = 0; i < np; ++i) {
        double acc = 0;
        for (int j = 0; j < np; ++j)
          for (int l = 0; l < np; ++l) {
            x[0] = node[0][i];
            x[1] = node[1][j];
            x[2] = node[2][l];
            double s = host_spacing(p, 1.0, x);
            acc += wt[1][j] * wt[2][l] / (s * s * s);
          }
        total += wt[0][i] * acc;
      }
    }
    return total;
  }
  const double r0 = p->geometry == MPSPH_ANNULUS ? p->r_in : 0.0, r1 = p->r_out;
  const int MR = d == 2 ? 128 : 64, MT = d == 2 ? 64 : 16, MP = 32;
  for (int mr = 0; mr < MR; ++mr)
    for (int qr = 0; qr < 8; ++qr) {
      double r = r0 + (mr + xg[qr]) * (r1 - r0) / MR, wr = wg[qr] * (r1 - r0) / MR;
      for (int mt = 0; mt < MT; ++mt)
        for (int qt = 0; qt < 8; ++qt) {
          double th = (mt + xg[qt]) * (d == 2 ? 2 * pi : pi) / MT, wth = wg[qt] * (d == 2 ? 2 * pi : pi) / MT;
          if (d == 2) {
            double x[2] = {p->centre[0] + r * std::cos(th), p->centre[1] + r * std::sin(th)};
            total += wr * wth * r * std::pow(host_spacing(p, 1.0, x), -2);
          } else {
            for (int mp = 0; mp < MP; ++mp)
              for (int qp = 0; qp < 8; ++qp) {
                double ph = (mp + xg[qp]) * 2 * pi / MP, wph = wg[qp] * 2 * pi / MP;
                double x[3] = {p->centre[0] + r * std::sin(th) * std::cos(ph),
                               p->centre[1] + r * std::sin(th) * std::sin(ph), p->centre[2] + r * std::cos(th)};
                total += wr * wth * wph * r * r * std::sin(th) * std::pow(host_spacing(p, 1.0, x), -3);
              }
          }
        }
    }
  return total;
}

// Boundary features of a region (the order the header documents) with the integral, at s0 = 1,
// of s^-k over each: k = dim - 1 on a feature surface, 1 on a feature curve, 0 at a corner.
struct FeatureList {
  int n = 0;
  int type[MPSPH_MAX_FEATURES];
  int power[MPSPH_MAX_FEATURES];
  double I[MPSPH_MAX_FEATURES];
  void add(int t, int k, double v) {
    type[n] = t;
    power[n] = k;
    I[n] = v;
    ++n;
  }
};

// Panels per axis of the composite rule along box axis a: one per background-mesh cell for a
// gridded field (the interpolant is smooth inside a cell), else the given count.
int feature_panels(const mpsph_params *p, int a, int dflt) {
  return p->field == MPSPH_GRID ? std::max(p->grid_n[a] - 1, 1) : dflt;
}

// Integral of s^-k over the parallelogram o + u e1 + v e2 (u, v in [0,1]; e2 = 0 for a segment)
// with m1 x m2 panels of the 8-point Gauss-Legendre rule, s0 = 1.
double flat_integral(const mpsph_params *p, const double *o, const double *e1, const double *e2, int k, int m1,
                     int m2) {
  double xg[8], wg[8];
  gauss8(xg, wg);
  const int d = p->dim;
  double l1 = 0, l2 = 0;
  for (int a = 0; a < d; ++a) {
    l1 += e1[a] * e1[a];
    l2 += e2[a] * e2[a];
  }
  const bool seg = l2 == 0.0;
  const double meas = seg ? std::sqrt(l1) : std::sqrt(l1) * std::sqrt(l2);  // e1, e2 orthogonal
  if (!seg && m2 < 1) m2 = 1;
  const int n2 = seg ? 1 : 8 * m2;
  double total = 0.0;
  for (int i = 0; i < 8 * m1; ++i) {
    const double u = ((i >> 3) + xg[i & 7]) / m1, wu = wg[i & 7] / m1;
    double acc = 0.0;
    for (int j = 0; j < n2; ++j) {
      const double v = seg ? 0.0 : ((j >> 3) + xg[j & 7]) / m2, wv = seg ? 1.0 : wg[j & 7] / m2;
      double x[3] = {0, 0, 0};
      for (int a = 0; a < d; ++a) x[a] = o[a] + u * e1[a] + v * e2[a];
      acc += wv * std::pow(host_spacing(p, 1.0, x), -(double)k);
    }
    total += wu * acc;
  }
  return total * meas;
}

// Integral of s^-k over the sphere (dim 3) or circle (dim 2) of radius R about the region's
// centre, s0 = 1.
double round_integral(const mpsph_params *p, double R, int k) {
  double xg[8], wg[8];
  gauss8(xg, wg);
  const double pi = 3.14159265358979323846;
  const double *c = p->centre;
  double total = 0.0;
  if (p->dim == 2) {
    const int M = 256;
    for (int i = 0; i < 8 * M; ++i) {
      const double th = ((i >> 3) + xg[i & 7]) * 2 * pi / M, w = wg[i & 7] * 2 * pi / M;
      const double x[2] = {c[0] + R * std::cos(th), c[1] + R * std::sin(th)};
      total += w * R * std::pow(host_spacing(p, 1.0, x), -(double)k);
    }
    return total;
  }
  const int MT = 32, MP = 64;
  for (int i = 0; i < 8 * MT; ++i) {
    const double th = ((i >> 3) + xg[i & 7]) * pi / MT, wt = wg[i & 7] * pi / MT;
    double acc = 0.0;
    for (int j = 0; j < 8 * MP; ++j) {
      const double ph = ((j >> 3) + xg[j & 7]) * 2 * pi / MP, wp = wg[j & 7] * 2 * pi / MP;
      const double x[3] = {c[0] + R * std::sin(th) * std::cos(ph), c[1] + R * std::sin(th) * std::sin(ph),
                           c[2] + R * std::cos(th)};
      acc += wp * std::pow(host_spacing(p, 1.0, x), -(double)k);
    }
    total += wt * R * R * std::sin(th) * acc;
  }
  return total;
}

// The features of a region and their integrals at s0 = 1 (§2.3, Eq. 6: a surface integral on the
// feature surfaces and a line integral on the feature curves).
FeatureList feature_integrals(const mpsph_params *p) {
  FeatureList f;
  const int d = p->dim;
  if (p->geometry == MPSPH_PERIODIC) return f;
  if (p->geometry == MPSPH_BALL) {
    f.add(MPSPH_SURFACE, d - 1, round_integral(p, p->r_out, d - 1));
    return f;
  }
  if (p->geometry == MPSPH_ANNULUS) {
    f.add(MPSPH_SURFACE, 1, round_integral(p, p->r_in, 1));
    f.add(MPSPH_SURFACE, 1, round_integral(p, p->r_out, 1));
    return f;
  }
  const double *lo = p->lo, *hi = p->hi;
  auto corner_of = [&](int bits, double *x) {
    for (int a = 0; a < 3; ++a) x[a] = a < d ? ((bits >> a) & 1 ? hi[a] : lo[a]) : 0.0;
  };
  if (d == 2) {
    for (int a = 0; a < 2; ++a)
      for (int side = 0; side < 2; ++side) {
        const int b = 1 - a;
        double o[3] = {0, 0, 0}, e1[3] = {0, 0, 0}, e2[3] = {0, 0, 0};
        o[a] = side ? hi[a] : lo[a];
        o[b] = lo[b];
        e1[b] = hi[b] - lo[b];
        f.add(MPSPH_SURFACE, 1, flat_integral(p, o, e1, e2, 1, feature_panels(p, b, 256), 0));
      }
    for (int c = 0; c < 4; ++c) f.add(MPSPH_FIXED, 0, 1.0);
    return f;
  }
  for (int a = 0; a < 3; ++a)
    for (int side = 0; side < 2; ++side) {
      const int b = (a + 1) % 3, c = (a + 2) % 3;
      double o[3], e1[3] = {0, 0, 0}, e2[3] = {0, 0, 0};
      corner_of(0, o);
      o[a] = side ? hi[a] : lo[a];
      e1[b] = hi[b] - lo[b];
      e2[c] = hi[c] - lo[c];
      f.add(MPSPH_SURFACE, 2, flat_integral(p, o, e1, e2, 2, feature_panels(p, b, 32), feature_panels(p, c, 32)));
    }
  for (int a = 0; a < 3; ++a) {
    const int b = a == 0 ? 1 : 0, c = a == 2 ? 1 : 2;  // the two other axes, lower first
    for (int sc = 0; sc < 2; ++sc)
      for (int sb = 0; sb < 2; ++sb) {
        double o[3], e1[3] = {0, 0, 0}, e2[3] = {0, 0, 0};
        corner_of(0, o);
        o[b] = sb ? hi[b] : lo[b];
        o[c] = sc ? hi[c] : lo[c];
        e1[a] = hi[a] - lo[a];
        f.add(MPSPH_CURVE, 1, flat_integral(p, o, e1, e2, 1, feature_panels(p, a, 256), 0));
      }
  }
  for (int c = 0; c < 8; ++c) f.add(MPSPH_FIXED, 0, 1.0);
  return f;
}

// Bounds of s over the bounding box, and a Lipschitz constant of s (domain units).
// Bounds of the RBF field s = s0 exp(f), f(x) = sum_k c_k G_k(x), G_k = exp(-|x - x_k|^2 / (2 w^2)),
// over the box, from f and grad f on a grid: every point of the box lies within rho (half a grid
// cell's diagonal) of a node n, and |hess G| <= 1 / w^2 everywhere, so with Hf = sum |c_k| / w^2
//   f(x) <= f(n) + |grad f(n)| rho + Hf rho^2 / 2   (Taylor), likewise for the minimum, and
//   |grad f(x)| <= |grad f(n)| + Hf rho.
// Each bound is also capped by its grid-free form (sum of the positive / negative c_k, and
// |grad f| <= sum |c_k| / (w sqrt(e))).  The Lipschitz constant of s is smax * max |grad f|.
constexpr int kRbfBlocks = 512;   // blocks of the device's evaluation (rbf_extremes)
struct RbfGrid {
  int d, nr, m, nodes;             // m^d nodes
  double lo[3], step[3], rho, hess, inv2w2, w2;
  double centre[3 * kMaxRbf], coeff[kMaxRbf];
};

RbfGrid rbf_grid(const mpsph_params *p) {
  RbfGrid r;
  r.d = p->dim;
  r.nr = p->n_rbf;
  r.m = r.d == 3 ? 64 : 256;   // grid nodes per axis
  r.nodes = r.d == 3 ? r.m * r.m * r.m : r.m * r.m;
  r.w2 = p->rbf_width * p->rbf_width;
  r.inv2w2 = 1.0 / (2.0 * r.w2);
  double rho2 = 0, abs_sum = 0;
  for (int a = 0; a < 3; ++a) {
    r.lo[a] = a < r.d ? p->lo[a] : 0.0;
    r.step[a] = a < r.d ? (p->hi[a] - p->lo[a]) / (r.m - 1) : 0.0;
    rho2 += 0.25 * r.step[a] * r.step[a];
  }
  r.rho = std::sqrt(rho2);
  for (int k = 0; k < r.nr; ++k) {
    for (int a = 0; a < 3; ++a) r.centre[3 * k + a] = a < r.d ? p->rbf_centre[k * r.d + a] : 0.0;
    r.coeff[k] = p->rbf_coeff[k];
    abs_sum += std::fabs(p->rbf_coeff[k]);
  }
  r.hess = abs_sum / r.w2;
  return r;
}

// f and |grad f| at a node (x fastest).
__host__ __device__ void rbf_node(const RbfGrid &r, int node, double *fn, double *gn) {
  const int idx[3] = {node % r.m, node / r.m % r.m, node / (r.m * r.m)};
  const double x[3] = {r.lo[0] + idx[0] * r.step[0], r.lo[1] + idx[1] * r.step[1], r.lo[2] + idx[2] * r.step[2]};
  double f = 0, g[3] = {0, 0, 0};
  for (int k = 0; k < r.nr; ++k) {
    double dv[3], r2 = 0;
    for (int a = 0; a < 3; ++a) {
      dv[a] = x[a] - r.centre[3 * k + a];
      r2 += dv[a] * dv[a];
    }
    const double t = r.coeff[k] * exp(-r2 * r.inv2w2);
    f += t;
    for (int a = 0; a < 3; ++a) g[a] -= t * dv[a];
  }
  *fn = f;
  *gn = sqrt(g[0] * g[0] + g[1] * g[1] + g[2] * g[2]) / r.w2;
}

// The bounds from the three extremes over the nodes: max f + reach, min f - reach and max |grad f|.
void rbf_bounds_from(const mpsph_params *p, double s0, double fmax, double fmin, double gmax, double *smin, double *smax,
                     double *lip) {
  double pos = 0, neg = 0, abs_sum = 0;
  for (int k = 0; k < p->n_rbf; ++k) {
    pos += std::max(p->rbf_coeff[k], 0.0);
    neg += std::min(p->rbf_coeff[k], 0.0);
    abs_sum += std::fabs(p->rbf_coeff[k]);
  }
  const double w = p->rbf_width, Lf = abs_sum / (w * std::exp(0.5));
  const RbfGrid r = rbf_grid(p);
  fmax = std::min(pos, fmax);
  fmin = std::max(neg, fmin);
  gmax = std::min(Lf, gmax + r.hess * r.rho);
  *smin = s0 * std::exp(fmin);
  *smax = s0 * std::exp(fmax);
  *lip = *smax * gmax;
}

void rbf_bounds(const mpsph_params *p, double s0, double *smin, double *smax, double *lip) {
  const RbfGrid r = rbf_grid(p);
  double fmax = -INFINITY, fmin = INFINITY, gmax = 0;
  for (int node = 0; node < r.nodes; ++node) {
    double f, gn;
    rbf_node(r, node, &f, &gn);
    const double reach = gn * r.rho + 0.5 * r.hess * r.rho * r.rho;
    fmax = std::max(fmax, f + reach);
    fmin = std::min(fmin, f - reach);
    gmax = std::max(gmax, gn);
  }
  rbf_bounds_from(p, s0, fmax, fmin, gmax, smin, smax, lip);
}

bool spacing_bounds(const mpsph_params *p, double s0, double *smin, double *smax, double *lip) {
  if (p->field == MPSPH_GRID) {
    // the interpolant stays within the node extremes; its slope along an axis is bounded by the
    // largest node difference along that axis over the spacing
    const int d = p->dim;
    size_t nodes = 1;
    for (int a = 0; a < d; ++a) nodes *= (size_t)p->grid_n[a];
    double lo = INFINITY, hi = 0.0, l2 = 0.0;
    for (size_t k = 0; k < nodes; ++k) {
      lo = std::min(lo, p->grid_s[k]);
      hi = std::max(hi, p->grid_s[k]);
    }
    size_t stride = 1;
    for (int a = 0; a < d; ++a) {
      const double hs = (p->hi[a] - p->lo[a]) / (p->grid_n[a] - 1);
      double m = 0.0;
      for (size_t k = 0; k < nodes; ++k) {
        const size_t ia = (k / stride) % (size_t)p->grid_n[a];
        if (ia + 1 < (size_t)p->grid_n[a]) m = std::max(m, std::fabs(p->grid_s[k + stride] - p->grid_s[k]));
      }
      l2 += (m / hs) * (m / hs);
      stride *= (size_t)p->grid_n[a];
    }
    *smin = s0 * lo;
    *smax = s0 * hi;
    *lip = s0 * std::sqrt(l2);
    return *smin > 0 && std::isfinite(*smax);
  }
  switch (p->field) {
    case MPSPH_UNIFORM:
      *smin = *smax = s0;
      *lip = 0;
      break;
    case MPSPH_RADIAL_LINEAR: {
      double rmax, rmin = box_dist_range(p, p->fcentre, &rmax);
      double a = s0 * (1 + p->fa * (rmin - p->fb)), b = s0 * (1 + p->fa * (rmax - p->fb));
      *smin = std::min(a, b);
      *smax = std::max(a, b);
      *lip = s0 * std::fabs(p->fa);
      break;
    }
    case MPSPH_SPHERE_DISTANCE: {
      double rmax, rmin = box_dist_range(p, p->fcentre, &rmax);
      double dlo = (p->fb >= rmin && p->fb <= rmax) ? 0.0 : std::min(std::fabs(rmin - p->fb), std::fabs(rmax - p->fb));
      double dhi = std::max(std::fabs(rmin - p->fb), std::fabs(rmax - p->fb));
      double a = s0 * (1 + p->fa * dlo), b = s0 * (1 + p->fa * dhi);
      *smin = std::min(a, b);
      *smax = std::max(a, b);
      *lip = s0 * std::fabs(p->fa);
      break;
    }
    default:
      rbf_bounds(p, s0, smin, smax, lip);
  }
  return *smin > 0 && std::isfinite(*smax);
}

// bounds: smin, smax and Lipschitz constant where the caller has them (null: computed here).
int derive(const mpsph_params *p, int64_t n, double s0, Derived *d, const double *bounds = nullptr) {
  d->dim = p->dim;
  double L = 0;
  for (int a = 0; a < p->dim; ++a) L = std::max(L, p->hi[a] - p->lo[a]);
  d->L = L;
  for (int a = 0; a < 3; ++a) d->lo[a] = a < p->dim ? p->lo[a] : 0.0;
  if (bounds) {
    d->smin = bounds[0];
    d->smax = bounds[1];
    d->lip = bounds[2];
    if (!(d->smin > 0) || !std::isfinite(d->smax)) return MPSPH_E_INVALID;
  } else if (!spacing_bounds(p, s0, &d->smin, &d->smax, &d->lip)) {
    return MPSPH_E_INVALID;
  }
  int k = p->cell_log2;
  if (k < 0) {
    // cells of about 0.75 of the smallest cut-off radius; at most 2^24 cells, and not many more
    // cells than particles
    double rc_min = p->kappa * p->tau * d->smin;
    double target = L / (0.75 * rc_min) + 1.0;
    k = (int)std::lround(std::log2(std::max(target, 2.0)));
    int kmax = p->dim == 3 ? 8 : 12;
    while (k > 1 && std::pow(2.0, p->dim * k) > 8.0 * std::max<int64_t>(n, 64)) --k;
    k = std::min(std::max(k, 1), kmax);
  }
  if (p->dim * k > 24) return MPSPH_E_UNSUPPORTED;
  // x sub-cells: up to 2^MPSPH_XSUB per cell while the cell table stays within 4 entries per
  // particle (its fill is part of every step) and the key within 26 bits
  int xe = 0;
  while (xe < MPSPH_XSUB && p->dim * k + xe < 26 &&
         std::pow(2.0, p->dim * k + xe + 1) <= 4.0 * (double)std::max<int64_t>(n, 1))
    ++xe;
  d->xe = xe;
  d->k = k;
  d->gmax = (1 << k) - 1;
  // walls at cells 0 and 2^k - 1 (offset 0); a periodic box wraps after 2^k cells
  const double span = p->geometry == MPSPH_PERIODIC ? (double)(1 << k) : (double)d->gmax;
  d->cs = L / span;
  d->inv_cs = span / L;
  for (int a = 0; a < 3; ++a) d->xhi[a] = a < p->dim ? (p->hi[a] - p->lo[a]) * d->inv_cs : 0.0;
  // neighbour search bound: j interacts only if r < kappa (h_i + h_j)/2 and h_j <= h_i + L_h r
  // (L_h = tau * Lipschitz(s)), so r < kappa h_i / (1 - kappa L_h / 2).
  double Lh = p->tau * d->lip;
  double fac = 1e30;
  if (p->kappa * Lh / 2 < 0.95) fac = p->kappa / (1.0 - p->kappa * Lh / 2);
  d->search_fac = std::max(fac, p->kappa) * (1.0 + 1e-4);
  // minimum images are unique only while the cut-off stays below half the period
  if (p->geometry == MPSPH_PERIODIC && !(p->kappa * p->tau * d->smax < 0.5 * L)) return MPSPH_E_UNSUPPORTED;
  return MPSPH_OK;
}

// Mean spacing over particles distributed by the target density, int s^(1-d) / int s^-d, by midpoints.  Up to a range
// of about 1:8 over the region a coarse lattice is within 8 %.  Beyond, most particles lie where the field is fine, in parts
// that it misses (cube graded 1:60 from a sphere of 0.05: 2.5 times the mean, its rows four times too wide and a step
// of 262,144 particles 2650 us): fields of the distance to a point are sampled along rays from there, with
// steps that grow from the finest place (64 x 128 points, within 2 % up to 1:200), the others on a finer lattice.  A
// correction by less than 1.6 is left out: it moves rows only from about one to two per cut-off, and in graded
// fields one is the faster (262,144 particles, cube 1:8: 306 us per step against 353; 10^6, 1:30: 1711 against 1895).
double mean_spacing(const mpsph_params *p, double s0, const Derived &dv) {
  const int d = p->dim;
  if (p->field == MPSPH_UNIFORM) return s0;
  double w = 0.0, ws = 0.0, lo = INFINITY, hi = 0.0;
  const auto add = [&](const double *x, double weight) {
    for (int a = 0; a < d; ++a)
      if (!(x[a] >= p->lo[a] && x[a] <= p->hi[a])) return;
    if (!inside_region(p, x)) return;
    const double s = host_spacing(p, s0, x), v = weight / (d == 2 ? s * s : s * s * s);
    w += v;
    ws += v * s;
    lo = std::min(lo, s);
    hi = std::max(hi, s);
  };
  const auto lattice = [&](int m) {
    w = ws = 0.0;
    for (int iz = 0; iz < (d == 3 ? m : 1); ++iz)
      for (int iy = 0; iy < m; ++iy)
        for (int ix = 0; ix < m; ++ix) {
          const int idx[3] = {ix, iy, iz};
          double x[3] = {0, 0, 0};
          for (int a = 0; a < d; ++a) x[a] = p->lo[a] + (p->hi[a] - p->lo[a]) * (idx[a] + 0.5) / m;
          add(x, 1.0);
        }
  };
  lattice(d == 2 ? 24 : 8);
  const double coarse = w > 0 && std::isfinite(ws / w) ? ws / w : dv.smin;
  double rmax = 0.0;
  if (p->field == MPSPH_RADIAL_LINEAR || p->field == MPSPH_SPHERE_DISTANCE) {
    // a lattice that shows 1:5 misses the finest places of a range of 1:6 to 1:12 (from spheres of 0.05 on)
    if (hi > 5.0 * lo && box_dist_range(p, p->fcentre, &rmax) == 0.0) {
      constexpr int kRays = 64, kSteps = 64;
      const double pi = 3.14159265358979323846;
      const double fine = p->field == MPSPH_SPHERE_DISTANCE ? std::min(std::max(p->fb, 0.0), rmax) : (p->fa > 0 ? 0.0 : rmax);
      w = ws = 0.0;
      for (int side = -1; side <= 1; side += 2) {
        const double len = side < 0 ? fine : rmax - fine;
        if (!(len > 0)) continue;
        const double first = std::min(0.1 * dv.smin / (s0 * std::fabs(p->fa)), 0.5 * len), q = std::pow(len / first, 1.0 / (kSteps - 1));
        double t0 = 0.0, t1 = first;
        for (int k = 0; k < kSteps; ++k, t0 = t1, t1 *= q) {
          const double r = fine + side * 0.5 * (t0 + t1), weight = (t1 - t0) * (d == 2 ? r : r * r);
          for (int m = 0; m < kRays; ++m) {
            const double z = d == 2 ? 0.0 : 1.0 - (2.0 * m + 1.0) / kRays, c = std::sqrt(1.0 - z * z);
            const double ph = d == 2 ? (m + 0.5) * 2.0 * pi / kRays : (m + 0.5) * pi * (3.0 - std::sqrt(5.0));
            const double x[3] = {p->fcentre[0] + r * c * std::cos(ph), p->fcentre[1] + r * c * std::sin(ph), p->fcentre[2] + r * z};
            add(x, weight);
          }
        }
      }
    } else if (hi > 5.0 * lo) {
      lattice(d == 2 ? 512 : 64);
    }
  } else if (dv.smax > 8.0 * dv.smin) {
    // a background mesh by its nodes, Gaussians by a third of their width
    double m = 0.0;
    for (int a = 0; a < d; ++a)
      m = std::max(m, p->field == MPSPH_GRID ? (double)p->grid_n[a] : 3.0 * (p->hi[a] - p->lo[a]) / p->rbf_width);
    const double most = p->field == MPSPH_RBF_EXP ? (d == 2 ? 128 : 32) : (d == 2 ? 512 : 64);
    lattice((int)std::min(std::max(m, d == 2 ? 24.0 : 8.0), most));
  }
  if (!(w > 0) || !std::isfinite(ws / w)) return coarse;
  const double mean = ws / w;
  return mean < 1.6 * coarse && coarse < 1.6 * mean ? coarse : mean;
}

// Search rows: a row about as wide as the cut-off of a mean particle, whatever the cell size.
// The rule's cells follow the finest one, which in a graded field makes the rows of most particles
// narrow: a row costs as much as six candidates, the candidates fall by less.  Measured per step at 4
// lanes with rows of one and two cells: graded cube, 1M particles 1280 and 936 us, ball 1:3, 262,144
// particles 462 and 346; with a mean cut-off of 0.93, 1.95 and 3.9 rows (8192 particles, uniform) 88, 82 and 105.
int search_rows_rule(const mpsph_params *p, double s0, const Derived &d) {
  const double rc = p->kappa * p->tau * mean_spacing(p, s0, d) * d.inv_cs;
  const int rb = (int)std::floor(std::log2(std::max(rc / 1.05, 1e-3)));
  return std::min(std::max(rb, -1), d.k);
}

// x sub-cells of the search grid, and coarser rows where the table would be much larger than the
// particle count (at most 8 entries per particle or 2^20).
void fit_search(int dim, int64_t n, Derived *d) {
  const double most = std::max(8.0 * (double)std::max<int64_t>(n, 1), 1048576.0);
  auto bits = [&] { return d->k + d->xb + (dim - 1) * (d->k - d->rb); };
  d->xb = 0;
  while (std::pow(2.0, bits()) > most && d->rb < d->k) ++d->rb;
  // x sub-cells: up to 2^MPSPH_XSUB per cell while the table stays within 4 entries per particle (its scan is
  // part of every step)
  while (d->xb < MPSPH_XSUB && bits() < 26 && std::pow(2.0, bits() + 1) <= 4.0 * (double)std::max<int64_t>(n, 1)) ++d->xb;
}

// Cells that the separation of two candidates stays below: the reach of the pair loops (the largest cut-off of the
// box, a search row and a sub-cell), at most the grid, at most half of it in a periodic box (minimum image).
double separation_bound(const mpsph_params *p, const Derived &d) {
  const double reach = p->kappa * p->tau * d.smax * d.inv_cs * 1.001 + std::pow(2.0, std::max(d.rb, 0)) + 1.0;
  return std::min(reach, std::pow(2.0, p->geometry == MPSPH_PERIODIC ? d.k - 1 : d.k));
}
// Whether separations may reach 2^31 units of the fixed-point coordinates, whose difference would then be taken
// for a smaller one.
bool wide_field(const mpsph_params *p, const Derived &d) { return separation_bound(p, d) > std::ldexp(1.0, 31 - d.fb); }
// Bits of the fixed-point coordinates' fraction: 27, or 26 for separations of 16 to 32 cells; more in periodic boxes of
// few cells, whose period the coordinates' wrap has to divide.  Wider domains load cells as well instead of
// taking fewer bits: against 64-bit separations of particles 0.6 cells apart fixed-point ones are off by 5.5e-8 at 27
// and 26 bits, 5.8e-8 at 25, 7.6e-8 at 24 and 1.3e-7 at 23; (cell, offset) pairs of FP32 offsets by 5.8e-8.
int fixed_fraction(const mpsph_params *p, const Derived &d) {
  const int fb = separation_bound(p, d) <= 16.0 ? 27 : 26;
  return p->geometry == MPSPH_PERIODIC ? std::max(fb, 32 - d.k) : fb;
}

struct EventHook : LaunchHook {
  struct Rec {
    const char *name;
    hipEvent_t a, b;
  };
  hipStream_t stream = nullptr;
  bool on = false;
  bool pairs_only = false;   // record only the pair passes (kernels named pass_*)
  bool open = false;         // the last begin() recorded an event
  std::vector<Rec> pending;
  std::vector<hipEvent_t> pool;
  std::vector<std::string> names;
  std::vector<int64_t> launches;
  std::vector<double> ms;
  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e;
    (void)hipEventCreate(&e);
    return e;
  }
  void begin(const char *name) override {
    open = on && (!pairs_only || std::strncmp(name, "pass_", 5) == 0);
    if (!open) return;
    Rec r{name, get(), get()};
    (void)hipEventRecord(r.a, stream);
    pending.push_back(r);
  }
  void end() override {
    if (!open) return;
    open = false;
    (void)hipEventRecord(pending.back().b, stream);
  }
  void collect() {
    (void)hipStreamSynchronize(stream);
    for (auto &r : pending) {
      float t = 0;
      (void)hipEventElapsedTime(&t, r.a, r.b);
      size_t k = 0;
      for (; k < names.size(); ++k)
        if (names[k] == r.name) break;
      if (k == names.size()) {
        names.emplace_back(r.name);
        launches.push_back(0);
        ms.push_back(0);
      }
      launches[k] += 1;
      ms[k] += t;
      pool.push_back(r.a);
      pool.push_back(r.b);
    }
    pending.clear();
  }
  void reset() {
    names.clear();
    launches.clear();
    ms.clear();
  }
  ~EventHook() override {
    for (auto &r : pending) {
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
    for (auto e : pool) (void)hipEventDestroy(e);
  }
};


void split_cell(double X, int *c, float *o) {
  double f = std::floor(X);
  *c = (int)f;
  *o = (float)(X - f);
  if (*o >= 1.0f) {
    *o = 0.0f;
    *c += 1;
  }
}

// Surface-tension strength reported for a step (the kernels evaluate the same ramp in FP32).
double sigma_at(const mpsph_params *p, int64_t step, int64_t t0_auto = -1) {
  int64_t t0i = p->t0, t1i = p->t1;
  if (p->t0 == -2) {
    if (t0_auto < 0) return p->sigma0;
    const double th = p->theta > 0 ? p->theta : 0.2;
    t0i = t0_auto;
    // the same single-precision rounding as the kernels (round half to even)
    t1i = t0_auto + std::max<int64_t>(1, (int64_t)std::rint((float)th * (float)t0_auto));
  }
  if (t0i < 0) return p->sigma0;
  double t = (double)step, t0 = (double)t0i, t1 = (double)t1i;
  if (t <= t0) return p->sigma0;
  if (t <= t1) return p->sigma0 * (1.0 - (t - t0) / (t1 - t0));
  return 0.0;
}

// dt2 / dt1: with the velocity reset, v~ = a dt1 / 2 (Eq. 26) and nu = nu_coeff r_c |v~| (Eq. 21),
// so the three criteria of Eq. 29 are c_acc sqrt(m), (2 c_vel / dt1) m and
// (2 c_visc / (nu_coeff dt1)) m in m = r_c / |a|; their minima over the particles are reached at
// the same m = (dt1 / c_acc)^2, which gives dt2 = dt1 min(1, 2 min(c_vel, c_visc/nu_coeff) / c_acc^2).
double dt2_factor(const mpsph_params *p) {
  double c = p->c_vel;
  if (p->nu_coeff > 0) c = std::min(c, p->c_visc / p->nu_coeff);
  return std::min(1.0, 2.0 * c / (p->c_acc * p->c_acc));
}

// One domain of a context: its parameters (RBF arrays copied), derived grid and device constants.
struct Domain {
  mpsph_params p{};
  std::vector<double> rbf_centre, rbf_coeff;
  Derived d{};
  double s0 = 0;
  int64_t n = 0, off = 0;
  uint32_t ncells = 0, cellbase = 0;   // cells of the exported cell table
  uint32_t scells = 0, sbase = 0;      // cells of the search table
  int blk0 = 0, nblk = 0, row0 = 0, nrow = 0;
  size_t rbf0 = 0;  // first RBF term of this domain in the packed RBF arrays
  std::vector<double> gphi, gs;  // background-mesh node values (level set, field)
  size_t gphi0 = 0, gs0 = 0;     // first node of this domain in the packed device arrays
  int uidx = 0;     // index of the domain in the caller's list
  int64_t uoff = 0, xoff = 0;  // first row / first float of the domain in the caller's arrays

  Domain() = default;
  Domain(const Domain &o) { *this = o; }
  Domain(Domain &&o) noexcept = default;
  Domain &operator=(Domain &&o) noexcept = default;
  // p's RBF pointers refer to this domain's own copies of the arrays
  Domain &operator=(const Domain &o) {
    if (this == &o) return *this;
    p = o.p;
    rbf_centre = o.rbf_centre;
    rbf_coeff = o.rbf_coeff;
    d = o.d;
    s0 = o.s0;
    n = o.n;
    off = o.off;
    ncells = o.ncells;
    cellbase = o.cellbase;
    scells = o.scells;
    sbase = o.sbase;
    blk0 = o.blk0;
    nblk = o.nblk;
    row0 = o.row0;
    nrow = o.nrow;
    rbf0 = o.rbf0;
    gphi = o.gphi;
    gs = o.gs;
    gphi0 = o.gphi0;
    gs0 = o.gs0;
    uidx = o.uidx;
    uoff = o.uoff;
    xoff = o.xoff;
    if (!rbf_centre.empty()) {
      p.rbf_centre = rbf_centre.data();
      p.rbf_coeff = rbf_coeff.data();
    }
    p.grid_phi = gphi.empty() ? nullptr : gphi.data();
    p.grid_s = gs.empty() ? nullptr : gs.data();
    return *this;
  }
};

// Most pair-kernel blocks of a domain whose step the viscous pass closes (at 256 its end, 9.4 us longer, is no
// cheaper than finalize), and the fewest block partials per reduction row otherwise.
constexpr int64_t kFusedBlocks = 128, kRowBlocks = 256;

// Domains of one dimension occupy consecutive internal domain, particle and block ranges.
struct Group {
  int D = 0;
  bool periodic = false;  // some domain of the group is a periodic box
  bool kappa2 = true;     // every domain's cut-off is the kernel's support, kappa = 2
  int nwide = 0;          // wide domains (Derived::wide)
  int d0 = 0, nd = 0;   // internal domains
  int i0 = 0, i1 = 0;   // internal particles
  int b0 = 0, nb = 0;   // pair-kernel blocks
};

// Cells of the domain's two tables and the coordinates of its pair loops, for its cell size and search rows (d.rb).
void fit_grid(Domain *dm) {
  fit_search(dm->p.dim, dm->n, &dm->d);
  dm->d.fb = fixed_fraction(&dm->p, dm->d);
  dm->d.wide = wide_field(&dm->p, dm->d);
  dm->ncells = (uint32_t)1u << (dm->p.dim * dm->d.k + dm->d.xe);
  dm->scells = (uint32_t)1u << (dm->d.k + dm->d.xb + (dm->p.dim - 1) * (dm->d.k - dm->d.rb));
}

// Parameters copied into a domain; s0 normalised and the grid derived.  n is the domain's count.
int make_domain(const mpsph_params *params, int64_t n, Domain *dm) {
  if (!valid_params(params) || n < 0 || n > (int64_t)1 << 30) return MPSPH_E_INVALID;
  dm->p = *params;
  dm->n = n;
  if (params->field == MPSPH_RBF_EXP && params->n_rbf > 0) {
    dm->rbf_centre.assign(params->rbf_centre, params->rbf_centre + params->n_rbf * params->dim);
    dm->rbf_coeff.assign(params->rbf_coeff, params->rbf_coeff + params->n_rbf);
    dm->p.rbf_centre = dm->rbf_centre.data();
    dm->p.rbf_coeff = dm->rbf_coeff.data();
  } else {
    dm->p.n_rbf = 0;
    dm->p.rbf_centre = nullptr;
    dm->p.rbf_coeff = nullptr;
  }
  size_t nodes = 1;
  for (int a = 0; a < params->dim; ++a) nodes *= (size_t)std::max(params->grid_n[a], 1);
  dm->gphi.clear();
  dm->gs.clear();
  if (params->geometry == MPSPH_LEVELSET) dm->gphi.assign(params->grid_phi, params->grid_phi + nodes);
  if (params->field == MPSPH_GRID) dm->gs.assign(params->grid_s, params->grid_s + nodes);
  dm->p.grid_phi = dm->gphi.empty() ? nullptr : dm->gphi.data();
  dm->p.grid_s = dm->gs.empty() ? nullptr : dm->gs.data();
  double s0 = params->s0;
  if (!(s0 > 0)) {
    double I = field_integral_unit(&dm->p);
    if (!(I > 0) || !std::isfinite(I)) return MPSPH_E_INVALID;
    s0 = std::pow(I / (double)std::max<int64_t>(n, 1), 1.0 / params->dim);
  }
  dm->s0 = s0;
  int rc = derive(&dm->p, n, s0, &dm->d);
  if (rc) return rc;
  dm->d.rb = search_rows_rule(&dm->p, s0, dm->d);
  fit_grid(dm);
  return MPSPH_OK;
}

// Workspace layout of a context (byte offsets, 256-aligned).
struct Layout {
  int ndom = 0;
  Group grp[2];  // 2D domains, then 3D domains
  std::vector<int> internal;  // caller's domain index -> internal index
  int64_t n = 0;
  uint32_t ncells = 0;  // cells of all domains (exported cell table)
  uint32_t scells = 0;  // cells of the search table
  int nblocks_pair = 0, nrows = 0;
  // lanes per particle in the forward pair kernels of 2D and of 3D domains
  int lanes = MPSPH_LANES, lanes3 = MPSPH_LANES_3D;
  int lanes_of(int dim) const { return dim == 3 ? lanes3 : lanes; }
  int64_t chunk = 1;  // block partials per first-level reduction row
  bool fused = false; // the viscous pass closes the step (StepEnd)
  size_t n_rbf = 0;
  size_t bytes = 0;
  size_t s_key, s_off, s_ct, s_id, s_cell, w_key, w_pos, w_fix, w_jaux, w_id, counts, sums, cstart, acc, rho, nn, aabs, at, v,
      partials, partials2, groups, metrics, dtslots, stepctr, bad, paircount, queue, doms, vscale, rbf_c, rbf_o, rbf_k,
      gphi, gs, domdone, rbf_red;
};

// Orders the domains internally (2D before 3D, otherwise as given), assigns particle offsets,
// cell bases, pair-kernel blocks (lanes per particle) and reduction rows, and lays out the
// workspace.  doms must be in the caller's order.
int plan(std::vector<Domain> &doms, int lanes, Layout *out) {
  Layout L;
  L.ndom = (int)doms.size();
  int64_t all = 0;
  for (const auto &dm : doms) all += dm.n;
  // lanes 0: a context that was never configured; the wider groups only where the thread indices allow them
  L.lanes = lanes > 0 ? lanes : MPSPH_LANES;
  L.lanes3 = lanes > 0 ? lanes : (all * MPSPH_LANES_3D < ((int64_t)1 << 31) ? MPSPH_LANES_3D : MPSPH_LANES);
  const int most = std::max(L.lanes, doms.empty() || std::none_of(doms.begin(), doms.end(), [](const Domain &d) { return d.p.dim == 3; }) ? 0 : L.lanes3);
  int64_t uoff = 0, xoff = 0;
  for (int d = 0; d < L.ndom; ++d) {
    doms[d].uidx = d;
    doms[d].uoff = uoff;
    doms[d].xoff = xoff;
    uoff += doms[d].n;
    xoff += doms[d].n * doms[d].p.dim;
  }
  std::stable_sort(doms.begin(), doms.end(), [](const Domain &a, const Domain &b) { return a.p.dim < b.p.dim; });
  L.internal.assign(L.ndom, 0);
  for (int d = 0; d < L.ndom; ++d) L.internal[doms[d].uidx] = d;
  uint64_t cells = 0, scells = 0;
  int64_t n = 0;
  int64_t blocks = 0;
  size_t nrbf = 0, ngphi = 0, ngs = 0;
  for (int gi = 0; gi < 2; ++gi) {
    L.grp[gi].D = 2 + gi;
    L.grp[gi].d0 = 0;
  }
  for (int d = 0; d < L.ndom; ++d) {
    Domain &dm = doms[d];
    Group &g = L.grp[dm.p.dim - 2];
    if (g.nd == 0) {
      g.d0 = d;
      g.i0 = g.i1 = (int)n;
      g.b0 = (int)blocks;
    }
    dm.off = n;
    dm.cellbase = (uint32_t)cells;
    dm.sbase = (uint32_t)scells;
    dm.blk0 = (int)blocks;
    dm.nblk = std::max(1, (int)((dm.n * L.lanes_of(dm.p.dim) + kBlock - 1) / kBlock));   // an empty domain's one block closes its step
    dm.rbf0 = nrbf;
    dm.gphi0 = ngphi;
    dm.gs0 = ngs;
    ngphi += dm.gphi.size();
    ngs += dm.gs.size();
    n += dm.n;
    cells += dm.ncells;
    scells += dm.scells;
    blocks += dm.nblk;
    nrbf += (size_t)dm.p.n_rbf;
    // thread indices of the pair kernels (particles x lanes) stay below 2^31, indices of the search table below 2^32:
    // no larger than 2^(dim-1) times the cells (rows of half a cell) or 4 times the particles per domain
    // (fit_search), it stays so within the other limits
    if (n > ((int64_t)1 << 30) || n * most >= ((int64_t)1 << 31) || cells > ((uint64_t)1 << 28) ||
        scells >= ((uint64_t)1 << 32) || blocks > ((int64_t)1 << 30))
      return MPSPH_E_UNSUPPORTED;
    g.nd += 1;
    g.i1 = (int)n;
    g.nb += dm.nblk;
    g.periodic |= dm.p.geometry == MPSPH_PERIODIC;
    g.kappa2 &= dm.p.kappa == 2.0;
    g.nwide += dm.d.wide ? 1 : 0;
  }
  // first-level reduction: rows of at most `chunk` block partials, never straddling domains
  const int64_t chunk = std::max<int64_t>(kRowBlocks, (blocks + kReduceBlocks - 1) / kReduceBlocks);
  L.fused = n > 0;
  for (const auto &dm : doms) L.fused = L.fused && dm.nblk <= kFusedBlocks;
  int rows = 0;
  for (auto &dm : doms) {
    dm.row0 = rows;
    dm.nrow = (int)((dm.nblk + chunk - 1) / chunk);
    rows += dm.nrow;
  }
  L.n = n;
  L.ncells = (uint32_t)cells;
  L.scells = (uint32_t)scells;
  L.nblocks_pair = (int)blocks;
  L.nrows = rows;
  L.chunk = chunk;
  L.n_rbf = nrbf;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align_up(std::max<size_t>(bytes, 4));
    return at;
  };
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  L.s_key = take(nn * 4);
  L.s_off = take(nn * 16);
  L.s_ct = take(nn * 4);
  L.s_id = take(nn * 4);
  L.w_key = take(nn * 4);
  L.w_pos = take(nn * 16);
  L.w_jaux = take(nn * 4);
  L.w_id = take(nn * 4);
  L.s_cell = take(nn * 4);
  L.w_fix = take(nn * 16);
  L.cstart = take(((size_t)L.scells + 1) * 4);
  L.sums = take(cell_sum_words(L.scells) * 4);
  L.acc = take(nn * 16);
  // debug exports only
  const size_t nd = !doms.empty() && doms[0].p.debug ? nn : 0;
  L.rho = take(nd * 4);
  L.nn = take(nd * 4);
  L.aabs = take(nd * 4);
  L.at = take(nd * 16);
  L.v = take(nd * 16);
  L.partials = take((size_t)std::max(L.nblocks_pair, 1) * kNumPartials * 8);
  L.partials2 = take((size_t)std::max(L.nrows, 1) * kNumPartials * 8);
  L.groups = take((size_t)std::max(L.nrows, 1) * sizeof(int4));
  // what a load clears, in one range: metrics, step counter, validation flag, cell counts
  L.metrics = take((size_t)L.ndom * 32 * 8);
  L.stepctr = take(8);
  L.bad = take(4);
  L.counts = take(cell_count_words(L.scells) * 4);
  L.dtslots = take((size_t)L.ndom * kDtWords * 4);
  L.domdone = take((size_t)L.ndom * 4);
  L.paircount = take(8);
  L.queue = take(32 * 4);                   // work queues of the persistent pair passes (2 x 16 words)
  L.doms = take((size_t)L.ndom * sizeof(DomDev));
  L.vscale = take((size_t)L.ndom * 4);
  L.rbf_c = take(std::max<size_t>(nrbf, 1) * 3 * 4);
  L.rbf_o = take(std::max<size_t>(nrbf, 1) * 3 * 4);
  L.rbf_k = take(std::max<size_t>(nrbf, 1) * 4);
  L.rbf_red = take(nrbf > 0 ? (size_t)kRbfBlocks * 3 * 8 : 0);
  L.gphi = take(std::max<size_t>(ngphi, 1) * 4);
  L.gs = take(std::max<size_t>(ngs, 1) * 4);
  L.bytes = o;
  *out = L;
  return MPSPH_OK;
}

// Device constants of a domain (grid, region and field in cell units; step constants).
DomDev domain_device(const Domain &dm, const int *rbf_c, const float *rbf_o, const float *rbf_k, const float *gphi,
                     const float *gsv) {
  const mpsph_params &p = dm.p;
  const double cs = dm.d.cs, ics = dm.d.inv_cs;
  const int D = p.dim;
  DomDev dd;
  std::memset(&dd, 0, sizeof(dd));
  GridDev &g = dd.g;
  g.k = dm.d.k;
  g.n = (int)(dm.off + dm.n);
  g.gmax = dm.d.gmax;
  g.geometry = p.geometry;
  for (int a = 0; a < 3; ++a) {
    double Xhi = a < D ? (p.hi[a] - p.lo[a]) * ics : 0.0;
    split_cell(Xhi, &g.whi_c[a], &g.whi_o[a]);
    if (g.whi_c[a] > g.gmax) {
      g.whi_c[a] = g.gmax;
      g.whi_o[a] = 0.f;
    }
    double Xc = a < D ? (p.centre[a] - p.lo[a]) * ics : 0.0;
    split_cell(Xc, &g.gc_c[a], &g.gc_o[a]);
  }
  g.r_in = (float)(p.r_in * ics);
  g.r_out = (float)(p.r_out * ics);
  g.seeded = p.seeded ? 1 : 0;
  // 3D row tiles of 16 x 16 rows (fewer when the grid is smaller)
  g.xe = (uint32_t)dm.d.xe;
  g.ly = D == 3 ? (uint32_t)std::min(MPSPH_TILE_LY, g.k) : 0u;
  g.lz = D == 3 ? (uint32_t)std::min(MPSPH_TILE_LZ, g.k) : 0u;
  g.rb = dm.d.rb;
  g.skr = (uint32_t)(g.k - g.rb);
  g.xb = (uint32_t)dm.d.xb;
  g.sly = D == 3 ? std::min((uint32_t)MPSPH_TILE_LY, g.skr) : 0u;
  g.slz = D == 3 ? std::min((uint32_t)MPSPH_TILE_LZ, g.skr) : 0u;
  g.rowinv = std::ldexp(1.f, -g.rb);
  g.fx = std::ldexp(1.f, (int)g.xb);
  g.rfx = std::ldexp(1.f, g.rb + (int)g.xb);
  g.fb = dm.d.fb;
  g.funit = std::ldexp(1.f, -g.fb);
  g.wide = dm.d.wide ? 1 : 0;
  // background mesh: node spacing (hi - lo) / (n - 1) in cell units
  for (int a = 0; a < 3; ++a) {
    const int na = a < D ? std::max(p.grid_n[a], 2) : 2;
    g.gn[a] = na;
    g.ginv[a] = a < D ? (double)(na - 1) / ((p.hi[a] - p.lo[a]) * ics) : 1.0;
  }
  g.phi = p.geometry == MPSPH_LEVELSET ? gphi + dm.gphi0 : nullptr;
  FieldDev &f = dd.f;
  f.kind = p.field;
  f.s0 = (float)(dm.s0 * ics);
  f.g = (float)(p.fa * cs);
  f.b = (float)(p.fb * ics);
  for (int a = 0; a < 3; ++a) {
    double Xc = a < D ? (p.fcentre[a] - p.lo[a]) * ics : 0.0;
    split_cell(Xc, &f.fc_c[a], &f.fc_o[a]);
  }
  f.n_rbf = p.n_rbf;
  f.e2 = p.field == MPSPH_RBF_EXP ? (float)(cs * cs / (2.0 * p.rbf_width * p.rbf_width)) : 0.f;
  f.rbf_c = rbf_c + 3 * dm.rbf0;
  f.rbf_o = rbf_o + 3 * dm.rbf0;
  f.rbf_k = rbf_k + dm.rbf0;
  for (int a = 0; a < 3; ++a) {
    f.gn[a] = g.gn[a];
    f.ginv[a] = g.ginv[a];
  }
  f.gs = p.field == MPSPH_GRID ? gsv + dm.gs0 : nullptr;
  StepDev &sp = dd.sp;
  sp.kappa = (float)p.kappa;
  sp.tau = (float)p.tau;
  sp.inv_tau = (float)(1.0 / p.tau);
  sp.p0c = (float)(p.p0 * std::pow(cs, D - 2));
  sp.nu_coeff = (float)p.nu_coeff;
  sp.c_acc = (float)p.c_acc;
  sp.c_vel = (float)p.c_vel;
  sp.c_visc = (float)p.c_visc;
  sp.search_fac = (float)dm.d.search_fac;
  sp.hmax = (float)(p.tau * dm.d.smax / cs * (1.0 + 1e-5));
  sp.alpha = (float)(D == 2 ? 7.0 / (4.0 * M_PI) : 21.0 / (16.0 * M_PI));
  sp.dt2_factor = (float)dt2_factor(&p);
  sp.sigma0 = (float)p.sigma0;
  sp.t0 = p.t0 < 0 ? -1.f : (float)p.t0;
  sp.t1 = (float)p.t1;
  sp.auto_t0 = p.t0 == -2 ? 1 : 0;
  sp.t0_window = p.t0_window > 0 ? p.t0_window : 50;
  sp.t0_tol = (float)(p.t0_tol > 0 ? p.t0_tol : 1e-3);
  sp.theta = (float)(p.theta > 0 ? p.theta : 0.2);
  dd.cellbase = dm.cellbase;
  dd.sbase = dm.sbase;
  dd.off = (int)dm.off;
  dd.n = (int)dm.n;
  dd.uoff = (int)dm.uoff;
  dd.xoff = dm.xoff;
  dd.blk0 = dm.blk0;
  dd.nblk = dm.nblk;
  dd.row0 = dm.row0;
  dd.nrow = dm.nrow;
  for (int a = 0; a < 3; ++a) {
    dd.lo[a] = dm.d.lo[a];
    dd.xhi[a] = dm.d.xhi[a];
  }
  dd.cs = cs;
  dd.inv_cs = ics;
  return dd;
}

}  // namespace

struct mpsph_ctx {
  std::vector<Domain> dom;
  Layout L;
  hipStream_t stream = nullptr;
  char *ws = nullptr;
  size_t ws_cap = 0;  // bytes of the workspace
  bool owns = false;
  bool loaded = false;
  bool poisoned = false;
  int64_t steps_done = 0;
  EventHook hook;
  // step graph: nsteps steps captured once on a private stream, replayed on `stream`
  hipStream_t cap_stream = nullptr;
  hipGraphExec_t graph_exec = nullptr;
  int32_t graph_steps = 0;
  // device memory of the gradient driver (checkpoints, step records, adjoint arrays), grown on
  // demand by mpsph_grad and freed with the context
  char *gmem = nullptr;
  size_t gbytes = 0;
  // device whose static scratch array is the workspace (mpsph_create_static), -1 otherwise
  int static_dev = -1;
  // pair-kernel variant (mpsph_set_pair_variant): MPSPH_PAIRS_DEFAULT, _PERSISTENT or _TILE
  int variant = MPSPH_PAIRS_DEFAULT;
  int cus = 256;   // compute units of the device (the persistent grid holds kQueueBlocksPerCU per CU)
  template <typename T>
  T *at(size_t off) {
    return reinterpret_cast<T *>(ws + off);
  }
};

namespace {

// Extremes of the sampled RBF field: per block the largest f + reach, the smallest f - reach and the largest
// |grad f| (out[3 b ...]).  FP64; about 10 operations and one exponential per node and term.
__global__ __launch_bounds__(kBlock) void rbf_extremes(RbfGrid r, double *__restrict__ out) {
  __shared__ double red[3][kBlock / kWave];
  double hi = -INFINITY, lo = INFINITY, gmax = 0.0;
  for (int node = blockIdx.x * kBlock + threadIdx.x; node < r.nodes; node += kRbfBlocks * kBlock) {
    double f, gn;
    rbf_node(r, node, &f, &gn);
    const double reach = gn * r.rho + 0.5 * r.hess * r.rho * r.rho;
    hi = fmax(hi, f + reach);
    lo = fmin(lo, f - reach);
    gmax = fmax(gmax, gn);
  }
  for (int off = kWave / 2; off > 0; off >>= 1) {
    hi = fmax(hi, __shfl_xor(hi, off, kWave));
    lo = fmin(lo, __shfl_xor(lo, off, kWave));
    gmax = fmax(gmax, __shfl_xor(gmax, off, kWave));
  }
  if ((threadIdx.x & (kWave - 1)) == 0) {
    red[0][threadIdx.x / kWave] = hi;
    red[1][threadIdx.x / kWave] = lo;
    red[2][threadIdx.x / kWave] = gmax;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double x = red[threadIdx.x][0];
    for (int w = 1; w < kBlock / kWave; ++w) {
      const double y = red[threadIdx.x][w];
      x = threadIdx.x == 1 ? fmin(x, y) : fmax(x, y);
    }
    out[3 * blockIdx.x + threadIdx.x] = x;
  }
}

// The same extremes on the device: an optimisation loop sets new coefficients before every gradient, and
// the 262,144 nodes times 32 terms took the host 67 of the 70 ms of a gradient of 8192 particles
// (a gradient of four steps now takes 0.9 ms).
// In: the field's grid and terms; out: 3 doubles per block.
bool rbf_bounds_device(mpsph_ctx *ctx, const mpsph_params *p, double s0, double *bounds) {
  const RbfGrid r = rbf_grid(p);
  double *dev = ctx->at<double>(ctx->L.rbf_red);
  rbf_extremes<<<kRbfBlocks, kBlock, 0, ctx->stream>>>(r, dev);
  double h[kRbfBlocks][3];
  if (hipGetLastError() != hipSuccess ||
      hipMemcpyAsync(h, dev, sizeof(h), hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
      hipStreamSynchronize(ctx->stream) != hipSuccess)
    return false;
  double fmax = -INFINITY, fmin = INFINITY, gmax = 0;
  for (int b = 0; b < kRbfBlocks; ++b) {
    fmax = std::max(fmax, h[b][0]);
    fmin = std::min(fmin, h[b][1]);
    gmax = std::max(gmax, h[b][2]);
  }
  rbf_bounds_from(p, s0, fmax, fmin, gmax, &bounds[0], &bounds[1], &bounds[2]);
  return true;
}

int fail(mpsph_ctx *c, int code) {
  if (c && code == MPSPH_E_DEVICE) c->poisoned = true;
  return code;
}

#define HIP_OK(expr)                                            \
  do {                                                          \
    if ((expr) != hipSuccess) return fail(ctx, MPSPH_E_DEVICE); \
  } while (0)

// The arrays one step orders its particles into and works on: the context's own, or those of a
// gradient's record, which a step then fills in place.  slots and perm lie in acc until the density
// pass writes it.
struct WorkView {
  uint32_t *key;
  float4 *pos, *fix;
  uint32_t *jaux, *id, *cstart, *slots, *perm;
  float4 *acc;
  uint32_t *dts;
};
WorkView work_view(mpsph_ctx *ctx) {
  const Layout &L = ctx->L;
  uint32_t *a = ctx->at<uint32_t>(L.acc);
  return WorkView{ctx->at<uint32_t>(L.w_key), ctx->at<float4>(L.w_pos), ctx->at<float4>(L.w_fix), ctx->at<uint32_t>(L.w_jaux),
                  ctx->at<uint32_t>(L.w_id), ctx->at<uint32_t>(L.cstart), a, a + std::max<int64_t>(L.n, 1),
                  ctx->at<float4>(L.acc), ctx->at<uint32_t>(L.dtslots)};
}

// Orders the state by search cell: the slots of every cell and the search table.
// keep: the state's counts stay, for an order that no step follows.
hipError_t order_state(mpsph_ctx *ctx, const WorkView &w, hipStream_t st, LaunchHook *hk, bool keep = false) {
  const Layout &L = ctx->L;
  return cell_order(ctx->at<uint32_t>(L.s_cell), ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.counts),
                    ctx->at<uint32_t>(L.sums), w.cstart, w.slots, (int)L.n, L.scells, keep, st, hk);
}

bool dbg_context(const mpsph_ctx *ctx) { return ctx->dom[0].p.debug != 0; }

bool any_wide(const mpsph_ctx *ctx) { return ctx->L.grp[0].nwide + ctx->L.grp[1].nwide > 0; }

// The variant a step's launches take: the persistent and the staged ones serve narrow domains only.
int launch_variant(const mpsph_ctx *ctx) { return any_wide(ctx) ? MPSPH_PAIRS_DEFAULT : ctx->variant; }

// Whether the viscous pass closes the step (not the persistent launches: their blocks are not co-resident).
bool fused_end(const mpsph_ctx *ctx) { return ctx->L.fused && launch_variant(ctx) != MPSPH_PAIRS_PERSISTENT; }

// The step's end for a launch whose first domain is d0.
StepEnd step_end(mpsph_ctx *ctx, int d0) {
  const Layout &L = ctx->L;
  return StepEnd{d0, ctx->at<uint32_t>(L.domdone), ctx->at<double>(L.metrics) + (size_t)d0 * 32, ctx->at<int64_t>(L.stepctr)};
}

// The gather of one dimension group.
template <int D>
void launch_group(mpsph_ctx *ctx, const WorkView &w, const Group &gr, int nreset, hipStream_t st, EventHook *hk) {
  const Layout &L = ctx->L;
  if (hk) hk->begin("reorder_field");
  const int nt = std::max(gr.i1 - gr.i0, nreset);
  reorder_field<D><<<(nt + kBlock - 1) / kBlock, kBlock, 0, st>>>(
      ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, gr.i0, gr.i1, nreset, w.slots, w.cstart,
      ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.s_key), ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct),
      ctx->at<uint32_t>(L.s_id), w.key, w.pos, w.fix, w.jaux, w.id, w.perm, w.dts);
  if (hk) hk->end();
}

// launch(wide, b0, nb) for the blocks of every run of domains of one kind, wide or narrow, of a group: as a rule the
// whole group.
template <typename F>
void launch_kinds(const mpsph_ctx *ctx, const Group &gr, F &&launch) {
  if (gr.nwide == 0 || gr.nwide == gr.nd) {
    launch(gr.nwide > 0, gr.b0, gr.nb);
    return;
  }
  for (int d = gr.d0, e; d < gr.d0 + gr.nd; d = e) {
    int nb = 0;
    for (e = d; e < gr.d0 + gr.nd && ctx->dom[e].d.wide == ctx->dom[d].d.wide; ++e) nb += ctx->dom[e].nblk;
    launch(ctx->dom[d].d.wide, ctx->dom[d].blk0, nb);
  }
}

template <int D, int L_, bool PER>
void launch_pass1_l(mpsph_ctx *ctx, const WorkView &w, const Group &gr, hipStream_t st) {
  const Layout &L = ctx->L;
  const bool dbg = ctx->dom[0].p.debug != 0;
  auto kern = dbg ? pass_density_force<D, L_, PER, true, false, false>
                  : (gr.kappa2 ? pass_density_force<D, L_, PER, false, true, false>
                               : pass_density_force<D, L_, PER, false, false, false>);
  if constexpr (D == 3 && !PER)
    if (launch_variant(ctx) == MPSPH_PAIRS_TILE) kern = dbg ? pass_density_force_tile<L_, true> : pass_density_force_tile<L_, false>;
  const auto kwide = dbg ? pass_density_force<D, L_, PER, true, false, true> : pass_density_force<D, L_, PER, false, false, true>;
  launch_kinds(ctx, gr, [&](bool wide, int b0, int nb) {
    (wide ? kwide : kern)<<<nb, kBlock, 0, st>>>(
        b0, ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, ctx->at<int64_t>(L.stepctr), w.key, w.pos, w.fix, w.jaux,
        w.cstart, w.acc,
        dbg ? ctx->at<float>(L.rho) : nullptr, dbg ? ctx->at<float>(L.nn) : nullptr,
        dbg ? ctx->at<float>(L.aabs) : nullptr, w.dts + (size_t)gr.d0 * kDtWords,
        ctx->at<double>(L.metrics) + (size_t)gr.d0 * 32, ctx->at<double>(L.partials));
  });
}

template <int D>
void launch_pass1(mpsph_ctx *ctx, const WorkView &w, const Group &gr, hipStream_t st, EventHook *hk) {
  if (hk) hk->begin("pass_density_force");
  const int sel = ctx->L.lanes_of(D) * 2 + (gr.periodic ? 1 : 0);
  switch (sel) {
    case 4: launch_pass1_l<D, 2, false>(ctx, w, gr, st); break;
    case 5: launch_pass1_l<D, 2, true>(ctx, w, gr, st); break;
    case 16: launch_pass1_l<D, 8, false>(ctx, w, gr, st); break;
    case 17: launch_pass1_l<D, 8, true>(ctx, w, gr, st); break;
    case 9: launch_pass1_l<D, 4, true>(ctx, w, gr, st); break;
    default: launch_pass1_l<D, 4, false>(ctx, w, gr, st);
  }
  if (hk) hk->end();
}

template <int D, int L_, bool PER>
void launch_pass2_l(mpsph_ctx *ctx, const WorkView &w, const Group &gr, hipStream_t st, float4 *at_o, float4 *v_o) {
  const Layout &L = ctx->L;
  auto kern = fused_end(ctx) ? (gr.kappa2 ? pass_viscous_integrate<D, L_, PER, true, true, false>
                                          : pass_viscous_integrate<D, L_, PER, true, false, false>)
                             : (gr.kappa2 ? pass_viscous_integrate<D, L_, PER, false, true, false>
                                          : pass_viscous_integrate<D, L_, PER, false, false, false>);
  const auto kwide = fused_end(ctx) ? pass_viscous_integrate<D, L_, PER, true, false, true>
                                    : pass_viscous_integrate<D, L_, PER, false, false, true>;
  launch_kinds(ctx, gr, [&](bool wide, int b0, int nb) {
    (wide ? kwide : kern)<<<nb, kBlock, 0, st>>>(
        b0, ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, w.key, w.pos, w.fix, w.jaux, w.id, w.cstart, w.acc,
        w.dts + (size_t)gr.d0 * kDtWords, ctx->at<uint32_t>(L.s_key), ctx->at<float4>(L.s_off),
        ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id), ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.counts), at_o,
        v_o, ctx->at<double>(L.partials), step_end(ctx, gr.d0));
  });
}

template <int D>
void launch_pass2(mpsph_ctx *ctx, const WorkView &w, const Group &gr, hipStream_t st, EventHook *hk, float4 *at_rec = nullptr,
                  float4 *v_rec = nullptr) {
  const Layout &L = ctx->L;
  const bool dbg = ctx->dom[0].p.debug != 0;
  float4 *at_o = at_rec ? at_rec : (dbg ? ctx->at<float4>(L.at) : nullptr);
  float4 *v_o = v_rec ? v_rec : (dbg ? ctx->at<float4>(L.v) : nullptr);
  if (hk) hk->begin("pass_viscous_integrate");
  const int sel = L.lanes_of(D) * 2 + (gr.periodic ? 1 : 0);
  switch (sel) {
    case 4: launch_pass2_l<D, 2, false>(ctx, w, gr, st, at_o, v_o); break;
    case 5: launch_pass2_l<D, 2, true>(ctx, w, gr, st, at_o, v_o); break;
    case 16: launch_pass2_l<D, 8, false>(ctx, w, gr, st, at_o, v_o); break;
    case 17: launch_pass2_l<D, 8, true>(ctx, w, gr, st, at_o, v_o); break;
    case 9: launch_pass2_l<D, 4, true>(ctx, w, gr, st, at_o, v_o); break;
    default: launch_pass2_l<D, 4, false>(ctx, w, gr, st, at_o, v_o);
  }
  if (hk) hk->end();
}

// Persistent launches of the pair passes (pair-kernel variant MPSPH_PAIRS_PERSISTENT; see
// pass_density_force_queue): one launch per pass serves both dimension groups.
constexpr int kQueueBlocksPerCU = 8;   // blocks of the pair kernels resident per CU (8 waves per SIMD)
int queue_grid(const mpsph_ctx *ctx, int nb) { return std::max(1, std::min(nb, ctx->cus * kQueueBlocksPerCU)); }

template <int DM, int L_, int L3_, bool PER>
void launch_pass1_queue_l(mpsph_ctx *ctx, int b0, int nb2, int nb, hipStream_t st) {
  const Layout &L = ctx->L;
  const bool dbg = ctx->dom[0].p.debug != 0;
  auto kern = dbg ? pass_density_force_queue<DM, L_, L3_, PER, true> : pass_density_force_queue<DM, L_, L3_, PER, false>;
  kern<<<queue_grid(ctx, nb), kBlock, 0, st>>>(
      b0, nb2, nb, ctx->at<uint32_t>(L.queue), ctx->at<DomDev>(L.doms), L.ndom, ctx->at<int64_t>(L.stepctr),
      ctx->at<uint32_t>(L.w_key), ctx->at<float4>(L.w_pos), ctx->at<float4>(L.w_fix), ctx->at<uint32_t>(L.w_jaux),
      ctx->at<uint32_t>(L.cstart), ctx->at<float4>(L.acc), dbg ? ctx->at<float>(L.rho) : nullptr, dbg ? ctx->at<float>(L.nn) : nullptr,
      dbg ? ctx->at<float>(L.aabs) : nullptr, ctx->at<uint32_t>(L.dtslots), ctx->at<double>(L.metrics),
      ctx->at<double>(L.partials));
}

template <int DM, int L_, int L3_, bool PER>
void launch_pass2_queue_l(mpsph_ctx *ctx, int b0, int nb2, int nb, hipStream_t st) {
  const Layout &L = ctx->L;
  const bool dbg = ctx->dom[0].p.debug != 0;
  pass_viscous_integrate_queue<DM, L_, L3_, PER><<<queue_grid(ctx, nb), kBlock, 0, st>>>(
      b0, nb2, nb, ctx->at<uint32_t>(L.queue) + 16, ctx->at<DomDev>(L.doms), L.ndom, ctx->at<uint32_t>(L.w_key),
      ctx->at<float4>(L.w_pos), ctx->at<float4>(L.w_fix), ctx->at<uint32_t>(L.w_jaux), ctx->at<uint32_t>(L.w_id),
      ctx->at<uint32_t>(L.cstart), ctx->at<float4>(L.acc), ctx->at<uint32_t>(L.dtslots), ctx->at<uint32_t>(L.s_key),
      ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id), ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.counts),
      dbg ? ctx->at<float4>(L.at) : nullptr, dbg ? ctx->at<float4>(L.v) : nullptr, ctx->at<double>(L.partials),
      step_end(ctx, 0));
}

template <int DM>
void launch_queue_dm(mpsph_ctx *ctx, int pass, int b0, int nb2, int nb, bool per, hipStream_t st) {
  const Layout &L = ctx->L;
#define MPSPH_QUEUE_CASE(LN, LN3)                                                  \
  if (pass == 1 && per) launch_pass1_queue_l<DM, LN, LN3, true>(ctx, b0, nb2, nb, st); \
  else if (pass == 1) launch_pass1_queue_l<DM, LN, LN3, false>(ctx, b0, nb2, nb, st);  \
  else if (per) launch_pass2_queue_l<DM, LN, LN3, true>(ctx, b0, nb2, nb, st);         \
  else launch_pass2_queue_l<DM, LN, LN3, false>(ctx, b0, nb2, nb, st);
  if constexpr (DM == 5) {
    if (L.lanes != L.lanes3) {   // never configured
      MPSPH_QUEUE_CASE(MPSPH_LANES, MPSPH_LANES_3D)
      return;
    }
  }
  switch (L.lanes_of(DM)) {
    case 2: MPSPH_QUEUE_CASE(2, 2) break;
    case 8: MPSPH_QUEUE_CASE(8, 8) break;
    default: MPSPH_QUEUE_CASE(4, 4)
  }
#undef MPSPH_QUEUE_CASE
}

void launch_pairs_queue(mpsph_ctx *ctx, hipStream_t st, EventHook *hk) {
  const Layout &L = ctx->L;
  const Group &g2 = L.grp[0], &g3 = L.grp[1];
  for (int pass = 1; pass <= 2; ++pass) {
    if (hk) hk->begin(pass == 1 ? "pass_density_force" : "pass_viscous_integrate");
    if (g2.nb > 0 && g3.nb > 0) {
      launch_queue_dm<5>(ctx, pass, 0, g2.nb, g2.nb + g3.nb, g2.periodic || g3.periodic, st);
    } else {
      if (g2.nb > 0) launch_queue_dm<2>(ctx, pass, g2.b0, g2.nb, g2.nb, g2.periodic, st);
      if (g3.nb > 0) launch_queue_dm<3>(ctx, pass, g3.b0, 0, g3.nb, g3.periodic, st);
    }
    if (hk) hk->end();
  }
}

// The step's end where the viscous pass does not hold it.
void launch_step_end(mpsph_ctx *ctx, const WorkView &w, hipStream_t st, EventHook *hk) {
  const Layout &L = ctx->L;
  if (fused_end(ctx)) return;
  if (hk) hk->begin("finalize");
  finalize<<<L.nrows, kBlock, 0, st>>>(ctx->at<DomDev>(L.doms), ctx->at<int4>(L.groups), ctx->at<double>(L.partials),
                                       ctx->at<double>(L.partials2), w.dts, step_end(ctx, 0));
  if (hk) hk->end();
}

// Whether one launch per kernel serves both dimension groups: batches of both dimensions, at the lanes of a
// context that was never configured, without wide domains or the debug exports (their kernels come one per dimension).
bool mixed_launch(const mpsph_ctx *ctx) {
  const Layout &L = ctx->L;
  return L.grp[0].nb > 0 && L.grp[1].nb > 0 && ctx->variant == MPSPH_PAIRS_DEFAULT && !any_wide(ctx) && !dbg_context(ctx) &&
         L.lanes == MPSPH_LANES && L.lanes3 == MPSPH_LANES_3D;
}

void launch_mixed(mpsph_ctx *ctx, const WorkView &w, hipStream_t st, EventHook *hk) {
  const Layout &L = ctx->L;
  const Group &g2 = L.grp[0], &g3 = L.grp[1];
  const DomDev *doms = ctx->at<DomDev>(L.doms);
  const bool per = g2.periodic || g3.periodic, k2 = g2.kappa2 && g3.kappa2;
  const int nreset = L.ndom * kDtSlots;
  const int nblk2 = (std::max(g2.i1 - g2.i0, nreset) + kBlock - 1) / kBlock, nblk3 = (g3.i1 - g3.i0 + kBlock - 1) / kBlock;
  if (hk) hk->begin("reorder_field");
  reorder_field_mixed<<<nblk2 + nblk3, kBlock, 0, st>>>(
      g3.i0, nblk2, doms, L.ndom, 0, g3.i1, nreset, w.slots, w.cstart, ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.s_key),
      ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id), w.key, w.pos, w.fix, w.jaux, w.id, w.perm,
      w.dts);
  if (hk) hk->end();
  if (hk) hk->begin("pass_density_force");
  auto p1 = per ? (k2 ? pass_density_force_mixed<true, true> : pass_density_force_mixed<true, false>)
                : (k2 ? pass_density_force_mixed<false, true> : pass_density_force_mixed<false, false>);
  p1<<<g2.nb + g3.nb, kBlock, 0, st>>>(g2.nb, doms, L.ndom, ctx->at<int64_t>(L.stepctr), w.key, w.pos, w.fix, w.jaux, w.cstart,
                                       w.acc, nullptr, nullptr, nullptr, w.dts, ctx->at<double>(L.metrics),
                                       ctx->at<double>(L.partials));
  if (hk) hk->end();
  if (hk) hk->begin("pass_viscous_integrate");
  auto p2 = fused_end(ctx)
                ? (per ? (k2 ? pass_viscous_integrate_mixed<true, true, true> : pass_viscous_integrate_mixed<true, true, false>)
                       : (k2 ? pass_viscous_integrate_mixed<false, true, true> : pass_viscous_integrate_mixed<false, true, false>))
                : (per ? (k2 ? pass_viscous_integrate_mixed<true, false, true> : pass_viscous_integrate_mixed<true, false, false>)
                       : (k2 ? pass_viscous_integrate_mixed<false, false, true>
                             : pass_viscous_integrate_mixed<false, false, false>));
  p2<<<g2.nb + g3.nb, kBlock, 0, st>>>(g2.nb, doms, L.ndom, w.key, w.pos, w.fix, w.jaux, w.id, w.cstart, w.acc, w.dts,
                                       ctx->at<uint32_t>(L.s_key), ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct),
                                       ctx->at<uint32_t>(L.s_id), ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.counts),
                                       nullptr, nullptr, ctx->at<double>(L.partials), step_end(ctx, 0));
  if (hk) hk->end();
}

// Enqueues nsteps steps of every domain on stream st.  No host synchronisation, no memset and
// no host-side state read, so the same launches can be captured into a graph and replayed.
// Each kernel is launched once per non-empty dimension group, or once for both.
int enqueue(mpsph_ctx *ctx, int nsteps, hipStream_t st, EventHook *hk) {
  const Layout &L = ctx->L;
  const int n = (int)L.n, ndom = L.ndom;
  const WorkView w = work_view(ctx);
  for (int s = 0; s < nsteps; ++s) {
    if (n > 0) {
      if (order_state(ctx, w, st, hk) != hipSuccess)
        return fail(ctx, MPSPH_E_DEVICE);
      if (mixed_launch(ctx)) {
        launch_mixed(ctx, w, st, hk);
        launch_step_end(ctx, w, st, hk);
        if (hipGetLastError() != hipSuccess) return fail(ctx, MPSPH_E_DEVICE);
        continue;
      }
      int nreset = ndom * kDtSlots;  // the first launch resets every domain's time-step slots
      for (const Group &gr : L.grp) {
        if (gr.i1 <= gr.i0) continue;
        if (gr.D == 2) launch_group<2>(ctx, w, gr, nreset, st, hk);
        else launch_group<3>(ctx, w, gr, nreset, st, hk);
        nreset = 0;
      }
      if (launch_variant(ctx) == MPSPH_PAIRS_PERSISTENT) {
        launch_pairs_queue(ctx, st, hk);
      } else {
        for (const Group &gr : L.grp) {
          if (gr.nb <= 0) continue;
          if (gr.D == 2) launch_pass1<2>(ctx, w, gr, st, hk);
          else launch_pass1<3>(ctx, w, gr, st, hk);
        }
        for (const Group &gr : L.grp) {
          if (gr.nb <= 0) continue;
          if (gr.D == 2) launch_pass2<2>(ctx, w, gr, st, hk);
          else launch_pass2<3>(ctx, w, gr, st, hk);
        }
      }
    }
    launch_step_end(ctx, w, st, hk);
    if (hipGetLastError() != hipSuccess) return fail(ctx, MPSPH_E_DEVICE);
  }
  return MPSPH_OK;
}

void drop_graph(mpsph_ctx *ctx) {
  if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
  ctx->graph_exec = nullptr;
  ctx->graph_steps = 0;
}

void fill_metrics(const mpsph_ctx *ctx, int dmi, const double *m, mpsph_metrics_t *out) {
  const Domain &dm = ctx->dom[dmi];
  const double cs = dm.d.cs;
  std::memset(out, 0, sizeof(*out));
  out->step = ctx->steps_done - 1;
  out->pairs = (int64_t)m[P_PAIRS];
  out->interface_pairs = (int64_t)m[P_IFC] / 2;
  out->candidates = (int64_t)m[P_CAND];
  out->n_normal = (int64_t)m[P_NNORM];
  out->n_elr = (int64_t)m[P_NELR];
  out->nonfinite = (int64_t)(m[P_NONFIN1] + m[P_NONFIN2]);
  out->n_feature = (int64_t)m[P_NFEAT];
  out->residual_l2 = m[P_NNORM] > 0 ? std::sqrt(m[P_E2] / m[P_NNORM]) : 0.0;
  out->residual_linf = m[P_EMAX];
  out->pairs_total = (int64_t)m[18];
  out->candidates_total = (int64_t)m[19];
  out->kinetic = m[P_KE] * cs * cs;
  out->dt1 = m[16];
  out->dt2 = m[17];
  const int64_t t0a = m[kAutoT0] > 0 ? (int64_t)m[kAutoT0] - 1 : -1;
  out->sigma = sigma_at(&dm.p, std::max<int64_t>(ctx->steps_done - 1, 0), t0a);
  out->interface_particles = (int64_t)m[P_IFCP];
  out->t0 = dm.p.t0 == -2 ? t0a : dm.p.t0;
  if (m[P_NELR] > 0) {
    double mean = m[P_ELR] / m[P_NELR];
    out->elr_mean = mean;
    out->elr_std = std::sqrt(std::max(0.0, m[P_ELR2] / m[P_NELR] - mean * mean));
    out->elr_min = m[P_ELRMIN];
    out->elr_max = m[P_ELRMAX];
  }
}

int batch_check(int32_t ndom, const mpsph_params *params, const int64_t *n) {
  if (ndom < 1 || ndom > 4096 || !params || !n) return MPSPH_E_INVALID;
  for (int d = 0; d < ndom; ++d) {
    if (!valid_params(&params[d]) || n[d] < 0 || n[d] > (int64_t)1 << 30) return MPSPH_E_INVALID;
    if (params[d].debug != params[0].debug) return MPSPH_E_INVALID;
  }
  return MPSPH_OK;
}

int build_domains(int32_t ndom, const mpsph_params *params, const int64_t *n, std::vector<Domain> *doms, Layout *L) {
  int rc = batch_check(ndom, params, n);
  if (rc) return rc;
  doms->resize(ndom);
  for (int d = 0; d < ndom; ++d)
    if ((rc = make_domain(&params[d], n[d], &(*doms)[d])) != MPSPH_OK) return rc;
  return plan(*doms, 0, L);
}

// Re-derives every domain's cell grid -- the cell exponent of the size rule plus kdelta for
// domains whose cell_log2 was left to the library, the caller's value otherwise -- and plans
// the workspace for `lanes` lanes per particle.
int replan(std::vector<Domain> &doms, int kdelta, int lanes, Layout *L, int kabs = -1) {
  std::stable_sort(doms.begin(), doms.end(), [](const Domain &a, const Domain &b) { return a.uidx < b.uidx; });
  for (auto &dm : doms) {
    mpsph_params q = dm.p;
    if (kabs >= 1) {
      q.cell_log2 = kabs;
    } else if (q.cell_log2 < 0) {
      Derived r;
      int rc = derive(&q, dm.n, dm.s0, &r);
      if (rc) return rc;
      q.cell_log2 = std::min(std::max(r.k + kdelta, 1), q.dim == 3 ? 8 : 12);
    }
    int rc = derive(&q, dm.n, dm.s0, &dm.d);
    if (rc) return rc;
    dm.d.rb = search_rows_rule(&q, dm.s0, dm.d);   // by the cells alone: the same exponent gives the same rows again
    fit_grid(&dm);
  }
  return plan(doms, lanes, L);
}


// Zeroes the workspace and uploads the domain table, the reduction row groups and the RBF
// terms of the current layout.
int setup_device(mpsph_ctx *ctx) {
  const Layout &L = ctx->L;
  const int ndom = L.ndom;
  // a zeroed workspace keeps every table entry a valid index before its first write
  HIP_OK(hipMemset(ctx->ws, 0, L.bytes));
  std::vector<DomDev> dd(ndom);
  std::vector<int4> groups;
  std::vector<int> rc3(3 * std::max<size_t>(L.n_rbf, 1), 0);
  std::vector<float> ro3(3 * std::max<size_t>(L.n_rbf, 1), 0.f), rk(std::max<size_t>(L.n_rbf, 1), 0.f);
  for (int d = 0; d < ndom; ++d) {
    const Domain &dm = ctx->dom[d];
    dd[d] = domain_device(dm, ctx->at<int>(L.rbf_c), ctx->at<float>(L.rbf_o), ctx->at<float>(L.rbf_k),
                          ctx->at<float>(L.gphi), ctx->at<float>(L.gs));
    for (int r = 0; r < dm.nrow; ++r) {
      const int64_t a = dm.blk0 + (int64_t)r * L.chunk;
      groups.push_back(make_int4(d, (int)a, (int)std::min<int64_t>(a + L.chunk, dm.blk0 + dm.nblk), 0));
    }
    for (int t = 0; t < dm.p.n_rbf; ++t) {
      const size_t kk = dm.rbf0 + t;
      for (int a = 0; a < dm.p.dim; ++a)
        split_cell((dm.p.rbf_centre[t * dm.p.dim + a] - dm.p.lo[a]) * dm.d.inv_cs, &rc3[kk * 3 + a], &ro3[kk * 3 + a]);
      rk[kk] = (float)dm.p.rbf_coeff[t];
    }
  }
  HIP_OK(hipMemcpy(ctx->at<DomDev>(L.doms), dd.data(), dd.size() * sizeof(DomDev), hipMemcpyHostToDevice));
  if (!groups.empty())
    HIP_OK(hipMemcpy(ctx->at<int4>(L.groups), groups.data(), groups.size() * sizeof(int4), hipMemcpyHostToDevice));
  HIP_OK(hipMemcpy(ctx->at<int>(L.rbf_c), rc3.data(), rc3.size() * 4, hipMemcpyHostToDevice));
  HIP_OK(hipMemcpy(ctx->at<float>(L.rbf_o), ro3.data(), ro3.size() * 4, hipMemcpyHostToDevice));
  HIP_OK(hipMemcpy(ctx->at<float>(L.rbf_k), rk.data(), rk.size() * 4, hipMemcpyHostToDevice));
  // background-mesh values: the level set in cell units, the field's relative spacing as given
  for (int d = 0; d < ndom; ++d) {
    const Domain &dm = ctx->dom[d];
    if (!dm.gphi.empty()) {
      std::vector<float> v(dm.gphi.size());
      for (size_t k = 0; k < v.size(); ++k) v[k] = (float)(dm.gphi[k] * dm.d.inv_cs);
      HIP_OK(hipMemcpy(ctx->at<float>(L.gphi) + dm.gphi0, v.data(), v.size() * 4, hipMemcpyHostToDevice));
    }
    if (!dm.gs.empty()) {
      std::vector<float> v(dm.gs.begin(), dm.gs.end());
      HIP_OK(hipMemcpy(ctx->at<float>(L.gs) + dm.gs0, v.data(), v.size() * 4, hipMemcpyHostToDevice));
    }
  }
  return MPSPH_OK;
}

// Re-plans the context for a cell size (rule + kdelta, or kabs >= 1 for every domain) and a
// lane count, growing a library-owned workspace when needed, and resets the device tables.
// The loaded state is lost.  A configuration that does not fit a caller workspace returns
// MPSPH_E_NOMEM and leaves the context unchanged.
int reconfigure(mpsph_ctx *ctx, const std::vector<Domain> &base, int kdelta, int kabs, int lanes) {
  std::vector<Domain> doms = base;
  Layout Lc;
  int rc = replan(doms, kdelta, lanes, &Lc, kabs);
  if (rc) return rc;
  if (Lc.bytes > ctx->ws_cap) {
    if (!ctx->owns) return MPSPH_E_NOMEM;
    (void)hipStreamSynchronize(ctx->stream);
    (void)hipFree(ctx->ws);
    ctx->ws = nullptr;
    ctx->ws_cap = 0;
    if (hipMalloc((void **)&ctx->ws, Lc.bytes) != hipSuccess) return fail(ctx, MPSPH_E_DEVICE);
    ctx->ws_cap = Lc.bytes;
  }
  drop_graph(ctx);
  ctx->dom = doms;
  ctx->L = Lc;
  ctx->loaded = false;
  ctx->steps_done = 0;
  return setup_device(ctx);
}

// ------------------------------------------------------------------------------------------
// Gradient driver: forward with checkpoints, loss, and the reverse sweep.  Every step of a segment
// of ckpt steps is recorded (its sorted state and results), then the segment's steps are reversed
// from last to first.  The last segment is recorded as the forward pass runs it; the others start
// again from their checkpoints.  A recorded step writes its arrays in place, the last of a segment
// the context's own, so that no copy is made and the exports refer to the last step recorded.
// 262,144 particles, 4 steps, a checkpoint every 2, with copies of every array and all segments
// recomputed 4.10 ms, this way and with five reverse kernels a step 3.01; 8,192 particles 1.30 and 0.93 ms.
// ------------------------------------------------------------------------------------------

// Most particles of a 3D gradient whose loss and adjoint pair kernels take 16 lanes per particle: at 8 the
// grid leaves SIMDs with a single wave (8,192 particles), whose loops are a chain of latencies.  Gradient of 4
// steps at 8 / 16 lanes: 2,000 particles 647 / 582 us, 4,096 691 / 620, 8,192 615 / 569, 16,384 606 / 590, 24,000
// 728 / 723, 65,536 995 / 1026.
constexpr int kAdjSmall = 16384;

struct GradPlan {
  int nck = 0, ckpt = 0;
  size_t ck0 = 0, ck_stride = 0, ck_key = 0, ck_off = 0, ck_ct = 0, ck_id = 0, ck_cell = 0;
  size_t tp0 = 0, tp_stride = 0, tp_perm = 0, tp_wkey = 0, tp_wpos = 0, tp_wfix = 0, tp_wjaux = 0, tp_acc = 0, tp_at = 0,
         tp_v = 0, tp_cstart = 0, tp_dts = 0;
  size_t xbar = 0, xacc = 0, abv = 0, vtb = 0, fbar = 0, sbar = 0, e = 0, dtc = 0, pa = 0, pb = 0, cpart = 0, slots = 0,
         out = 0, mback = 0;
  size_t bytes = 0;
};

GradPlan grad_plan(int64_t n, uint32_t ncells, int nck, int ckpt, int nb1, int nbp, int nrow) {
  GradPlan P;
  P.nck = nck;
  P.ckpt = ckpt;
  const size_t nn = (size_t)std::max<int64_t>(n, 1);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align_up(std::max<size_t>(bytes, 4));
    return at;
  };
  // checkpoint: the state arrays (key, offsets, type | colour, id)
  size_t c = 0;
  auto ctake = [&](size_t bytes) {
    size_t at = c;
    c += align_up(bytes);
    return at;
  };
  P.ck_key = ctake(nn * 4);
  P.ck_off = ctake(nn * 16);
  P.ck_ct = ctake(nn * 4);
  P.ck_id = ctake(nn * 4);
  P.ck_cell = ctake(nn * 4);
  P.ck_stride = c;
  P.ck0 = take(P.ck_stride * nck);
  size_t t = 0;
  auto ttake = [&](size_t bytes) {
    size_t at = t;
    t += align_up(bytes);
    return at;
  };
  P.tp_perm = ttake(nn * 4);
  P.tp_wkey = ttake(nn * 4);
  P.tp_wpos = ttake(nn * 16);
  P.tp_wfix = ttake(nn * 16);
  P.tp_wjaux = ttake(nn * 4);
  P.tp_acc = ttake(nn * 16);
  P.tp_at = ttake(nn * 16);
  P.tp_v = ttake(nn * 16);
  P.tp_cstart = ttake(((size_t)ncells + 1) * 4);
  P.tp_dts = ttake(kDtWords * 4);
  P.tp_stride = t;
  P.tp0 = take(P.tp_stride * ckpt);
  P.xbar = take(nn * 16);
  P.xacc = take(nn * 16);
  P.abv = take(nn * 16);
  P.vtb = take(nn * 16);
  P.fbar = take(nn * 16);
  P.sbar = take(nn * 4);
  P.e = take(nn * 4);
  P.dtc = take(nn * 4);
  P.pa = take((size_t)std::max(nb1, 1) * 8);
  P.pb = take((size_t)std::max(nbp, 1) * 2 * 8);
  P.cpart = take((size_t)std::max(nrow, 1) * kMaxRbf * 8);
  P.slots = take((kDtWords + 1) * 4);   // time-step slots of the reverse sweep, index of the minimum
  P.out = take((1 + kMaxRbf) * 8);      // loss, c-bar
  P.mback = take(32 * 8);
  P.bytes = o;
  return P;
}

struct GradRun {
  mpsph_ctx *ctx;
  GradPlan P;
  hipStream_t st;
  const Group *gr;
  int nb1;
  int lanes; // of the loss and adjoint pair kernels: MPSPH_ADJ_LANES or MPSPH_ADJ_LANES_SMALL
  int nbp;   // blocks of those kernels
  int nrow;  // rows of coefficient sums: waves of adj_field
  char *g;
  template <typename T>
  T *at(size_t off) {
    return reinterpret_cast<T *>(g + off);
  }
  uint32_t *minslots() { return at<uint32_t>(P.slots); }
  uint32_t *argmin() { return at<uint32_t>(P.slots) + kDtWords; }
  // Record slot m as a step's work arrays; slots, perm and ids in its acc until that is written.
  WorkView slot_view(int m) {
    char *b = g + P.tp0 + P.tp_stride * m;
    const int64_t nn = std::max<int64_t>(ctx->L.n, 1);
    uint32_t *a = reinterpret_cast<uint32_t *>(b + P.tp_acc);
    return WorkView{reinterpret_cast<uint32_t *>(b + P.tp_wkey),   reinterpret_cast<float4 *>(b + P.tp_wpos),
                    reinterpret_cast<float4 *>(b + P.tp_wfix),     reinterpret_cast<uint32_t *>(b + P.tp_wjaux),
                    a + 2 * nn,                                    reinterpret_cast<uint32_t *>(b + P.tp_cstart),
                    a,                                             a + nn,
                    reinterpret_cast<float4 *>(a),                 reinterpret_cast<uint32_t *>(b + P.tp_dts)};
  }
  // Step m of a recorded segment, last: its last one, in the context's arrays.
  WorkView step_view(int m, bool last) {
    WorkView w = last ? work_view(ctx) : slot_view(m);
    w.id = ctx->at<uint32_t>(ctx->L.w_id);
    w.perm = at<uint32_t>(P.tp0 + P.tp_stride * m + P.tp_perm);
    return w;
  }
  // the debug exports of a recorded step's v and a~ need them in the context
  float4 *at_of(int m, bool last) {
    return last && dbg_context(ctx) ? ctx->at<float4>(ctx->L.at) : at<float4>(P.tp0 + P.tp_stride * m + P.tp_at);
  }
  float4 *v_of(int m, bool last) {
    return last && dbg_context(ctx) ? ctx->at<float4>(ctx->L.v) : at<float4>(P.tp0 + P.tp_stride * m + P.tp_v);
  }
  TapeView tape(const WorkView &w, const float4 *at_w, const float4 *v_w) {
    return TapeView{w.key, w.pos, w.fix, w.jaux, w.cstart, w.perm, w.acc, at_w, v_w, w.dts};
  }
  StateView state() {
    const Layout &L = ctx->L;
    return StateView{ctx->at<uint32_t>(L.s_key), ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id),
                     ctx->at<uint32_t>(L.s_cell)};
  }
  StateView checkpoint(int k) {
    char *c = g + P.ck0 + P.ck_stride * k;
    return StateView{reinterpret_cast<uint32_t *>(c + P.ck_key), reinterpret_cast<float4 *>(c + P.ck_off),
                     reinterpret_cast<uint32_t *>(c + P.ck_ct), reinterpret_cast<uint32_t *>(c + P.ck_id),
                     reinterpret_cast<uint32_t *>(c + P.ck_cell)};
  }
};

// Copies the context's state to checkpoint k; metrics: with the step's metrics.
int save_state(GradRun &R, int k, bool metrics) {
  mpsph_ctx *ctx = R.ctx;
  const Layout &L = ctx->L;
  copy_state<<<R.nb1, kBlock, 0, R.st>>>(R.checkpoint(k), R.state(), (int)L.n, metrics ? R.at<double>(R.P.mback) : nullptr,
                                         ctx->at<double>(L.metrics), nullptr, nullptr, 0);
  HIP_OK(hipGetLastError());
  return MPSPH_OK;
}

// The context's state from checkpoint k, whose next step is number t.
int restore_state(GradRun &R, int k, int64_t t, bool metrics) {
  mpsph_ctx *ctx = R.ctx;
  const Layout &L = ctx->L;
  HIP_OK(hipMemsetAsync(ctx->at<uint32_t>(L.counts), 0, cell_count_words(L.scells) * 4, R.st));
  copy_state<<<R.nb1, kBlock, 0, R.st>>>(R.state(), R.checkpoint(k), (int)L.n, metrics ? ctx->at<double>(L.metrics) : nullptr,
                                         R.at<double>(R.P.mback), ctx->at<uint32_t>(L.counts), ctx->at<int64_t>(L.stepctr), t);
  HIP_OK(hipGetLastError());
  return MPSPH_OK;
}

// Runs and records the len steps of a segment.
template <int D>
int record_segment(GradRun &R, int len) {
  mpsph_ctx *ctx = R.ctx;
  for (int m = 0; m < len; ++m) {
    const bool last = m == len - 1;
    const WorkView w = R.step_view(m, last);
    if (order_state(ctx, w, R.st, nullptr) != hipSuccess) return fail(ctx, MPSPH_E_DEVICE);
    launch_group<D>(ctx, w, *R.gr, kDtSlots, R.st, nullptr);
    launch_pass1<D>(ctx, w, *R.gr, R.st, nullptr);
    launch_pass2<D>(ctx, w, *R.gr, R.st, nullptr, R.at_of(m, last), R.v_of(m, last));
    launch_step_end(ctx, w, R.st, nullptr);
    HIP_OK(hipGetLastError());
  }
  return MPSPH_OK;
}

// Field adjoint of a step (or of the loss): x-bar in the previous state order, c-bar sums.
template <int D>
void field_backward(GradRun &R, const TapeView &tv, bool first) {
  adj_field<D><<<R.nrow, kWave, 0, R.st>>>(R.ctx->at<DomDev>(R.ctx->L.doms), tv, R.at<float4>(R.P.xacc), R.at<float>(R.P.sbar),
                                           R.at<float4>(R.P.xbar), R.at<double>(R.P.cpart), first ? 1 : 0, R.minslots(),
                                           R.argmin());
}

// Adjoint of the loss at the current state: x-bar (state order) and the first share of c-bar.  The
// final state is ordered into record slot m, which no recorded step occupies; its counts stay.
template <int D>
int loss_backward(GradRun &R, double lam, int m) {
  mpsph_ctx *ctx = R.ctx;
  const Layout &L = ctx->L;
  const Domain &dm = ctx->dom[0];
  const int n = (int)L.n;
  const DomDev *dom = ctx->at<DomDev>(L.doms);
  const WorkView w = R.slot_view(m);
  if (order_state(ctx, w, R.st, nullptr, true) != hipSuccess)
    return fail(ctx, MPSPH_E_DEVICE);
  launch_group<D>(ctx, w, *R.gr, kDtSlots, R.st, nullptr);
  const int nbp = R.nbp;
  const bool small = R.lanes == MPSPH_ADJ_LANES_SMALL, wide = dm.d.wide;
  const auto density = small ? (wide ? loss_density<D, MPSPH_ADJ_LANES_SMALL, true> : loss_density<D, MPSPH_ADJ_LANES_SMALL, false>)
                             : (wide ? loss_density<D, MPSPH_ADJ_LANES, true> : loss_density<D, MPSPH_ADJ_LANES, false>);
  const auto grad = small ? (wide ? loss_grad<D, MPSPH_ADJ_LANES_SMALL, true> : loss_grad<D, MPSPH_ADJ_LANES_SMALL, false>)
                          : (wide ? loss_grad<D, MPSPH_ADJ_LANES, true> : loss_grad<D, MPSPH_ADJ_LANES, false>);
  density<<<nbp, kBlock, 0, R.st>>>(dom, w.key, w.fix, w.jaux, w.cstart, R.at<float>(R.P.e),
                                                       R.at<double>(R.P.pb));
  loss_value<<<1, kLossThreads, 0, R.st>>>(R.at<double>(R.P.pb), nbp, 1.0 / n, lam, R.at<double>(R.P.out));
  // every neighbour j whose support reaches k: r < kappa h_j <= kappa h_k / (1 - kappa L_h)
  const double Lh = dm.p.tau * dm.d.lip;
  const double kl = dm.p.kappa * Lh;
  const float reach = kl < 0.95 ? (float)(dm.p.kappa / (1.0 - kl) * (1.0 + 1e-4)) : 1e30f;
  grad<<<nbp, kBlock, 0, R.st>>>(dom, w.key, w.fix, w.jaux, w.cstart, R.at<float>(R.P.e),
                                                    (float)(2.0 / n), (float)(lam / n), reach, R.at<float4>(R.P.xacc),
                                                    R.at<float>(R.P.sbar));
  field_backward<D>(R, R.tape(w, nullptr, nullptr), true);
  HIP_OK(hipGetLastError());
  return MPSPH_OK;
}

// Reverse of step m of the recorded segment (step index t of the run).
template <int D>
int step_backward(GradRun &R, int m, bool last, int64_t t) {
  mpsph_ctx *ctx = R.ctx;
  const Layout &L = ctx->L;
  const DomDev *dom = ctx->at<DomDev>(L.doms);
  const TapeView tv = R.tape(R.step_view(m, last), R.at_of(m, last), R.v_of(m, last));
  const int nbp = R.nbp;
  adj_drift<D><<<R.nb1, kBlock, 0, R.st>>>(dom, tv, R.at<float4>(R.P.xbar), R.at<float4>(R.P.xacc),
                                           R.at<float4>(R.P.abv), R.at<float4>(R.P.vtb), R.at<float>(R.P.dtc), R.minslots(),
                                           R.at<double>(R.P.pa));
  const bool small = R.lanes == MPSPH_ADJ_LANES_SMALL, wide = ctx->dom[0].d.wide;
  const auto visc = small ? (wide ? adj_visc<D, MPSPH_ADJ_LANES_SMALL, true> : adj_visc<D, MPSPH_ADJ_LANES_SMALL, false>)
                          : (wide ? adj_visc<D, MPSPH_ADJ_LANES, true> : adj_visc<D, MPSPH_ADJ_LANES, false>);
  const auto force = small ? (wide ? adj_force<D, MPSPH_ADJ_LANES_SMALL, true> : adj_force<D, MPSPH_ADJ_LANES_SMALL, false>)
                           : (wide ? adj_force<D, MPSPH_ADJ_LANES, true> : adj_force<D, MPSPH_ADJ_LANES, false>);
  visc<<<nbp, kBlock, 0, R.st>>>(dom, tv, R.at<float4>(R.P.abv), R.at<float4>(R.P.vtb),
                                                   R.at<float4>(R.P.xacc), R.at<float>(R.P.sbar),
                                                   R.at<float4>(R.P.fbar), R.at<float>(R.P.dtc), R.minslots(), R.argmin(),
                                                   R.at<double>(R.P.pb));
  adj_time_step<D><<<1, kTimeStepThreads, 0, R.st>>>(dom, tv, R.at<double>(R.P.pa), R.nb1, R.at<double>(R.P.pb), nbp,
                                                     (float)dt2_factor(&ctx->dom[0].p), R.argmin(), R.at<float>(R.P.sbar),
                                                     R.at<float4>(R.P.fbar));
  force<<<nbp, kBlock, 0, R.st>>>(dom, tv, (float)t, R.at<float4>(R.P.fbar),
                                                    R.at<float4>(R.P.xacc), R.at<float>(R.P.sbar));
  field_backward<D>(R, tv, false);
  HIP_OK(hipGetLastError());
  return MPSPH_OK;
}

template <int D>
int grad_run(mpsph_ctx *ctx, int nsteps, int ckpt, double lam, double *loss_out, double *grad_coeff,
             float *d_grad_pos) {
  const Layout &L = ctx->L;
  const Domain &dm = ctx->dom[0];
  const int n = (int)L.n;
  GradRun R;
  R.ctx = ctx;
  R.st = ctx->stream;
  R.gr = &L.grp[D - 2];
  R.nb1 = (n + kBlock - 1) / kBlock;
  R.lanes = D == 3 && n <= kAdjSmall ? MPSPH_ADJ_LANES_SMALL : MPSPH_ADJ_LANES;
  R.nbp = (int)(((int64_t)n * R.lanes + kBlock - 1) / kBlock);
  R.nrow = (n + kWave - 1) / kWave;
  const int nseg = nsteps > 0 ? (nsteps + ckpt - 1) / ckpt : 0;
  const int seg_len = std::min(ckpt, std::max(nsteps, 1));
  // checkpoints: the starts of all segments but the last, and the final state, which they replace
  const int nck = std::max(nseg, 1);
  R.P = grad_plan(n, L.scells, nck, seg_len, R.nb1, R.nbp, R.nrow);
  if (ctx->gbytes < R.P.bytes) {
    if (ctx->gmem) (void)hipFree(ctx->gmem);
    ctx->gmem = nullptr;
    ctx->gbytes = 0;
    if (hipMalloc((void **)&ctx->gmem, R.P.bytes) != hipSuccess) return MPSPH_E_NOMEM;
    ctx->gbytes = R.P.bytes;
  }
  R.g = ctx->gmem;
  const int64_t t0 = ctx->steps_done;
  EventHook *hk = ctx->hook.on ? &ctx->hook : nullptr;
  const bool coeff = n > 0 && dm.p.field == MPSPH_RBF_EXP && dm.p.n_rbf > 0;
  int rc = MPSPH_OK;
  double out[1 + kMaxRbf] = {0.0};
  if (hk) hk->begin("grad_forward");
  if (n == 0 && (rc = enqueue(ctx, nsteps, R.st, nullptr)) != MPSPH_OK) return rc;
  for (int sg = 0; n > 0 && sg < nseg; ++sg) {
    const int len = std::min(ckpt, nsteps - sg * ckpt);
    const bool again = sg < nseg - 1;   // recomputed for its record
    if (again) {
      if ((rc = save_state(R, sg, false)) != MPSPH_OK || (rc = enqueue(ctx, len, R.st, nullptr)) != MPSPH_OK) return rc;
    } else {
      if (sg == 0 && d_grad_pos)   // the start's ids
        HIP_OK(hipMemcpyAsync(R.checkpoint(0).id, R.state().id, (size_t)n * 4, hipMemcpyDeviceToDevice, R.st));
      if ((rc = record_segment<D>(R, len)) != MPSPH_OK) return rc;
    }
  }
  if (nseg > 1 && n > 0 && (rc = save_state(R, nseg - 1, true)) != MPSPH_OK) return rc;
  if (hk) hk->end();
  if (hk) hk->begin("grad_backward");
  if (n > 0) {
    if ((rc = loss_backward<D>(R, lam, seg_len - 1)) != MPSPH_OK) return rc;
    for (int sg = nseg - 1; sg >= 0; --sg) {
      const int len = std::min(ckpt, nsteps - sg * ckpt);
      const int64_t t = t0 + (int64_t)sg * ckpt;
      if (sg < nseg - 1 &&
          ((rc = restore_state(R, sg, t, false)) != MPSPH_OK || (rc = record_segment<D>(R, len)) != MPSPH_OK))
        return rc;
      for (int m = len - 1; m >= 0; --m)
        if ((rc = step_backward<D>(R, m, m == len - 1, t + m)) != MPSPH_OK) return rc;
    }
    if (coeff)
      adj_sum_coeff<<<dm.p.n_rbf, kCoeffSumThreads, 0, R.st>>>(R.at<double>(R.P.cpart), R.nrow, dm.p.n_rbf,
                                                              R.at<double>(R.P.out) + 1);
    if (d_grad_pos)
      adj_store_pos<D><<<R.nb1, kBlock, 0, R.st>>>(n, nseg > 0 ? R.checkpoint(0).id : R.state().id, R.at<float4>(R.P.xbar),
                                                   (float)dm.d.inv_cs, d_grad_pos);
    // back to the state after the last step
    if (nseg > 1 && (rc = restore_state(R, nseg - 1, t0 + nsteps, true)) != MPSPH_OK) return rc;
  }
  if (hk) hk->end();
  HIP_OK(hipGetLastError());
  if (n > 0)
    HIP_OK(hipMemcpyAsync(out, R.at<double>(R.P.out), (1 + (coeff ? dm.p.n_rbf : 0)) * 8, hipMemcpyDeviceToHost, R.st));
  HIP_OK(hipStreamSynchronize(R.st));
  ctx->steps_done = t0 + nsteps;
  if (loss_out) *loss_out = out[0];
  if (grad_coeff && dm.p.field == MPSPH_RBF_EXP)
    for (int m = 0; m < dm.p.n_rbf; ++m) grad_coeff[m] = out[1 + m];
  return MPSPH_OK;
}

}  // namespace

// Workspace of mpsph_create_static: one array per GPU, for callers that cannot allocate device
// memory.  Host code never uses the array's name as an address: the device address of each
// GPU's copy comes from hipGetSymbolAddress, taken once per device with that device current.
constexpr size_t kScratchBytes = size_t(64) << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) char scratch[kScratchBytes];

struct ScratchTable {
  std::mutex mu;
  char *ptr[kMaxDevices] = {};
  bool busy[kMaxDevices] = {};
};
ScratchTable &scratch_table() {
  static ScratchTable t;
  return t;
}

extern "C" {

const char *mpsph_strerror(int status) {
  if (status < 0 || status > MPSPH_E_SCRATCH) return "unknown status";
  return kErr[status];
}

int mpsph_field_scale(const mpsph_params *params, int64_t n, double *s0_out) {
  if (!valid_params(params) || n <= 0 || !s0_out) return MPSPH_E_INVALID;
  double I = field_integral_unit(params);
  if (!(I > 0) || !std::isfinite(I)) return MPSPH_E_INVALID;
  *s0_out = std::pow(I / (double)n, 1.0 / params->dim);
  return MPSPH_OK;
}

int mpsph_field_bounds(const mpsph_params *params, int64_t n, double *out) {
  if (!valid_params(params) || n <= 0 || !out) return MPSPH_E_INVALID;
  double s0 = params->s0;
  if (!(s0 > 0)) {
    const double I = field_integral_unit(params);
    if (!(I > 0) || !std::isfinite(I)) return MPSPH_E_INVALID;
    s0 = std::pow(I / (double)n, 1.0 / params->dim);
  }
  double smin, smax, lip;
  if (!spacing_bounds(params, s0, &smin, &smax, &lip)) return MPSPH_E_INVALID;
  out[0] = s0;
  out[1] = smin;
  out[2] = smax;
  out[3] = lip;
  return MPSPH_OK;
}

int mpsph_feature_budget(const mpsph_params *params, int64_t n, mpsph_features_t *out) {
  if (!valid_params(params) || n <= 0 || !out) return MPSPH_E_INVALID;
  if (params->geometry == MPSPH_LEVELSET) return MPSPH_E_UNSUPPORTED;
  const int d = params->dim;
  const double Iv = field_integral_unit(params);
  if (!(Iv > 0) || !std::isfinite(Iv)) return MPSPH_E_INVALID;
  const FeatureList f = feature_integrals(params);
  // n = sum_k c_k u^k with u = 1/s0: the volume term (k = dim) plus every feature's term
  double coef[4] = {0, 0, 0, 0};
  coef[d] = Iv;
  for (int i = 0; i < f.n; ++i) {
    if (!(f.I[i] > 0) || !std::isfinite(f.I[i])) return MPSPH_E_INVALID;
    coef[f.power[i]] += f.I[i];
  }
  const double target = (double)n - coef[0];
  if (!(target > 0)) return MPSPH_E_INVALID;
  // Newton from the volume-only root, which lies at or above the root: the polynomial is convex
  // and increasing for u > 0, so the iterates decrease monotonically onto it
  double u = std::pow(target / Iv, 1.0 / d);
  for (int it = 0; it < 200; ++it) {
    double g = -target, dg = 0.0;
    for (int k = 1; k <= d; ++k) {
      g += coef[k] * std::pow(u, k);
      dg += k * coef[k] * std::pow(u, k - 1);
    }
    const double du = g / dg;
    u -= du;
    if (std::fabs(du) <= 1e-15 * u) break;
  }
  if (!(u > 0) || !std::isfinite(u)) return MPSPH_E_INVALID;
  *out = mpsph_features_t{};
  out->s0 = 1.0 / u;
  out->mass_volume = Iv * std::pow(u, d);
  out->n_features = f.n;
  int64_t used = 0;
  for (int i = 0; i < f.n; ++i) {
    out->type[i] = f.type[i];
    out->mass[i] = f.I[i] * std::pow(u, f.power[i]);
    out->count[i] = f.power[i] == 0 ? 1 : (int64_t)std::llround(out->mass[i]);
    used += out->count[i];
  }
  out->n_volume = n - used;
  return out->n_volume >= 0 ? MPSPH_OK : MPSPH_E_INVALID;
}

size_t mpsph_batch_workspace_bytes(int32_t ndom, const mpsph_params *params, const int64_t *n) {
  std::vector<Domain> doms;
  Layout L;
  if (build_domains(ndom, params, n, &doms, &L) != MPSPH_OK) return 0;
  return L.bytes;
}

size_t mpsph_workspace_bytes(const mpsph_params *params, int64_t n) {
  return mpsph_batch_workspace_bytes(1, params, &n);
}

int mpsph_batch_create(int32_t ndom, const mpsph_params *params, const int64_t *n, void *d_workspace,
                       size_t workspace_bytes, void *hip_stream, mpsph_ctx **out) {
  if (!out) return MPSPH_E_INVALID;
  *out = nullptr;
  mpsph_ctx *ctx = new (std::nothrow) mpsph_ctx();
  if (!ctx) return MPSPH_E_NOMEM;
  int rc = build_domains(ndom, params, n, &ctx->dom, &ctx->L);
  if (rc) {
    delete ctx;
    return rc;
  }
  const Layout &L = ctx->L;
  ctx->stream = (hipStream_t)hip_stream;
  ctx->hook.stream = ctx->stream;
  {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) ==
                                                hipSuccess && cus > 0)
      ctx->cus = cus;
  }
  if (d_workspace) {
    if (workspace_bytes < L.bytes || ((uintptr_t)d_workspace & 255)) {
      delete ctx;
      return MPSPH_E_NOMEM;
    }
    ctx->ws = (char *)d_workspace;
  } else {
    if (hipMalloc((void **)&ctx->ws, L.bytes) != hipSuccess) {
      delete ctx;
      return MPSPH_E_NOMEM;
    }
    ctx->owns = true;
  }
  ctx->ws_cap = d_workspace ? workspace_bytes : L.bytes;
  if ((rc = setup_device(ctx)) != MPSPH_OK) {
    mpsph_destroy(ctx);
    return rc;
  }
  *out = ctx;
  return MPSPH_OK;
}

int mpsph_create(const mpsph_params *params, int64_t n, void *d_workspace, size_t workspace_bytes, void *hip_stream,
                 mpsph_ctx **out) {
  return mpsph_batch_create(1, params, &n, d_workspace, workspace_bytes, hip_stream, out);
}

int mpsph_create_static(const mpsph_params *params, int64_t n, void *hip_stream, mpsph_ctx **out) {
  if (!out) return MPSPH_E_INVALID;
  *out = nullptr;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return MPSPH_E_DEVICE;
  if (dev < 0 || dev >= kMaxDevices) return MPSPH_E_UNSUPPORTED;
  ScratchTable &t = scratch_table();
  std::lock_guard<std::mutex> lock(t.mu);
  if (!t.ptr[dev]) {
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MPSPH_E_DEVICE;
    t.ptr[dev] = static_cast<char *>(p);
  }
  if (t.busy[dev]) return MPSPH_E_STATE;
  const size_t need = mpsph_workspace_bytes(params, n);
  if (need == 0) return MPSPH_E_INVALID;
  if (need > kScratchBytes) return MPSPH_E_SCRATCH;
  // the workspace is zeroed by the set-up of the context, so nothing of an earlier context that
  // used the array survives
  const int rc = mpsph_batch_create(1, params, &n, t.ptr[dev], kScratchBytes, hip_stream, out);
  if (rc != MPSPH_OK) return rc;
  (*out)->static_dev = dev;
  t.busy[dev] = true;
  return MPSPH_OK;
}

int mpsph_configure(mpsph_ctx *ctx, int32_t cell_log2, int32_t lanes) {
  if (!ctx || (lanes != 2 && lanes != 4 && lanes != 8) || cell_log2 == 0 || cell_log2 < -1 || cell_log2 > 12)
    return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  for (const Domain &dm : ctx->dom)
    if (cell_log2 > 0 && dm.p.dim * cell_log2 > 24) return MPSPH_E_UNSUPPORTED;
  const std::vector<Domain> base = ctx->dom;
  return reconfigure(ctx, base, 0, cell_log2, lanes);
}

int mpsph_set_pair_variant(mpsph_ctx *ctx, int32_t variant) {
  if (!ctx || variant < MPSPH_PAIRS_DEFAULT || variant > MPSPH_PAIRS_TILE) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  if (variant != ctx->variant) drop_graph(ctx);   // a captured graph holds the other kernels
  ctx->variant = variant;
  return MPSPH_OK;
}

int mpsph_autotune(mpsph_ctx *ctx, const float *d_pos, const int32_t *d_colour, const int32_t *d_type,
                   int32_t warm_steps, int32_t probe_steps, int32_t *cell_log2_out, int32_t *lanes_out) {
  if (!ctx || probe_steps < 1 || probe_steps > 1000 || warm_steps < 0 || warm_steps > 10000) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  bool rule = false;
  for (const Domain &dm : ctx->dom) rule |= dm.p.cell_log2 < 0;
  const std::vector<Domain> base = ctx->dom;
  struct Pick {
    int kd, lanes;
    float ms;
  } best{0, MPSPH_LANES, INFINITY};
  // applies a configuration: plan, workspace, device tables, and the caller's state loaded
  auto apply = [&](int kd, int lanes) -> int {
    int rc = reconfigure(ctx, base, kd, -1, lanes);
    if (rc) return rc;
    return mpsph_load(ctx, d_pos, d_colour, d_type);
  };
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return fail(ctx, MPSPH_E_DEVICE);
  int rc = MPSPH_OK;
  const int lanes_c[3] = {2, 4, 8};
  for (int kd = rule ? -1 : 0; kd <= (rule ? 1 : 0) && rc == MPSPH_OK; ++kd) {
    for (int li = 0; li < 3; ++li) {
      int a = apply(kd, lanes_c[li]);
      if (a == MPSPH_E_NOMEM || a == MPSPH_E_UNSUPPORTED) continue;  // does not fit: not a candidate
      if (a != MPSPH_OK) {
        rc = a;
        break;
      }
      // untimed steps first: the first steps after a load (state still in load order, dense
      // initial neighbourhoods) are not representative of a run
      if ((a = enqueue(ctx, std::max(warm_steps, 1), ctx->stream, nullptr)) != MPSPH_OK) {
        rc = a;
        break;
      }
      if (hipEventRecord(e0, ctx->stream) != hipSuccess || enqueue(ctx, probe_steps, ctx->stream, nullptr) ||
          hipEventRecord(e1, ctx->stream) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
        rc = fail(ctx, MPSPH_E_DEVICE);
        break;
      }
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      if (ms < best.ms) best = Pick{kd, lanes_c[li], ms};
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc == MPSPH_OK) rc = apply(best.kd, best.lanes);
  if (rc != MPSPH_OK) return rc;
  if (cell_log2_out) *cell_log2_out = ctx->dom[ctx->L.internal[0]].d.k;
  if (lanes_out) *lanes_out = ctx->L.lanes;
  return MPSPH_OK;
}

int mpsph_load(mpsph_ctx *ctx, const float *d_pos, const int32_t *d_colour, const int32_t *d_type) {
  if (!ctx) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  const int n = (int)L.n;
  if (n > 0 && (!d_pos || !d_colour)) return MPSPH_E_INVALID;
  HIP_OK(hipMemsetAsync(ctx->ws + L.metrics, 0, L.dtslots - L.metrics, ctx->stream));
  for (const Group &gr : L.grp) {
    if (gr.i1 <= gr.i0) continue;
    auto kern = gr.D == 2 ? load_kernel<2> : load_kernel<3>;
    kern<<<(gr.i1 - gr.i0 + kBlock - 1) / kBlock, kBlock, 0, ctx->stream>>>(
        ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, gr.i0, gr.i1, d_pos, d_colour, d_type, ctx->at<uint32_t>(L.s_key),
        ctx->at<float4>(L.s_off), ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id), ctx->at<uint32_t>(L.s_cell), ctx->at<uint32_t>(L.counts), ctx->at<int>(L.bad));
    HIP_OK(hipGetLastError());
  }
  int bad = 0;
  HIP_OK(hipMemcpyAsync(&bad, ctx->at<int>(L.bad), 4, hipMemcpyDeviceToHost, ctx->stream));
  HIP_OK(hipStreamSynchronize(ctx->stream));
  ctx->steps_done = 0;
  if (bad) {
    ctx->loaded = false;
    return MPSPH_E_INVALID;
  }
  ctx->loaded = true;
  return MPSPH_OK;
}

int mpsph_step(mpsph_ctx *ctx, int32_t nsteps) {
  if (!ctx || nsteps < 0) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded) return MPSPH_E_STATE;
  int rc = enqueue(ctx, nsteps, ctx->stream, ctx->hook.on ? &ctx->hook : nullptr);
  if (rc == MPSPH_OK) ctx->steps_done += nsteps;
  return rc;
}

int mpsph_step_graph(mpsph_ctx *ctx, int32_t nsteps) {
  if (!ctx || nsteps < 0) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded) return MPSPH_E_STATE;
  if (nsteps == 0) return MPSPH_OK;
  if (!ctx->graph_exec || ctx->graph_steps != nsteps) {
    drop_graph(ctx);
    if (!ctx->cap_stream) HIP_OK(hipStreamCreateWithFlags(&ctx->cap_stream, hipStreamNonBlocking));
    HIP_OK(hipStreamBeginCapture(ctx->cap_stream, hipStreamCaptureModeThreadLocal));
    const int rc = enqueue(ctx, nsteps, ctx->cap_stream, nullptr);
    hipGraph_t graph = nullptr;
    const hipError_t ec = hipStreamEndCapture(ctx->cap_stream, &graph);
    if (rc != MPSPH_OK || ec != hipSuccess || !graph) {
      if (graph) (void)hipGraphDestroy(graph);
      return fail(ctx, MPSPH_E_DEVICE);
    }
    const hipError_t ei = hipGraphInstantiate(&ctx->graph_exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (ei != hipSuccess) {
      ctx->graph_exec = nullptr;
      return fail(ctx, MPSPH_E_DEVICE);
    }
    ctx->graph_steps = nsteps;
  }
  EventHook *hk = ctx->hook.on ? &ctx->hook : nullptr;
  if (hk) hk->begin("step_graph");
  HIP_OK(hipGraphLaunch(ctx->graph_exec, ctx->stream));
  if (hk) hk->end();
  ctx->steps_done += nsteps;
  return MPSPH_OK;
}

int mpsph_domain_count(mpsph_ctx *ctx, int32_t *ndom, int64_t *n_total) {
  if (!ctx) return MPSPH_E_INVALID;
  if (ndom) *ndom = ctx->L.ndom;
  if (n_total) *n_total = ctx->L.n;
  return MPSPH_OK;
}

int mpsph_domain_metrics(mpsph_ctx *ctx, int32_t first, int32_t count, mpsph_metrics_t *out) {
  if (!ctx || !out || first < 0 || count < 1 || first + count > ctx->L.ndom) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  std::vector<double> m((size_t)ctx->L.ndom * 32);
  HIP_OK(hipMemcpyAsync(m.data(), ctx->at<double>(ctx->L.metrics), m.size() * 8, hipMemcpyDeviceToHost,
                        ctx->stream));
  HIP_OK(hipStreamSynchronize(ctx->stream));
  bool nonfinite = false;
  for (int d = 0; d < count; ++d) {
    const int k = ctx->L.internal[first + d];
    fill_metrics(ctx, k, m.data() + (size_t)k * 32, &out[d]);
    nonfinite |= out[d].nonfinite != 0;
  }
  return nonfinite ? MPSPH_E_NONFINITE : MPSPH_OK;
}

int mpsph_metrics(mpsph_ctx *ctx, mpsph_metrics_t *out) { return mpsph_domain_metrics(ctx, 0, 1, out); }

int mpsph_store(mpsph_ctx *ctx, float *d_pos, int32_t *d_type) {
  if (!ctx) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  for (const Group &gr : L.grp) {
    if (gr.i1 <= gr.i0) continue;
    auto kern = gr.D == 2 ? store_kernel<2> : store_kernel<3>;
    kern<<<(gr.i1 - gr.i0 + kBlock - 1) / kBlock, kBlock, 0, ctx->stream>>>(
        ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, gr.i0, gr.i1, ctx->at<uint32_t>(L.s_key), ctx->at<float4>(L.s_off),
        ctx->at<uint32_t>(L.s_ct), ctx->at<uint32_t>(L.s_id), d_pos, d_type);
    HIP_OK(hipGetLastError());
  }
  HIP_OK(hipStreamSynchronize(ctx->stream));
  return MPSPH_OK;
}

int mpsph_debug_fields(mpsph_ctx *ctx, int32_t which, float *d_out) {
  if (!ctx || !d_out || which < 0 || which > MPSPH_F_X0) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded || ctx->steps_done == 0) return MPSPH_E_STATE;
  const bool needs_debug = which == MPSPH_F_RHO || which == MPSPH_F_A_ABS || which == MPSPH_F_AT ||
                           which == MPSPH_F_V || which == MPSPH_F_DR || which == MPSPH_F_NN;
  if (needs_debug && !ctx->dom[0].p.debug) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  const float4 *vec = ctx->at<float4>(L.acc);
  const float *sc = ctx->at<float>(L.rho);
  const float *vscale = nullptr;
  if (which == MPSPH_F_NN) sc = ctx->at<float>(L.nn);
  if (which == MPSPH_F_A_ABS) sc = ctx->at<float>(L.aabs);
  if (which == MPSPH_F_AT) vec = ctx->at<float4>(L.at);
  if (which == MPSPH_F_V) vec = ctx->at<float4>(L.v);
  if (which == MPSPH_F_DR) vec = ctx->at<float4>(L.v);
  if (which == MPSPH_F_VT || which == MPSPH_F_DR) {
    // by the first time step of the exported step itself (the metrics may be another step's after a gradient):
    // v~ = a dt1 / 2 (Eq. 26 after the velocity reset; fixed particles carry a = 0), and the drift is v dt2, the
    // product the integrator forms (Eq. 28)
    std::vector<float> vs(L.ndom), slots((size_t)L.ndom * kDtWords);
    HIP_OK(hipMemcpyAsync(slots.data(), ctx->at<float>(L.dtslots), slots.size() * 4, hipMemcpyDeviceToHost, ctx->stream));
    HIP_OK(hipStreamSynchronize(ctx->stream));
    for (int d = 0; d < L.ndom; ++d) {
      float d1 = INFINITY;
      for (int q = 0; q < kDtSlots; ++q) d1 = std::min(d1, slots[(size_t)d * kDtWords + q * kDtStride]);
      d1 = std::isfinite(d1) ? d1 : 0.f;
      vs[d] = d1 * (which == MPSPH_F_VT ? 0.5f : (float)dt2_factor(&ctx->dom[d].p));
    }
    HIP_OK(hipMemcpyAsync(ctx->at<float>(L.vscale), vs.data(), vs.size() * 4, hipMemcpyHostToDevice, ctx->stream));
    vscale = ctx->at<float>(L.vscale);
  }
  for (const Group &gr : L.grp) {
    if (gr.i1 <= gr.i0) continue;
    auto kern = gr.D == 2 ? dump_kernel<2> : dump_kernel<3>;
    kern<<<(gr.i1 - gr.i0 + kBlock - 1) / kBlock, kBlock, 0, ctx->stream>>>(
        ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, gr.i0, gr.i1, which, ctx->at<uint32_t>(L.w_key),
        ctx->at<float4>(L.w_pos), ctx->at<uint32_t>(L.w_id), sc, vec, vscale ? vscale + gr.d0 : nullptr, d_out);
    HIP_OK(hipGetLastError());
  }
  HIP_OK(hipStreamSynchronize(ctx->stream));
  return MPSPH_OK;
}

int mpsph_debug_cells(mpsph_ctx *ctx, uint32_t *d_key, uint32_t *d_cell_start, int64_t *ncells, int32_t *cell_log2) {
  if (!ctx) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  if (ncells) *ncells = ctx->L.ncells;
  if (cell_log2) *cell_log2 = ctx->dom[ctx->L.internal[0]].d.k;
  if ((d_key || d_cell_start) && (!ctx->loaded || ctx->steps_done == 0)) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  const int n = (int)L.n;
  try {
    std::vector<uint32_t> k(n), out;
    if (n > 0 && (d_key || d_cell_start))
      HIP_OK(hipMemcpyAsync(k.data(), ctx->at<uint32_t>(L.w_key), 4 * (size_t)n, hipMemcpyDeviceToHost, ctx->stream));
    if (d_key && n > 0) {
      // keys of the last step's start in load order: scatter w_key by w_id
      std::vector<uint32_t> id(n);
      out.resize(n);
      HIP_OK(hipMemcpyAsync(id.data(), ctx->at<uint32_t>(L.w_id), 4 * (size_t)n, hipMemcpyDeviceToHost, ctx->stream));
      HIP_OK(hipStreamSynchronize(ctx->stream));
      for (int i = 0; i < n; ++i) out[id[i]] = k[i];
      HIP_OK(hipMemcpyAsync(d_key, out.data(), 4 * (size_t)n, hipMemcpyHostToDevice, ctx->stream));
    }
    HIP_OK(hipStreamSynchronize(ctx->stream));
    if (d_cell_start) {
      // lower bound of every cell in the sorted keys, from the counts (the search order is another)
      out.assign((size_t)L.ncells + 1, 0u);
      for (int i = 0; i < n; ++i) ++out[(size_t)k[i] + 1];
      for (size_t c = 0; c < (size_t)L.ncells; ++c) out[c + 1] += out[c];
      HIP_OK(hipMemcpyAsync(d_cell_start, out.data(), 4 * out.size(), hipMemcpyHostToDevice, ctx->stream));
      HIP_OK(hipStreamSynchronize(ctx->stream));
    }
  } catch (const std::bad_alloc &) {
    return MPSPH_E_NOMEM;
  }
  return MPSPH_OK;
}

int mpsph_debug_search(mpsph_ctx *ctx, uint32_t *d_start, uint32_t *d_order, int64_t *ncells, int32_t *rows_log2,
                       int32_t *xsub_log2) {
  if (!ctx) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  const Derived &d = ctx->dom[L.internal[0]].d;
  if (ncells) *ncells = L.scells;
  if (rows_log2) *rows_log2 = d.rb;
  if (xsub_log2) *xsub_log2 = d.xb;
  if ((d_start || d_order) && (!ctx->loaded || ctx->steps_done == 0)) return MPSPH_E_STATE;
  if (d_start)
    HIP_OK(hipMemcpyAsync(d_start, ctx->at<uint32_t>(L.cstart), 4 * ((size_t)L.scells + 1), hipMemcpyDeviceToDevice, ctx->stream));
  if (d_order)
    HIP_OK(hipMemcpyAsync(d_order, ctx->at<uint32_t>(L.w_id), 4 * (size_t)L.n, hipMemcpyDeviceToDevice, ctx->stream));
  HIP_OK(hipStreamSynchronize(ctx->stream));
  return MPSPH_OK;
}

int mpsph_debug_pairs(mpsph_ctx *ctx, int64_t cap, uint32_t *d_i, uint32_t *d_j, int64_t *count) {
  if (!ctx || cap < 0 || !count || (cap > 0 && (!d_i || !d_j))) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded || ctx->steps_done == 0) return MPSPH_E_STATE;
  const Layout &L = ctx->L;
  unsigned long long *cnt = ctx->at<unsigned long long>(L.paircount);
  HIP_OK(hipMemsetAsync(cnt, 0, 8, ctx->stream));
  for (const Group &gr : L.grp) {
    if (gr.i1 <= gr.i0) continue;
    for (const bool wide : {false, true}) {
      if (gr.nwide == (wide ? 0 : gr.nd)) continue;
      auto kern = gr.D == 2 ? (wide ? (gr.periodic ? dump_pairs<2, true, true> : dump_pairs<2, false, true>)
                                    : (gr.periodic ? dump_pairs<2, true, false> : dump_pairs<2, false, false>))
                            : (wide ? (gr.periodic ? dump_pairs<3, true, true> : dump_pairs<3, false, true>)
                                    : (gr.periodic ? dump_pairs<3, true, false> : dump_pairs<3, false, false>));
      // two lanes per particle
      kern<<<(int)((2 * (int64_t)(gr.i1 - gr.i0) + kBlock - 1) / kBlock), kBlock, 0, ctx->stream>>>(
          ctx->at<DomDev>(L.doms) + gr.d0, gr.nd, gr.i0, gr.i1, ctx->at<uint32_t>(L.w_key), ctx->at<float4>(L.w_fix),
          ctx->at<uint32_t>(L.w_id), ctx->at<uint32_t>(L.cstart), (unsigned long long)cap, d_i, d_j, cnt);
      HIP_OK(hipGetLastError());
    }
  }
  unsigned long long total = 0;
  HIP_OK(hipMemcpyAsync(&total, cnt, 8, hipMemcpyDeviceToHost, ctx->stream));
  HIP_OK(hipStreamSynchronize(ctx->stream));
  *count = (int64_t)total;
  return MPSPH_OK;
}

int mpsph_set_field_coeff(mpsph_ctx *ctx, int32_t domain, const double *coeff) {
  if (!ctx || !coeff || domain < 0 || domain >= ctx->L.ndom) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  const int k = ctx->L.internal[domain];
  Domain &dm = ctx->dom[k];
  if (dm.p.field != MPSPH_RBF_EXP) return MPSPH_E_INVALID;
  for (int m = 0; m < dm.p.n_rbf; ++m)
    if (!std::isfinite(coeff[m])) return MPSPH_E_INVALID;
  std::vector<double> saved = dm.rbf_coeff;
  dm.rbf_coeff.assign(coeff, coeff + dm.p.n_rbf);
  dm.p.rbf_coeff = dm.rbf_coeff.data();
  // bounds of the field, search radius and h_max for the new coefficients on the same grid
  mpsph_params q = dm.p;
  q.cell_log2 = dm.d.k;
  Derived nd;
  double bounds[3];
  const bool sampled = q.n_rbf > 0;
  if (sampled && !rbf_bounds_device(ctx, &q, dm.s0, bounds)) return fail(ctx, MPSPH_E_DEVICE);
  if (derive(&q, dm.n, dm.s0, &nd, sampled ? bounds : nullptr) != MPSPH_OK) {
    dm.rbf_coeff = saved;
    dm.p.rbf_coeff = dm.rbf_coeff.data();
    return MPSPH_E_UNSUPPORTED;
  }
  nd.rb = dm.d.rb;   // the search grid stays too, and the fixed-point coordinates of the last step
  nd.xb = dm.d.xb;
  nd.fb = dm.d.fb;
  nd.wide = wide_field(&q, nd);
  if (nd.wide != dm.d.wide) {
    ctx->L.grp[dm.p.dim - 2].nwide += nd.wide ? 1 : -1;
    drop_graph(ctx);   // it holds the other passes
  }
  dm.d = nd;
  const Layout &L = ctx->L;
  const DomDev dd = domain_device(dm, ctx->at<int>(L.rbf_c), ctx->at<float>(L.rbf_o), ctx->at<float>(L.rbf_k),
                                  ctx->at<float>(L.gphi), ctx->at<float>(L.gs));
  std::vector<float> rk(std::max(dm.p.n_rbf, 1));
  for (int m = 0; m < dm.p.n_rbf; ++m) rk[m] = (float)coeff[m];
  HIP_OK(hipStreamSynchronize(ctx->stream));
  HIP_OK(hipMemcpy(ctx->at<DomDev>(L.doms) + k, &dd, sizeof(DomDev), hipMemcpyHostToDevice));
  if (dm.p.n_rbf > 0)
    HIP_OK(hipMemcpy(ctx->at<float>(L.rbf_k) + dm.rbf0, rk.data(), (size_t)dm.p.n_rbf * 4, hipMemcpyHostToDevice));
  return MPSPH_OK;
}

int mpsph_grad(mpsph_ctx *ctx, int32_t nsteps, int32_t ckpt_every, double lambda, double *loss_out,
               double *grad_coeff_out, float *d_grad_pos) {
  if (!ctx || nsteps < 0 || ckpt_every < 1 || !std::isfinite(lambda)) return MPSPH_E_INVALID;
  if (ctx->poisoned || !ctx->loaded) return MPSPH_E_STATE;
  // the gradient driver allocates its checkpoint memory; a static-scratch context must not
  if (ctx->static_dev >= 0) return MPSPH_E_UNSUPPORTED;
  const Domain &dm = ctx->dom[0];
  if (ctx->L.ndom != 1 || dm.p.geometry != MPSPH_BOX || dm.p.t0 == -2 || dm.p.seeded ||
      (dm.p.field != MPSPH_RBF_EXP && dm.p.field != MPSPH_UNIFORM))
    return MPSPH_E_UNSUPPORTED;
  return dm.p.dim == 2 ? grad_run<2>(ctx, nsteps, ckpt_every, lambda, loss_out, grad_coeff_out, d_grad_pos)
                       : grad_run<3>(ctx, nsteps, ckpt_every, lambda, loss_out, grad_coeff_out, d_grad_pos);
}

int mpsph_profile(mpsph_ctx *ctx, int32_t enable) {
  if (!ctx || enable < 0 || enable > 2) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  ctx->hook.collect();
  if (enable) ctx->hook.reset();
  ctx->hook.on = enable != 0;
  ctx->hook.pairs_only = enable == 2;
  return MPSPH_OK;
}

int mpsph_profile_read(mpsph_ctx *ctx, int32_t cap, const char **names, int64_t *launches, double *ms, int32_t *count) {
  if (!ctx || cap < 0 || !count) return MPSPH_E_INVALID;
  if (ctx->poisoned) return MPSPH_E_STATE;
  ctx->hook.collect();
  int m = (int)ctx->hook.names.size();
  *count = m;
  for (int i = 0; i < m && i < cap; ++i) {
    if (names) names[i] = ctx->hook.names[i].c_str();
    if (launches) launches[i] = ctx->hook.launches[i];
    if (ms) ms[i] = ctx->hook.ms[i];
  }
  return MPSPH_OK;
}

void mpsph_destroy(mpsph_ctx *ctx) {
  if (!ctx) return;
  (void)hipStreamSynchronize(ctx->stream);
  drop_graph(ctx);
  if (ctx->cap_stream) (void)hipStreamDestroy(ctx->cap_stream);
  if (ctx->owns && ctx->ws) (void)hipFree(ctx->ws);
  if (ctx->gmem) (void)hipFree(ctx->gmem);
  if (ctx->static_dev >= 0) {
    ScratchTable &t = scratch_table();
    std::lock_guard<std::mutex> lock(t.mu);
    t.busy[ctx->static_dev] = false;
  }
  delete ctx;
}

}  // extern "C"
