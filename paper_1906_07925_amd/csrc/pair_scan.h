// Neighbour candidate scans and lane-group helpers of the pair passes, their adjoints and the
// pair dump (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mpsph_device.h"

namespace mpsph {

// Neighbour candidates
//
// Particle i's candidates are the particles of every x-run of search rows (fixed y, z) that meets the
// ball of radius rs around it, the run taken at x sub-cell resolution; in the search order (x
// fastest) each run is one contiguous range of the sorted arrays.  A group of L lanes works on
// one particle (scan_group_table below).
// ------------------------------------------------------------------------------------------
// Lanes per particle of the pair kernels of a context that was never configured (mpsph_configure and
// mpsph_autotune choose 2, 4 or 8), and of the adjoint's pair kernels.  Measured per step at 4 / 8 lanes:
// 3D 8192 particles 77 / 70 us, 20,011 87 / 74, 100,003 157 / 142, 10^6 775 / 695, 2M 2316 / 2184; 2D 4096
// 47 / 46, 262,144 125 / 137.  A 2D particle has 20 neighbours: at 8 lanes its slots are three rounds and
// the row table and the epilogue of twice the blocks cost more than the shorter loops save.  (16 lanes:
// 8192 particles 65, 100,003 151, 10^6 835 us.)
#ifndef MPSPH_LANES
#define MPSPH_LANES 4
#endif
#ifndef MPSPH_LANES_3D
#define MPSPH_LANES_3D 8
#endif
#ifndef MPSPH_ADJ_LANES
#define MPSPH_ADJ_LANES 8
#endif
// The adjoint's pair kernels of small 3D gradients (kAdjSmall).
#ifndef MPSPH_ADJ_LANES_SMALL
#define MPSPH_ADJ_LANES_SMALL 16
#endif

// Separation of two particles from their fixed-point coordinates, in units of 2^-fb cells: the integer
// difference is exact, in a periodic box of the minimum image (the coordinates' wrap divides the
// period), and is rounded once, by the conversion.  Two VALU operations per axis; with (cell, offset)
// pairs x took four (ten with a minimum image), and y and z needed their row's offsets from the table.
// Per step, with rows of the same width: 2M-particle graded cube 2458 -> 2174 us (viscous pass 1339 ->
// 1068, whose flags load went with the x cell in it), periodic 37^3 box 436 -> 110 us.
struct FixedPos {
  int x, y, z;
};
__device__ __forceinline__ FixedPos fixed_of(const float4 &p) {
  return FixedPos{(int)__float_as_uint(p.x), (int)__float_as_uint(p.y), (int)__float_as_uint(p.z)};
}
__device__ __forceinline__ float fixed_diff(int a, float b) { return (float)(int)((uint32_t)a - __float_as_uint(b)); }

// What the scan needs of the group's particle: x cell and offset, search row and offset in rows.
struct OwnRow {
  int cx, ry, rz;
  float ox, oy, oz;
};
// c: cells of the particle (from its key), p: its fixed-point coordinates.
__device__ __forceinline__ void row_and_offset(int c, int fix, const GridDev &g, int &r, float &o) {
  const float f = (float)((uint32_t)fix & ((1u << g.fb) - 1u)) * g.funit;   // offset in the cell
  if (g.rb >= 0) {
    r = c >> g.rb;
    o = ((float)(c & ((1 << g.rb) - 1)) + f) * g.rowinv;
  } else {
    const float t = f * g.rowinv;
    const int i = (int)t;
    r = (c << -g.rb) + i;
    o = t - (float)i;
  }
}
template <int D>
__device__ __forceinline__ OwnRow own_row(const int *c, const FixedPos &p, const GridDev &g) {
  OwnRow o;
  o.cx = c[0];
  o.ox = (float)((uint32_t)p.x & ((1u << g.fb) - 1u)) * g.funit;
  row_and_offset(c[1], p.y, g, o.ry, o.oy);
  o.rz = 0;
  o.oz = 0.f;
  if constexpr (D == 3) row_and_offset(c[2], p.z, g, o.rz, o.oz);
  return o;
}

// A particle's position and its neighbours' as the pair loops take separations from them: in units of
// `unit` cells, the same on every axis.
// Narrow domains (every separation below 2^(31 - fb) cells) take the difference of the fixed-point
// coordinates.  In wide ones (GridDev::wide) particles may be further apart, and that difference is the
// separation but for a multiple of the coordinates' range: the neighbour's key, loaded as well, has the
// cells that tell which.  Separations inside the range come out the same bit for bit.
// PER: the launch may hold periodic boxes.
template <int D, bool PER, bool WIDE>
struct PairPos {
  FixedPos x;
  OwnRow row;
  float h, unit;
  BufRes rp;
  struct Nb {
    float4 p;
  };
  // Of particle i and the sorted arrays of its context.
  __device__ __forceinline__ PairPos(const GridDev &g, uint32_t cellbase, int i, const uint32_t *__restrict__ wkey,
                                     const float4 *__restrict__ wfix) {
    int c[3];
    unpack_key<D>(wkey[i] - cellbase, g, c);
    const float4 p = wfix[i];
    x = fixed_of(p);
    row = own_row<D>(c, x, g);
    h = p.w;
    unit = g.funit;
    rp = buf_res(wfix, 16, (uint32_t)g.n);
  }
  __device__ __forceinline__ Nb fetch(uint32_t j) const { return Nb{buf_f4(rp, j)}; }
  // dz only in 3D
  __device__ __forceinline__ void sep(const Nb &nb, float &dx, float &dy, float &dz) const {
    dx = fixed_diff(x.x, nb.p.x);
    dy = fixed_diff(x.y, nb.p.y);
    if constexpr (D == 3) dz = fixed_diff(x.z, nb.p.z);
  }
};
template <int D, bool PER>
struct PairPos<D, PER, true> : PairPos<D, PER, false> {
  using Narrow = PairPos<D, PER, false>;
  int c[3];
  const GridDev &g;
  uint32_t cellbase;
  BufRes rk;
  struct Nb {
    float4 p;
    uint32_t key;
  };
  __device__ __forceinline__ PairPos(const GridDev &gr, uint32_t cb, int i, const uint32_t *__restrict__ wkey,
                                     const float4 *__restrict__ wfix)
      : Narrow(gr, cb, i, wkey, wfix), g(gr), cellbase(cb) {
    unpack_key<D>(wkey[i] - cb, g, c);
    rk = buf_res(wkey, 4, (uint32_t)g.n);
  }
  __device__ __forceinline__ Nb fetch(uint32_t j) const { return Nb{buf_f4(Narrow::rp, j), buf_u32(rk, j)}; }
  __device__ __forceinline__ float axis(int ci, int cj, float t) const {
    constexpr float kRange = 4294967296.f;   // of the coordinates, in their units
    const float cell = (float)(1u << g.fb), P = (float)(g.gmax + 1) * cell;
    int dc = ci - cj;
    if (PER && g.geometry == 0) {            // the cells' minimum image, at most one cell from the particles'
      const int p = g.gmax + 1;
      dc = dc >= p / 2 ? dc - p : (dc < -(p / 2) ? dc + p : dc);
    }
    float d = fmaf(rintf(((float)dc * cell - t) * (1.f / kRange)), kRange, t);
    if (PER && g.geometry == 0) d = d > 0.5f * P ? d - P : (d < -0.5f * P ? d + P : d);
    return d;
  }
  __device__ __forceinline__ void sep(const Nb &nb, float &dx, float &dy, float &dz) const {
    int cj[3];
    unpack_key<D>(nb.key - cellbase, g, cj);
    dx = axis(c[0], cj[0], fixed_diff(Narrow::x.x, nb.p.x));
    dy = axis(c[1], cj[1], fixed_diff(Narrow::x.y, nb.p.y));
    if constexpr (D == 3) dz = axis(c[2], cj[2], fixed_diff(Narrow::x.z, nb.p.z));
  }
};

// Value of lane l - o (o < 16) within the lane's row of 16 lanes, through a DPP row shift (no
// LDS round trip and no lane arithmetic); lanes l < o of the row get 0.  Used for prefix sums
// inside groups of at most 16 lanes, where the lanes that would read across the group's start
// discard the value.
__device__ __forceinline__ uint32_t lane_up(uint32_t x, int o) {
  switch (o) {   // the shift is an immediate of the instruction
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, true);
    case 4: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, true);
    default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, true);
  }
}
// The value of the group's last lane (L lanes, L <= 16), in every lane of the group, through
// ds_swizzle in its bit-mask mode: source lane = (lane & ~(L - 1)) | (L - 1) within 32 lanes.
template <int L>
__device__ __forceinline__ uint32_t group_last(uint32_t x) {
  static_assert(L >= 2 && L <= 16 && (L & (L - 1)) == 0, "groups of 2 to 16 lanes");
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (0x1F & ~(L - 1)) | ((L - 1) << 5));
}

// Rows per chunk of the LDS row table at 4 lanes per particle (scaled with the lanes, so that
// the table of a 256-thread block stays below 19 KB and 8 blocks fit a CU's LDS).
#ifndef MPSPH_ROW_TABLE
#define MPSPH_ROW_TABLE 36
#endif
template <int L>
constexpr int row_table_rows() {
  return MPSPH_ROW_TABLE * L / 4 < L + 2 ? L + 2 : MPSPH_ROW_TABLE * L / 4;
}
// Entries between two rows of one group's column (one more than the groups of a block, so that
// the columns of a wave's groups start in different banks).
template <int L>
constexpr int row_table_stride() {
  return kBlock / L + 1;
}

// Candidate scan with a row table in LDS (the pair passes, their adjoints and the pair dump).
//
// The group's L lanes take L rows at a time (each reads its row's range from the cell table)
// and lay out the non-empty ones in a table in LDS: base index, end of the run in the flattened
// slot order of the particle's candidates.  Then the group visits the slots L at a
// time, lane l taking every L-th one and advancing through the table as its slot index passes
// the end of a row.  A lane's loop ends with the slots of its own group (no wave-wide rounds of
// rows).  A table holds at most C - 1 rows and an end marker; a particle with more non-empty
// rows is scanned in several chunks.  With CUT the particle's own slot is cut out of its row
// (the row becomes the runs before and after it), so the particle itself is never a slot.
// The end marker (end of run 2^32 - 1) stops a lane's walk through the table when it looks one
// round ahead past the chunk's slots.
// In a periodic box (PER) a row whose run crosses the end of the x axis is taken as two runs, so a
// particle near that end has its rows twice, the second time for the part beyond it.
// tab: the group's column of the table, entry e at tab[e * stride]; C > L + 1.
// body(j) is called for every slot.  The return value is the group's candidate count (the particle
// itself excluded), the same in every lane of the group.
// The row's base index goes through remap(ry, rz, a) (a: the global index of the row's first
// candidate) before it enters the table, so that the slots can index a staged copy of the
// neighbours; self is the particle's own index in that numbering.
// A body may also come in two parts, fetch(j) -> payload (the slot's neighbour loads) and
// use(payload) (its arithmetic): the scan then issues the loads of a lane's next slot round before
// the arithmetic of the current one, so that their latency overlaps it.  A fetch past the chunk's end
// gets an index that may lie outside the arrays: bounds-checked loads, and no use() follows.
struct IdentityRemap {
  __device__ __forceinline__ uint32_t operator()(int, int, uint32_t a) const { return a; }
};
template <typename FetchF, typename UseF>
struct SplitBody {
  FetchF fetch;
  UseF use;
};
// The two-part body when PIPE, else one body that loads and computes in turn (fewer registers
// live across the loop: the kernels that could not hold a second round's loads in 64 registers
// without spilling take it).
template <bool PIPE, typename FetchF, typename UseF>
__device__ __forceinline__ auto pair_body(FetchF fetch, UseF use) {
  if constexpr (PIPE)
    return SplitBody<FetchF, UseF>{fetch, use};
  else
    return [=](uint32_t j) { use(fetch(j)); };
}
template <typename T>
struct IsSplitBody {
  static constexpr bool value = false;
};
template <typename F, typename U>
struct IsSplitBody<SplitBody<F, U>> {
  static constexpr bool value = true;
};
template <int D, int L, int C, bool PER = false, bool CUT = true, typename BodyF, typename RemapF = IdentityRemap>
__device__ __forceinline__ uint32_t scan_group_table(uint32_t self, int sub, uint2 *tab, int stride, const OwnRow &own,
                                                     float rs, const GridDev &g, uint32_t sbase,
                                                     const uint32_t *__restrict__ cstart, BodyF &&body,
                                                     RemapF remap = RemapF()) {
  static_assert(C > L + 1, "a table chunk holds at least one round of rows (one of them split) and the end marker");
  // one lane per particle is not supported: with no cross-lane operation in the loop nest the
  // compiler merged the chunk loop with the table loop and took the chunk loop's exit mask from a
  // compare of the divergent inner loop, and such a build listed some candidates twice (the same
  // build with the chunk bound passed through a width-1 shuffle listed each once)
  static_assert(L >= 2, "at least two lanes per particle");
  static_assert(L <= 16, "a group's prefix sums use row shifts within 16 lanes");
  rs = fminf(fmaxf(rs, 0.f), 2.f * (float)g.gmax + 2.f) * g.rowinv;   // in rows from here on
  const float rs2 = rs * rs;
  const bool per = PER && g.geometry == 0;
  const int P = 1 << g.skr;
  int z0 = D == 3 ? own.rz + (int)floorf(own.oz - rs) : 0;
  int z1 = D == 3 ? own.rz + (int)floorf(own.oz + rs) : 0;
  int y0 = own.ry + (int)floorf(own.oy - rs);
  int y1 = own.ry + (int)floorf(own.oy + rs);
  if (per) {
    if (y1 - y0 + 1 > P) {
      y0 = own.ry - P / 2;
      y1 = y0 + P - 1;
    }
    if (D == 3 && z1 - z0 + 1 > P) {
      z0 = own.rz - P / 2;
      z1 = z0 + P - 1;
    }
  } else {
    y0 = max(0, y0);
    y1 = min(P - 1, y1);
    if (D == 3) {
      z0 = max(0, z0);
      z1 = min(P - 1, z1);
    }
  }
  const int ny = y1 - y0 + 1;
  const int nrows = ny * (z1 - z0 + 1);
  const float inv_ny = 1.f / (float)ny;
  const uint32_t nmax = (uint32_t)g.n;
  const float fxr = g.rfx;                        // x sub-cells per row width
  const float oxs = own.ox * g.fx;                // offset in x sub-cells
  const int xi = own.cx << g.xb;
  const int xlast = ((g.gmax + 1) << g.xb) - 1;
  const uint32_t kx = g.k + g.xb;
  int nq = nrows;
  if (PER && per && (xi + (int)floorf(oxs - rs * fxr) < 0 || xi + (int)floorf(oxs + rs * fxr) > xlast)) nq = 2 * nrows;
  uint32_t total = 0;   // candidates of the group (the particle itself only without CUT)
  int q0 = 0;
  while (q0 < nq) {
    // table of the next chunk of rows: whole rounds of L rows while a round surely fits
    uint32_t ne = 0, run = 0;
    while (q0 < nq && ne + L + 1u < (uint32_t)C) {
      int q = q0 + sub;
      const bool in = q < nq;
      bool beyond = false;                        // the part of a periodic row past the end of the x axis
      if (PER && q >= nrows) {
        beyond = true;
        q -= nrows;
      }
      const int qz = (int)(((float)q + 0.5f) * inv_ny);   // q / ny, exact for nz = 1 and for ny, nz <= 2^9
      const int cz = z0 + qz, cy = y0 + (q - qz * ny);
      float ez = 0.f;
      if constexpr (D == 3) {
        const float lo = (float)(cz - own.rz) - own.oz, hi = lo + 1.f;
        ez = lo > 0.f ? lo : (hi < 0.f ? -hi : 0.f);
      }
      const float lo = (float)(cy - own.ry) - own.oy, hi = lo + 1.f;
      const float ey = lo > 0.f ? lo : (hi < 0.f ? -hi : 0.f);
      const float d2 = ey * ey + ez * ez;
      bool hit = in && d2 < rs2;
      // the hardware square root (about 1 ulp) is enough: the callers' reach rs exceeds every
      // range test of the bodies by a relative 1e-4
      const float wx = fast_sqrt(fmaxf(rs2 - d2, 0.f)) * fxr;
      int x0 = xi + (int)floorf(oxs - wx);
      int x1 = xi + (int)floorf(oxs + wx);
      if (PER && per) {
        if (x1 - x0 > xlast) {                    // the run covers the period: one run, nothing beyond
          x0 = 0;
          x1 = xlast;
          hit = hit && !beyond;
        } else if (beyond) {                      // at most one end is crossed
          if (x0 < 0) {
            x0 += xlast + 1;
            x1 = xlast;
          } else if (x1 > xlast) {
            x0 = 0;
            x1 -= xlast + 1;
          } else {
            hit = false;
          }
        }
      }
      x0 = max(0, x0);
      x1 = min(xlast, x1);
      const int cyw = PER && per ? cy & (P - 1) : cy;
      uint32_t kb;
      if constexpr (D == 3)
        kb = (uint32_t)x0 | (search_row(cyw, PER && per ? cz & (P - 1) : cz, g) << kx);
      else
        kb = (uint32_t)x0 | ((uint32_t)cyw << kx);
      kb += sbase;
      uint32_t a = 0u, b = 0u;
      if (hit) {
        a = cstart[kb];
        b = min(cstart[kb + (uint32_t)(x1 - x0) + 1u], nmax);
      }
      const uint32_t len = b > a ? b - a : 0u;
      // the particle's own slot is cut out of its row, which becomes the runs before and after it
      // (len1 and len2 candidates; a row without the particle keeps len1 = len)
      uint32_t base = 0u, len1 = len, len2 = 0u;
      if (len > 0u) {
        base = remap(cy, cz, a);
        const uint32_t o = self - base;   // >= len unless the particle lies in this run
        if (CUT && o < len) {
          len1 = o;
          len2 = len - o - 1u;
        }
      }
      const uint32_t lsum = len1 + len2, nl = (len1 > 0u ? 1u : 0u) + (len2 > 0u ? 1u : 0u);
      // prefix sums over the group of the candidates and of the table entries
      uint32_t incl = lsum, nz = nl;
#pragma unroll
      for (int o = 1; o < L; o <<= 1) {
        const uint32_t v = lane_up(incl, o), w = lane_up(nz, o);
        if (sub >= o) {
          incl += v;
          nz += w;
        }
      }
      if (nl > 0u) {
        uint32_t end = run + incl - lsum, en = ne + nz - nl;   // the lane's first slot and entry
        if (len1 > 0u) {
          end += len1;
          tab[en++ * (uint32_t)stride] = make_uint2(base - (end - len1), end);
        }
        if (len2 > 0u) {
          end += len2;
          tab[en * (uint32_t)stride] = make_uint2(base + len1 + 1u - (end - len2), end);
        }
      }
      run += group_last<L>(incl);
      ne += group_last<L>(nz);
      q0 += L;
    }
    // end marker (ne < C): base -run, so that slot t past the end maps to index t - run
    if (sub == 0) tab[ne * (uint32_t)stride] = make_uint2(0u - run, 0xFFFFFFFFu);
    total += run;
    // the chunk's slots, L at a time; slot t of row e is candidate base_e + t
    uint32_t t = (uint32_t)sub;
    const uint2 *rp = tab;
    uint2 row = *rp;           // row of the last located slot
    const auto locate = [&](uint32_t tt) -> uint32_t {
      while (tt >= row.y) {
        rp += stride;
        row = *rp;
      }
      return row.x + tt;
    };
    if constexpr (IsSplitBody<typename std::decay<BodyF>::type>::value) {
      // one round ahead: the loads of slot t + L are issued before the arithmetic of slot t; two
      // payloads used in turn (the loop is unrolled twice), so that none is copied.  The wave runs the
      // rounds of its longest group: as a loop that each lane left by itself, the exit's merge of the
      // two payloads made every other round wait for all loads before it issued the next ones
      bool v = t < run;
      if (__builtin_amdgcn_ballot_w64(v)) {
        auto pa = body.fetch(locate(t));
        while (true) {
          t += L;
          auto pb = body.fetch(locate(t));
          if (v) body.use(pa);
          v = t < run;
          if (!__builtin_amdgcn_ballot_w64(v)) break;
          t += L;
          pa = body.fetch(locate(t));
          if (v) body.use(pb);
          v = t < run;
          if (!__builtin_amdgcn_ballot_w64(v)) break;
        }
      }
    } else {
      for (; t < run; t += L) body(locate(t));
    }
  }
  return CUT ? total : (total > 0u ? total - 1u : 0u);
}

// Sum / minimum across the L lanes of a group (fixed butterfly order: lane l combines with lane
// l ^ o for o = L/2, ..., 1).  The partner's value comes through ds_swizzle in its bit-mask mode
// (and-mask 31, xor-mask o), which needs no per-lane address arithmetic; groups never straddle
// the 32-lane halves the swizzle works in (L <= 32).
template <int O>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
  static_assert(O > 0 && O < 32, "swizzle xor masks stay within 32 lanes");
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (O << 10));
}
template <int L>
__device__ __forceinline__ float group_sum(float x) {
  static_assert(L <= 32, "a group fits in 32 lanes");
  if constexpr (L >= 32) x += __uint_as_float(xor_lane<16>(__float_as_uint(x)));
  if constexpr (L >= 16) x += __uint_as_float(xor_lane<8>(__float_as_uint(x)));
  if constexpr (L >= 8) x += __uint_as_float(xor_lane<4>(__float_as_uint(x)));
  if constexpr (L >= 4) x += __uint_as_float(xor_lane<2>(__float_as_uint(x)));
  if constexpr (L >= 2) x += __uint_as_float(xor_lane<1>(__float_as_uint(x)));
  return x;
}
template <int L>
__device__ __forceinline__ uint32_t group_sum_u(uint32_t x) {
  static_assert(L <= 32, "a group fits in 32 lanes");
  if constexpr (L >= 32) x += xor_lane<16>(x);
  if constexpr (L >= 16) x += xor_lane<8>(x);
  if constexpr (L >= 8) x += xor_lane<4>(x);
  if constexpr (L >= 4) x += xor_lane<2>(x);
  if constexpr (L >= 2) x += xor_lane<1>(x);
  return x;
}
template <int L>
__device__ __forceinline__ float group_min(float x) {
  static_assert(L <= 32, "a group fits in 32 lanes");
  if constexpr (L >= 32) x = fminf(x, __uint_as_float(xor_lane<16>(__float_as_uint(x))));
  if constexpr (L >= 16) x = fminf(x, __uint_as_float(xor_lane<8>(__float_as_uint(x))));
  if constexpr (L >= 8) x = fminf(x, __uint_as_float(xor_lane<4>(__float_as_uint(x))));
  if constexpr (L >= 4) x = fminf(x, __uint_as_float(xor_lane<2>(__float_as_uint(x))));
  if constexpr (L >= 2) x = fminf(x, __uint_as_float(xor_lane<1>(__float_as_uint(x))));
  return x;
}

// First time step (Eq. 29 with v = 0): minimum over the domain's slots, every lane gets it.
__device__ __forceinline__ float read_dt1(const uint32_t *slots) {
  float v = __uint_as_float(slots[(threadIdx.x & (kDtSlots - 1)) * kDtStride]);
  for (int off = kWave / 2; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off, kWave));
  v = v < INFINITY ? v : 0.f;
  // the same value in every lane: held as a wave-uniform (scalar) value
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}

}  // namespace mpsph
