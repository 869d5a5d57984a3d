// Reverse-mode (adjoint) kernels of the relaxation step and of the relaxation loss (gfx950).
//
// Notation (cell units, one step, the forward kernels in mpsph.hip compute the same values):
//   s_i field spacing, h_i = tau s_i, P_i = p0c s_i^(2d), H = h_ij = (h_i + h_j)/2, q = r/H,
//   u = 1 - q/2, g(r, H) = 5 alpha H^-(d+2) u^3 (= -W'(r, H)/r),  u_ij = X_i - X_j,
//   F_i = sum_j M_ij B_ij (P_i + P_j) g u_ij, a = Pi F (force mapping, Eq. 18, 23, 30),
//   T1 = min_i c_acc sqrt(kappa h_i / |a_i|), T2 = f T1 (Eq. 29), v~ = T1 a / 2 (Eq. 26),
//   eta_i = nu_coeff kappa tau s_i^(1-d) |v~_i| (Eq. 21-22),
//   K_ij = -Hm(eta_i, eta_j) (s_i^(2d) + s_j^(2d)) g, A~_i = sum_j M_ij K_ij (v~_i - v~_j) (Eq. 20),
//   a~ = Pi A~, Delta = T2 (v~ + T2 a~ / 2) (Eq. 27-28), X' = clamp(X + Delta).
// M_ij = [type_j >= type_i] is the interaction mask, B_ij = 1 + sigma [C_i != C_j] (Eq. 24).
// The pair sums are symmetric in everything but the mask, so the adjoint of a pair sum is a
// gather over the same neighbours: particle k collects, for every neighbour j, the terms of the
// pair (k, j) (mask M_kj) and of the pair (j, k) (mask M_jk) -- no atomics, a fixed order.
//
// Loss (after the last step, all n particles):
//   L = (1/n) sum_i e_i^2 + (lambda / n) sum_{i<j, C_i != C_j} w(r_ij / h_ij),
//   e_i = rho_i / rho_t,i - 1 = alpha tau^-d sum_j w(r_ij / h_i) - 1 (Eq. 17, self included),
//   w(q) = (1 - q/2)^4 (1 + 2q), w'(q) = -5 q (1 - q/2)^3.
// Piecewise-constant parts (pair sets, masks, re-tagging, the particle attaining T1) are held
// fixed; the clamp passes the gradient where the coordinate stays inside the box.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mpsph_device.h"
#include "pair_scan.h"

// Waves per SIMD the viscous adjoint is compiled for; 0 leaves it to the compiler.  With the
// particle's own data scoped to the pair loop and its per-group values in LDS, and the neighbour
// loads issued one slot round ahead (three loads held for the next round), 5 waves (89 VGPRs in
// 3D) need no scratch memory; at 6 waves it spills 10 registers.  Reverse sweep of the
// 2^20-particle RBF cube over 50 steps, with the pair terms in spacings: 106.7 ms at 5 waves, 109.4 ms at
// 6 with the spills, 107.4 ms with one round of loads at 6 waves.
#ifndef MPSPH_ADJ_WAVES
#define MPSPH_ADJ_WAVES 5
#endif
#if MPSPH_ADJ_WAVES > 0
#define MPSPH_ADJ_OCCUPANCY __attribute__((amdgpu_waves_per_eu(MPSPH_ADJ_WAVES, MPSPH_ADJ_WAVES)))
#else
#define MPSPH_ADJ_OCCUPANCY
#endif

namespace mpsph {

constexpr int kMaxRbf = 64;

// One step of the forward record: the sorted state the step started from and its results.
struct TapeView {
  const uint32_t *wkey;
  const float4 *wpos;    // offsets, h
  const float4 *wfix;    // fixed-point coordinates, h
  const uint32_t *wjaux; // colour | type << 30
  const uint32_t *cstart;
  const uint32_t *perm;  // state index of each sorted index
  const float4 *acc;     // a (after the force mapping), e = rho_t nu_coeff r_c |a|
  const float4 *at;      // a~ after the force mapping
  const float4 *v;       // v_{n+1/2}
  const uint32_t *dts;   // time-step slots of the step
};

template <int D>
__device__ __forceinline__ float pow2d(float s) {  // s^(2d)
  return powd<D>(s * s);
}

// The pair adjoints take the kernel's derivatives from one common factor, with 2H = h_i + h_j,
// u = 1 - r / 2H and w = (2H)^-(d+3) u^2:
//   g = C w u 2H / 2,  dg/dr = -(3/2) C w,  dg/dH = C w (3 - (d+5) u),  C = 5 alpha 2^(d+3),
// and spacings as h^2d = tau^2d s^2d; every factor common to a particle's pairs is applied once to its
// sums.  Bound by the issue of vector instructions: at 262,144 particles the
// viscous adjoint took 161 us and the force adjoint 122 with g, dg/dr and dg/dH formed one by one in
// spacings, 151 and 110 this way.
template <int D>
__device__ __forceinline__ float slope_scale(float alpha) {
  return (D == 3 ? 320.f : 160.f) * alpha;
}

// w from i = 1 / 2H and u.
template <int D>
__device__ __forceinline__ float slope_factor(float i, float u) {
  const float i2 = i * i;
  return (D == 3 ? i2 * i2 * i2 : i2 * i2 * i) * (u * u);
}

// The RBF table of a field, entry m in lane m of the wave (kMaxRbf of them at most).  Read from there
// by readlane into scalar registers: 7 loads per wave instead of 7 for every Gaussian.
struct RbfTable {
  int c[3];
  float o[3], k;
};
static_assert(kMaxRbf <= kWave, "one table entry per lane");
template <int D>
__device__ __forceinline__ RbfTable rbf_table(const FieldDev &f, int nr) {
  RbfTable r{};
  const int m = threadIdx.x & (kWave - 1);
  if (m < nr) {
#pragma unroll
    for (int a = 0; a < D; ++a) {
      r.c[a] = f.rbf_c[m * 3 + a];
      r.o[a] = f.rbf_o[m * 3 + a];
    }
    r.k = f.rbf_k[m];
  }
  return r;
}

// Gaussians [m0, m0 + kRbfChunk) of the RBF field at X, zero past the last one, with their share of
// the exponent e and of its gradient ge.  By whole waves.
constexpr int kRbfChunk = 32;
template <int D>
__device__ __forceinline__ void rbf_chunk(const RbfTable &r, float e2, int m0, int nr, const int *c, const float *o,
                                          float *gauss, float &e, float *ge) {
#pragma unroll
  for (int t = 0; t < kRbfChunk; ++t) {
    const int m = m0 + t;
    gauss[t] = 0.f;
    if (m < nr) {   // uniform
      float dv[3], r2 = 0.f;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        dv[a] = (float)(c[a] - __builtin_amdgcn_readlane(r.c[a], m)) +
                (o[a] - __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r.o[a]), m)));
        r2 += dv[a] * dv[a];
      }
      gauss[t] = __expf(-r2 * e2);
      const float k = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(r.k), m)) * gauss[t];
      e += k;
#pragma unroll
      for (int a = 0; a < D; ++a) ge[a] -= 2.f * e2 * k * dv[a];
    }
  }
}

// Minimum of non-negative floats over the block into *dst: one atomic per block.  The callers
// spread their blocks over the kDtSlots lines of a slot array: device-wide atomics on one line
// take 12 ns each (262,144 particles: the drift adjoint 17.6 us on one address, 8.3 on 16 lines).
__device__ __forceinline__ void block_min_atomic(float v, uint32_t *dst) {
  __shared__ float wmin[kBlock / kWave];
  for (int off = kWave / 2; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off, kWave));
  if ((threadIdx.x & (kWave - 1)) == 0) wmin[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    float m = wmin[0];
    for (int w = 1; w < kBlock / kWave; ++w) m = fminf(m, wmin[w]);
    if (m < INFINITY) atomic_min_pos(dst, m);
  }
}

// Minimum over the slots, as bits; every lane of the wave takes part and gets it.
__device__ __forceinline__ uint32_t slots_min(const uint32_t *slots) {
  uint32_t m = slots[(threadIdx.x & (kDtSlots - 1)) * kDtStride];
#pragma unroll
  for (int o = kDtSlots / 2; o > 0; o >>= 1) m = min(m, (uint32_t)__shfl_xor((int)m, o, kWave));
  return __builtin_amdgcn_readfirstlane(m);
}

// Drift and velocity adjoint, one thread per particle (sorted order of the step).
//   xbar_next: adjoint of the positions after the step (this step's order)
//   xacc <- identity part of the position adjoint, abv <- adjoint of A~ (before the viscous
//   pair sum), vtb <- direct part of the adjoint of v~, dtc <- the particle's candidate of T1.
template <int D>
__global__ __launch_bounds__(kBlock) void adj_drift(const DomDev *__restrict__ dom, TapeView tp,
                                                    const float4 *__restrict__ xbar_next, float4 *__restrict__ xacc,
                                                    float4 *__restrict__ abv, float4 *__restrict__ vtb,
                                                    float *__restrict__ dtc, uint32_t *__restrict__ minslots,
                                                    double *__restrict__ partials) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  const GridDev &g = dom->g;
  const StepDev &sp = dom->sp;
  const float dt1 = read_dt1(tp.dts);
  const float dt2 = dt1 * sp.dt2_factor;
  double part[1] = {0.0};
  const int ops[1] = {0};
  float c1 = INFINITY;   // the particle's candidate of T1
  if (i < dom->n) {
    int ci[3];
    unpack_key<D>(tp.wkey[i], g, ci);
    const float4 pi = tp.wpos[i];
    const float oi[3] = {pi.x, pi.y, pi.z};
    const int ti = aux_type(tp.wjaux[i]);
    const float4 xb4 = xbar_next[i], v4 = tp.v[i], at4 = tp.at[i];
    const float xb[3] = {xb4.x, xb4.y, xb4.z}, vv[3] = {v4.x, v4.y, v4.z}, av[3] = {at4.x, at4.y, at4.z};
    float xd[3] = {0.f, 0.f, 0.f}, db[3] = {0.f, 0.f, 0.f}, ab[3] = {0.f, 0.f, 0.f};
    double t2 = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      float keep = 1.f;
      if (ti != 3) {
        // the drift of the forward pass, to find the coordinates the wall clamp fixed
        const float x = oi[a] + vv[a] * dt2;
        const float fl = floorf(x);
        int c = ci[a] + (int)fl;
        float o = x - fl;
        if (o >= 1.f) {
          o = 0.f;
          c += 1;
        }
        if (c < 0 || c > g.whi_c[a] || (c == g.whi_c[a] && o > g.whi_o[a])) keep = 0.f;
      }
      xd[a] = keep * xb[a];
      if (ti != 3) {
        db[a] = xd[a];
        ab[a] = 0.5f * dt2 * dt2 * db[a];
        t2 += (double)db[a] * (double)(vv[a] + 0.5f * dt2 * av[a]);
      }
    }
    project_feature<D>(g, ti, ci, oi, ab);
    xacc[i] = make_float4(xd[0], xd[1], xd[2], 0.f);
    abv[i] = make_float4(ab[0], ab[1], ab[2], __int_as_float(ti));   // the type for the viscous pass
    vtb[i] = make_float4(dt2 * db[0], dt2 * db[1], dt2 * db[2], 0.f);
    part[0] = t2;
    // candidate of the first time step (as in the forward pass, from the stored a)
    const float4 a4 = tp.acc[i];
    const float am2 = a4.x * a4.x + a4.y * a4.y + (D == 3 ? a4.z * a4.z : 0.f);
    if (ti != 3 && am2 > 0.f) c1 = sp.c_acc * fast_sqrt(sp.kappa * pi.w * fast_rsq(am2));   // as the density pass
    dtc[i] = c1;
  }
  block_min_atomic(c1, minslots + (blockIdx.x & (kDtSlots - 1)) * kDtStride);
  block_reduce_write<1>(part, ops, partials + blockIdx.x);
}

// Viscous adjoint, L lanes per particle.  Gathers over the neighbours j of k the terms of the
// pairs (k, j) and (j, k) of A~ = sum M K (v~_k - v~_j):
//   v~bar_k += K (M_kj Abar_k - M_jk Abar_j),  Kbar = (M_kj Abar_k - M_jk Abar_j).(v~_k - v~_j)
// and Kbar's share of eta_k, s_k, X_k; then eta -> v~, s; a-bar = T1/2 v~bar; T1-bar partials.
// fbar receives Pi a-bar, the adjoint of the force before the mapping but for the share of the
// time step in the particle attaining T1 (adj_time_step).
template <int D, int L, bool WIDE>
__global__ __launch_bounds__(kBlock) MPSPH_ADJ_OCCUPANCY void adj_visc(const DomDev *__restrict__ dom, TapeView tp,
                                                   const float4 *__restrict__ abv, const float4 *__restrict__ vtb,
                                                   float4 *__restrict__ xacc, float *__restrict__ sbar,
                                                   float4 *__restrict__ fbar, const float *__restrict__ dtc,
                                                   const uint32_t *__restrict__ minslots, uint32_t *__restrict__ argmin,
                                                   double *__restrict__ partials) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const GridDev &g = dom->g;
  const StepDev &sp = dom->sp;
  const int local = lb * kBlock + threadIdx.x;
  const int i = local / L, sub = local % L;
  __shared__ uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  // per lane group, the particle's (a, e) and (a~-bar, d h^(2d)/dh): read from LDS by the
  // pair terms instead of being held in registers across the pair loop
  __shared__ float4 gdat[kBlock / L][2];
  const float dt1 = read_dt1(tp.dts);
  const uint32_t tmin = slots_min(minslots);
  const float hdt = 0.5f * dt1;
  double part[1] = {0.0};
  const int ops[1] = {0};
  if (i < dom->n && sub == 0) {
    const float4 ai = tp.acc[i];
    const float4 abi = abv[i];
    const float hi = tp.wpos[i].w;
    gdat[threadIdx.x / L][0] = ai;
    gdat[threadIdx.x / L][1] = make_float4(abi.x, abi.y, abi.z, (2.f * (float)D) * pow2d<D>(hi) / hi);
  }
  __syncthreads();
  if (i < dom->n) {
    float vb[3] = {0.f, 0.f, 0.f}, xb[3] = {0.f, 0.f, 0.f}, eb = 0.f, sb = 0.f;
    {
    // the pair sum; the particle's own data is scoped to it (the epilogue reads it again), so
    // that the kernel fits its register budget without spilling
    const PairPos<D, false, WIDE> pos(g, 0u, i, tp.wkey, tp.wfix);
    const float unit = pos.unit;
    const int ti = aux_type(tp.wjaux[i]);
    const float hi = pos.h;
    const float h2di = pow2d<D>(hi);
    const float4 *gd = gdat[threadIdx.x / L];
    const float ei = gd[0].w;
    const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
    const float kh = 0.5f * sp.kappa;
    if (hdt * ei > 0.f) {
      const BufRes racc = buf_res(tp.acc, 16, (uint32_t)g.n), rabv = buf_res(abv, 16, (uint32_t)g.n);
      struct Nb {
        typename PairPos<D, false, WIDE>::Nb p;
        float4 a4, ab;   // ab.w: the neighbour's type
      };
      // the neighbour's loads (bounds-checked: slots past the arrays read zeros) are issued one
      // slot round ahead of the pair's arithmetic
      const auto fetch = [&](uint32_t jr) {
        return Nb{pos.fetch(jr), buf_f4(racc, jr), buf_f4(rabv, jr)};
      };
      const auto use = [&](const Nb &nb) {
        const float4 pj = nb.p.p, aj4 = nb.a4, abj = nb.ab;
        // separations in units of pos.unit cells
        float dx, dy, dz = 0.f;
        pos.sep(nb.p, dx, dy, dz);
        float r2 = dx * dx + dy * dy;
        if constexpr (D == 3) r2 += dz * dz;
        const float rinv = fast_rsq(r2);
        const float r = r2 * rinv * unit;   // NaN at zero separation
        const float hs = hi + pj.w;
        const float ej = aj4.w;
        // e_j = 0: the pair's K and every derivative of it vanish
        if (!(r > 0.f && r < kh * hs && ej > 0.f)) return;
        const int tj = __float_as_int(abj.w);
        const float mkj = tj >= ti ? 1.f : 0.f, mjk = ti >= tj ? 1.f : 0.f;
        const float4 ai = gd[0], abi = gd[1];
        const float wv[3] = {mkj * abi.x - mjk * abj.x, mkj * abi.y - mjk * abj.y, mkj * abi.z - mjk * abj.z};
        const float i2h = fast_rcp(hs);
        const float u = fmaf(-r, i2h, 1.f);
        const float w = slope_factor<D>(i2h, u), uh = u * hs;
        const float sw = powd_add<D>(pj.w * pj.w, h2di) * w;
        const float rat = ej * fast_rcp(ei + ej);
        const float K = rat * (sw * uh);
        vb[0] = fmaf(K, wv[0], vb[0]);
        vb[1] = fmaf(K, wv[1], vb[1]);
        if constexpr (D == 3) vb[2] = fmaf(K, wv[2], vb[2]);
        const float dvx = ai.x - aj4.x, dvy = ai.y - aj4.y, dvz = ai.z - aj4.z;
        const float kb = wv[0] * dvx + wv[1] * dvy + (D == 3 ? wv[2] * dvz : 0.f);
        const float m = kb * rat;
        eb = fmaf(m, K, eb);
        sb = fmaf(m, fmaf(abi.w, w * uh, sw * fmaf(-(float)(D + 5), u, 3.f)), sb);
        const float cx = m * sw * rinv;
        xb[0] = fmaf(cx, dx, xb[0]);
        xb[1] = fmaf(cx, dy, xb[1]);
        if constexpr (D == 3) xb[2] = fmaf(cx, dz, xb[2]);
      };
      scan_group_table<D, L, row_table_rows<L>()>((uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row,
                                                  rs, g, 0u, tp.cstart, pair_body<true>(fetch, use));
    }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      vb[a] = group_sum<L>(vb[a]);
      xb[a] = group_sum<L>(xb[a]);
    }
    eb = group_sum<L>(eb);
    sb = group_sum<L>(sb);
    if (sub == 0) {
      // the particle's own data again, through an index the compiler cannot tie to i, so that
      // neither values nor addresses stay live across the pair loop
      const int io = __shfl(i, (int)(threadIdx.x & (kWave - 1)));
      const float4 po = tp.wpos[io];
      const float si = po.w * sp.inv_tau;
      const uint32_t xo = tp.wjaux[io];
      const int ti = aux_type(xo);
      const float4 ai = tp.acc[io];
      // the factors common to the particle's pairs
      const float fe = -hdt * slope_scale<D>(sp.alpha) * pow2d<D>(sp.inv_tau), fv = fe * ai.w, fs = fv * hdt;
      eb *= fe;
      sb *= fs * sp.tau;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        vb[a] *= fv;
        xb[a] *= -3.f * fs;
      }
      const float vti[3] = {hdt * ai.x, hdt * ai.y, hdt * ai.z};
      const float4 vd = vtb[io];
      float vt[3] = {vd.x + vb[0], vd.y + vb[1], vd.z + vb[2]};
      const float vm2 = vti[0] * vti[0] + vti[1] * vti[1] + (D == 3 ? vti[2] * vti[2] : 0.f);
      if (vm2 > 0.f && eb != 0.f) {
        // eta = nu_coeff kappa tau s^(1-d) |v~|
        const float vm = sqrtf(vm2);
        const float c0 = sp.nu_coeff * sp.kappa * sp.tau * (D == 3 ? 1.f / (si * si) : 1.f / si);
        const float f = eb * c0 / vm;
#pragma unroll
        for (int a = 0; a < D; ++a) vt[a] = fmaf(f, vti[a], vt[a]);
        sb = fmaf(eb * c0 * (float)(1 - D) / si, vm, sb);
      }
      float ab[3] = {0.f, 0.f, 0.f};
      const float av[3] = {ai.x, ai.y, ai.z};
      double t1 = 0.0;
      if (ti != 3) {
#pragma unroll
        for (int a = 0; a < D; ++a) {
          ab[a] = hdt * vt[a];
          t1 += 0.5 * (double)av[a] * (double)vt[a];
        }
      }
      int co[3];
      unpack_key<D>(tp.wkey[io], g, co);
      const float oo[3] = {po.x, po.y, po.z};
      project_feature<D>(g, ti, co, oo, ab);
      fbar[io] = make_float4(ab[0], ab[1], ab[2], __uint_as_float(xo));   // the flags for the force adjoint
      sbar[io] = sb;
      const float4 x0 = xacc[io];
      xacc[io] = make_float4(x0.x + xb[0], x0.y + xb[1], x0.z + xb[2], 0.f);
      // tmin stays infinite where no particle has a force: none attains T1 then
      if (tmin != kInfBits && __float_as_uint(dtc[io]) == tmin) atomicMin(argmin, (uint32_t)io);
      part[0] = t1;
    }
  }
  block_reduce_write<1, L>(part, ops, partials + lb);   // first lanes of the groups
}

// Time-step adjoint, one block: T1-bar + f T2-bar from the partials (fixed order), and its share in
// the particle that attains T1: F-bar += Pi dT1/da T1-bar, s-bar += dT1/ds T1-bar.  Bound by the latency
// of its loads; the partials lie one after the other (8,192 of them 5 us; 14 us at kNumPartials doubles
// apart in a block of 256).
constexpr int kTimeStepThreads = 1024;
template <int D>
__global__ __launch_bounds__(kTimeStepThreads) void adj_time_step(const DomDev *__restrict__ dom, TapeView tp,
                                                                  const double *__restrict__ pa, int na,
                                                                  const double *__restrict__ pb, int nb, float f,
                                                                  const uint32_t *__restrict__ argmin,
                                                                  float *__restrict__ sbar, float4 *__restrict__ fbar) {
  __shared__ double red[kTimeStepThreads / kWave];
  const float dt1 = read_dt1(tp.dts);   // by whole waves
  double x = 0.0, y = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < na; b += kTimeStepThreads) x += pa[b];
#pragma unroll 8
  for (int b = threadIdx.x; b < nb; b += kTimeStepThreads) y += pb[b];
  y += (double)f * x;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) y += __shfl_xor(y, o, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = y;
  __syncthreads();
  const uint32_t i = *argmin;
  if (threadIdx.x != 0 || i >= (uint32_t)dom->n) return;   // no particle with a force: no time step to adjoin
  double t1bar = red[0];
#pragma unroll
  for (int w = 1; w < kTimeStepThreads / kWave; ++w) t1bar += red[w];
  const GridDev &g = dom->g;
  int ci[3];
  unpack_key<D>(tp.wkey[i], g, ci);
  const float4 pi = tp.wpos[i], a4 = tp.acc[i], f0 = fbar[i];
  const float oi[3] = {pi.x, pi.y, pi.z};
  const float tb = (float)t1bar;
  // T1 = c_acc sqrt(kappa h / |a|): dT1/da = -T1 a / (2 |a|^2), dT1/ds = T1 / (2 s)
  const float am2 = a4.x * a4.x + a4.y * a4.y + (D == 3 ? a4.z * a4.z : 0.f);
  const float c = -0.5f * dt1 * tb / am2;
  float ff[3] = {c * a4.x, c * a4.y, D == 3 ? c * a4.z : 0.f};
  project_feature<D>(g, aux_type(tp.wjaux[i]), ci, oi, ff);
  fbar[i] = make_float4(f0.x + ff[0], f0.y + ff[1], f0.z + ff[2], f0.w);
  sbar[i] += 0.5f * dt1 * tb / (pi.w * dom->sp.inv_tau);
}

// Force adjoint, L lanes per particle: for every neighbour j, with W = M_kj Fbar_k - M_jk Fbar_j
// and w = B (P_k + P_j) g(r, H):
//   X-bar_k += w W + B (P_k + P_j) dg/dr (u.W) u / r
//   s-bar_k += (u.W) B [2d p0c s_k^(2d-1) g + (P_k + P_j) dg/dH tau / 2]
template <int D, int L, bool WIDE>
__global__ __launch_bounds__(kBlock) void adj_force(const DomDev *__restrict__ dom, TapeView tp, float tstep,
                                                    const float4 *__restrict__ fbar, float4 *__restrict__ xacc,
                                                    float *__restrict__ sbar) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const GridDev &g = dom->g;
  const StepDev &sp = dom->sp;
  const int local = lb * kBlock + threadIdx.x;
  const int i = local / L, sub = local % L;
  __shared__ uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  if (i >= dom->n) return;
  const PairPos<D, false, WIDE> pos(g, 0u, i, tp.wkey, tp.wfix);
  const float unit = pos.unit;
  const uint32_t ai = tp.wjaux[i];
  const int ti = aux_type(ai);
  const float hi = pos.h;
  const float h2di = pow2d<D>(hi);
  const float dh2di = (2.f * (float)D) * h2di / hi;
  const float4 fi = fbar[i];
  const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
  const float kh = 0.5f * sp.kappa, unit3 = -3.f * unit;
  const float opb = 1.f + sigma_of(sp, tstep);   // surface tension of the step (Eq. 24-25)
  float xb[3] = {0.f, 0.f, 0.f}, sb = 0.f;
  const BufRes rfb = buf_res(fbar, 16, (uint32_t)g.n);
  struct Nb {
    typename PairPos<D, false, WIDE>::Nb p;
    float4 f;   // f.w: the neighbour's type and colour
  };
  // the neighbour's loads (bounds-checked: slots past the arrays read zeros) are issued one slot
  // round ahead of the pair's arithmetic
  const auto fetch = [&](uint32_t jr) { return Nb{pos.fetch(jr), buf_f4(rfb, jr)}; };
  const auto use = [&](const Nb &nb) {
    const float4 pj = nb.p.p, fj = nb.f;
    const uint32_t aj = __float_as_uint(fj.w);
    // separations in units of pos.unit cells
    float dx, dy, dz = 0.f;
    pos.sep(nb.p, dx, dy, dz);
    float r2 = dx * dx + dy * dy;
    if constexpr (D == 3) r2 += dz * dz;
    const float rinv = fast_rsq(r2);
    const float r = r2 * rinv * unit;   // NaN at zero separation
    const float hs = hi + pj.w;
    if (!(r > 0.f && r < kh * hs)) return;
    const int tj = aux_type(aj);
    const float mkj = tj >= ti ? 1.f : 0.f, mjk = ti >= tj ? 1.f : 0.f;
    const float wf[3] = {mkj * fi.x - mjk * fj.x, mkj * fi.y - mjk * fj.y, mkj * fi.z - mjk * fj.z};
    const float i2h = fast_rcp(hs);
    const float u = fmaf(-r, i2h, 1.f), uh = u * hs;
    const float bw = (colour_differs(aj, ai) ? opb : 1.f) * slope_factor<D>(i2h, u);
    const float x = powd_add<D>(pj.w * pj.w, h2di) * bw;
    const float uw = dx * wf[0] + dy * wf[1] + (D == 3 ? dz * wf[2] : 0.f);
    const float cw = x * uh, cr = x * uw * (rinv * unit3);
    xb[0] = fmaf(cw, wf[0], fmaf(cr, dx, xb[0]));
    xb[1] = fmaf(cw, wf[1], fmaf(cr, dy, xb[1]));
    if constexpr (D == 3) xb[2] = fmaf(cw, wf[2], fmaf(cr, dz, xb[2]));
    sb = fmaf(uw, fmaf(dh2di, bw * uh, x * fmaf(-(float)(D + 5), u, 3.f)), sb);
  };
  scan_group_table<D, L, row_table_rows<L>()>((uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row, rs, g,
                                              0u, tp.cstart, pair_body<true>(fetch, use));
#pragma unroll
  for (int a = 0; a < 3; ++a) xb[a] = group_sum<L>(xb[a]);
  sb = group_sum<L>(sb);
  if (sub == 0) {
    // the factors common to the particle's pairs
    const float fx = 0.5f * slope_scale<D>(sp.alpha) * sp.p0c * pow2d<D>(sp.inv_tau);
    const float4 x0 = xacc[i];
    xacc[i] = make_float4(fmaf(fx, xb[0], x0.x), fmaf(fx, xb[1], x0.y), fmaf(fx, xb[2], x0.z), 0.f);
    sbar[i] = fmaf(fx * sp.tau * unit, sb, sbar[i]);
  }
}

// Field adjoint and hand-over to the previous step, one thread per particle:
//   X-bar_k += s-bar_k grad s(X_k),  c-bar_m += s-bar_k ds/dc_m = s-bar_k s_k G_m(X_k),
// X-bar written at the particle's index in the previous state order (perm).  Each wave keeps its
// sums of c-bar in row cpart[row * kMaxRbf + m], added to over the steps of the sweep (set by the
// loss, the first of them).  Also clears the time-step slots for the step that is reversed next.
// One wave per block: 8,192 particles are 128 CUs' work instead of 32 blocks'.  Bound by the
// latency of the Gaussians and of the reduction, which halves the sums a lane holds at each exchange
// (32 exchanges for 32 sums instead of 192): with the table in lanes 21 -> 8.7 us at
// 8,192 particles, 38 -> 23 us at 262,144.
template <int D>
__global__ __launch_bounds__(kWave) void adj_field(const DomDev *__restrict__ dom, TapeView tp,
                                                   const float4 *__restrict__ xacc, const float *__restrict__ sbar,
                                                   float4 *__restrict__ xbar_prev, double *__restrict__ cpart, int first,
                                                   uint32_t *__restrict__ minslots, uint32_t *__restrict__ argmin) {
  const int lane = threadIdx.x, i = blockIdx.x * kWave + lane;
  const GridDev &g = dom->g;
  const FieldDev &f = dom->f;
  if (blockIdx.x == 0) {
    if (lane < kDtSlots) minslots[lane * kDtStride] = kInfBits;
    if (lane == kDtSlots) *argmin = 0xffffffffu;
  }
  const bool act = i < dom->n;
  int ci[3] = {0, 0, 0};
  float oi[3] = {0.f, 0.f, 0.f}, sb = 0.f;
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  uint32_t to = 0u;
  if (act) {
    unpack_key<D>(tp.wkey[i], g, ci);
    const float4 pi = tp.wpos[i];
    oi[0] = pi.x;
    oi[1] = pi.y;
    oi[2] = pi.z;
    sb = sbar[i];
    x = xacc[i];
    to = tp.perm[i];
  }
  const int nr = f.kind == 3 ? f.n_rbf : 0;   // other fields: no gradient, no coefficients
  float gauss[kRbfChunk], e = 0.f, ge[3] = {0.f, 0.f, 0.f};
  const RbfTable tab = rbf_table<D>(f, nr);
  for (int m0 = 0; m0 < nr; m0 += kRbfChunk) rbf_chunk<D>(tab, f.e2, m0, nr, ci, oi, gauss, e, ge);
  const float w = sb * (f.s0 * __expf(e));
  if (act) xbar_prev[to] = make_float4(fmaf(w, ge[0], x.x), fmaf(w, ge[1], x.y), fmaf(w, ge[2], x.z), 0.f);
  for (int m0 = 0; m0 < nr; m0 += kRbfChunk) {
    if (nr > kRbfChunk) {   // the first loop left the last chunk's
      float e1 = 0.f, g1[3] = {0.f, 0.f, 0.f};
      rbf_chunk<D>(tab, f.e2, m0, nr, ci, oi, gauss, e1, g1);
    }
    // the first exchange passes the FP32 terms, sums are FP64
    double v[kRbfChunk / 2];
    const bool upper = (lane & (kWave / 2)) != 0;
#pragma unroll
    for (int t = 0; t < kRbfChunk / 2; ++t) {
      const float lo = w * gauss[t], hi = w * gauss[t + kRbfChunk / 2];
      v[t] = (double)(upper ? hi : lo) + (double)__shfl_xor(upper ? lo : hi, kWave / 2, kWave);
    }
    int m = m0 + (upper ? kRbfChunk / 2 : 0);
#pragma unroll
    for (int h = kRbfChunk / 4, o = kWave / 4; h > 0; h >>= 1, o >>= 1) {
      const bool up = (lane & o) != 0;
#pragma unroll
      for (int t = 0; t < h; ++t) {
        const double keep = up ? v[t + h] : v[t], give = up ? v[t] : v[t + h];
        v[t] = keep + __shfl_xor(give, o, kWave);
      }
      m += up ? h : 0;
    }
#pragma unroll
    for (int o = kWave / 2 / kRbfChunk; o > 0; o >>= 1) v[0] += __shfl_xor(v[0], o, kWave);
    if ((lane & (kWave / kRbfChunk - 1)) == 0 && m < nr) {
      double *c = cpart + (size_t)blockIdx.x * kMaxRbf + m;
      *c = first ? v[0] : *c + v[0];
    }
  }
}

// c-bar[m] = sum over the rows of cpart[row][m]: one block per coefficient, each thread summing
// every 256th row in order, then a fixed tree over the threads (deterministic).
constexpr int kCoeffSumThreads = 256;
__global__ __launch_bounds__(kCoeffSumThreads) void adj_sum_coeff(const double *__restrict__ cpart, int rows,
                                                                  int n_rbf, double *__restrict__ cbar) {
  __shared__ double red[kCoeffSumThreads];
  const int m = blockIdx.x;
  if (m >= n_rbf) return;  // block-uniform
  double s = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < rows; b += kCoeffSumThreads) s += cpart[(size_t)b * kMaxRbf + m];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = kCoeffSumThreads / 2; off > 0; off >>= 1) {
    if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) cbar[m] = red[0];
}

// Loss, first pass (L lanes per particle, sorted order of the final state):
//   e_k = alpha tau^-d sum_{r < kappa h_k} w(r / h_k) - 1 (self included), and the ordered
//   interface sum sum_{C_j != C_k, r < kappa H} w(r / H); block partials of sum e^2 (slot 0)
//   and of the interface sum (slot 1).
template <int D, int L, bool WIDE>
__global__ __launch_bounds__(kBlock) void loss_density(const DomDev *__restrict__ dom, const uint32_t *__restrict__ wkey,
                                                       const float4 *__restrict__ wfix, const uint32_t *__restrict__ wjaux,
                                                       const uint32_t *__restrict__ cstart, float *__restrict__ e_out,
                                                       double *__restrict__ partials) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const GridDev &g = dom->g;
  const StepDev &sp = dom->sp;
  const int local = lb * kBlock + threadIdx.x;
  const int i = local / L, sub = local % L;
  __shared__ uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  double part[2] = {0.0, 0.0};
  const int ops[2] = {0, 0};
  if (i < dom->n) {
    const PairPos<D, false, WIDE> pos(g, 0u, i, wkey, wfix);
    const float unit = pos.unit;
    const uint32_t ai = wjaux[i];
    const float hi = pos.h, ihi = fast_rcp(hi);
    const float rci = sp.kappa * hi, rci2 = rci * rci;
    const float rs = fminf(sp.search_fac * hi, sp.kappa * 0.5f * (hi + sp.hmax)) * 1.0001f;
    const float kh = 0.5f * sp.kappa;
    float ws = 0.f, wi = 0.f;
    const BufRes raux = buf_res(wjaux, 4, (uint32_t)g.n);
    struct Nb {
      typename PairPos<D, false, WIDE>::Nb p;
      uint32_t a;
    };
    const auto fetch = [&](uint32_t jr) { return Nb{pos.fetch(jr), buf_u32(raux, jr)}; };
    const auto use = [&](const Nb &nb) {
      const float4 pj = nb.p.p;
      const uint32_t aj = nb.a;
      float dx, dy, dz = 0.f;
      pos.sep(nb.p, dx, dy, dz);
      dx *= unit;
      dy *= unit;
      dz *= unit;
      float r2 = dx * dx + dy * dy;
      if constexpr (D == 3) r2 += dz * dz;
      const float r = sqrtf(r2);
      if (r2 < rci2) {
        const float q = r * ihi, u = fmaf(-0.5f, q, 1.f);
        ws += u * u * u * u * fmaf(2.f, q, 1.f);
      }
      const float hij = kh * (hi + pj.w);
      if (colour_differs(aj, ai) && r2 < hij * hij) {
        const float q = r * sp.kappa * fast_rcp(hij), u = fmaf(-0.5f, q, 1.f);
        wi += u * u * u * u * fmaf(2.f, q, 1.f);
      }
    };
    scan_group_table<D, L, row_table_rows<L>()>((uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row, rs, g,
                                                0u, cstart, pair_body<true>(fetch, use));
    ws = group_sum<L>(ws);
    wi = group_sum<L>(wi);
    if (sub == 0) {
      const float A = sp.alpha * (D == 3 ? sp.inv_tau * sp.inv_tau * sp.inv_tau : sp.inv_tau * sp.inv_tau);
      const float e = A * (1.f + ws) - 1.f;
      e_out[i] = e;
      part[0] = (double)e * (double)e;
      part[1] = (double)wi;
    }
  }
  block_reduce_write<2, L>(part, ops, partials + 2 * (size_t)lb);   // first lanes of the groups
}

// Loss, gradient pass: with ebar = 2 e / n and the interface weight cl = lambda / n,
//   X-bar_k = sum_j u_kj (-5) [ebar_k A u_k^3 / h_k^2 + ebar_j A u_j^3 / h_j^2 + cl [C_j != C_k] u^3 / H^2]
//   s-bar_k = tau sum_j [ebar_k A 5 q_k^2 u_k^3 / h_k + cl [C_j != C_k] 2.5 q^2 u^3 / H]
// (u_k = 1 - r / (2 h_k) inside the support of particle k, etc.).  The search radius covers
// every j whose support reaches k: r < kappa h_j <= kappa h_k / (1 - kappa L_h).
template <int D, int L, bool WIDE>
__global__ __launch_bounds__(kBlock) void loss_grad(const DomDev *__restrict__ dom, const uint32_t *__restrict__ wkey,
                                                    const float4 *__restrict__ wfix, const uint32_t *__restrict__ wjaux,
                                                    const uint32_t *__restrict__ cstart, const float *__restrict__ e,
                                                    float ebar_scale, float cl, float reach_fac,
                                                    float4 *__restrict__ xacc, float *__restrict__ sbar) {
  const int lb = xcd_block(blockIdx.x, gridDim.x);
  const GridDev &g = dom->g;
  const StepDev &sp = dom->sp;
  const int local = lb * kBlock + threadIdx.x;
  const int i = local / L, sub = local % L;
  __shared__ uint2 rowtab[row_table_rows<L>() * row_table_stride<L>()];
  if (i >= dom->n) return;
  const PairPos<D, false, WIDE> pos(g, 0u, i, wkey, wfix);
  const float unit = pos.unit;
  const uint32_t ai = wjaux[i];
  const float hi = pos.h, ihi = fast_rcp(hi);
  const float A = sp.alpha * (D == 3 ? sp.inv_tau * sp.inv_tau * sp.inv_tau : sp.inv_tau * sp.inv_tau);
  const float ebi = ebar_scale * e[i];
  const float rs = fminf(reach_fac * hi, sp.kappa * sp.hmax) * 1.0001f;
  const float kh = 0.5f * sp.kappa;
  float xb[3] = {0.f, 0.f, 0.f}, sb = 0.f;
  const BufRes raux = buf_res(wjaux, 4, (uint32_t)g.n);
  const BufRes re = buf_res(e, 4, (uint32_t)g.n);
  struct Nb {
    typename PairPos<D, false, WIDE>::Nb p;
    uint32_t a, e;
  };
  const auto fetch = [&](uint32_t jr) { return Nb{pos.fetch(jr), buf_u32(raux, jr), buf_u32(re, jr)}; };
  const auto use = [&](const Nb &nb) {
    const float4 pj = nb.p.p;
    const uint32_t aj = nb.a;
    float dx, dy, dz = 0.f;
    pos.sep(nb.p, dx, dy, dz);
    dx *= unit;
    dy *= unit;
    dz *= unit;
    float r2 = dx * dx + dy * dy;
    if constexpr (D == 3) r2 += dz * dz;
    if (!(r2 > 0.f)) return;
    const float r = sqrtf(r2);
    float cx = 0.f;
    const float qi = r * ihi;
    if (qi < sp.kappa) {
      const float u = fmaf(-0.5f, qi, 1.f), u3 = u * u * u;
      cx += ebi * A * u3 * ihi * ihi;
      sb = fmaf(ebi * A * 5.f * qi * qi * u3 * ihi, sp.tau, sb);
    }
    const float ihj = fast_rcp(pj.w), qj = r * ihj;
    if (qj < sp.kappa) {
      const float u = fmaf(-0.5f, qj, 1.f);
      cx += ebar_scale * __uint_as_float(nb.e) * A * u * u * u * ihj * ihj;
    }
    const float hij = kh * (hi + pj.w);
    if (colour_differs(aj, ai) && r2 < hij * hij) {
      const float ih = sp.kappa * fast_rcp(hij), q = r * ih, u = fmaf(-0.5f, q, 1.f), u3 = u * u * u;
      cx += cl * u3 * ih * ih;
      sb = fmaf(cl * 2.5f * q * q * u3 * ih, sp.tau, sb);
    }
    cx *= -5.f;
    xb[0] = fmaf(cx, dx, xb[0]);
    xb[1] = fmaf(cx, dy, xb[1]);
    if constexpr (D == 3) xb[2] = fmaf(cx, dz, xb[2]);
  };
  scan_group_table<D, L, row_table_rows<L>()>((uint32_t)i, sub, rowtab + threadIdx.x / L, row_table_stride<L>(), pos.row, rs, g,
                                              0u, cstart, pair_body<true>(fetch, use));
#pragma unroll
  for (int a = 0; a < 3; ++a) xb[a] = group_sum<L>(xb[a]);
  sb = group_sum<L>(sb);
  if (sub == 0) {
    xacc[i] = make_float4(xb[0], xb[1], xb[2], 0.f);
    sbar[i] = sb;
  }
}

constexpr int kLossThreads = 1024;
// Loss value from the first loss pass's partials: sum e^2 / n + lambda sum_ifc / (2 n).
__global__ __launch_bounds__(kLossThreads) void loss_value(const double *__restrict__ pb, int nb, double inv_n, double lam,
                                                  double *__restrict__ out) {
  __shared__ double r0[kLossThreads], r1[kLossThreads];
  double x = 0.0, y = 0.0;
#pragma unroll 4
  for (int b = threadIdx.x; b < nb; b += kLossThreads) {
    x += pb[2 * (size_t)b];
    y += pb[2 * (size_t)b + 1];
  }
  r0[threadIdx.x] = x;
  r1[threadIdx.x] = y;
  __syncthreads();
  for (int w = kLossThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      r0[threadIdx.x] += r0[threadIdx.x + w];
      r1[threadIdx.x] += r1[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = r0[0] * inv_n + lam * 0.5 * r1[0] * inv_n;
}

// State arrays of a run (a checkpoint or the context's).
struct StateView {
  uint32_t *key;
  float4 *off;
  uint32_t *ct, *id, *cell;
};

// Copies a state, and the metrics where both pointers are given.  A state that becomes the context's
// (counts given, all zero on entry) has its particles counted by cell again, as the load does it, and
// the step counter set to t.  One launch: a copy of each array costs 3 us of its own at 8,192
// particles.
__global__ __launch_bounds__(kBlock) void copy_state(StateView to, StateView from, int n, double *__restrict__ m_to,
                                                     const double *__restrict__ m_from, uint32_t *__restrict__ counts,
                                                     int64_t *__restrict__ stepctr, int64_t t) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (m_to && i < 32) m_to[i] = m_from[i];
  if (counts && i == 0) *stepctr = t;
  if (i >= n) return;
  // all loads before the first store, which the compiler could not move them across
  const uint32_t cell = from.cell[i], key = from.key[i], ct = from.ct[i], id = from.id[i];
  const float4 o = from.off[i];
  const float w = counts ? __uint_as_float(atomicAdd(&counts[cell], 1u)) : o.w;
  to.key[i] = key;
  to.ct[i] = ct;
  to.id[i] = id;
  to.cell[i] = cell;
  to.off[i] = make_float4(o.x, o.y, o.z, w);
}

// Positions adjoint of the first step's start state to the caller's layout (domain units).
template <int D>
__global__ __launch_bounds__(kBlock) void adj_store_pos(int n, const uint32_t *__restrict__ sid,
                                                        const float4 *__restrict__ xbar, float inv_cs,
                                                        float *__restrict__ out) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const float4 x = xbar[i];
  const float xv[3] = {x.x, x.y, x.z};
  const uint32_t id = sid[i];
#pragma unroll
  for (int a = 0; a < D; ++a) out[(size_t)id * D + a] = xv[a] * inv_cs;
}

}  // namespace mpsph
