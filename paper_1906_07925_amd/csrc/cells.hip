// Counting order of the particles by cell key (gfx950, wave64).
//
// The cell table itself is the sort: whoever writes a particle's key (the load, the integrator)
// adds it to its cell's count and keeps its arrival number, and one step then needs
//   cell_sums   sums of tiles of kScanTile counts (large tables only)
//   cell_scan   exclusive prefix of the counts = the cell table
//   cell_place  every particle's index to slot cstart[key] + arrival; the counts back to zero
// (cell_order_small does all of it in one block for small sets)
// The arrival order inside a cell depends on timing; the gather that follows ranks each
// particle among its cell's slots by index, so the final order is that of a stable sort by key.
// Bound by launch latency up to ~10^5 particles and beyond by the table's bytes (12 per entry; at
// most 4 entries per particle by the sub-cell rule, 8 per particle or 2^20 a domain by the rows) and one atomic per
// particle.
// Measured per step (scan, place and gather, against radix passes with their gather and gap fill):
// 4096 particles 9.4 us against 54, 262,144 in 2D 25 against 98, 2M with 4M cells 56 against 133.
#include "cells.h"

#include <algorithm>

namespace mpsph {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;   // counts per thread, four 16-byte loads
constexpr uint32_t kScanTile = kScanThreads * kScanItems;
// Tables of up to this many tiles are scanned by one launch, whose blocks publish their sums: at 16 tiles 4.7 us
// against 7.9 with every block adding up the counts before its tile (seeded ball of 20000, 4 steps 287 ->
// 271 us).  Larger tables have a launch of cell_sums first: waiting for the sums of 256 tiles takes as long as
// that launch (annulus of 2^18 particles 304 us against 298).
constexpr uint32_t kPublishTiles = 64;
// Polls of a tile's sum before a block adds the tile up itself, so that no block depends on another
// one having started.
constexpr int kSumPolls = 1024;
constexpr uint32_t kSumReady = 0x80000000u;   // sums stay below 2^31

__device__ __forceinline__ uint32_t wave_inclusive(uint32_t x, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(x, o, 64);
    if (lane >= o) x += u;
  }
  return x;
}

// Sum over the block, in every thread.  lds: kScanThreads / 64 words.
__device__ __forceinline__ uint32_t block_sum(uint32_t x, uint32_t *lds) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = x;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / 64; ++w) t += lds[w];
  return t;
}

__global__ __launch_bounds__(kScanThreads) void cell_sums(const uint4 *__restrict__ counts, uint32_t *__restrict__ sums) {
  __shared__ uint32_t lds[kScanThreads / 64];
  const uint4 *c = counts + (size_t)blockIdx.x * (kScanTile / 4);
  uint32_t s = 0;
#pragma unroll
  for (int q = 0; q < kScanItems / 4; ++q) {
    const uint4 v = c[q * kScanThreads + threadIdx.x];
    s += v.x + v.y + v.z + v.w;
  }
  s = block_sum(s, lds);
  if (threadIdx.x == 0) sums[blockIdx.x] = kSumReady | s;
}

// One tile per block.  With publish a block stores its tile's sum for the others; it adds up the sums of
// the tiles before it as they appear.  sums is all zero on entry, or filled by cell_sums; cell_place
// clears it.
__global__ __launch_bounds__(kScanThreads) void cell_scan(const uint4 *__restrict__ counts, uint32_t *__restrict__ sums,
                                                          uint32_t *__restrict__ cstart, uint32_t ncells, uint32_t n,
                                                          int publish) {
  __shared__ uint32_t lds[2][kScanThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  // each thread's counts are consecutive
  uint32_t v[kScanItems];
  const uint4 *c = counts + (size_t)blockIdx.x * (kScanTile / 4) + (size_t)threadIdx.x * (kScanItems / 4);
#pragma unroll
  for (int q = 0; q < kScanItems / 4; ++q) {
    const uint4 u = c[q];
    v[4 * q] = u.x;
    v[4 * q + 1] = u.y;
    v[4 * q + 2] = u.z;
    v[4 * q + 3] = u.w;
  }
  uint32_t own = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) own += v[q];
  const uint32_t incl = wave_inclusive(own, lane);
  if (lane == 63) lds[1][w] = incl;
  __syncthreads();
  if (publish && threadIdx.x == 0) {
    uint32_t t = kSumReady;
#pragma unroll
    for (int ww = 0; ww < kScanThreads / 64; ++ww) t += lds[1][ww];
    __hip_atomic_store(&sums[blockIdx.x], t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // everything before the tile
  uint32_t before = 0;
  for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kScanThreads) {
    uint32_t x = 0;
    for (int k = 0; k < kSumPolls && x == 0; ++k) x = __hip_atomic_load(&sums[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (x == 0)
      for (uint32_t q = 0; q < kScanTile / 4; ++q) {
        const uint4 u = counts[(size_t)t * (kScanTile / 4) + q];
        x += u.x + u.y + u.z + u.w;
      }
    before += x & ~kSumReady;
  }
  before = block_sum(before, lds[0]);
  uint32_t run = before + incl - own;
  for (int ww = 0; ww < w; ++ww) run += lds[1][ww];
  const uint32_t c0 = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const uint32_t t = v[q];
    v[q] = run;
    run += t;
  }
  if (c0 + kScanItems <= ncells) {
    uint4 *o = reinterpret_cast<uint4 *>(cstart + c0);
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) o[q] = make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  } else {
#pragma unroll
    for (int q = 0; q < kScanItems; ++q)
      if (c0 + q < ncells) cstart[c0 + q] = v[q];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) cstart[ncells] = n;
}

__global__ __launch_bounds__(256) void cell_place(const uint32_t *__restrict__ keys, const float4 *__restrict__ off,
                                                  const uint32_t *__restrict__ cstart, uint4 *__restrict__ counts,
                                                  uint32_t nquads, uint32_t *__restrict__ sums, uint32_t nsums,
                                                  uint32_t *__restrict__ slots, int n) {
  const uint32_t t = blockIdx.x * 256u + threadIdx.x, stride = gridDim.x * 256u;
  for (uint32_t q = t; q < nquads; q += stride) counts[q] = make_uint4(0u, 0u, 0u, 0u);
  for (uint32_t q = t; q < nsums; q += stride) sums[q] = 0u;
  if (t >= (uint32_t)n) return;
  const uint32_t at = cstart[keys[t]] + __float_as_uint(off[t].w);
  if (at < (uint32_t)n) slots[at] = t;
}

// Scan, place and clearing of a set whose table is one tile, in one block: a 16-byte load of the
// counts per thread and up to kSmallItems particles.  Latency only: the particles' keys are loaded with
// the counts, and what a second launch would cost (its start and the gap before it) is saved.
constexpr int kSmallThreads = 1024, kSmallItems = 4;
__global__ __launch_bounds__(kSmallThreads) void cell_order_small(const uint32_t *__restrict__ keys,
                                                                  const float4 *__restrict__ off, uint4 *counts,
                                                                  uint32_t *cstart, uint32_t *__restrict__ slots, uint32_t n,
                                                                  uint32_t ncells, int keep) {
  static_assert(kScanTile == 4 * kSmallThreads, "one load per thread");
  __shared__ uint32_t lds[kSmallThreads / 64];
  const uint32_t tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const uint4 v = counts[tid];
  uint32_t key[kSmallItems], arr[kSmallItems];
#pragma unroll
  for (int q = 0; q < kSmallItems; ++q) {
    const uint32_t t = tid + (uint32_t)q * kSmallThreads;
    if (t < n) {
      key[q] = keys[t];
      arr[q] = __float_as_uint(off[t].w);
    }
  }
  if (!keep) counts[tid] = make_uint4(0u, 0u, 0u, 0u);
  const uint32_t own = v.x + v.y + v.z + v.w;
  const uint32_t incl = wave_inclusive(own, lane);
  if (lane == 63) lds[w] = incl;
  __syncthreads();
  uint32_t run = incl - own;
#pragma unroll
  for (int ww = 0; ww < kSmallThreads / 64; ++ww) run += ww < w ? lds[ww] : 0u;
  const uint32_t at = tid * 4u;
  const uint4 u = make_uint4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
  if (at + 4u <= ncells) {
    *reinterpret_cast<uint4 *>(cstart + at) = u;
  } else {
    if (at < ncells) cstart[at] = u.x;
    if (at + 1u < ncells) cstart[at + 1u] = u.y;
    if (at + 2u < ncells) cstart[at + 2u] = u.z;
  }
  if (tid == 0) cstart[ncells] = n;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSmallItems; ++q) {
    const uint32_t t = tid + (uint32_t)q * kSmallThreads;
    if (t < n) {
      const uint32_t to = cstart[key[q]] + arr[q];
      if (to < n) slots[to] = t;
    }
  }
}

size_t cell_sum_words(uint32_t ncells) { return ((size_t)ncells + kScanTile - 1) / kScanTile; }
size_t cell_count_words(uint32_t ncells) { return cell_sum_words(ncells) * kScanTile; }

hipError_t cell_order(const uint32_t *keys, const float4 *off, uint32_t *counts, uint32_t *sums, uint32_t *cstart,
                      uint32_t *slots, int n, uint32_t ncells, bool keep, hipStream_t stream, LaunchHook *hook) {
  const uint32_t tiles = (uint32_t)cell_sum_words(ncells);
  const uint4 *c4 = reinterpret_cast<const uint4 *>(counts);
  // One block for up to 4,096 particles with a table of one tile: 3.4 us in place of two launches of 2.5
  // and 1.8 us with a gap between them (a call of one step of 1,024 particles 94 -> 90.5 us).  With a table of 4
  // tiles the block takes 6.3 us and a step is 1 us slower than with the two launches.
  if (n > 0 && n <= kSmallThreads * kSmallItems && tiles == 1) {
    if (hook) hook->begin("cell_scan");
    cell_order_small<<<1, kSmallThreads, 0, stream>>>(keys, off, reinterpret_cast<uint4 *>(counts), cstart, slots, (uint32_t)n,
                                                      ncells, keep ? 1 : 0);
    if (hook) hook->end();
    return hipGetLastError();
  }
  if (hook) hook->begin("cell_scan");
  if (tiles > kPublishTiles) cell_sums<<<tiles, kScanThreads, 0, stream>>>(c4, sums);
  cell_scan<<<tiles, kScanThreads, 0, stream>>>(c4, sums, cstart, ncells, (uint32_t)n, tiles <= kPublishTiles ? 1 : 0);
  if (hook) hook->end();
  if (hook) hook->begin("cell_place");
  cell_place<<<(n + 255) / 256, 256, 0, stream>>>(keys, off, cstart, reinterpret_cast<uint4 *>(counts),
                                                  keep ? 0u : tiles * (kScanTile / 4), sums, tiles, slots, n);
  if (hook) hook->end();
  return hipGetLastError();
}

}  // namespace mpsph
