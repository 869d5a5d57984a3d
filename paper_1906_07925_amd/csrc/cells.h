// Host interface of the counting order of the particles by cell key.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mpsph {

// Optional per-launch hook (event timing); begin() before a launch, end() after it.
struct LaunchHook {
  virtual void begin(const char *name) = 0;
  virtual void end() = 0;
  virtual ~LaunchHook() = default;
};

// Entries of the count array for ncells cells: whole tiles of the scan, the rest zero.
size_t cell_count_words(uint32_t ncells);
// Words of the tile sums, all zero before and after an order.
size_t cell_sum_words(uint32_t ncells);

// From the particles counted per cell (counts[key]) and each one's arrival number in its cell (the bits of
// off[i].w): the cell table cstart[c] = particles in cells below c
// (c <= ncells), and the particles grouped by cell, slots[s] for s in [cstart[c], cstart[c + 1])
// naming those of cell c in an unspecified order.  Leaves counts all zero, or with keep as they are.
// Enqueued on stream.
hipError_t cell_order(const uint32_t *keys, const float4 *off, uint32_t *counts, uint32_t *sums, uint32_t *cstart,
                      uint32_t *slots, int n, uint32_t ncells, bool keep, hipStream_t stream, LaunchHook *hook);

}  // namespace mpsph
