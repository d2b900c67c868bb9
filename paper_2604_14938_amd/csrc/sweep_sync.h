// The flags by which the blocks of one launch step together through the sweeps
// of an iteration.  Every function here is run by one wavefront of its block,
// all lanes together; W gives the lanes and the agent-scope memory operations.
#pragma once

#include <stdint.h>

namespace vofpc {

constexpr int kSyncMaxBlocks = 1024;   // blocks at most
constexpr int kSyncRow = kSyncMaxBlocks;
constexpr int kSyncWords = 2 * kSyncRow + 2;   // two rows of barrier flags; blocks that came, blocks that take part
// Polls of a flag before a wait is given up: seconds of running.  Polls and not
// a clock: time in which the whole launch was off the device does not count.
constexpr uint32_t kSyncWaitPolls = 1u << 22;

// Barrier `epoch` (1, 2, ...) of the blocks 0 .. nb - 1, this one `id`.  Returns
// in `any` whether some block brought `mine`.  The flags alternate between two
// rows, so a block that runs ahead cannot overwrite a flag that is still to be
// read.  False when a block's flag did not come within `polls` polls.
template <class W>
__device__ __forceinline__ bool sync_barrier(W w, uint32_t *flag, int id, int nb, uint32_t epoch, bool mine, bool &any,
                                             uint32_t polls = kSyncWaitPolls) {
  uint32_t *row = flag + (epoch & 1) * kSyncRow;
  if (w.lane() == 0) w.store(row + id, (epoch << 1) | (mine ? 1u : 0u));
  bool a = false, ok = true;
  for (int i = w.lane(); i < nb && ok; i += W::kLanes) {
    uint32_t v = w.load(row + i);
    for (uint32_t k = 0; (v >> 1) != epoch && k < polls; ++k) v = w.load(row + i);
    ok = (v >> 1) == epoch;
    a = a || (ok && (v & 1u));
  }
  any = w.any(a);
  return !w.any(!ok);
}

}  // namespace vofpc
