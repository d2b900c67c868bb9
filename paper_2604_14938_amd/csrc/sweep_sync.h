// The flags by which the blocks of one launch step together through the sweeps
// of an iteration.  Every function here is run by one wavefront of its block,
// all lanes together; W gives the lanes and the agent-scope memory operations.
//
// A block takes part from the sweep after it was let in.  The first block to
// come leads: it waits a little for the others (sync_enter), starts the sweeps
// with those that are there, and at every barrier lets in those that have come
// since.  So every block that another one waits for is running, however few of
// an ordinary launch's blocks find room, and a chip that was busy at the start
// is in use from the first sweep after its blocks do find room.
#pragma once

#include <stdint.h>

namespace vofpc {

constexpr int kSyncMaxBlocks = 1024;   // blocks at most
constexpr int kSyncRow = kSyncMaxBlocks;
constexpr int kSyncWords = 3 * kSyncRow + 1;   // two rows of barrier flags, the letters, the count of blocks that came
constexpr int kSyncLetter = 2 * kSyncRow, kSyncCame = 3 * kSyncRow;   // places of the last two
constexpr uint32_t kSyncClosed = 0x80000000u;  // in the count: the sweeps are over
constexpr uint32_t kSyncEnd = 0xffffffffu;     // letter of a block that came too late
// Polls of a flag before a wait is given up: seconds of running.  Polls and not
// a clock: time in which the whole launch was off the device does not count.
constexpr uint32_t kSyncWaitPolls = 1u << 22;
// Polls for which the leader waits for the others before the first sweep, about
// 50 us; on an idle chip all come within a few.
constexpr uint32_t kSyncGatherPolls = 64;

// A flag: the epoch, the number of blocks after it (the leader's flag alone),
// and whether the block brought its verdict.  A letter: the epoch after which
// the block takes part, the number of blocks up to it, and a set low bit.
__device__ __forceinline__ uint32_t sync_word(uint32_t epoch, uint32_t blocks, bool bit) {
  return (epoch << 12) | (blocks << 1) | (bit ? 1u : 0u);
}
__device__ __forceinline__ int sync_blocks(uint32_t word) { return (int)((word >> 1) & 0x7ffu); }

// The flags of barrier `epoch` by the blocks 0 .. nb - 1: whether some block
// brought its verdict, and the number of blocks after it.  False when a flag did
// not come within `polls` polls.
template <class W>
__device__ __forceinline__ bool sync_wait(W w, uint32_t *flag, int nb, uint32_t epoch, bool &any, int &next,
                                          uint32_t polls) {
  const uint32_t *row = flag + (epoch & 1) * kSyncRow;
  bool a = false, ok = true;
  int n = 0;
  for (int i = w.lane(); i < nb && ok; i += W::kLanes) {
    uint32_t v = w.load(row + i);
    for (uint32_t k = 0; (v >> 12) != epoch && k < polls; ++k) v = w.load(row + i);
    ok = (v >> 12) == epoch;
    a = a || (ok && (v & 1u));
    if (i == 0) n = sync_blocks(v);
  }
  any = w.any(a);
  next = w.first(n);
  return !w.any(!ok);
}

// Barrier `epoch` (1, 2, ...) of the blocks 0 .. nb - 1, this one `id`; nb is
// then the number of blocks of the next sweep, of at most `want`.  Returns in
// `any` whether some block brought `mine`.  The flags alternate between two
// rows, so a block that runs ahead cannot overwrite a flag that is still to be
// read, also by a block that the leader has just let in: it takes part in the
// next barrier.  False when a wait failed.
template <class W>
__device__ __forceinline__ bool sync_barrier(W w, uint32_t *flag, int id, int &nb, int want, uint32_t epoch, bool mine,
                                             bool &any, uint32_t polls = kSyncWaitPolls) {
  int next = nb;
  if (id == 0 && nb < want) {
    const int came = (int)w.first((int)w.load(flag + kSyncCame));
    next = came < want ? came : want;
    for (int i = nb + w.lane(); i < next; i += W::kLanes) w.store(flag + kSyncLetter + i, sync_word(epoch, nb, true));
  }
  if (w.lane() == 0) w.store(flag + (epoch & 1) * kSyncRow + id, sync_word(epoch, id == 0 ? next : 0, mine));
  return sync_wait(w, flag, nb, epoch, any, nb, polls);
}

// This block's number, the barrier after which it takes part (0: from the
// start) and the number of blocks then; -1 when the sweeps ended first.  The
// wait for the letter ends because the leader runs, and writes one to every
// block that has come before it ends (sync_close).
template <class W>
__device__ __forceinline__ int sync_enter(W w, uint32_t *flag, int want, int &epoch, int &nb,
                                          uint32_t gather = kSyncGatherPolls) {
  epoch = 0;
  nb = 1;
  const uint32_t k = (uint32_t)w.first(w.lane() == 0 ? (int)w.fetch_add(flag + kSyncCame, 1u) : 0);
  if (k & kSyncClosed) return -1;
  if (k == 0) {
    for (uint32_t p = 0; p < gather && nb < want; ++p) nb = w.first((int)w.load(flag + kSyncCame));
    if (nb > want) nb = want;
    for (int i = 1 + w.lane(); i < nb; i += W::kLanes) w.store(flag + kSyncLetter + i, sync_word(0, nb, true));
    return 0;
  }
  uint32_t letter = 0;
  while (letter == 0) letter = (uint32_t)w.first((int)w.load(flag + kSyncLetter + k));
  if (letter == kSyncEnd) return -1;
  epoch = (int)(letter >> 12);
  nb = sync_blocks(letter);
  if (epoch > 0) {
    bool any;
    if (!sync_wait(w, flag, nb, (uint32_t)epoch, any, nb, kSyncWaitPolls) || !any) return -1;
  }
  return (int)k;
}

// The leader's last act: blocks that were not let in (nb were) are told to end.
template <class W>
__device__ __forceinline__ void sync_close(W w, uint32_t *flag, int nb) {
  const int came = w.first(w.lane() == 0 ? (int)w.fetch_or(flag + kSyncCame, kSyncClosed) : 0);
  for (int i = nb + w.lane(); i < came; i += W::kLanes) w.store(flag + kSyncLetter + i, kSyncEnd);
}

}  // namespace vofpc
