// The sweep flags with host threads for blocks (one lane each).
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#define __device__
#define __forceinline__ inline
#include "sweep_sync.h"

using namespace vofpc;

#define CHECK(c)                                              \
  do {                                                        \
    if (!(c)) {                                               \
      std::printf("line %d: %s\n", __LINE__, #c);             \
      std::exit(1);                                           \
    }                                                         \
  } while (0)

struct HostSync {
  static constexpr int kLanes = 1;
  int lane() const { return 0; }
  uint32_t load(const uint32_t *a) const {
    std::this_thread::yield();
    return __atomic_load_n(a, __ATOMIC_SEQ_CST);
  }
  void store(uint32_t *a, uint32_t v) const { __atomic_store_n(a, v, __ATOMIC_SEQ_CST); }
  uint32_t fetch_add(uint32_t *a, uint32_t v) const { return __atomic_fetch_add(a, v, __ATOMIC_SEQ_CST); }
  uint32_t fetch_or(uint32_t *a, uint32_t v) const { return __atomic_fetch_or(a, v, __ATOMIC_SEQ_CST); }
  bool any(bool b) const { return b; }
  int first(int v) const { return v; }
};

// a flag that arrives with the last poll
struct LastPoll : HostSync {
  uint32_t *left;
  uint32_t load(const uint32_t *a) const { return (*left)-- ? 0 : *a; }
};

static void last_poll() {
  std::vector<uint32_t> flag(kSyncWords, 0);
  uint32_t left = 5;   // the first load and four polls find nothing
  LastPoll w;
  w.left = &left;
  bool any = false;
  int nb = 1;
  CHECK(sync_barrier(w, flag.data(), 0, nb, 1, 1, true, any, 5) && any && nb == 1);
  left = 6;
  CHECK(!sync_barrier(w, flag.data(), 0, nb, 1, 2, true, any, 5));
}

// `want` blocks sweep `cells` cells `sweeps` times (or until the verdict after
// `stop` sweeps), the blocks from `there` on only come once sweep `from` has
// begun (or all are through): every cell is done once in every sweep, from
// values of the sweep before, whoever does it; late blocks do their share.
static void iterate(int want, int there, int cells, int sweeps, int stop, int from) {
  std::vector<uint32_t> flag(kSyncWords, 0);
  std::vector<std::atomic<int>> done(cells);   // sweeps done of each cell
  for (auto &d : done) d = 0;
  std::atomic<int> begun{0}, through{0}, wrong{0}, outputs{0};
  std::vector<int> work(want, 0);
  const int last = stop < sweeps ? stop : sweeps;
  const bool all_come = from + 5 < last;
  auto block = [&](int) {
    int e = 0, nb = 0;
    const int id = sync_enter(HostSync(), flag.data(), want, e, nb, there < want ? 1000 : 1 << 30);
    if (id < 0) return;
    int in = nb, s = e;
    bool ok = true;
    while (s < sweeps) {
      if (id == 0) begun = s + 1;
      if (id == 0 && all_come && s == from + 2)   // the late ones are at the door
        while (HostSync().load(&flag[kSyncCame]) < (uint32_t)want) {
        }
      for (int c = id; c < cells; c += nb) {
        if (done[c].fetch_add(1) != s) ++wrong;
        ++work[id];
      }
      ++s;
      if (s == sweeps) break;
      bool more;
      ok = sync_barrier(HostSync(), flag.data(), id, in, want, s, s < stop, more);
      if (!ok || !more) break;
      nb = in;
    }
    if (id == 0 && in < want) sync_close(HostSync(), flag.data(), in);
    if (!ok) ++wrong;
    for (int c = id; c < cells; c += nb) ++outputs;
    if (id == 0) through = s;
  };
  std::vector<std::thread> t;
  for (int i = 0; i < want; ++i)
    t.emplace_back([&, i] {
      while (i >= there && begun < from && through == 0) std::this_thread::yield();
      block(i);
    });
  for (auto &x : t) x.join();
  CHECK(wrong == 0);
  CHECK(through == last);
  CHECK(outputs == cells);
  for (auto &d : done) CHECK(d == last);
  if (all_come)
    for (int i = 0; i < want && i < cells; ++i) CHECK(work[i] > 0);
}

static void missing_block() {
  std::vector<uint32_t> flag(kSyncWords, 0);
  std::vector<std::thread> t;
  std::atomic<int> gave_up{0};
  for (int id = 0; id < 2; ++id)   // block 2 never comes
    t.emplace_back([&, id] {
      bool any;
      int nb = 3;
      if (!sync_barrier(HostSync(), flag.data(), id, nb, 3, 1, false, any, 1000)) ++gave_up;
    });
  for (auto &x : t) x.join();
  CHECK(gave_up == 2);
}

int main() {
  last_poll();
  missing_block();
  for (int rep = 0; rep < 20; ++rep) {
    iterate(1, 1, 7, 30, 100, 0);
    iterate(5, 5, 23, 60, 100, 0);      // all there
    iterate(5, 5, 23, 60, 17, 0);
    iterate(6, 1, 40, 100, 1000, 3);    // late, in the middle
    iterate(6, 3, 40, 100, 90, 20);
    iterate(6, 3, 2, 60, 1000, 5);     // more blocks than cells
    iterate(6, 2, 40, 12, 100, 11);     // about the last sweep
    iterate(6, 2, 40, 12, 6, 6);        // about the verdict
    iterate(6, 2, 40, 5, 100, 9);       // too late
  }
  std::printf("ok\n");
  return 0;
}
