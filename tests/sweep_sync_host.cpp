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
  bool any(bool b) const { return b; }
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
  CHECK(sync_barrier(w, flag.data(), 0, 1, 1, true, any, 5) && any);
  left = 6;
  CHECK(!sync_barrier(w, flag.data(), 0, 1, 2, true, any, 5));
}

static void agreement(int nb, int epochs) {
  std::vector<uint32_t> flag(kSyncWords, 0);
  std::vector<std::thread> t;
  std::atomic<int> wrong{0};
  for (int id = 0; id < nb; ++id)
    t.emplace_back([&, id] {
      for (int e = 1; e <= epochs; ++e) {
        bool any = false;
        const bool ok = sync_barrier(HostSync(), flag.data(), id, nb, e, (e * 7 + id) % (nb + 3) == 0, any);
        bool want = false;
        for (int i = 0; i < nb; ++i) want = want || (e * 7 + i) % (nb + 3) == 0;
        if (!ok || any != want) ++wrong;
      }
    });
  for (auto &x : t) x.join();
  CHECK(wrong == 0);
}

static void missing_block() {
  std::vector<uint32_t> flag(kSyncWords, 0);
  std::vector<std::thread> t;
  std::atomic<int> gave_up{0};
  for (int id = 0; id < 2; ++id)   // block 2 never comes
    t.emplace_back([&, id] {
      bool any;
      if (!sync_barrier(HostSync(), flag.data(), id, 3, 1, false, any, 1000)) ++gave_up;
    });
  for (auto &x : t) x.join();
  CHECK(gave_up == 2);
}

int main() {
  last_poll();
  agreement(1, 50);
  agreement(5, 200);
  missing_block();
  std::printf("ok\n");
  return 0;
}
