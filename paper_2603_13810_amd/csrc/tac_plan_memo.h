// Plans that a thread has asked for lately, by geometry.
#pragma once
#include <cstdint>
#include <cstring>

namespace tac {

// In sets of four, so that the layers of a network do not turn each other out (two of them in one place: a choice each, every pass).  One per thread
// (static thread_local): holds geometry only, 64 plans at most.
template <int N, class Plan>
struct PlanMemo {
  struct Entry {
    int key[N];
    Plan plan;
    bool used;
  };
  struct Set {
    Entry entry[4];
    unsigned oldest;
  };
  Set sets[16];

  // The plan of a geometry; choose(plan) forms one that is not there.  nullptr: it found none, and nothing is kept.
  template <class Choose>
  const Plan* of(const int (&key)[N], Choose&& choose) {
    uint32_t hash = 2166136261u;
    for (int v : key) hash = (hash ^ (uint32_t)v) * 16777619u;
    Set& set = sets[(hash >> 16) & 15];
    for (Entry& x : set.entry)
      if (x.used && !std::memcmp(x.key, key, sizeof(key))) return &x.plan;
    Entry& e = set.entry[set.oldest++ & 3];
    e.used = false;
    if (!choose(e.plan)) return nullptr;
    std::memcpy(e.key, key, sizeof(key));
    e.used = true;
    return &e.plan;
  }
};

}  // namespace tac
