// PlanMemory on a simulated runtime: memory that is handed out never overlaps a live piece, nor one released since the
// last device synchronisation (a launch may still read it).  Prints what fails and returns 1.
#include <stdio.h>
#include <stdlib.h>

#include <chrono>
#include <future>
#include <map>
#include <random>
#include <vector>

#include "plan_memory.h"

namespace {

struct Fake {
  using Error = int;
  using Stream = int*;
  static constexpr Error kSuccess = 0, kOutOfMemory = 2;
  static std::map<char*, size_t> blocks;
  static size_t used, limit;
  static Error last;
  static int syncs, copies_to_fail, streams;
  static bool (*while_freeing)();
  static bool free_blocked;
  static std::mutex mu;

  static Error malloc(void** p, size_t n) {
    std::lock_guard<std::mutex> lock(mu);
    if (used + n > limit) return last = kOutOfMemory;
    char* c = static_cast<char*>(::malloc(n));
    blocks[c] = n;
    used += n;
    *p = c;
    return kSuccess;
  }
  static void free(void* p) {
    if (while_freeing && !while_freeing()) free_blocked = true;
    std::lock_guard<std::mutex> lock(mu);
    used -= blocks.at(static_cast<char*>(p));
    blocks.erase(static_cast<char*>(p));
    ::free(p);
  }
  static Error device_synchronize();
  static void clear_error() { last = kSuccess; }
  static Error stream_create(Stream* s) {
    ++streams;
    *s = new int(streams);
    return kSuccess;
  }
  static Error copy(void*, const void*, size_t, Stream) { return copies_to_fail > 0 ? --copies_to_fail, last = 1 : 0; }
  static Error stream_synchronize(Stream) { return kSuccess; }
};
std::map<char*, size_t> Fake::blocks;
size_t Fake::used = 0, Fake::limit = ~size_t(0);
Fake::Error Fake::last = 0;
int Fake::syncs = 0, Fake::copies_to_fail = 0, Fake::streams = 0;
bool (*Fake::while_freeing)() = nullptr;
bool Fake::free_blocked = false;
std::mutex Fake::mu;

using Memory = pkv::PlanMemory<Fake>;
std::map<char*, size_t> live, released;  // handed out, by address; released since the last synchronisation
int failures = 0;

#define CHECK(x)                                            \
  do {                                                      \
    if (!(x)) {                                             \
      printf("line %d: %s\n", __LINE__, #x);                \
      ++failures;                                           \
    }                                                       \
  } while (0)

Fake::Error Fake::device_synchronize() {
  ++syncs;
  released.clear();
  return kSuccess;
}

bool clear_of(const std::map<char*, size_t>& m, char* p, size_t n) {
  auto it = m.lower_bound(p);
  if (it != m.end() && it->first < p + n) return false;
  if (it == m.begin()) return true;
  --it;
  return it->first + it->second <= p;
}

char* take(Memory& m, size_t n) {
  void* p = nullptr;
  if (m.allocate(n, &p) != Fake::kSuccess) return nullptr;
  char* c = static_cast<char*>(p);
  auto b = Fake::blocks.upper_bound(c);
  CHECK(b != Fake::blocks.begin());
  --b;
  CHECK(c + n <= b->first + b->second);  // inside an allocation
  CHECK((c - b->first) % 256 == 0);
  CHECK(clear_of(live, c, n));
  CHECK(clear_of(released, c, n));
  live[c] = n;
  return c;
}

void give(Memory& m, char* p) {
  const size_t n = live.at(p);
  live.erase(p);
  released[p] = n;
  m.release(p);
  // What went back to the runtime was synchronised by it.
  for (auto it = released.begin(); it != released.end();) {
    auto b = Fake::blocks.upper_bound(it->first);
    const bool inside = b != Fake::blocks.begin() && (--b, it->first < b->first + b->second);
    it = inside ? std::next(it) : released.erase(it);
  }
}

void random_plans(uint32_t seed, size_t largest) {
  Memory m;
  std::mt19937 rng(seed);
  std::vector<char*> held;
  for (int i = 0; i < 4000; ++i) {
    if (!held.empty() && rng() % 100 < 48) {
      const size_t k = rng() % held.size();
      give(m, held[k]);
      held.erase(held.begin() + long(k));
    } else if (char* p = take(m, 1 + rng() % largest)) {
      held.push_back(p);
    } else {
      CHECK(!"allocation failed");
    }
  }
  for (char* p : held) give(m, p);
  CHECK(Fake::used == 0);
}

// Plans of 100 KB that live for one restore, every 20th of them kept: what is kept must not hold slabs back.
void kept_plans() {
  Memory m;
  std::vector<char*> kept;
  const int before = Fake::syncs;
  for (int i = 0; i < 4000; ++i) {
    char* p = take(m, 100 << 10);
    if (i % 20 == 0 && kept.size() < 50)
      kept.push_back(p);
    else
      give(m, p);
  }
  const size_t bytes = kept.size() * (100 << 10);
  CHECK(Fake::used <= 2 * bytes + 2 * Memory::kSlab);
  CHECK(Fake::syncs - before <= 4000 / 20 + 2);  // one for each half slab of released plans at most
  for (char* p : kept) give(m, p);
  CHECK(Fake::used == 0);
}

void little_memory() {
  Memory m;
  Fake::limit = size_t(1) << 20;  // no room for a slab
  char* a = take(m, 100 << 10);
  CHECK(a != nullptr);
  CHECK(Fake::last == Fake::kSuccess);
  void* p = nullptr;
  CHECK(m.allocate(2 << 20, &p) == Fake::kOutOfMemory);
  CHECK(Fake::last == Fake::kSuccess);  // the next launch does not report it
  if (a) give(m, a);
  // Room for one slab: when it is full, released plans make place, short of half a slab too.
  Fake::limit = Memory::kSlab;
  std::vector<char*> all;
  for (int i = 0; i < 4; ++i) all.push_back(take(m, 1 << 20));
  CHECK(all.back() != nullptr);
  give(m, all[1]);
  all[1] = take(m, 900 << 10);
  CHECK(all[1] != nullptr);
  for (char* c : all)
    if (c) give(m, c);
  Fake::limit = ~size_t(0);
  CHECK(Fake::used == 0);
}

// Another thread makes a plan while one waits in free.
Memory* shared = nullptr;
bool makes_a_plan() {
  Fake::while_freeing = nullptr;
  auto other = std::async(std::launch::async, [] {
    void* p = nullptr;
    return shared->allocate(1000, &p) == Fake::kSuccess;
  });
  const bool done = other.wait_for(std::chrono::seconds(5)) == std::future_status::ready;
  if (!done) {
    printf("a plan build waits for another plan's free\n");
    exit(1);
  }
  return other.get();
}

void free_without_lock() {
  Memory m;
  shared = &m;
  void *small = nullptr, *big = nullptr;
  CHECK(m.allocate(1000, &small) == 0 && m.allocate(3 << 20, &big) == 0);
  Fake::while_freeing = makes_a_plan;
  m.release(big);  // an allocation of its own
  CHECK(!Fake::free_blocked);
}

void upload_after_reset() {
  Memory m;
  char from[4] = {}, to[4];
  CHECK(m.upload(to, from, 4) == 0);
  const int streams = Fake::streams;
  CHECK(m.upload(to, from, 4) == 0 && Fake::streams == streams);  // the stream is kept
  Fake::copies_to_fail = 1;
  CHECK(m.upload(to, from, 4) == 0 && Fake::streams == streams + 1);
  Fake::copies_to_fail = 2;
  CHECK(m.upload(to, from, 4) == 1 && Fake::last == Fake::kSuccess);
  Fake::copies_to_fail = 0;
  CHECK(m.upload(to, from, 4) == 0);
}

}  // namespace

int main() {
  for (uint32_t seed = 1; seed <= 6; ++seed) random_plans(seed, seed % 2 ? 300 << 10 : 2 << 20);
  kept_plans();
  little_memory();
  upload_after_reset();
  free_without_lock();
  printf("%d failures\n", failures);
  return failures != 0;
}
