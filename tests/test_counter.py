"""The arrival counters of cut items (csrc/pa_counter.h), the very code that the
kernels run, compiled for the host: of n parts exactly one, the last, is told to
merge and the counter is left at 0, whatever the word held beforehand (what an
earlier call left with any 1, 2 or 4 of its bytes written over, the residue of
calls that overlapped, random bytes) and however the parts' atomics interleave;
and the next call finds the word in order."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_09345_amd", "csrc")

SOURCE = r"""
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <random>
#include <thread>
#include <vector>
#include "pa_counter.h"
using namespace pa;

#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf("\n"); std::exit(1); } } while (0)

struct Plain {  // parts one after the other
  uint64_t v;
  int ops = 0;
  uint64_t fetch_add(uint64_t x) { ++ops; uint64_t o = v; v += x; return o; }
  bool swap(uint64_t& e, uint64_t x) { ++ops; if (v == e) { v = x; return true; } e = v; return false; }
  void store(uint64_t x) { ++ops; v = x; }
};

static uint64_t g_call = 12345;

static void in_turn(uint64_t start, int n, const char* what) {
  Plain w{start};
  for (int again = 0; again < 2; ++again) {  // the call, and the one after it
    const CounterKey key = counter_key(g_call++);
    CHECK(key.step * key.inverse == 1, "inverse");
    for (int i = 0; i < n; ++i) {
      const bool last = counter_arrive(w, key, n);
      CHECK(last == (i == n - 1), "%s: start %016llx n %d: part %d told %d", what, (unsigned long long)start, n, i, last);
    }
    CHECK(w.v == 0, "%s: left %016llx", what, (unsigned long long)w.v);
  }
}

// Parts in threads, one atomic at a time in the order that `pick` chooses.
struct Baton {
  std::mutex mu;
  std::condition_variable cv;
  int turn = -1;  // the part whose atomic may run
  std::vector<int> waiting, done;
  uint64_t v;
};
struct Shared {
  Baton& b;
  int id;
  template <typename F> auto step(F f) {
    std::unique_lock<std::mutex> l(b.mu);
    b.waiting[id] = 1;
    b.cv.notify_all();
    b.cv.wait(l, [&] { return b.turn == id; });
    b.turn = -1;
    b.waiting[id] = 0;
    return f();
  }
  uint64_t fetch_add(uint64_t x) { return step([&] { uint64_t o = b.v; b.v += x; return o; }); }
  bool swap(uint64_t& e, uint64_t x) {
    return step([&] { if (b.v == e) { b.v = x; return true; } e = b.v; return false; });
  }
  void store(uint64_t x) { step([&] { b.v = x; return 0; }); }
};

static void interleaved(uint64_t start, int n, std::mt19937_64& rng) {
  Baton b;
  b.v = start;
  b.waiting.assign(n, 0);
  b.done.assign(n, 0);
  const CounterKey key = counter_key(g_call++);
  std::vector<int> last(n, 0);
  std::vector<std::thread> t;
  for (int i = 0; i < n; ++i)
    t.emplace_back([&, i] {
      Shared w{b, i};
      const bool l = counter_arrive(w, key, n);
      std::unique_lock<std::mutex> lk(b.mu);
      last[i] = l;
      b.done[i] = 1;
      b.cv.notify_all();
    });
  int steps = 0;
  for (;;) {
    std::unique_lock<std::mutex> l(b.mu);
    b.cv.wait(l, [&] {
      if (b.turn != -1) return false;
      for (int i = 0; i < n; ++i) if (!b.waiting[i] && !b.done[i]) return false;
      return true;
    });
    std::vector<int> can;
    for (int i = 0; i < n; ++i) if (b.waiting[i]) can.push_back(i);
    if (can.empty()) break;
    CHECK(++steps < 100 * n, "no end");
    b.turn = can[rng() % can.size()];
    b.cv.notify_all();
  }
  for (auto& x : t) x.join();
  int merges = 0;
  for (int x : last) merges += x;
  CHECK(merges == 1 && b.v == 0, "start %016llx n %d: %d merges, left %016llx", (unsigned long long)start, n, merges,
        (unsigned long long)b.v);
}

int main() {
  std::mt19937_64 rng(7);
  const int ns[] = {2, 3, 8, 13, 16, 32, 1024};
  for (int n : ns) {
    in_turn(0, n, "fresh");
    Plain one{0};
    const CounterKey key = counter_key(g_call++);
    for (int i = 0; i < n; ++i) counter_arrive(one, key, n);
    CHECK(one.ops == n + 1, "an atomic per part and one store, not %d", one.ops);
    // what a call left (0), with bytes written over
    for (int size : {1, 2, 4})
      for (int at = 0; at + size <= 8; ++at)
        for (int pat = 0; pat < (size == 1 ? 256 : 64); ++pat) {
          const uint32_t fixed[] = {0u, 1u, 5u, 0x3f80u, 0xffffffffu, 0x3f803f80u, 0x7fc0u, 0x10000u};
          const uint32_t x = size == 1 ? (uint32_t)pat : pat < 8 ? fixed[pat] : (uint32_t)rng();
          uint64_t v = 0;
          std::memcpy(reinterpret_cast<char*>(&v) + at, &x, size);
          in_turn(v, n, "written over");
          // and the same bytes within a word of ones, of a count and of noise
          for (uint64_t base : std::initializer_list<uint64_t>{~0ull, counter_key(g_call - 1).step * 3, rng()}) {
            v = base;
            std::memcpy(reinterpret_cast<char*>(&v) + at, &x, size);
            in_turn(v, n, "written over");
          }
        }
    // residues of earlier calls that never completed, every count
    for (int k = 1; k < n; ++k) in_turn(counter_key(g_call - 5).step * (uint64_t)k, n, "residue");
    for (int i = 0; i < 2000; ++i) in_turn(rng(), n, "random");
  }
  for (int i = 0; i < 600; ++i) interleaved(i % 3 ? rng() : 0, 2, rng);
  for (int i = 0; i < 400; ++i) interleaved(i % 3 ? counter_key(g_call - 2).step * (1 + rng() % 3) : rng(), 3 + i % 3, rng);
  std::printf("ok\n");
}
"""


def test_every_overwrite_and_interleaving(tmp_path):
    src = tmp_path / "counter.cpp"
    src.write_text(SOURCE)
    exe = str(tmp_path / "counter")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-pthread", "-I", CSRC, str(src), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-500:] + r.stderr[-500:]
