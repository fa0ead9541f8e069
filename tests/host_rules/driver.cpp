// Checks of the rules in csrc/rules.h, on the CPU.  One check per command-line
// name; exits 0 when it holds.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <random>
#include <thread>
#include <vector>

#include "chip_gate.h"
#include "rules.h"

using namespace gabp;

namespace {

// The LDS words of the check sums of a resident solve, as its waves touch them.
// Between two workgroup barriers (an epoch) nothing orders the waves, so a word
// that wave 0 writes in an epoch must not be read in it by another wave.
// A decision on check q is early or late:
//   early: wave 0 writes q's word; barrier; every wave reads it; the sweep
//          follows, with two barriers in it;
//   late:  the sweep's first barrier; wave 0 writes; its second barrier; every
//          wave reads.
// Either kind may follow either.  All sequences of `len` decisions are tried.
int sum_words() {
  const int len = 12;
  for (unsigned kinds = 0; kinds < (1u << len); ++kinds) {
    for (uint32_t q0 : {1u, 2u, 0xfffffffau}) {
      std::vector<uint32_t> wr, rd;  // words written by wave 0 and read by the others in the current epoch
      bool ok = true;
      auto barrier = [&] {
        for (uint32_t w : wr)
          for (uint32_t r : rd) ok = ok && w != r;
        wr.clear();
        rd.clear();
      };
      for (int k = 0; k < len; ++k) {
        const uint32_t w = sum_word(q0 + (uint32_t)k);
        if (w >= (uint32_t)kSumWords) return 1;
        const bool late = (kinds >> k) & 1u;
        if (late) barrier();
        wr.push_back(w);
        barrier();
        rd.push_back(w);
        if (!late) {
          barrier();
          barrier();
        }
      }
      barrier();
      if (!ok) {
        std::printf("a word is written while it may still be read: decisions %03x (bit k: check k late)\n", kinds);
        return 1;
      }
    }
  }
  return 0;
}

// A partial keeps every bit on its way, and a word that has not been written for
// check q is never taken for check q's.
int partials() {
  uint64_t r = 88172645463325252ull;
  auto carry = [](uint64_t bits) {
    for (uint32_t q = kFirstCheck; q < kFirstCheck + 16; ++q) {
      const uint64_t w = pack_partial(bits, q);
      if (!partial_sent(w, q) || partial_bits(w) != bits) return false;
    }
    return true;
  };
  // zero, the smallest subnormal, one and its neighbours, the largest, infinity, a NaN
  for (uint64_t bits : {0ull, 1ull, 0x3ff0000000000000ull, 0x3ff0000000000001ull, 0x3fefffffffffffffull,
                        0x7fefffffffffffffull, 0x7ff0000000000000ull, 0x7ff8000000000000ull})
    if (!carry(bits)) return 1;
  for (int k = 0; k < 100000; ++k) {
    r ^= r << 13;
    r ^= r >> 7;
    r ^= r << 17;
    if (!carry(r & ~kSignBit)) {
      std::printf("bits %016llx do not survive\n", (unsigned long long)(r & ~kSignBit));
      return 1;
    }
  }
  std::vector<uint64_t> set(4, 0);  // as a launch finds them
  for (uint32_t q = kFirstCheck; q < kFirstCheck + 4096; ++q) {
    uint64_t& w = set[partial_set(q)];
    if (partial_sent(w, q)) {
      std::printf("check %u is taken for sent before it was\n", q);
      return 1;
    }
    w = pack_partial(r, q);
    if (!partial_sent(w, q)) return 1;
  }
  return 0;
}

// Every team that an item can be given exists on the grid (one that does not would
// leave the item to nobody), and teams are powers of two up to the largest.
int teams() {
  for (int grid = 1; grid <= 1100; ++grid)
    for (int64_t units : {(int64_t)0, (int64_t)1, (int64_t)9, (int64_t)64, (int64_t)513, (int64_t)1 << 40})
      for (double cost : {0.0, 1.0, 1e3, 1e30})
        for (double share : {0.0, 1.0, 1e3}) {
          const int T = team_for(cost, share, units, grid);
          if (T < 1 || (T & (T - 1)) || T > kMaxTeam || grid / T < 1) {
            std::printf("team of %d on a grid of %d\n", T, grid);
            return 1;
          }
        }
  // a large item on a large grid still gets the largest team, a small one none
  return team_for(1e9, 1.0, 1 << 20, 1024) == kMaxTeam && team_for(0.4, 1.0, 1 << 20, 1024) == 1 ? 0 : 1;
}

// An item that no team shares is at most a third of an even share (or a single
// right-hand side), one that a team shares likewise per workgroup of the largest
// team it can have, and the group is the largest such one.
int groups() {
  const double share = 1000.0;
  for (int grid : {1, 2, 7, 256, 1024})
    for (int64_t nsl : {(int64_t)1, (int64_t)16, (int64_t)100, (int64_t)4000})
      for (int64_t ncls : {(int64_t)1, (int64_t)2, (int64_t)9})
        for (double unit = 0.5; unit < 1e7; unit *= 1.07) {
          auto per_workgroup = [&](int g) {
            const int64_t units = nsl * g / ncls;
            const bool alone = team_for(unit * g, share, units, grid) == 1;
            return unit * g / (alone ? 1 : team_for(unit * g, 0.0, units, grid));
          };
          const int g = group_for(unit, share, nsl, ncls, grid);
          bool ok = g == 1 || g == 2 || g == 4 || g == 8;
          ok = ok && (g == 1 || per_workgroup(g) <= share / 3.0);
          for (int bigger = 2 * g; ok && bigger <= kMaxGroup; bigger *= 2) ok = per_workgroup(bigger) > share / 3.0;
          if (!ok) {
            std::printf("group of %d: unit %g, %lld slices in %lld classes, grid %d\n", g, unit, (long long)nsl,
                        (long long)ncls, grid);
            return 1;
          }
        }
  // alone at 8 right-hand sides just above a third of a share: 4
  return group_for(0.342 * share / 8, share, 40, 1, 1024) == 4 ? 0 : 1;
}

// Launches that wait for each other's places are never inside together: all but
// one of those inside fit on the chip, one that asks for more than the chip is
// inside alone, threads enter in order, and one that gives up holds nobody up.
int gate() {
  using std::chrono::milliseconds;
  const milliseconds forever(60000);
  const int64_t room = 256;
  {  // one thread alone has nobody to keep waiting
    ChipGate g;
    if (g.shared() || !ChipPlace(g, room, room, forever).in() || g.shared()) return 1;
    std::thread([&] { g.shared(); }).join();
    if (!g.shared()) return 1;
  }
  {  // in any mix, seen through what the threads know to be inside
    ChipGate g;
    std::mutex m;
    std::vector<int64_t> inside;
    std::atomic<int> bad{0};
    auto work = [&](unsigned seed) {
      std::mt19937 r(seed);
      const int64_t needs[] = {1, 31, 124, 200, room, room + 1};
      for (int k = 0; k < 300; ++k) {
        const int64_t need = needs[r() % 6];
        ChipPlace p(g, need, room, forever);
        if (!p.in()) ++bad;
        {
          std::lock_guard<std::mutex> lk(m);
          inside.push_back(need);
          int64_t sum = 0, most = 0;
          for (int64_t v : inside) {
            sum += v;
            most = std::max(most, v);
          }
          if (sum - most > room || (most > room && inside.size() > 1)) ++bad;
        }
        if (r() % 4) p.issued();
        if (r() % 3 == 0) std::this_thread::yield();
        std::lock_guard<std::mutex> lk(m);
        inside.erase(std::find(inside.begin(), inside.end(), need));
      }
    };
    std::vector<std::thread> t;
    for (unsigned i = 0; i < 12; ++i) t.emplace_back(work, i);
    for (auto& x : t) x.join();
    if (bad) {
      std::printf("%d launches inside that cannot all end\n", bad.load());
      return 1;
    }
  }
  {  // one beyond the chip, and only behind launches that have been issued; then in order
    ChipGate g;
    auto a = std::make_unique<ChipPlace>(g, room, room, forever);
    if (ChipPlace(g, room, room, milliseconds(20)).in()) return 1;  // a is not issued yet
    a->issued();
    auto b = std::make_unique<ChipPlace>(g, room, room, milliseconds(20));
    if (!b->in()) return 1;
    b->issued();
    if (ChipPlace(g, 1, room, milliseconds(20)).in()) return 1;  // a second one beyond it
    std::mutex m;
    std::vector<int> order;
    std::vector<std::thread> t;
    for (int i = 0; i < 5; ++i) {
      t.emplace_back([&, i] {
        // the third gives up while it waits
        ChipPlace p(g, i == 1 ? room + 1 : room, room, i == 2 ? milliseconds(1) : forever);
        std::lock_guard<std::mutex> lk(m);
        if (p.in()) order.push_back(i);
      });
      std::this_thread::sleep_for(milliseconds(150));  // in line before the next
    }
    a.reset();
    b.reset();
    for (auto& x : t) x.join();
    // each enters before the next may; they note it one after the other but for the issue of two at once
    std::vector<int> sorted = order;
    std::sort(sorted.begin(), sorted.end());
    if (sorted != std::vector<int>({0, 1, 3, 4}) || order[0] != 0 || order[1] != 1) {
      std::printf("order of %zu threads\n", order.size());
      return 1;
    }
    if (!ChipPlace(g, room + 1, room, milliseconds(0)).in()) return 1;  // everything was given back
  }
  return 0;
}

// Failures in a row are tried 1, 2, 4, ... 64 calls apart, and a success starts
// anew.
int backoff() {
  Backoff b;
  std::vector<int> tried;
  for (int call = 0; call < 400; ++call)
    if (!b.skip()) {
      tried.push_back(call);
      b.failed();
    }
  if (tried != std::vector<int>({0, 2, 5, 10, 19, 36, 69, 134, 199, 264, 329, 394})) return 1;
  while (b.skip()) {
  }
  b.succeeded();
  if (b.skip()) return 1;
  b.failed();
  return b.skip() && !b.skip() ? 0 : 1;
}

}  // namespace

int main(int argc, char** argv) {
  const char* name = argc > 1 ? argv[1] : "";
  int bad = 2;
  if (!std::strcmp(name, "sum_words")) bad = sum_words();
  if (!std::strcmp(name, "partials")) bad = partials();
  if (!std::strcmp(name, "teams")) bad = teams();
  if (!std::strcmp(name, "groups")) bad = groups();
  if (!std::strcmp(name, "gate")) bad = gate();
  if (!std::strcmp(name, "backoff")) bad = backoff();
  if (!bad) std::printf("ok: %s\n", name);
  return bad;
}
