// Small rules that the kernels and the host code share, in plain C++, so that
// host tests can include them without a device compiler.
#pragma once

#include <algorithm>
#include <cstdint>

#ifdef __HIPCC__
#define GABP_HD __host__ __device__
#else
#define GABP_HD
#endif

namespace gabp {

// Which of two LDS words receives the sum of check q's partials in the
// resident solve.  A late decision leaves a sweep by reading the word after the
// sweep's last workgroup barrier, and the next sweep's early decision has wave
// 0 write its sum before the next barrier, so consecutive checks must not share
// a word.  Two words are enough: the sums of checks q and q + 2 always have the
// barrier of check q + 1's sum between the last read and the write.
constexpr int kSumWords = 2;
GABP_HD constexpr uint32_t sum_word(uint32_t q) { return q & 1u; }

// Partial sums of a check travel without a wait between them and the barrier
// arrival: each word says itself whether it has arrived.  A partial is a sum of
// squares, so its sign bit is free: it holds bit 2 of the check's number, and
// the value keeps all its bits.  One bit is enough.  There are four sets of
// words, taken by the check number mod 4; a set is written for check q only
// after everyone has read check q - 4 from it, whose bit is the other one; and
// a launch finds zeros, while its first four checks (numbers 4 to 7) carry a 1.
constexpr uint32_t kFirstCheck = 4;
constexpr uint64_t kSignBit = 1ull << 63;
GABP_HD constexpr uint32_t partial_set(uint32_t q) { return q & 3u; }
GABP_HD constexpr uint64_t partial_tag(uint32_t q) { return (uint64_t)((q >> 2) & 1u) << 63; }
GABP_HD constexpr uint64_t pack_partial(uint64_t bits, uint32_t q) { return (bits & ~kSignBit) | partial_tag(q); }
GABP_HD constexpr bool partial_sent(uint64_t word, uint32_t q) { return (word & kSignBit) == partial_tag(q); }
GABP_HD constexpr uint64_t partial_bits(uint64_t word) { return word & ~kSignBit; }

// Members of the team that runs a batched item of the given cost, where an even
// share of the work per workgroup is `share`: enough to bring it to half a
// share, at most one wave per 64-lane unit of its passes, and never more than
// the `grid` workgroups that are launched.  Half a share: the items behind the
// first then even out what the estimates miss (a quarter, half, one share: 192
// systems of up to 16384 rows 9.0, 8.0, 8.3 ms; 600 of up to 32768 rows 40, 43,
// 46 ms).  One unit per wave: with at least two or four, the 192 systems take
// 7.7 and 10.0 ms, 20 of them 1.1, 1.5 and 2.1 ms.
constexpr int kMaxTeam = 64;
constexpr int kTeamWaves = 8;  // waves of a batched workgroup
inline int team_for(double cost, double share, int64_t units, int grid) {
  int T = 1;
  while (T < kMaxTeam && 2 * T <= grid && T * kTeamWaves < units && cost / T > 0.5 * share) T *= 2;
  return T;
}

// Right-hand sides per work item of a system (8, 4, 2 or 1), one of which costs
// `unit`; nsl / ncls: 64-row slices per pass of one right-hand side.  The
// largest group whose item is not long next to the makespan: at most a third of
// an even share per workgroup that runs it, which is one where the item gets no
// team, else as many as the largest team it can have.  (Dividing by that team
// where none is given left items of up to half a share whole: 3000 equal
// systems with 8 right-hand sides 63.1 instead of 62.1 ms.)
constexpr int kMaxGroup = 8;
inline int group_for(double unit, double share, int64_t nsl, int64_t ncls, int grid) {
  int g = kMaxGroup;
  for (; g > 1; g >>= 1) {
    const int64_t units = nsl * g / ncls;
    const int T = team_for(unit * g, share, units, grid) == 1 ? 1 : team_for(unit * g, 0.0, units, grid);
    if (unit * g / T <= share / 3.0) break;
  }
  return g;
}

// A handle whose launch found no place on the chip does not try again at once:
// it leaves out 1, 2, 4, ... 64 calls after each failure in a row, so that a chip
// that stays out of reach (another process, a stream with few compute units)
// costs at most the limit of one roll call in 65 solves, and a single failure
// one call on the slower path.
struct Backoff {
  int wait = 0, left = 0;
  bool skip() { return left > 0 && left-- > 0; }
  void failed() { left = wait = std::min(64, std::max(1, 2 * wait)); }
  void succeeded() { wait = 0; }
};

}  // namespace gabp
