// Small rules that the kernels and the host code share, in plain C++, so that
// host tests can include them without a device compiler.
#pragma once

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

}  // namespace gabp
