// One-workgroup solve of a small system: every sweep of the synchronous
// iteration of Alg. 2 (Ch. 3 Sec. 3.3), the fused residual checks and the stop
// rule run inside a single launch of 1024 lanes.
//
// A small system (n <= 1024 rows, E <= 4096 directed slots, or rows of at most
// 6 slots) spends more time in kernel launches and host polling than in
// arithmetic when every sweep is a launch of its own.  Here the whole state
// stays on chip: messages pass through LDS to the slots that receive them (one
// division each, see small.h), which keep those of the last two rounds in
// registers; a row's aggregate stays with its lane.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "small.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

// A slot per lane: rows of any length.  Checked sweeps to the same measure (two
// divisions a slot before): G(600, 1800) 5.4 -> 3.3 us, a tree of 777 nodes 3.9 ->
// 2.2 us, a star of 600 (one row sum of 599 terms in CSR order) 19.7 -> 15 us.
template <int K>
__global__ __launch_bounds__(kSB) void k_small(SmallArgs A) {
  extern __shared__ __align__(16) double sm[];
  __shared__ int s_bad[3];
  constexpr int S = kSB * K;
  const int tid = threadIdx.x;
  const int n = A.n, E = A.E;
  if (E < 0 || E > S || n < 1 || n > kSB) return;  // never run past the lanes' slots
  // set-up: the entries and the slots' rows in LDS
  double* s_a = sm;                  // [S]
  int* s_row = (int*)(sm + 2 * S);   // [S]
  uint32_t meta[K];
  double aa[K], am[K];
  int rlo = 0, rhi = 0;
  double dr = 1.0, br = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int s = tid + k * kSB;
    meta[k] = (uint32_t)s << 20;
    aa[k] = am[k] = 0.0;
    if (s < E) {
      meta[k] = pack_slot(0, A.col[s]) | ((uint32_t)A.rev[s] << 20);
      aa[k] = A.a[s];
      s_a[s] = aa[k];
    }
  }
  if (tid < n) {
    rlo = A.off_ptr[tid];
    rhi = A.off_ptr[tid + 1];
    dr = A.diag[tid];
    br = A.rhs[tid];
    for (int s = rlo; s < rhi; ++s) s_row[s] = tid;
  }
  if (tid < 3) s_bad[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int s = tid + k * kSB;
    if (s < E) {
      meta[k] |= pack_slot(s_row[s], 0);
      am[k] = s_a[slot_mir(meta[k])];
    }
  }
  __syncthreads();
  small_loop<K, true>(A, n, E, sm, s_bad, meta, aa, am, rlo, rhi, dr, br);
}

// Rows of at most KR slots: lane i owns row i and adds its messages as it
// takes them, so a sweep is: send the messages of round t; barrier; take them,
// publish the row's mean.  With two message buffers by parity (PAIR) that one
// barrier is enough; where they do not fit in LDS (rows of 5 or 6 slots, n >
// 768), a second one keeps a fast wave from overwriting what a slow one reads.
// Bound by VALU issue: 16 waves share four SIMDs, so every instruction of a lane
// costs 16 cycles a sweep.  Checked FP64 sweeps, against a kernel that kept the
// messages in registers and formed each from the aggregates of two rounds (two
// divisions a slot): 32 x 32 grid 2.96 -> 2.04 us (57 sweeps to 1e-10: 187 -> 125
// us the solve), 8^3 grid 3.0 -> 1.83 us, 10^3 grid (two barriers) 4.5 -> 2.7.
// Rows are NR apart in LDS, a constant, so that a lane's slots have constant
// offsets from one address.  A slot that a row does not have reads -0.0 and
// sends to a cell that nothing reads, so no lane is masked off in the loop (a
// branch per slot would also keep its divisions from overlapping).
template <int KR, bool PAIR>
constexpr int kRowsMax = KR == 6 && PAIR ? 768 : kSB;
template <int KR, bool PAIR>
constexpr int kRowsBuf = KR * kRowsMax<KR, PAIR> + 64;  // messages of a round, the cells that nothing reads
template <int KR, bool PAIR>
constexpr size_t kRowsLds =
    sizeof(double) * ((PAIR ? 4 : 2) * kRowsBuf<KR, PAIR> + 2 * kParts + 2 * kRowsMax<KR, PAIR>);
static_assert(kRowsLds<4, true> <= 160 * 1024 - 64 && kRowsLds<6, true> <= 160 * 1024 - 64, "LDS of a CU");

template <int KR, bool PAIR>
__global__ __launch_bounds__(kSB) void k_small_rows(SmallArgs A) {
  using V2 = vec2<double>;
  extern __shared__ __align__(16) double sm[];
  __shared__ int s_bad[3];  // non-finite messages by sweep mod 3
  constexpr int NR = kRowsMax<KR, PAIR>, NB = kRowsBuf<KR, PAIR>;
  const int tid = threadIdx.x;
  const int n = A.n;
  if (n < 1 || n > NR) return;
  V2* msg = (V2*)sm;                       // [PAIR ? 2 : 1][NB], slot k of row r at k NR + r
  double* s_red = sm + (PAIR ? 4 : 2) * NB;  // [2][kParts] residual partials by sweep parity
  double* gX = s_red + 2 * kParts;           // [2][NR] means by round parity
  const bool own = tid < n;
  // a wave without rows only waits at the barriers
  const bool on = __builtin_amdgcn_readfirstlane(tid & ~63) < n;
  int rlo = 0, deg = 0;
  double dr = 1.0, br = 0.0;
  if (own) {
    rlo = A.off_ptr[tid];
    deg = min(A.off_ptr[tid + 1] - rlo, KR);  // the host sends only rows of at most KR slots
    dr = A.diag[tid];
    br = A.rhs[tid];
  }
  // the slots: column and mirror slot packed, the entries of both
  uint32_t meta[KR];
  double aa[KR], am[KR];
  double mP0[KR], mH0[KR], mP1[KR], mH1[KR];  // messages of the even and the odd rounds
  double* s_a = sm;                           // set-up only: [KR][NR], then the columns
  int* s_col = (int*)(sm + KR * NR);
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    meta[k] = 0;
    aa[k] = am[k] = 0.0;
    mP0[k] = mH0[k] = mP1[k] = mH1[k] = 0.0;
    int c = -1;
    if (k < deg) {
      c = A.col[rlo + k];
      meta[k] = (uint32_t)c;
      aa[k] = A.a[rlo + k];
    }
    if (own) {
      s_a[k * NR + tid] = aa[k];
      s_col[k * NR + tid] = c;
    }
  }
  if (tid < 3) s_bad[tid] = 0;
  store_parts(own ? br * br : 0.0, s_red);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < KR; ++k) {
    int m = KR * NR + (tid & 63);
    if (k < deg) {
      const int c = (int)meta[k];
#pragma unroll
      for (int q = 0; q < KR; ++q)
        if (s_col[q * NR + c] == tid) m = q * NR + c;
      am[k] = s_a[m < KR * NR ? m : 0];
    }
    meta[k] |= (uint32_t)m << 10;
  }
  // the row's aggregates of the last two rounds and its mean of the last (round 0: the prior)
  double o1P = dr, o1h = br, o2P = 0.0, o2h = 0.0, x1 = br / dr;
  if (own) gX[tid] = x1;
  SmallStop stop(A, uni_r(sqrt(sum_parts(s_red))));
  __syncthreads();
  if (on) {
#pragma unroll
    for (int k = 0; k < KR; ++k)
      if (k >= deg) msg[k * NR + tid] = msg[(PAIR ? NB : 0) + k * NR + tid] = V2{-0.0, -0.0};
  } else if ((tid & 15) == 0) {
    s_red[tid >> 4] = s_red[kParts + (tid >> 4)] = 0.0;
  }
  int T = 0;                                  // the last round whose aggregates were formed
  bool ck = stop.exact ? stop.M == 0 : true;  // the next sweep checks the last round
  bool pending = false;                       // a check whose partials are about to cross a barrier

  // One sweep; its parity is a compile-time constant, so that the messages of
  // the two parities need no selects.  Returns true when the solve ends.
  auto sweep = [&](auto odd_c, const int t) -> bool {
    constexpr bool ODD = decltype(odd_c)::value;
    constexpr int p1 = ODD ? 0 : 1, pn = ODD ? 1 : 0;  // parities of rounds t-1 and t
    const bool upd = t <= stop.M;
    V2* buf = msg + (PAIR && ODD ? NB : 0);
    if (upd && on) {
#pragma unroll
      for (int k = 0; k < KR; ++k) {
        const double av = am[k];
        const double inv = 1.0 / (o1P - (ODD ? mP0[k] : mP1[k]));
        buf[fresh(meta[k]) >> 10] = V2{-av * av * inv, -av * (o1h - (ODD ? mH0[k] : mH1[k])) * inv};
        // one slot's division at a time: interleaved, they would not fit 128 registers
        if (KR > 4) __builtin_amdgcn_sched_barrier(0);
      }
    }
    lds_barrier_r();
    if (s_bad[(t + 2) % 3]) {  // sweep t-1 met a non-finite message: as the multi-launch path, it ends the solve
      stop.err |= kErrNonfinite;
      return true;
    }
    // the check of round t-2, made by sweep t-1
    if (pending && stop.decide(sum_parts(s_red + p1 * kParts), t - 2)) return true;
    pending = ck;
    if (!upd && !ck) return true;
    if (tid == 0) s_bad[(t + 1) % 3] = 0;  // read before this barrier, set after the next
    if (on) {
      double P = dr, h = br, acc = 0.0;
      if (ck) acc = br - dr * x1;  // the row's residual in round t-1
#pragma unroll
      for (int k = 0; k < KR; ++k) {
        if (ck) acc -= aa[k] * gX[p1 * NR + slot_row(fresh(meta[k]))];
        if (upd) {
          const V2 m = buf[k * NR + tid];
          P += m.x;
          h += m.y;
          if (ODD) {
            mP1[k] = m.x;
            mH1[k] = m.y;
          } else {
            mP0[k] = m.x;
            mH0[k] = m.y;
          }
        }
      }
      if (ck) store_parts(own ? acc * acc : 0.0, s_red + pn * kParts);
      if (upd) {
        if (!(isfinite(P) && isfinite(h))) {  // a non-finite message leaves no finite sum
#pragma unroll
          for (int k = 0; k < KR; ++k)
            if (!(isfinite(ODD ? mP1[k] : mP0[k]) && isfinite(ODD ? mH1[k] : mH0[k]))) s_bad[t % 3] = 1;
        }
        o2P = o1P;
        o2h = o1h;
        o1P = P;
        o1h = h;
      }
    }
    ck = upd && stop.next(t);
    if (ck && on) {
      x1 = o1h / o1P;
      gX[pn * NR + tid] = x1;
    }
    if (upd) T = t;
    if (!PAIR) lds_barrier_r();
    return false;
  };
  for (int t = 1;; t += 2) {
    if (sweep(std::true_type{}, t)) break;
    if (sweep(std::false_type{}, t + 1)) break;
  }

  const int ret = stop.conv >= 0 ? stop.conv : stop.M;  // round whose means are returned
  if (own) store_row(A, tid, ret, T, o1P, o1h, o2P, o2h);
  if (A.cin_out) {
#pragma unroll
    for (int k = 0; k < KR; ++k)
      if (k < deg) {
        ((V2*)A.cin_out)[rlo + k] = V2{mP0[k], mH0[k]};
        ((V2*)A.cin_out)[(size_t)A.E + rlo + k] = V2{mP1[k], mH1[k]};
      }
  }
  if (tid == 0) stop.store(A.st);
}

template <int K>
hipError_t launch_slots(const SmallArgs& a, hipStream_t s) {
  const uint32_t lds = (uint32_t)small_lds(a.n, K);
  (void)hipFuncSetAttribute((const void*)k_small<K>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_small<K>, dim3(1), dim3(kSB), lds, s, a);
  return hipGetLastError();
}

template <int KR, bool PAIR>
hipError_t launch_rows(const SmallArgs& a, hipStream_t s) {
  constexpr uint32_t lds = (uint32_t)kRowsLds<KR, PAIR>;
  (void)hipFuncSetAttribute((const void*)k_small_rows<KR, PAIR>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds);
  hipLaunchKernelGGL((k_small_rows<KR, PAIR>), dim3(1), dim3(kSB), lds, s, a);
  return hipGetLastError();
}

}  // namespace

bool small_fits(int64_t n, int64_t E) { return n >= 1 && n <= kSmallLanes && E <= (int64_t)kSmallLanes * 4; }

bool small_rows_fit(int64_t n, int32_t max_deg) { return n >= 1 && n <= kSmallLanes && max_deg >= 1 && max_deg <= 6; }

hipError_t launch_small(const SmallArgs& a, hipStream_t s) {
  if (small_rows_fit(a.n, a.max_deg)) {  // a lane per row
    if (a.max_deg <= 4) return launch_rows<4, true>(a, s);
    if (a.n <= kRowsMax<6, true>) return launch_rows<6, true>(a, s);
    return launch_rows<6, false>(a, s);
  }
  if (!small_fits(a.n, a.E)) return hipErrorInvalidValue;
  if (a.E <= kSB) return launch_slots<1>(a, s);
  if (a.E <= 2 * kSB) return launch_slots<2>(a, s);
  return launch_slots<4>(a, s);
}

}  // namespace gabp
