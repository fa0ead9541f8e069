// The sweep loop of the one-workgroup solves (small.hip, noalloc.hip): a slot
// per lane, messages exchanged through LDS.
//
// What bounds a sweep on one CU is FP64 arithmetic, above all divisions (13
// FP64 instructions of 4 cycles each per wave).  A message lives in the slot
// that receives it, and the row that sends it forms it from its aggregate and
// the message it got back,
//     in^(t) at (j, i) = F(A_i^(t-1), in^(t-1) at (i, j)),
// one division, and stores it at the mirror slot: the values of the compact
// recurrence of compact.hip, which takes two divisions a slot because there a
// slot must not be written from another row.  A sweep is two phases, each
// ended by a workgroup barrier:
//   1. slot lanes: the messages of round t into LDS, and the a_ji x_i terms of
//      the check of round t-1;
//   2. slot lanes take their new messages into registers; row lanes add them
//      in CSR order after the diagonal, publish the aggregate and the mean, and
//      form the residual of round t-1.
// The stop decision on a check falls a phase later, when its partial sums have
// crossed the barrier on their own.
//
// Products and sums are separately rounded, as in the sweep kernels: for a
// matrix whose stored halves agree exactly, x, the variances and the messages
// equal those of the multi-launch compact path bit for bit; only the residual
// norm is summed in another order.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gabp_internal.h"
#include "wave.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

constexpr int kSB = kSmallLanes;  // lanes of the one workgroup
constexpr int kSW = kSB / 64;     // its waves

// Sums over the workgroup on the matrix cores, whose issue slots are free (16
// waves of a sweep are bound by VALU issue; a DPP reduction takes 36 of those).
// The instruction multiplies four 4 x 4 blocks.  Block b takes the lanes l with
// (l >> 2) & 3 = b: the first product sums over the quarters of the wave, the
// second over the four lanes side by side, and all 16 lanes get the sum.
__device__ __forceinline__ double sum_of_16(double v) {
  const double rows = __builtin_amdgcn_mfma_f64_4x4x4f64(v, 1.0, 0.0, 0, 0, 0);
  return __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, rows, 0.0, 0, 0, 0);
}
constexpr int kParts = kSB / 16;  // partial sums of the workgroup
__device__ __forceinline__ void store_parts(double v, double* red) {
  v = sum_of_16(v);
  const int l = threadIdx.x;
  if ((l & 0x33) == 0) red[(l >> 6) * 4 + ((l >> 2) & 3)] = v;
}
__device__ __forceinline__ double sum_parts(const double* red) {
  const int l = threadIdx.x;
  const vec2<double>* r = (const vec2<double>*)red + 2 * ((l & 3) | ((l >> 2) & 12));
  const vec2<double> u = r[0], v = r[1];
  return uni_r(sum_of_16((u.x + u.y) + (v.x + v.y)));
}
static_assert(kParts == 64, "four partial sums to each of 16 lanes");

// Which rounds are checked, and the decision on a checked round.  The relative
// residual is formed as the multi-launch finish forms it, but only near a
// threshold: a sum of squares clearly above (tol |b|)^2 cannot pass, one
// clearly below (1e8 |b|)^2 cannot diverge (margins far above the rounding of
// sqrt and the division); the decisions are the exact ones.
struct SmallStop {
  double tol, bnorm, conv_pre, div_pre;
  double last_tot = 0.0, prev_tot = 0.0;
  int last_round = -1, prev_round = -1, conv = -1, err = 0;
  int M, ce, jm = 0;  // jm: t mod ce
  bool exact;
  __device__ __forceinline__ SmallStop(const SmallArgs& A, double bn) {
    tol = A.tol;
    M = A.max_iter;
    ce = max(1, A.check_every);
    exact = !(tol > 0.0);
    bnorm = bn;
    const double scale = bn > 0.0 ? bn : 1.0;
    conv_pre = tol >= 0.0 ? (tol * scale) * (tol * scale) * (1.0 + 1e-6) : -1.0;
    if (tol > 0.0 && !(conv_pre > 1e-280 && conv_pre < 1e280)) conv_pre = INFINITY;  // out of range: always exact
    conv_pre = uni_r(conv_pre);
    div_pre = uni_r((kDivergeLimit * scale) * (kDivergeLimit * scale) * (1.0 - 1e-6));
  }
  // to round t = 1, 2, ...: does sweep t+1 check it?
  __device__ __forceinline__ bool next(int t) {
    jm = jm + 1 == ce ? 0 : jm + 1;
    return t == M || (t < M && !exact && jm == 0);
  }
  __device__ __forceinline__ double rel_of(double tot) const {
    const double rn = sqrt(tot);
    return bnorm > 0.0 ? rn / bnorm : rn;
  }
  // the decision on `round` from its residual's sum of squares; true: the solve ends
  __device__ __forceinline__ bool decide(double tot, int round) {
    prev_tot = last_tot;
    prev_round = last_round;
    last_tot = tot;
    last_round = round;
    if (tot <= conv_pre && rel_of(tot) <= tol) conv = round;
    else if (!(tot < div_pre) && !(rel_of(tot) <= kDivergeLimit)) err |= kErrDiverged;
    return conv >= 0 || err != 0;
  }
  __device__ __forceinline__ void store(DevStatus* out) const {
    DevStatus st{};
    st.done = 1;
    st.conv_round = conv;
    st.error = err;
    st.last_rel = last_round >= 0 ? rel_of(last_tot) : -1.0;
    st.last_round = last_round;
    st.prev_rel = prev_round >= 0 ? rel_of(prev_tot) : -1.0;
    st.prev_round = prev_round;
    *out = st;
  }
};

// A row's results: the means of round `ret`, the aggregates of rounds T and
// T - 1, of which ret is one.
__device__ __forceinline__ void store_row(const SmallArgs& A, int row, int ret, int T, double o1P, double o1h,
                                          double o2P, double o2h) {
  const bool prev = ret == T - 1;
  const double P = prev ? o2P : o1P, h = prev ? o2h : o1h;
  if (A.x_direct) A.x_direct[row] = h / P;
  if (A.var_direct) A.var_direct[row] = 1.0 / P;
  if (A.agg_out[0]) {
    ((vec2<double>*)A.agg_out[T % 3])[row] = vec2<double>{o1P, o1h};
    if (T >= 1) ((vec2<double>*)A.agg_out[(T - 1) % 3])[row] = vec2<double>{o2P, o2h};
  }
}

// Dynamic LDS of the loop, in its order: the messages [S], the a x terms [S],
// the residual partials of two sweeps, the rows' aggregates and means [n].
__host__ __device__ constexpr size_t small_lds(int n, int K) {
  return sizeof(double) * (3 * (size_t)kSB * K + 3 * (size_t)n + 2 * kParts);
}

// A slot: its row and column (10 bits each) and its mirror slot (12 bits).
static_assert(kSmallLanes <= 1024, "rows and columns are packed in 10 bits");
__device__ __forceinline__ uint32_t pack_slot(int row, int col) { return (uint32_t)row | ((uint32_t)col << 10); }
__device__ __forceinline__ int slot_row(uint32_t m) { return (int)(m & 1023u); }
__device__ __forceinline__ int slot_col(uint32_t m) { return (int)((m >> 10) & 1023u); }
__device__ __forceinline__ int slot_mir(uint32_t m) { return (int)(m >> 20); }

// A sweep unpacks its slots anew: LDS addresses kept across the sweeps would
// not fit 128 registers.
__device__ __forceinline__ uint32_t fresh(uint32_t m) {
  asm volatile("" : "+v"(m));
  return m;
}

// All sweeps.  Lane l owns the slots l, l + 1024, ... < E (meta, a: the entry
// of its own row, am: that of its mirror) and, below n, row l with the slots
// rlo .. rhi - 1, the diagonal dr and the right-hand side br; a slot s >= E has
// itself as mirror, row and column 0 and zero entries.  s_bad: three LDS words
// (non-finite messages by sweep mod 3), cleared by the caller; a barrier follows before they are used.  KEEP:
// the messages may be asked for (A.cin_out).
template <int K, bool KEEP>
__device__ __forceinline__ void small_loop(const SmallArgs& A, const int n, const int E, double* sm, int* s_bad,
                                           const uint32_t (&meta)[K], const double (&aa)[K], const double (&am)[K],
                                           const int rlo, const int rhi, const double dr, const double br) {
  using V2 = vec2<double>;
  constexpr int S = kSB * K;
  const int tid = threadIdx.x;
  const int w0 = __builtin_amdgcn_readfirstlane(tid & ~63);  // the wave's first lane
  V2* msg = (V2*)sm;                          // [S] messages, each in the slot that receives it
  double* sX = sm + 2 * S;                    // [S] a x terms of the check
  double* s_red = sm + 3 * S;                 // [2][kParts] residual partials by sweep parity
  V2* agg = (V2*)(sm + 3 * S + 2 * kParts);   // [n] aggregates {P~, h~} of the last round
  double* xm = sm + 3 * S + 2 * kParts + 2 * n;  // [n] means h~ / P~ of the last round
  const bool own = tid < n;
  // incoming messages of the even and of the odd rounds, the row's aggregates
  // of the last two rounds and its mean of the last
  double mP0[K], mH0[K], mP1[K], mH1[K];
  double o1P = dr, o1h = br, o2P = 0.0, o2h = 0.0, x1 = br / dr;
#pragma unroll
  for (int k = 0; k < K; ++k) mP0[k] = mH0[k] = mP1[k] = mH1[k] = 0.0;
  if (own) {  // round 0: the prior
    agg[tid] = V2{dr, br};
    xm[tid] = x1;
  }
  store_parts(own ? br * br : 0.0, s_red);
  __syncthreads();
  SmallStop stop(A, uni_r(sqrt(sum_parts(s_red))));
  int T = 0;                                   // the last round whose aggregates were formed
  bool ck = stop.exact ? stop.M == 0 : true;   // the next sweep checks the last round
  bool pending = false;                        // a check whose partials have crossed the last barrier

  // One sweep; its parity is a compile-time constant, so that the messages of
  // the two parities need no selects.  Returns true when the solve ends.
  auto sweep = [&](auto odd_c, const int t) -> bool {
    constexpr bool ODD = decltype(odd_c)::value;
    constexpr int p1 = ODD ? 0 : 1, pn = ODD ? 1 : 0;
    const bool upd = t <= stop.M;
    if (s_bad[(t + 2) % 3]) {  // sweep t-1 met a non-finite message: as the multi-launch path, it ends the solve
      stop.err |= kErrNonfinite;
      return true;
    }
    // the check of round t-2, made by sweep t-1
    if (pending && stop.decide(sum_parts(s_red + p1 * kParts), t - 2)) return true;
    pending = ck;
    if (!upd && !ck) return true;
    // 1. the messages of round t, to their receivers; the terms of the check.
    // A wave with any slot takes all lanes: the surplus ones write to themselves.
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (w0 + k * kSB < E) {
        const uint32_t mt = fresh(meta[k]);
        if (ck) sX[tid + k * kSB] = aa[k] * xm[slot_col(mt)];
        if (upd) {
          const V2 o = agg[slot_row(mt)];
          const double av = am[k];
          const double inv = 1.0 / (o.x - (ODD ? mP0[k] : mP1[k]));
          msg[slot_mir(mt)] = V2{-av * av * inv, -av * (o.y - (ODD ? mH0[k] : mH1[k])) * inv};
        }
      }
      // one slot's division at a time: interleaved, they would not fit 128 registers
      if (K > 2) __builtin_amdgcn_sched_barrier(0);
    }
    lds_barrier_r();
    if (tid == 0) s_bad[(t + 1) % 3] = 0;  // read before the last barrier, set after the next but one
    // 2. the slots' new messages; the rows' sums and residuals
    if (upd) {
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (w0 + k * kSB < E) {
          const V2 m = msg[tid + k * kSB];
          if (ODD) {
            mP1[k] = m.x;
            mH1[k] = m.y;
          } else {
            mP0[k] = m.x;
            mH0[k] = m.y;
          }
        }
    }
    double acc = 0.0;
    if (own) {
      double P = dr, h = br;
      if (ck) acc = br - dr * x1;
      // four slots' loads before their sums; what is left of the row in one step
      int j = rlo;
      for (; j + 4 <= rhi; j += 4) {
        V2 m[4];
        double ax[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          m[u] = msg[j + u];
          ax[u] = sX[j + u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          P += m[u].x;
          h += m[u].y;
          acc -= ax[u];
        }
      }
      if (j < rhi) {
        V2 m[3];
        double ax[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
          const int s = min(j + u, rhi - 1);
          m[u] = msg[s];
          ax[u] = sX[s];
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
          if (j + u < rhi) {
            P += m[u].x;
            h += m[u].y;
            acc -= ax[u];
          }
      }
      if (upd) {
        if (!(isfinite(P) && isfinite(h)))  // a non-finite message leaves no finite sum
          for (int s = rlo; s < rhi; ++s)
            if (!(isfinite(msg[s].x) && isfinite(msg[s].y))) s_bad[t % 3] = 1;
        agg[tid] = V2{P, h};
        o2P = o1P;
        o2h = o1h;
        o1P = P;
        o1h = h;
      }
    }
    if (ck) store_parts(own ? acc * acc : 0.0, s_red + pn * kParts);
    ck = upd && stop.next(t);
    if (ck && own) {
      x1 = o1h / o1P;
      xm[tid] = x1;
    }
    if (upd) T = t;
    lds_barrier_r();
    return false;
  };
  for (int t = 1;; t += 2) {
    if (sweep(std::true_type{}, t)) break;
    if (sweep(std::false_type{}, t + 1)) break;
  }

  const int ret = stop.conv >= 0 ? stop.conv : stop.M;  // round whose means are returned
  if (own) store_row(A, tid, ret, T, o1P, o1h, o2P, o2h);
  if (KEEP && A.cin_out) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int s = tid + k * kSB;
      if (s < E) {
        ((V2*)A.cin_out)[s] = V2{mP0[k], mH0[k]};
        ((V2*)A.cin_out)[(size_t)E + s] = V2{mP1[k], mH1[k]};
      }
    }
  }
  if (tid == 0) stop.store(A.st);
}

}  // namespace

}  // namespace gabp
