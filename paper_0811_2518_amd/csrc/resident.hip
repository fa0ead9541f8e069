// Resident solve of a mid-sized system: every sweep, residual check and stop
// decision of a plain FP64 compact solve in ONE launch whose workgroups stay on
// the chip, one per CU, with the messages in registers.
//
// What bounds the launch-per-sweep path on such systems: a sweep launch and
// its finish kernel cost 10-12 us of dispatch and drain whatever the size, and
// each sweep streams 44 B per slot (column, A_ij, one message pair in and out)
// although the chip's registers (128 MB) could hold the whole state.  Here
//   * a row's slots are dealt K at a time to consecutive lanes of one wave (a
//     chain; one lane for rows of at most K slots).  A lane keeps its slots'
//     columns, coefficients and the incoming messages of the last two rounds
//     in registers (the compact recurrence of compact.hip: in^(t) depends on
//     in^(t-2) of the same slot alone), so a sweep moves no message at all;
//   * the chain's lanes add their messages in turn, in CSR order after the
//     diagonal, so every sum is rounded as the sweep kernels round it; the last
//     lane of the chain holds the new aggregate and hands it back to the chain;
//   * only the node aggregates cross workgroups, in two buffers by round
//     parity.  They are stored with agent scope (written through) and gathered
//     with agent scope loads (past the L1, coherent across the XCDs), so no
//     cache is written back or invalidated between sweeps.  Neighbours of the
//     same workgroup are read from LDS;
//   * the sweeps are separated by a grid barrier over counters in memory: one
//     line per group of 8 workgroup ids (the XCD of a round-robin dispatch),
//     one root, one release line per group.  Measured alone on 256 workgroups:
//     1.84 us, against 3.76 us with one counter and 3.09 us with a flag per
//     workgroup polled by all; up to 32 workgroups one counter is the fastest
//     (1.0 us).
// The workgroups must all be resident at once for the barrier to end.  The
// host launches no more of them than the device holds, and the first barrier
// is a roll call with a time limit: if the device is busy with other work and
// not every workgroup has started in time, the launch ends without touching
// its outputs and the host takes the launch-per-sweep path instead.  Once the
// roll call has succeeded every workgroup is running, so later waits end.
//
// Measured against a launch per sweep and its finish kernel, whole solves to
// 1e-10: 181 x 173 grid with variances 669 -> 286 us, G(n, 4n) with n = 30011
// on frozen precisions 350 -> 160 us, 64^3 grid forward and adjoint 6.67 ->
// 1.94 ms (a checked mean-only sweep of its 1.5 M slots takes 6.3 us instead
// of 24), 29 x 23 grid on frozen precisions 1004 -> 201 us in one workgroup.
//
// The arithmetic is that of the compact sweep kernels operation for operation
// (products and sums separately rounded): x, the variances and the messages
// equal theirs bit for bit; only the residual norm is summed in another order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "gabp_internal.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

constexpr int kRL = kResLanes;
constexpr int kGroups = 8;
constexpr int kFlatBlocks = 32;  // at most this many workgroups share one counter

template <typename T>
using vec2 = T __attribute__((ext_vector_type(2)));
using u32x4 = uint32_t __attribute__((ext_vector_type(4)));

#define AGENT_LOAD(p) __hip_atomic_load((p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define AGENT_STORE(p, v) __hip_atomic_store((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define AGENT_ADD(p, v) __hip_atomic_fetch_add((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)

// Cache policy of an agent-scope access (the sc1 bit): loads pass the L1,
// stores are written through.
constexpr int kAgentPolicy = 16;

// Lane exchanges on the VALU (DPP); a lane without a source gets `old`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double old, double v) {
  const uint64_t o = __builtin_bit_cast(uint64_t, old), b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)b, CTRL, ROWS, 0xf, false);
  const uint32_t hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
constexpr int kRowShr = 0x110, kBcast15 = 0x142, kBcast31 = 0x143, kWaveShl1 = 0x130, kWaveShr1 = 0x138;
__device__ __forceinline__ double readlane_r(double v, int l) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)b, l);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double uni_r(double v) { return readlane_r(v, 0); }
// Sum over the first 16 lanes, over the wave: in scalar registers, in a fixed order.
__device__ __forceinline__ double sum16(double v) {
  v += dpp<kRowShr + 1, 0xf>(0.0, v);
  v += dpp<kRowShr + 2, 0xf>(0.0, v);
  v += dpp<kRowShr + 4, 0xf>(0.0, v);
  v += dpp<kRowShr + 8, 0xf>(0.0, v);
  return v;
}
__device__ __forceinline__ double wsum_r(double v) {
  v = sum16(v);
  v += dpp<kBcast15, 0xa>(0.0, v);
  v += dpp<kBcast31, 0xc>(0.0, v);
  return readlane_r(v, 63);
}

// Workgroup barrier ordering LDS only.
__device__ __forceinline__ void lds_barrier_r() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A node's aggregate record in the shared buffers.
struct RecBuf {
  __amdgpu_buffer_rsrc_t r;
};
__device__ __forceinline__ RecBuf rec_buf(void* base, int32_t n) {
  return RecBuf{__builtin_amdgcn_make_buffer_rsrc(base, 0, n * (int)sizeof(vec2<double>), 0x00027000)};
}
// off: byte offset; beyond the buffer the load returns zero without an access
__device__ __forceinline__ vec2<double> ld_rec(const RecBuf& b, uint32_t off) {
  return __builtin_bit_cast(vec2<double>, __builtin_amdgcn_raw_buffer_load_b128(b.r, (int)off, 0, kAgentPolicy));
}
constexpr uint32_t kNoRec = 0xfffffff0u;
__device__ __forceinline__ void st_rec(const RecBuf& b, int i, vec2<double> v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b.r, i * (int)sizeof(vec2<double>), 0,
                                         kAgentPolicy);
}

// Partial sums travel without a wait between them and the barrier arrival: the
// low two bits of a partial's mantissa (2^-50 of its value) carry the check's
// sequence number mod 4, and a reader waits until they match.  Two sets by the
// number's parity: a workgroup stores check s + 1 before the barrier that says
// every other has read check s, and check s + 2 after it.
__device__ __forceinline__ uint64_t tag_partial(double v, uint32_t seq) {
  return (__builtin_bit_cast(uint64_t, v) & ~3ull) | (seq & 3u);
}

enum GridState : int { kGo = 1, kAbort = 2 };
enum WaitResult : int { kWaitOk = 0, kWaitBad = 1, kWaitEnd = 2 };

// The workgroup's place in the grid barrier.
struct GridPos {
  uint32_t nb, grp, gsize, ngrp;
};
__device__ __forceinline__ GridPos grid_pos() {
  GridPos p;
  p.nb = gridDim.x;
  if (p.nb <= (uint32_t)kFlatBlocks) {
    p.grp = 0;
    p.gsize = p.nb;
    p.ngrp = 1;
  } else {
    p.grp = blockIdx.x % kGroups;
    p.ngrp = kGroups;
    p.gsize = (p.nb + kGroups - 1 - p.grp) / kGroups;
  }
  return p;
}

// One lane: arrive at barrier `ep` (1, 2, ...).  Counters hold arrivals in the
// low 40 bits and raised flags above.  Returns true for the last arrival of
// the whole grid, with the flags of all in *bad.
__device__ __forceinline__ bool grid_arrive(ResCtl* c, const GridPos& p, uint32_t ep, bool bad, bool* any_bad) {
  const uint64_t inc = 1ull + (bad ? (1ull << 40) : 0ull);
  const uint64_t mask = (1ull << 40) - 1;
  uint64_t v = AGENT_ADD(&c->grp[p.grp].v, inc) + inc;
  if ((v & mask) != (uint64_t)ep * p.gsize) return false;
  bool b = (v >> 40) != 0;
  if (p.ngrp > 1) {
    const uint64_t inc2 = 1ull + (b ? (1ull << 40) : 0ull);
    v = AGENT_ADD(&c->root.v, inc2) + inc2;
    if ((v & mask) != (uint64_t)ep * p.ngrp) return false;
    b = (v >> 40) != 0;
  }
  *any_bad = b;
  return true;
}

// One lane: wait for barrier `ep`.  The release word holds the barrier number
// and the flags raised before it, so every workgroup leaves it with the same
// answer.
__device__ __forceinline__ int grid_wait(ResCtl* c, const GridPos& p, uint32_t ep, bool last, bool any_bad,
                                         uint64_t limit) {
  const uint64_t word = (uint64_t)ep | (any_bad ? (1ull << 63) : 0ull);
  if (last)
    for (uint32_t k = 0; k < p.ngrp; ++k) AGENT_STORE(&c->rel[k].v, word);
  const uint64_t t0 = wall_clock64();
  for (;;) {
    const uint64_t v = AGENT_LOAD(&c->rel[p.grp].v);
    if ((v & ~(1ull << 63)) >= ep) return (v >> 63) ? kWaitBad : kWaitOk;
    if (wall_clock64() - t0 > limit) return kWaitEnd;
  }
}

// The roll call: the last arrival turns the state to kGo, a workgroup that has
// waited too long to kAbort, whichever comes first.
__device__ __forceinline__ bool roll_call(ResCtl* c, const GridPos& p, uint64_t limit) {
  bool any_bad = false;
  if (grid_arrive(c, p, 1, false, &any_bad)) {
    uint32_t want = 0;
    __hip_atomic_compare_exchange_strong(&c->state, &want, (uint32_t)kGo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
  }
  const uint64_t t0 = wall_clock64();
  for (;;) {
    const uint32_t s = AGENT_LOAD(&c->state);
    if (s) return s == kGo;
    if (wall_clock64() - t0 > limit) {
      uint32_t want = 0;
      __hip_atomic_compare_exchange_strong(&c->state, &want, (uint32_t)kAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// LANES lanes per workgroup, one workgroup per CU: 128 VGPRs at 1024 lanes, of
// which the messages of K slots take 8 K, so there A_ij, the neighbours and the
// rows' prior live in LDS; with fewer lanes they stay in registers too.
template <int LANES, int K, bool HONLY>
__global__ __launch_bounds__(LANES) void k_resident(ResArgs A) {
  constexpr bool REG = LANES < kRL;
  constexpr int NW = LANES / 64;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_red[2][16];
  __shared__ double s_tot;
  // non-finite message flags by sweep mod 3: sweep t sets [t % 3] and clears
  // [(t + 1) % 3], which no lane reads or sets until sweep t + 1
  __shared__ int s_bad[3];
  __shared__ int s_res;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = A.n;
  const int nb = gridDim.x;
  // workgroup id -> part of the rows, so that consecutive parts share an XCD
  const int b = (blockIdx.x % kGroups) * (nb / kGroups) + min((int)(blockIdx.x % kGroups), nb % kGroups) +
                (int)blockIdx.x / kGroups;
  const int r0 = A.blk[b].x, nrow = A.blk[b].y;
  const int cap = A.rows_cap;
  vec2<double>* s_agg = (vec2<double>*)smem;   // [2][cap] the workgroup's aggregates by round parity
  double* s_x = (double*)(s_agg + 2 * cap);    // [2][cap] and their means
  double* s_a = s_x + 2 * cap;                 // 1024 lanes only: [K][lanes] A_ij of the lane's slots,
  double* s_d = s_a + K * LANES;               // [lanes] A_ii and b_i of the lane's row,
  double* s_b = s_d + LANES;
  int* s_c = (int*)(s_b + LANES);              // [K][lanes] the slots' neighbours
  ResCtl* ctl = A.ctl;
  const GridPos gp = grid_pos();

  // ---- set-up: the lane's slots and row, the prior as round 0 --------------
  const int2 ld = A.lane[(size_t)b * LANES + tid];
  const int row = ld.x, pos = ld.y & 0xffff, len = ld.y >> 16;
  const bool own = row >= 0;
  const bool tail = own && pos == len - 1;
  int cnt = 0;
  int s0 = 0;
  double dr = 1.0, br = 0.0, ip = 0.0;
  if (own) {
    s0 = A.off_ptr[row] + pos * K;
    cnt = min(K, A.off_ptr[row + 1] - s0);
    dr = A.diag[row];
    br = A.rhs[A.inv ? A.inv[row] : row];
    if (HONLY) ip = A.inv_pt[row];
  }
  if (!REG) {
    s_d[tid] = dr;
    s_b[tid] = br;
  }
  int wmax = 1;  // longest chain of the wave
  while (__any(own && len > wmax)) ++wmax;
  // the slots' neighbours: a row of the same workgroup as ~(LDS index), else
  // the byte offset of its record; a slot the row does not have reads record 0
  // of the workgroup and contributes nothing
  int cc[K];
  double aa[K];
  // joint: incoming messages {P, h} of the even and the odd rounds; frozen
  // precisions: {g_in, g_out} and the h messages of the two parities
  double mP0[K], mH0[K], mP1[K], mH1[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    int c = ~0;
    double av = 0.0;
    mP0[k] = mH0[k] = mP1[k] = mH1[k] = 0.0;
    if (k < cnt) {
      c = A.col[s0 + k];
      c = (unsigned)(c - r0) < (unsigned)nrow ? ~(c - r0) : c * (int)sizeof(vec2<double>);
      av = A.a[s0 + k];
      if (HONLY) {
        const vec2<double> cf = ((const vec2<double>*)A.coef)[s0 + k];
        mP0[k] = cf.x;
        mP1[k] = cf.y;
      }
    }
    if (REG) {
      cc[k] = c;
      aa[k] = av;
    } else {
      s_c[k * LANES + tid] = c;
      s_a[k * LANES + tid] = av;
    }
  }
  const RecBuf buf0 = rec_buf(A.agg[0], n), buf1 = rec_buf(A.agg[1], n);
  // own aggregates of the last two rounds, and the mean of the last one
  double o1P = HONLY ? ip : dr, o1h = br, o2P = 0.0, o2h = 0.0;
  double x1 = HONLY ? br * ip : br / dr;
  // the record a neighbour gathers: {P~, h~}, or {mean, h~} with frozen precisions
  if (tail) {
    const vec2<double> v = {HONLY ? x1 : dr, br};
    if (nb > 1) st_rec(buf0, row, v);
    s_agg[row - r0] = v;
    if (!HONLY) s_x[row - r0] = x1;
  }
  if (tid < 3) s_bad[tid] = 0;
  if (tid == 0) s_res = 0;
  // the other control block is idle during this launch: cleared for the next one
  if (blockIdx.x == 0 && nb > 1)
    for (int i = tid; i < (int)(sizeof(ResCtl) / 8); i += LANES) ((uint64_t*)A.ctl_next)[i] = 0ull;
  // ||b||, and the roll call
  {
    const double v = wsum_r(tail ? br * br : 0.0);
    if (lane == 0) s_red[0][wave] = v;
  }
  uint32_t seq = 1;  // checks so far (the norm is the first): the partials' tag
  auto block_sum = [&](const double* red) -> double {
    return readlane_r(sum16(lane < NW ? red[lane] : 0.0), 15);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (nb > 1) {
    if (wave == 0) {
      const double v = block_sum(s_red[0]);
      if (tid == 0) {
        AGENT_STORE(&ctl->part[seq & 1][b], tag_partial(v, seq));
        s_res = roll_call(ctl, gp, A.roll_limit) ? 0 : 1;
      }
    }
    __syncthreads();
    if (s_res) return;
  }
  bool lost = false;
  // the sum of the workgroups' partials: formed by wave 0, read by all
  auto total = [&](const double* red) -> double {
    if (nb == 1) return block_sum(red);
    if (wave == 0) {
      constexpr int kPer = kResMaxBlocks / 64;
      uint64_t u[kPer];
#pragma unroll
      for (int j = 0; j < kPer; ++j)
        u[j] = lane + 64 * j < nb ? AGENT_LOAD(&ctl->part[seq & 1][lane + 64 * j]) : (seq & 3u);
      const uint64_t t0 = wall_clock64();
      bool late = false;
      double v = 0.0;
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        while ((u[j] & 3u) != (seq & 3u) && !late) {
          u[j] = AGENT_LOAD(&ctl->part[seq & 1][lane + 64 * j]);
          late = wall_clock64() - t0 > A.wait_limit;
        }
        v += __builtin_bit_cast(double, u[j] & ~3ull);
      }
      if (__any(late)) s_res = kWaitEnd;
      v = wsum_r(v);
      if (lane == 0) s_tot = v;
    }
    lds_barrier_r();
    if (s_res == kWaitEnd) lost = true;
    return uni_r(s_tot);
  };
  const double bnorm = uni_r(sqrt(total(s_red[0])));

  const bool exact = !(A.tol > 0.0);
  const double tol = exact ? -1.0 : A.tol;
  const int M = A.max_iter;
  const int ce = max(1, A.check_every);
  auto in_set = [&](int j) { return j == M || (j % ce) == 0; };
  auto rel_of = [&](double tot) {
    const double rn = sqrt(tot);
    return bnorm > 0.0 ? rn / bnorm : rn;
  };
  // the stop test forms the relative residual only near a threshold: a sum of
  // squares clearly above (tol |b|)^2 cannot pass, one clearly below
  // (1e8 |b|)^2 cannot diverge; the decisions are the exact ones
  const double scale = bnorm > 0.0 ? bnorm : 1.0;
  double conv_pre = tol >= 0.0 ? (tol * scale) * (tol * scale) * (1.0 + 1e-6) : -1.0;
  if (tol > 0.0 && !(conv_pre > 1e-280 && conv_pre < 1e280)) conv_pre = INFINITY;  // out of range: always exact
  conv_pre = uni_r(conv_pre);
  const double div_pre = uni_r((kDivergeLimit * scale) * (kDivergeLimit * scale) * (1.0 - 1e-6));
  double last_tot = 0.0, prev_tot = 0.0;
  int last_round = -1, prev_round = -1, conv = -1, err = 0;
  bool pending = false;  // a check whose partials are on their way
  uint32_t ep = 1;

  // One sweep: the gathers of round t-1, then the stop decision on the check
  // that the previous sweep made (round t-2; its partials arrive while the
  // gathers are in flight), then the update.  Returns true when the solve ends.
  auto sweep = [&](auto odd_c, const int t) -> bool {
    constexpr bool ODD = decltype(odd_c)::value;
    const bool upd = t <= M;
    const bool ck = exact ? (t == M + 1) : (t <= M + 1 && in_set(t - 1));
    const bool live = upd || ck;
    const bool ck_next = upd && (exact ? (t == M) : in_set(t));  // sweep t+1 checks round t
    constexpr int p1 = ODD ? 0 : 1, pn = ODD ? 1 : 0;
    const bool first = ODD && t == 1;
    int cr[K];
    vec2<double> g[K];
#pragma unroll
    for (int k = 0; k < K; ++k) cr[k] = REG ? cc[k] : s_c[k * LANES + tid];
    if (live && nb > 1) {
#pragma unroll
      for (int k = 0; k < K; ++k) g[k] = ld_rec(ODD ? buf0 : buf1, cr[k] < 0 ? kNoRec : (uint32_t)cr[k]);
    }
    if (pending) {
      const double tot = total(s_red[p1]);
      prev_tot = last_tot;
      prev_round = last_round;
      last_tot = tot;
      last_round = t - 2;
      pending = false;
      if (tot <= conv_pre && rel_of(tot) <= tol) conv = t - 2;
      else if (!(tot < div_pre) && !(rel_of(tot) <= kDivergeLimit)) err |= kErrDiverged;
      if (conv >= 0 || err || lost) return true;
    }
    if (!live) return true;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const vec2<double> l = s_agg[p1 * cap + (cr[k] < 0 ? ~cr[k] : 0)];
      if (nb == 1 || cr[k] < 0) g[k] = l;
    }
    bool bad = false;
    double ax[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double av = REG ? aa[k] : s_a[k * LANES + tid];
      ax[k] = 0.0;
      if (ck) {
        if (HONLY) {
          ax[k] = av * g[k].x;
        } else {
          double xc = s_x[p1 * cap + (cr[k] < 0 ? ~cr[k] : 0)];
          if (__any(cr[k] >= 0)) {
            const double q = g[k].y / g[k].x;
            if (cr[k] >= 0) xc = q;
          }
          ax[k] = av * xc;
        }
      }
      if (upd) {
        const bool has = k < cnt;
        if (HONLY) {
          double hout = 0.0;
          if (!first) hout = mP1[k] * (o2h - (ODD ? mH1[k] : mH0[k]));
          const double hn = mP0[k] * (g[k].y - hout);
          if (ODD) mH1[k] = hn;
          else mH0[k] = hn;
          bad |= has && !isfinite(hn);
        } else {
          // in^(t) = F(A_c^(t-1), out^(t-1)), out^(t-1) = F(A_own^(t-2), in^(t-2))
          double Pout = 0.0, hout = 0.0;
          if (!first) {
            const double inv_out = 1.0 / (o2P - (ODD ? mP1[k] : mP0[k]));
            Pout = -av * av * inv_out;
            hout = -av * (o2h - (ODD ? mH1[k] : mH0[k])) * inv_out;
          }
          const double inv_in = 1.0 / (g[k].x - Pout);
          const double Pn = -av * av * inv_in;
          const double hn = -av * (g[k].y - hout) * inv_in;
          if (ODD) {
            mP1[k] = Pn;
            mH1[k] = hn;
          } else {
            mP0[k] = Pn;
            mH0[k] = hn;
          }
          bad |= has && !(isfinite(Pn) && isfinite(hn));
        }
      }
      // one slot's divisions at a time: interleaved, they would not fit 128 registers
      if (!REG) __builtin_amdgcn_sched_barrier(0);
    }
    // row sums along the chain, in CSR order after the diagonal; the residual
    // of round t-1
    double P = REG ? dr : s_d[tid], h = REG ? br : s_b[tid], acc = 0.0;
    if (ck) acc = h - P * x1;
    for (int c = 0; c < wmax; ++c) {
      if (c > 0) {
        const double Pu = dpp<kWaveShr1, 0xf>(P, P), hu = dpp<kWaveShr1, 0xf>(h, h),
                     au = dpp<kWaveShr1, 0xf>(acc, acc);
        if (pos == c) {
          P = Pu;
          h = hu;
          acc = au;
        }
      }
      if (pos == c) {
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (k < cnt) {
            if (!HONLY) P += ODD ? mP1[k] : mP0[k];
            h += ODD ? mH1[k] : mH0[k];
            if (ck) acc -= ax[k];
          }
      }
    }
    if (upd) {
      for (int c = wmax - 2; c >= 0; --c) {  // the sums back to the head of the chain
        const double Pd = dpp<kWaveShl1, 0xf>(P, P), hd = dpp<kWaveShl1, 0xf>(h, h);
        if (pos == c && pos < len - 1) {
          P = Pd;
          h = hd;
        }
      }
      if (HONLY) P = ip;
      o2P = o1P;
      o2h = o1h;
      o1P = P;
      o1h = h;
      if (HONLY) x1 = h * ip;
      else if (ck_next) x1 = h / P;
      if (tail) {
        const vec2<double> v = {HONLY ? x1 : P, h};
        if (nb > 1) st_rec(ODD ? buf1 : buf0, row, v);
        s_agg[pn * cap + row - r0] = v;
        if (!HONLY) s_x[pn * cap + row - r0] = x1;
      }
    }
    if (tid == 0) s_bad[(t + 1) % 3] = 0;
    if (bad) s_bad[t % 3] = 1;
    if (ck) {
      const double v = wsum_r(tail ? acc * acc : 0.0);
      if (lane == 0) s_red[pn][wave] = v;
      ++seq;
      pending = true;
    }
    ++ep;
    if (nb == 1) {
      lds_barrier_r();
      if (s_bad[t % 3]) err |= kErrNonfinite;
    } else {
      // the wave's records have reached memory before the workgroup arrives
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      lds_barrier_r();
      if (wave == 0) {
        double v = 0.0;
        if (ck) v = block_sum(s_red[pn]);
        if (tid == 0) {
          if (ck) AGENT_STORE(&ctl->part[seq & 1][b], tag_partial(v, seq));
          bool any_bad = false;
          const bool last = grid_arrive(ctl, gp, ep, s_bad[t % 3] != 0, &any_bad);
          s_res = grid_wait(ctl, gp, ep, last, any_bad, A.wait_limit);
        }
      }
      lds_barrier_r();
      asm volatile("" ::: "memory");
      if (s_res == kWaitBad) err |= kErrNonfinite;
      if (s_res == kWaitEnd) lost = true;
    }
    return err != 0 || lost;  // a non-finite message ends the solve
  };
  for (int t = 1;; t += 2) {
    if (sweep(std::true_type{}, t)) break;
    if (sweep(std::false_type{}, t + 1)) break;
  }

  // ---- results: the returned round and the state it leaves -----------------
  // the own aggregates are of rounds T = min(conv + 1, M) and T - 1
  const int ret = conv >= 0 ? conv : M;
  const int T = min(ret + (conv >= 0 ? 1 : 0), M);
  const double rP = ret == T ? o1P : o2P, rh = ret == T ? o1h : o2h;
  if (tail) {
    const int out = A.inv ? A.inv[row] : row;
    A.x[out] = HONLY ? rh * ip : rh / rP;
    if (A.var) A.var[out] = HONLY ? ip : 1.0 / rP;
    if (A.agg_out[0] && !HONLY) {
      ((vec2<double>*)A.agg_out[T % 3])[row] = vec2<double>{o1P, o1h};
      if (T >= 1) ((vec2<double>*)A.agg_out[(T - 1) % 3])[row] = vec2<double>{o2P, o2h};
    }
  }
  if (A.cin_out && !HONLY) {
    const int s0 = own ? A.off_ptr[row] + pos * K : 0;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (k < cnt) {
        ((vec2<double>*)A.cin_out)[s0 + k] = vec2<double>{mP0[k], mH0[k]};
        ((vec2<double>*)A.cin_out)[(size_t)A.E + s0 + k] = vec2<double>{mP1[k], mH1[k]};
      }
  }
  if (blockIdx.x == 0 && tid == 0) {
    DevStatus st{};
    st.done = lost ? 2 : 1;
    st.conv_round = conv;
    st.error = err;
    st.last_rel = last_round >= 0 ? rel_of(last_tot) : -1.0;
    st.last_round = last_round;
    st.prev_rel = prev_round >= 0 ? rel_of(prev_tot) : -1.0;
    st.prev_round = prev_round;
    *A.st = st;
  }
}

using ResKernel = void (*)(ResArgs);
template <int LANES>
ResKernel res_kernel_l(int K, bool honly) {
  if (K == 4) return honly ? k_resident<LANES, 4, true> : k_resident<LANES, 4, false>;
  return honly ? k_resident<LANES, 6, true> : k_resident<LANES, 6, false>;
}
ResKernel res_kernel(int lanes, int K, bool honly) {
  if (lanes == 256) return res_kernel_l<256>(K, honly);
  if (lanes == 512) return res_kernel_l<512>(K, honly);
  return res_kernel_l<kRL>(K, honly);
}

uint32_t res_lds(int rows_cap, int lanes, int K) {
  size_t b = 2 * (size_t)rows_cap * (sizeof(vec2<double>) + sizeof(double));
  if (lanes == kRL) b += (size_t)lanes * (K * (sizeof(double) + sizeof(int)) + 2 * sizeof(double));
  return (uint32_t)b;
}

}  // namespace

// The plan: rows dealt to lanes in order, chains inside one wave, workgroups
// of `lanes` lanes (with XCD parts: no workgroup spans two of them, and every
// part gets the same number).  Empty when the system does not fit.
ResPlanHost plan_resident(const std::vector<int32_t>& op, int32_t n, int K, int lanes, int max_blocks,
                          const std::vector<int32_t>& parts) {
  ResPlanHost pl;
  pl.K = K;
  pl.lanes = lanes;
  auto chain = [&](int32_t r) { return std::max(1, (op[r + 1] - op[r] + K - 1) / K); };
  const size_t np = parts.size() > 1 ? parts.size() - 1 : 1;
  std::vector<std::vector<int2>> blk(np);       // {first row, rows} of every workgroup of a part
  std::vector<std::vector<int2>> lane(np);
  for (size_t p = 0; p < np; ++p) {
    const int32_t lo = np > 1 ? parts[p] : 0, hi = np > 1 ? parts[p + 1] : n;
    // the part's lanes in order (chains padded to the next wave where they
    // would cross its end), cut evenly into as few workgroups as hold them
    int64_t total = 0;
    for (int32_t r = lo; r < hi; ++r) {
      const int len = chain(r);
      if (len > 64) return ResPlanHost{};
      if (total % 64 + len > 64) total += 64 - total % 64;
      total += len;
    }
    const int64_t want = std::max<int64_t>(1, (total + lanes - 1) / lanes);
    // waves per workgroup, spread evenly
    int64_t waves = (total + 63) / 64;
    const int64_t per = std::max<int64_t>(1, (waves + want - 1) / want);
    int used = 0;
    int2 cur{lo, 0};
    std::vector<int2> ll;
    auto close = [&](int32_t next) {
      ll.resize(lanes, int2{-1, 1 << 16});
      lane[p].insert(lane[p].end(), ll.begin(), ll.end());
      blk[p].push_back(cur);
      ll.clear();
      cur = int2{next, 0};
      used = 0;
    };
    for (int32_t r = lo; r < hi; ++r) {
      const int len = chain(r);
      int at = used;
      if (at % 64 + len > 64) at += 64 - at % 64;
      if (at + len > per * 64) {
        close(r);
        at = 0;
      }
      ll.resize(at, int2{-1, 1 << 16});
      for (int q = 0; q < len; ++q) ll.push_back(int2{r, q | (len << 16)});
      used = at + len;
      ++cur.y;
    }
    if (cur.y > 0 || blk[p].empty()) close(hi);
  }
  size_t q = 0;
  for (auto& v : blk) q = std::max(q, v.size());
  if (q * np > (size_t)max_blocks) return ResPlanHost{};
  for (size_t p = 0; p < np; ++p) {
    for (; blk[p].size() < q;) {  // empty workgroups keep part p on XCD p
      blk[p].push_back(int2{np > 1 ? parts[p + 1] : n, 0});
      lane[p].resize(lane[p].size() + lanes, int2{-1, 1 << 16});
    }
    pl.blk.insert(pl.blk.end(), blk[p].begin(), blk[p].end());
    pl.lane.insert(pl.lane.end(), lane[p].begin(), lane[p].end());
  }
  for (const int2& v : pl.blk) pl.rows_cap = std::max(pl.rows_cap, v.y);
  return pl;
}

// Plain FP64 solves of the compact layout, unless an option asks for a step
// between the sweeps.
bool resident_mode(const Ctx* c) {
  constexpr int32_t kOther = GABP_FLAG_MULTI_LAUNCH | GABP_FLAG_TIME_SWEEPS | GABP_FLAG_POISON_STALE |
                             GABP_FLAG_PREDICT_ALL | GABP_FLAG_AITKEN | GABP_FLAG_STEFFENSEN | GABP_FLAG_SINGLE_LOOP;
  return c->opts.precision == GABP_FP64 && c->opts.gamma == 0.0 && !(c->opts.flags & kOther) &&
         (c->opts.layout == 0 || c->opts.layout == kLayoutCompact);
}

// Slots per lane and lanes per workgroup of a handle.  4 or 6 slots are a lane
// of 2-D and 3-D grids, whose rows then need no chain; longer rows take chains
// of 6.  Workgroups: one if it holds every row (no grid barrier: the 29 x 23
// grid's mean-only sweep takes 2.05 us in one workgroup, 3.09 us in three);
// else as small as the CU count allows, since a sweep of few waves per CU is
// bound by the latency of its dependent divisions and exchanges (measured at
// 256 / 512 / 1024 lanes, checked FP64 sweeps: 181 x 173 grid 4.58 / 4.93 /
// 5.65 us, G(n, 4n) with n = 30011 6.94 / 8.27 / 12.5 us).
gabp_status setup_resident(Ctx* c) {
  c->res = ResPlan{};
  if (c->n < 1 || c->E < 1 || !resident_mode(c)) return GABP_OK;
  int dev = 0, ncu = 0, khz = 0;
  GABP_HIP(c, hipGetDevice(&dev));
  GABP_HIP(c, hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  GABP_HIP(c, hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  const int K = c->max_degree <= 4 ? 4 : 6;
  const int max_blocks = std::min(ncu, kResMaxBlocks);
  // rows whose chains the lanes can hold, before the plan walks them
  if (c->max_degree > kResMaxChain * K || c->n > (int64_t)max_blocks * kRL ||
      c->E > (int64_t)max_blocks * kRL * K)
    return GABP_OK;
  const std::vector<int32_t>& parts = c->nparts > 0 ? c->part_start : std::vector<int32_t>{};
  ResPlanHost pl;
  for (int blocks : {1, max_blocks})
    for (int lanes : {256, 512, kRL}) {
      if (!pl.blk.empty() || c->E > (int64_t)blocks * lanes * K || c->n > (int64_t)blocks * lanes) continue;
      pl = plan_resident(c->off_ptr_h, c->n, K, lanes, blocks, blocks == 1 ? std::vector<int32_t>{} : parts);
    }
  if (pl.blk.empty()) return GABP_OK;
  const uint32_t lds = res_lds(pl.rows_cap, pl.lanes, K);
  for (bool honly : {false, true}) {
    if (honly && !(c->opts.flags & GABP_FLAG_REUSE_PRECISION)) break;
    const void* f = (const void*)res_kernel(pl.lanes, K, honly);
    GABP_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per = 0;
    GABP_HIP(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, pl.lanes, lds));
    if ((int64_t)per * ncu < (int64_t)pl.blk.size()) return GABP_OK;
  }
  // one allocation: control blocks (zero), workgroups, lanes
  const size_t nblk = pl.blk.size(), head = 2 * sizeof(ResCtl) + sizeof(int2) * nblk;
  std::vector<unsigned char> img(head + sizeof(int2) * pl.lane.size(), 0);
  std::memcpy(img.data() + 2 * sizeof(ResCtl), pl.blk.data(), sizeof(int2) * nblk);
  std::memcpy(img.data() + head, pl.lane.data(), sizeof(int2) * pl.lane.size());
  void* base = nullptr;
  const gabp_status r = dev_alloc(c, &base, img.size());
  if (r != GABP_OK) return r;
  GABP_HIP(c, hipMemcpyAsync(base, img.data(), img.size(), hipMemcpyHostToDevice, c->stream));
  GABP_HIP(c, hipStreamSynchronize(c->stream));
  c->res.K = K;
  c->res.lanes = pl.lanes;
  c->res.nb = (int32_t)pl.blk.size();
  c->res.rows_cap = pl.rows_cap;
  c->res.ctl_d = (ResCtl*)base;
  c->res.blk_d = (int2*)((char*)base + 2 * sizeof(ResCtl));
  c->res.lane_d = (int2*)((char*)base + head);
  c->res.khz = khz;
  return GABP_OK;
}

hipError_t launch_resident(Ctx* c, ResArgs a, bool honly, hipStream_t s) {
  ResPlan& p = c->res;
  a.n = c->n;
  a.E = (int32_t)c->E;
  a.blk = p.blk_d;
  a.lane = p.lane_d;
  a.rows_cap = p.rows_cap;
  a.ctl = p.ctl_d + p.phase;
  a.ctl_next = p.ctl_d + (p.phase ^ 1);
  p.phase ^= 1;
  a.roll_limit = (uint64_t)p.khz * kResRollMs;
  a.wait_limit = (uint64_t)p.khz * kResWaitMs;
  const uint32_t lds = res_lds(p.rows_cap, p.lanes, p.K);
  hipLaunchKernelGGL(res_kernel(p.lanes, p.K, honly), dim3(p.nb), dim3(p.lanes), lds, s, a);
  return hipGetLastError();
}

}  // namespace gabp
