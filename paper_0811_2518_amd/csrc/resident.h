// Resident solve of a mid-sized system: every sweep, residual check and stop
// decision of a compact-layout solve in ONE launch whose workgroups stay on the
// chip, one per CU, with the messages in registers.  The plain FP64 iteration,
// the single loop of Ch. 5 Sec. 5.3, and the refinement and loading loops with
// their inner solves (FP32 or FP64), freeze and FP64 residuals; synchronous or
// colour-serial sweeps.
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
//     workgroup polled by all; up to 64 workgroups one counter is the fastest
//     (1.0 us at 32 workgroups, 1.4 against 1.5 us at 64).
// The workgroups must all be resident at once for the barrier to end.  The
// host launches no more of them than the device holds and lets the process's
// threads launch in turn (chip_gate.h), and the first barrier is a roll call with
// a time limit: if the device is busy with other work and not every workgroup
// has started in time, the launch ends without touching its outputs and the host
// takes the launch-per-sweep path instead, with the same result, and leaves out
// a growing number of tries (rules.h).  Once the roll call has succeeded every
// workgroup is running, so later waits end; they have a limit all the same, and
// a workgroup that reaches it stores nothing and reports an error.
//
// Measured against a launch per sweep and its finish kernel, whole solves to
// 1e-10: 181 x 173 grid with variances 669 -> 267 us, G(n, 4n) with n = 30011
// on frozen precisions 350 -> 156 us, 64^3 grid forward and adjoint 6.65 ->
// 1.71 ms (a checked mean-only sweep of its 1.5 M slots takes 5.4 us instead
// of 24), 29 x 23 grid on frozen precisions 1004 -> 198 us in one workgroup.
// The loops of inner solves also lose the host's status reads (20-30 us each)
// and the launches between the phases: FP32 + refinement on G(n, 4n) with n =
// 130003 596 -> 355 us, the double loop on B^T B + 0.1 I with n = 30000 50.5 ->
// 27.7 ms.
//
// Colour-serial sweeps end a class with a grid barrier instead of a launch:
// 47^3 grid to 1e-10 (66 sweeps of 2 classes) 1.33 ms -> 756 us.
//
// The arithmetic is that of the compact and serial sweep kernels operation for
// operation (products and sums separately rounded): x, the variances and the
// messages equal theirs bit for bit; only the residual norm is summed in another
// order, in full FP64 (the words that carry its partial sums lose no bit, rules.h).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "gabp_internal.h"
#include "wave.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

constexpr int kRL = kResLanes;
constexpr int kGroups = 8;
constexpr int kFlatBlocks = 64;  // at most this many workgroups share one counter

using u32x4 = uint32_t __attribute__((ext_vector_type(4)));
using u32x2 = uint32_t __attribute__((ext_vector_type(2)));

#define AGENT_LOAD(p) __hip_atomic_load((p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define AGENT_STORE(p, v) __hip_atomic_store((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
#define AGENT_ADD(p, v) __hip_atomic_fetch_add((p), (v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)

// Cache policy of an agent-scope access (the sc1 bit): loads pass the L1,
// stores are written through.
constexpr int kAgentPolicy = 16;

// A buffer of n records that the workgroups share: a node's aggregates or x.
struct RecBuf {
  __amdgpu_buffer_rsrc_t r;
};
template <typename R>
__device__ __forceinline__ RecBuf rec_buf(void* base, int32_t n) {
  return RecBuf{__builtin_amdgcn_make_buffer_rsrc(base, 0, n * (int)sizeof(R), 0x00027000)};
}
// off: byte offset; beyond the buffer a load returns zero without an access
template <typename R>
__device__ __forceinline__ R ld_rec(const RecBuf& b, uint32_t off) {
  if constexpr (sizeof(R) == 16)
    return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b128(b.r, (int)off, 0, kAgentPolicy));
  else
    return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(b.r, (int)off, 0, kAgentPolicy));
}
template <typename R>
__device__ __forceinline__ void st_rec(const RecBuf& b, int i, R v) {
  if constexpr (sizeof(R) == 16)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b.r, i * (int)sizeof(R), 0, kAgentPolicy);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b.r, i * (int)sizeof(R), 0, kAgentPolicy);
}
constexpr uint32_t kNoRec = 0xfffffff0u;
__device__ __forceinline__ void st_rec(const RecBuf& b, int i, vec2<double> v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b.r, i * (int)sizeof(vec2<double>), 0,
                                         kAgentPolicy);
}

// A check's partial sum as it travels (rules.h).  Check s is read until the
// barrier after the one it was sent with has ended, and a workgroup stores check
// s + 4 into the same set of words after that.
__device__ __forceinline__ uint64_t tag_partial(double v, uint32_t seq) {
  return pack_partial(__builtin_bit_cast(uint64_t, v), seq);
}

constexpr int kErrLost = 1 << 30;  // beside the kErr* bits of a run, never stored

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
// low 40 bits and raised flags above (with one counter, by the parity of ep:
// the counter itself is what the others wait on, and a workgroup that is
// already one barrier ahead must not be heard early).  Returns true for the
// last arrival of the whole grid, with the flags of all in *bad.
constexpr uint64_t kCountMask = (1ull << 40) - 1;
__device__ __forceinline__ bool grid_arrive(ResCtl* c, const GridPos& p, uint32_t ep, bool bad, bool* any_bad) {
  const uint64_t inc = 1ull + (bad ? (1ull << (p.ngrp == 1 && (ep & 1) ? 52 : 40)) : 0ull);
  uint64_t v = AGENT_ADD(&c->grp[p.grp].v, inc) + inc;
  if ((v & kCountMask) != (uint64_t)ep * p.gsize) return false;
  bool b = (v >> 40) != 0;
  if (p.ngrp > 1) {
    const uint64_t inc2 = 1ull + (b ? (1ull << 40) : 0ull);
    v = AGENT_ADD(&c->root.v, inc2) + inc2;
    if ((v & kCountMask) != (uint64_t)ep * p.ngrp) return false;
    b = (v >> 40) != 0;
  }
  *any_bad = b;
  return true;
}

// The last arrival of the grid lets the others go.
__device__ __forceinline__ void grid_release(ResCtl* c, const GridPos& p, uint32_t ep, bool any_bad) {
  if (p.ngrp == 1) return;
  const uint64_t word = (uint64_t)ep | (any_bad ? (1ull << 63) : 0ull);
  for (uint32_t k = 0; k < p.ngrp; ++k) AGENT_STORE(&c->rel[k].v, word);
}

// One lane: wait for barrier `ep`: on the one counter, or on the group's
// release word, which holds the barrier number and the flags raised before it,
// so that every workgroup leaves it with the same answer.  The word is loaded
// after the clock, so a wave that was paused beyond the limit still sees a
// barrier that ended meanwhile.
__device__ __forceinline__ int grid_wait(ResCtl* c, const GridPos& p, uint32_t ep, uint64_t limit) {
  const uint64_t t0 = wall_clock64();
  for (;;) {
    const bool over = wall_clock64() - t0 > limit;
    if (p.ngrp == 1) {
      const uint64_t v = AGENT_LOAD(&c->grp[0].v);
      if ((v & kCountMask) >= (uint64_t)ep * p.gsize) return ((v >> (ep & 1 ? 52 : 40)) & 0xfff) ? kWaitBad : kWaitOk;
    } else {
      const uint64_t v = AGENT_LOAD(&c->rel[p.grp].v);
      if ((v & ~(1ull << 63)) >= ep) return (v >> 63) ? kWaitBad : kWaitOk;
    }
    if (over) return kWaitEnd;
  }
}

// The roll call: the last arrival turns the state to kGo, a workgroup that has
// waited too long to kAbort, whichever comes first.  With a limit of zero nobody
// waits, and nobody arrives last before the first has given up.
__device__ __forceinline__ bool roll_call(ResCtl* c, const GridPos& p, uint64_t limit) {
  bool any_bad = false;
  if (limit > 0 && grid_arrive(c, p, 1, false, &any_bad)) {
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

// What a launch runs.
enum ResMode : int {
  kResJoint = 0,   // plain sweeps
  kResFrozen = 1,  // mean-only sweeps on the handle's frozen precisions
  kResOuter = 2,   // refinement / loading loop around inner solves
  kResLoop = 3,    // the single loop: plain sweeps with damped feedback of the means
  kResOuterLoop = 4,  // refinement around single-loop inner solves (FP32)
  kResRefine = 5,  // kResOuter without frozen precisions (fewer registers)
  kResSerial = 6,  // colour-serial sweeps: the classes in turn, a grid barrier after each
  kResSerialOuter = 7  // refinement / loading loop around colour-serial inner solves
};
constexpr bool res_outer(int mode) {
  return mode == kResOuter || mode == kResOuterLoop || mode == kResRefine || mode == kResSerialOuter;
}

// Kernels whose stop decisions may fall a sweep late (see `run`): not with 1024
// lanes, whose 128 VGPRs the code for it overruns (64^3 grid, a checked sweep
// 9.2 us without it, 9.7 with it).
constexpr bool res_late(int mode, int lanes) {
  return lanes < kRL && (mode == kResJoint || mode == kResFrozen || mode == kResLoop);
}

// LANES lanes per workgroup, one workgroup per CU: 128 VGPRs at 1024 lanes, of
// which the FP64 messages of K slots take 8 K, so there A_ij, the neighbours
// and the rows' prior live in LDS; with fewer lanes they stay in registers too.
template <typename T, int LANES, int K, int MODE>
__global__ __launch_bounds__(LANES) void k_resident(ResArgs A) {
  constexpr bool OUTER = res_outer(MODE);
  constexpr bool SERIAL = MODE == kResSerial || MODE == kResSerialOuter;
  constexpr bool FEED = MODE == kResLoop || MODE == kResOuterLoop;
  constexpr bool LATE = res_late(MODE, LANES);
  constexpr bool REG = LANES < kRL;
  constexpr int NW = LANES / 64;
  using V2 = vec2<T>;
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ double s_red[3][16];  // by sweep parity, then the outer residual's
  // check sums by check number: the word that a late decision reads behind the
  // sweep's last barrier is not the one that the next sum is written to
  __shared__ double s_tot[kSumWords];
  // non-finite message flags by sweep mod 3: sweep t sets [t % 3] and clears
  // [(t + 1) % 3], which no lane reads or sets until sweep t + 1
  __shared__ int s_bad[3];
  __shared__ int s_res;
  __shared__ int s_late;  // nonzero: the wait for a check's partials ran out
  __shared__ __align__(16) uint64_t s_part[kResMaxBlocks];  // a check's partials, staged for a late decision
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = A.n;
  const int nb = gridDim.x;
  // workgroup id -> part of the rows, so that consecutive parts share an XCD
  const int b = (blockIdx.x % kGroups) * (nb / kGroups) + min((int)(blockIdx.x % kGroups), nb % kGroups) +
                (int)blockIdx.x / kGroups;
  const int r0 = A.blk[b].x, nrow = A.blk[b].y;
  const int cap = A.rows_cap;
  V2* s_agg = (V2*)smem;                       // [2][cap] the workgroup's aggregates by round parity
  double* s_xo = (double*)(s_agg + 2 * cap);   // [cap] outer loop: the iterate
  T* s_x = (T*)(s_xo + (OUTER ? cap : 0));     // [2][cap] the means of the last rounds
  V2* s_o3 = (V2*)(s_x + 2 * cap);             // [cap] late decisions: the aggregates of round t-2
  double* s_a = (double*)(s_o3 + (LATE ? cap : 0));  // 1024 lanes only: [K][lanes] A_ij of the lane's slots,
  double* s_d = s_a + K * LANES;               // [lanes] A_ii and b_i of the lane's row,
  double* s_b = s_d + LANES;
  int* s_c = (int*)(s_b + LANES);              // [K][lanes] the slots' neighbours
  ResCtl* ctl = A.ctl;
  const GridPos gp = grid_pos();

  // ---- set-up: the lane's slots and row ------------------------------------
  const int2 ld = A.lane[(size_t)b * LANES + tid];
  const int row = ld.x, pos = ld.y & 0xff, len = (ld.y >> 8) & 0xff;
  const int cls = ld.y >> 16;  // colour class (colour-serial)
  const bool own = row >= 0;
  const bool tail = own && pos == len - 1;
  int cnt = 0;
  int s0 = 0;
  double d64 = 1.0, b64 = 0.0;  // A_ii and b_i
  T din = 1, dchk = 1, ip = 0;  // the sweeps' diagonal, the checked one, the frozen 1 / P~
  if (own) {
    s0 = A.off_ptr[row] + pos * K;
    cnt = min(K, A.off_ptr[row + 1] - s0);
    b64 = A.rhs[A.inv ? A.inv[row] : row];
    din = ((const T*)A.diag)[row];
    d64 = OUTER ? A.d64[row] : (double)din;
    if (FEED) dchk = ((const T*)A.chk_diag)[row];
    if (MODE == kResFrozen || (MODE == kResOuter && A.frozen)) ip = ((const T*)A.inv_pt)[row];
  }
  if (!REG) {
    s_d[tid] = d64;
    s_b[tid] = b64;
  }
  int wmax = 1;  // longest chain of the wave
  while (__any(own && len > wmax)) ++wmax;
  // the slots' neighbours: a row of the same workgroup as ~(LDS index), else
  // the byte offset of its record; a slot the row does not have reads record 0
  // of the workgroup and contributes nothing
  int cc[K];
  double aa[K];
  uint32_t lowmask = 0;  // colour-serial: slots whose neighbour lies in an earlier class
  // joint: incoming messages {P, h} of the even and the odd rounds; frozen
  // precisions: {g_in, g_out} and the h messages of the two parities
  T mP0[K], mH0[K], mP1[K], mH1[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    int c = ~0;
    double av = 0.0;
    mP0[k] = mH0[k] = mP1[k] = mH1[k] = 0;
    if (k < cnt) {
      c = A.col[s0 + k];
      int local = c - r0;  // colour-serial: the workgroup's rows are a range of every class
      if constexpr (SERIAL) {
        int lo = 0, hi = A.ncls - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (A.cls_start[mid] <= c) lo = mid;
          else hi = mid - 1;
        }
        const int2 w = A.cls_tab[(size_t)b * (A.ncls + 1) + lo], w1 = A.cls_tab[(size_t)b * (A.ncls + 1) + lo + 1];
        local = (unsigned)(c - w.x) < (unsigned)(w1.y - w.y) ? w.y + c - w.x : -1;
        if (lo < cls) lowmask |= 1u << k;
      }
      c = (unsigned)local < (unsigned)nrow ? ~local : c * (int)sizeof(V2);
      av = A.a[s0 + k];
      if (MODE == kResFrozen || (MODE == kResOuter && A.frozen)) {
        const V2 cf = ((const V2*)A.coef)[s0 + k];
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
  // LDS index of the lane's row
  int lrow = row - r0;
  if constexpr (SERIAL) {
    const int2 w = own ? A.cls_tab[(size_t)b * (A.ncls + 1) + cls] : int2{0, 0};
    lrow = w.y + row - w.x;
  }
  auto slot_a = [&](int k) -> double { return REG ? aa[k] : s_a[k * LANES + tid]; };
  auto row_d = [&]() -> double { return REG ? d64 : s_d[tid]; };
  auto row_b = [&]() -> double { return REG ? b64 : s_b[tid]; };
  const RecBuf buf0 = rec_buf<V2>(A.agg[0], n), buf1 = rec_buf<V2>(A.agg[1], n);
  // own aggregates of the last two rounds, and the means of the last (two)
  T o1P = 0, o1h = 0, o2P = 0, o2h = 0, x1 = 0, x2 = 0;
  T rhs = (T)b64;  // right-hand side of the sweeps
  // round 0, the prior; the record a neighbour gathers is {P~, h~}, or
  // {mean, h~} with frozen precisions
  auto publish_prior = [&](bool honly) {
    o1P = honly ? ip : din;
    o1h = rhs;
    o2P = o2h = x2 = 0;
    x1 = honly ? rhs * ip : rhs / din;
    if (tail) {
      const V2 v = {honly ? x1 : din, rhs};
      if (nb > 1) st_rec<V2>(buf0, row, v);
      s_agg[lrow] = v;
      s_x[lrow] = x1;
    }
  };
  publish_prior(MODE == kResFrozen || (MODE == kResOuter && A.frozen));
  if (tid < 3) s_bad[tid] = 0;
  if (tid == 0) s_res = s_late = 0;
  // the other control block is idle during this launch: cleared for the next one
  if (blockIdx.x == 0 && nb > 1)
    for (int i = tid; i < (int)(sizeof(ResCtl) / 8); i += LANES) ((uint64_t*)A.ctl_next)[i] = 0ull;
  // ||b||, and the roll call
  {
    const double v = wsum_r(tail ? b64 * b64 : 0.0);
    if (lane == 0) s_red[0][wave] = v;
  }
  uint32_t seq = kFirstCheck;  // number of the last check (the norm is the first)
  uint32_t ep = 1;   // grid barriers so far
  auto block_sum = [&](const double* red) -> double {
    return readlane_r(sum16(lane < NW ? red[lane] : 0.0), 15);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (nb > 1) {
    if (wave == 0) {
      const double v = block_sum(s_red[0]);
      if (tid == 0) {
        AGENT_STORE(&ctl->part[partial_set(seq)][b], tag_partial(v, seq));
        s_res = roll_call(ctl, gp, A.roll_limit) ? 0 : 1;
      }
    }
    __syncthreads();
    if (s_res) return;
  }
  int err = 0;  // of the run; kErrLost: a wait of this workgroup ran out (all its waves agree)
  // the sum of check q's partials, formed by wave 0 and left in its word of
  // s_tot: from memory, or from the copy in s_part where `staged`.  True: a
  // wait ran out.
  auto sum_partials = [&](const uint32_t q, const bool staged) -> bool {
    constexpr int kPer = kResMaxBlocks / 64;
    const uint64_t* part = ctl->part[partial_set(q)];
    uint64_t u[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int i = lane + 64 * j;
      u[j] = i >= nb ? partial_tag(q) : staged ? s_part[i] : AGENT_LOAD(&part[i]);
    }
    const uint64_t t0 = wall_clock64();
    bool late = false;
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      while (!partial_sent(u[j], q) && !late) {
        const bool over = wall_clock64() - t0 > A.wait_limit;
        u[j] = AGENT_LOAD(&part[lane + 64 * j]);
        late = over && !partial_sent(u[j], q);
      }
      v += __builtin_bit_cast(double, partial_bits(u[j]));
    }
    v = wsum_r(v);
    if (lane == 0) s_tot[sum_word(q)] = v;
    return __any(late);
  };
  // the sum of the last check's partials (red: the waves' of one workgroup)
  auto total = [&](const double* red) -> double {
    if (nb == 1) return block_sum(red);
    if (wave == 0 && sum_partials(seq, false)) s_late = 1;
    lds_barrier_r();
    if (s_late) err |= kErrLost;
    return uni_r(s_tot[sum_word(seq)]);
  };
  // All workgroups: records stored before it are visible after it.  red
  // (nullable): the waves' partials of a check, sent along; flag: an LDS word,
  // nonzero where a message was not finite.  Returns whether any was.  sum
  // (nonzero): the check whose staged partials are added up meanwhile, into
  // its word of s_tot.
  auto grid_barrier = [&](const double* red, const int* flag, const uint32_t sum = 0) -> bool {
    ++ep;
    if (nb == 1) {
      lds_barrier_r();
      return flag && *flag;
    }
    // the wave's records have reached memory before the workgroup arrives
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier_r();
    if (wave == 0) {
      const double v = red ? block_sum(red) : 0.0;
      if (tid == 0) {
        if (red) AGENT_STORE(&ctl->part[partial_set(seq)][b], tag_partial(v, seq));
        bool any_bad = false;
        // (with one counter too the answer is awaited: polling at once delays the others' arrivals)
        if (grid_arrive(ctl, gp, ep, flag && *flag, &any_bad)) grid_release(ctl, gp, ep, any_bad);
      }
      const bool late = LATE && sum && sum_partials(sum, true);
      if (tid == 0) {
        const int r = grid_wait(ctl, gp, ep, A.wait_limit);
        s_res = late ? (int)kWaitEnd : r;
      }
    }
    lds_barrier_r();
    asm volatile("" ::: "memory");
    if (s_res == kWaitEnd) err |= kErrLost;
    return s_res == kWaitBad;
  };
  const double bnorm = uni_r(sqrt(total(s_red[0])));

  const int ce = max(1, A.check_every);
  // result of a run of sweeps (kept for the caller of the run)
  double last_rel = -1.0, prev_rel = -1.0;
  int last_round = -1, prev_round = -1, conv = -1;

  // Colour-serial sweeps (serial.hip) on the system with right-hand side `rhs`:
  // a slot holds the outgoing message of its row's last update (mP0, mH0), the
  // aggregates are updated in place, class by class.  As `run` below otherwise;
  // M >= 1.
  auto run_serial = [&](const double tol_in, const int M, const double norm) {
    const bool exact = !(tol_in > 0.0);
    const double tol = exact ? -1.0 : tol_in;
    auto in_set = [&](int j) { return j == M || (j % ce) == 0; };
    auto rel_of = [&](double tot) {
      const double rn = sqrt(tot);
      return norm > 0.0 ? rn / norm : rn;
    };
    bool pending = false;
    conv = last_round = prev_round = -1;
    last_rel = prev_rel = -1.0;
    err &= kErrLost;
    int nbar = 0;        // barriers of this run: the flag word in use
    double lsum = 0.0;   // the row's residual part of the earlier classes, from the last sweep
    for (int t = 1;; ++t) {
      if (pending) {
        const double rel = uni_r(rel_of(total(s_red[(t - 1) & 1])));
        prev_rel = last_rel;
        prev_round = last_round;
        last_rel = rel;
        last_round = t - 2;
        pending = false;
        if (rel <= tol) conv = t - 2;
        else if (!(rel <= kDivergeLimit)) err |= kErrDiverged;
        if (conv >= 0 || err) break;
      }
      const bool fin = t == M + 1;  // the residual of sweep M alone, every row at once
      const bool ck = exact ? fin : (t >= 2 && t <= M + 1 && in_set(t - 1));
      if (t > M && !ck) break;
      const bool first = t == 1, wl = !exact && t < M && in_set(t);
      double res = 0.0;  // the row's residual of round t-1
      const int ncls = fin ? 1 : A.ncls;
      for (int q = 0; q < ncls; ++q) {
        const bool act = own && (fin || cls == q);
        bool bad = false;
        if (__any(act)) {
          int cr[K];
          V2 g[K];
#pragma unroll
          for (int k = 0; k < K; ++k) cr[k] = REG ? cc[k] : s_c[k * LANES + tid];
          if (nb > 1) {
#pragma unroll
            for (int k = 0; k < K; ++k) g[k] = ld_rec<V2>(buf0, cr[k] < 0 || !act ? kNoRec : (uint32_t)cr[k]);
          }
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const V2 l = s_agg[cr[k] < 0 ? ~cr[k] : 0];
            if (nb == 1 || cr[k] < 0) g[k] = l;
          }
          T ax[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const T av = (T)slot_a(k);
            const bool low = !fin && ((lowmask >> k) & 1u);
            ax[k] = 0;
            if (low ? wl : ck) ax[k] = av * (g[k].y / g[k].x);
            if (act && !fin) {
              T Pin = 0, hin = 0;  // in the first sweep a later class has sent nothing yet
              if (!first || low) {
                const T inv = T(1) / (g[k].x - mP0[k]);
                Pin = -av * av * inv;
                hin = -av * (g[k].y - mH0[k]) * inv;
              }
              mP0[k] = Pin;  // kept in the slot until the row's aggregate is known
              mH0[k] = hin;
              bad |= k < cnt && !(isfinite(Pin) && isfinite(hin));
            }
            if (!REG) __builtin_amdgcn_sched_barrier(0);
          }
          T P = din, h = rhs;
          double Ls = 0.0, U = 0.0;
          for (int c = 0; c < wmax; ++c) {
            if (c > 0) {
              const T Pu = dpp<kWaveShr1, 0xf>(P, P), hu = dpp<kWaveShr1, 0xf>(h, h);
              const double Lu = dpp<kWaveShr1, 0xf>(Ls, Ls), Uu = dpp<kWaveShr1, 0xf>(U, U);
              if (pos == c) {
                P = Pu;
                h = hu;
                Ls = Lu;
                U = Uu;
              }
            }
            if (pos == c) {
#pragma unroll
              for (int k = 0; k < K; ++k)
                if (k < cnt) {
                  if (!fin) {
                    P += mP0[k];
                    h += mH0[k];
                  }
                  if (!fin && ((lowmask >> k) & 1u)) Ls += (double)ax[k];
                  else U += (double)ax[k];
                }
            }
          }
          if (act && ck) res = (double)rhs - (double)din * (double)(o1h / o1P) - (fin ? 0.0 : lsum) - U;
          if (!fin) {
            for (int c = wmax - 2; c >= 0; --c) {
              const T Pd = dpp<kWaveShl1, 0xf>(P, P), hd = dpp<kWaveShl1, 0xf>(h, h);
              if (pos == c && pos < len - 1) {
                P = Pd;
                h = hd;
              }
            }
            if (act) {
              if (wl) lsum = Ls;
              o2P = o1P;
              o2h = o1h;
              o1P = P;
              o1h = h;
              if (tail) {
                if (nb > 1) st_rec<V2>(buf0, row, V2{P, h});
                s_agg[lrow] = V2{P, h};
              }
#pragma unroll
              for (int k = 0; k < K; ++k) {  // out_{j->i} = F(agg_j, in_{i->j})
                const T av = (T)slot_a(k);
                const T inv = T(1) / (P - mP0[k]);
                const T Po = -av * av * inv, ho = -av * (h - mH0[k]) * inv;
                mP0[k] = Po;
                mH0[k] = ho;
                bad |= k < cnt && !(isfinite(Po) && isfinite(ho));
                if (!REG) __builtin_amdgcn_sched_barrier(0);
              }
            }
          }
        }
        ++nbar;
        if (tid == 0) s_bad[(nbar + 1) % 3] = 0;
        if (bad) s_bad[nbar % 3] = 1;
        const bool send = ck && q == ncls - 1;
        if (send) {
          const double v = wsum_r(tail ? res * res : 0.0);
          if (lane == 0) s_red[t & 1][wave] = v;
          ++seq;
          pending = true;
        }
        if (grid_barrier(send ? s_red[t & 1] : nullptr, &s_bad[nbar % 3])) err |= kErrNonfinite;
        if (err) break;
      }
      if (err) break;
    }
  };

  // Sweeps on the system with right-hand side `rhs` (round 0 published) to a
  // relative residual of tol (<= 0: exactly M sweeps): conv, err and the
  // rounds T = min(conv + 1, M) and T - 1 in the registers.
  auto run = [&](auto honly_c, const double tol_in, const int M, const double norm) {
    constexpr bool HONLY = decltype(honly_c)::value;
    const bool exact = !(tol_in > 0.0);
    const double tol = exact ? -1.0 : tol_in;
    auto in_set = [&](int j) { return j == M || (j % ce) == 0; };
    auto rel_of = [&](double tot) {
      const double rn = sqrt(tot);
      return norm > 0.0 ? rn / norm : rn;
    };
    // the stop test forms the relative residual only near a threshold: a sum of
    // squares clearly above (tol |b|)^2 cannot pass, one clearly below
    // (1e8 |b|)^2 cannot diverge; the decisions are the exact ones
    const double scale = norm > 0.0 ? norm : 1.0;
    double conv_pre = tol >= 0.0 ? (tol * scale) * (tol * scale) * (1.0 + 1e-6) : -1.0;
    if (tol > 0.0 && !(conv_pre > 1e-280 && conv_pre < 1e280)) conv_pre = INFINITY;  // out of range: always exact
    conv_pre = uni_r(conv_pre);
    const double div_pre = uni_r((kDivergeLimit * scale) * (kDivergeLimit * scale) * (1.0 - 1e-6));
    double last_tot = 0.0, prev_tot = 0.0;
    bool pending = false;  // a check whose partials are on their way
    conv = last_round = prev_round = -1;
    err &= kErrLost;
    // Early or late decisions.  Adding up the partials before the update makes
    // every wave wait for one; while no stop is in sight wave 0 only stages
    // them in LDS, adds them up while the barrier of the same sweep is under
    // way, and the decision on round t-2 falls at the end of sweep t.  If it
    // ends the run after all, the sweep is taken back: the aggregates of the
    // last three rounds are at hand (not the messages, so a run that leaves its
    // state behind decides early).  In sight: the next check would meet the
    // tolerance with a factor of 4 to spare if the residual kept its last rate.
    // Checked sweeps, early / late: 181 x 173 grid 4.3 / 4.0 us, on frozen
    // precisions 3.6 / 3.3; G(n, 4n) with n = 30011 6.8 / 6.3, frozen 5.6 / 5.1;
    // 24^3 grid 4.5 / 4.25; no gain on 16 workgroups (64 x 64 grid 3.5 / 3.55).
    const bool may_late = LATE && nb > 1 && (HONLY || (!A.cin_out && !A.agg_out[0]));
    bool far = false;
    auto decide = [&](const double tot, const int round) {
      prev_tot = last_tot;
      prev_round = last_round;
      last_tot = tot;
      last_round = round;
      if (tot <= conv_pre && rel_of(tot) <= tol) conv = round;
      else if (!(tot < div_pre) && !(rel_of(tot) <= kDivergeLimit)) err |= kErrDiverged;
      if (LATE) far = prev_round < 0 ? tot > 1e4 * conv_pre : tot * tot > 16.0 * conv_pre * prev_tot;
    };

    // One sweep: the gathers of round t-1, then the stop decision on the check
    // that the previous sweep made (round t-2; its partials arrive while the
    // gathers are in flight), then the update.  Returns true when the run ends.
    auto sweep = [&](auto odd_c, const int t) -> bool {
      constexpr bool ODD = decltype(odd_c)::value;
      const bool upd = t <= M;
      const bool ck = exact ? (t == M + 1) : (t <= M + 1 && in_set(t - 1));
      const bool live = upd || ck;
      const bool ck_next = upd && (exact ? (t == M) : in_set(t));  // sweep t+1 checks round t
      constexpr int p1 = ODD ? 0 : 1, pn = ODD ? 1 : 0;
      const bool first = ODD && t == 1;
      int cr[K];
      V2 g[K];
#pragma unroll
      for (int k = 0; k < K; ++k) cr[k] = REG ? cc[k] : s_c[k * LANES + tid];
      if (nb > 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) g[k] = ld_rec<V2>(ODD ? buf0 : buf1, cr[k] < 0 ? kNoRec : (uint32_t)cr[k]);
      }
      uint32_t late = 0;  // the check decided at the end of this sweep
      if (pending) {
        pending = false;
        if (LATE && may_late && far && live) {
          late = seq;
          if (wave == 0) {
            const __amdgpu_buffer_rsrc_t r =
                __builtin_amdgcn_make_buffer_rsrc(ctl->part, 0, (int)sizeof(ctl->part), 0x00027000);
            const int at = (int)(partial_set(seq) * sizeof(ctl->part[0]));
            for (int i = 0; i < nb; i += 128)
              __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)(s_part + i), 16,
                                                       lane * 16, at + i * 8, 0, kAgentPolicy);
          }
        } else {
          decide(total(s_red[p1]), t - 2);
        }
      }
      if (conv >= 0 || err || !live) return true;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const V2 l = s_agg[p1 * cap + (cr[k] < 0 ? ~cr[k] : 0)];
        if (nb == 1 || cr[k] < 0) g[k] = l;
      }
      bool bad = false;
      T ax[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const T av = (T)slot_a(k);
        ax[k] = 0;
        if (ck) {
          if (HONLY) {
            ax[k] = av * g[k].x;
          } else {
            T xc = s_x[p1 * cap + (cr[k] < 0 ? ~cr[k] : 0)];
            if (__any(cr[k] >= 0)) {
              const T q = g[k].y / g[k].x;
              if (cr[k] >= 0) xc = q;
            }
            ax[k] = av * xc;
          }
        }
        if (upd) {
          const bool has = k < cnt;
          if (HONLY) {
            T hout = 0;
            if (!first) hout = mP1[k] * (o2h - (ODD ? mH1[k] : mH0[k]));
            const T hn = mP0[k] * (g[k].y - hout);
            if (ODD) mH1[k] = hn;
            else mH0[k] = hn;
            bad |= has && !isfinite(hn);
          } else {
            // in^(t) = F(A_c^(t-1), out^(t-1)), out^(t-1) = F(A_own^(t-2), in^(t-2))
            T Pout = 0, hout = 0;
            if (!first) {
              const T inv_out = T(1) / (o2P - (ODD ? mP1[k] : mP0[k]));
              Pout = -av * av * inv_out;
              hout = -av * (o2h - (ODD ? mH1[k] : mH0[k])) * inv_out;
            }
            const T inv_in = T(1) / (g[k].x - Pout);
            const T Pn = -av * av * inv_in;
            const T hn = -av * (g[k].y - hout) * inv_in;
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
      T P, h;
      double acc = 0.0;
      if (OUTER || FEED) {
        P = din;
        h = rhs;
      } else {
        P = (T)row_d();
        h = (T)row_b();
      }
      if (ck) acc = (double)h - (double)(FEED ? dchk : P) * (double)x1;
      if (FEED) h = h + (din - dchk) * ((T(1) - (T)A.damp) * x2 + (T)A.damp * x1);
      for (int c = 0; c < wmax; ++c) {
        if (c > 0) {
          const T Pu = dpp<kWaveShr1, 0xf>(P, P), hu = dpp<kWaveShr1, 0xf>(h, h);
          const double au = dpp<kWaveShr1, 0xf>(acc, acc);
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
              if (ck) acc -= (double)ax[k];
            }
        }
      }
      if (upd) {
        for (int c = wmax - 2; c >= 0; --c) {  // the sums back to the head of the chain
          const T Pd = dpp<kWaveShl1, 0xf>(P, P), hd = dpp<kWaveShl1, 0xf>(h, h);
          if (pos == c && pos < len - 1) {
            P = Pd;
            h = hd;
          }
        }
        if (HONLY) P = ip;
        if (LATE && late && tail) s_o3[lrow] = V2{o2P, o2h};
        o2P = o1P;
        o2h = o1h;
        o1P = P;
        o1h = h;
        if (FEED) x2 = x1;
        if (HONLY) x1 = h * ip;
        else if (FEED || ck_next) x1 = h / P;
        if (tail) {
          const V2 v = {HONLY ? x1 : P, h};
          if (nb > 1) st_rec<V2>(ODD ? buf1 : buf0, row, v);
          s_agg[pn * cap + lrow] = v;
          if (!HONLY) s_x[pn * cap + lrow] = x1;
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
      const bool any_bad = grid_barrier(ck ? s_red[pn] : nullptr, &s_bad[t % 3], late);
      if (LATE && late) {
        if (err) return true;
        decide(uni_r(s_tot[sum_word(late)]), t - 2);
        if (conv >= 0 || err) {
          if (upd && tail) {  // the sweep taken back
            o1P = o2P;
            o1h = o2h;
            const V2 v = s_o3[lrow];
            o2P = v.x;
            o2h = v.y;
          }
          return true;
        }
      }
      if (any_bad) err |= kErrNonfinite;
      return err != 0;  // a non-finite message ends the solve
    };
    for (int t = 1;; t += 2) {
      if (sweep(std::true_type{}, t)) break;
      if (sweep(std::false_type{}, t + 1)) break;
    }
    last_rel = last_round >= 0 ? rel_of(last_tot) : -1.0;
    prev_rel = prev_round >= 0 ? rel_of(prev_tot) : -1.0;
  };

  // a workgroup that stopped waiting stores no result, and the host hears of it
  // from whichever workgroup it was
  auto give_up = [&]() -> bool {
    const bool lost = (err & kErrLost) != 0;
    if (lost && tid == 0) *A.lost = 1;
    return lost;
  };

  if constexpr (!OUTER) {
    constexpr bool HONLY = MODE == kResFrozen;
    const int M = A.max_iter;
    if constexpr (SERIAL) run_serial(A.tol, M, bnorm);
    else run(std::integral_constant<bool, HONLY>{}, A.tol, M, bnorm);
    if (give_up()) return;
    // ---- results: the returned round and the state it leaves ---------------
    // the own aggregates are of rounds T = min(conv + 1, M) and T - 1
    const int ret = conv >= 0 ? conv : M;
    const int T1 = min(ret + (conv >= 0 ? 1 : 0), M);
    const T rP = ret == T1 ? o1P : o2P, rh = ret == T1 ? o1h : o2h;
    if (tail) {
      const int out = A.inv ? A.inv[row] : row;
      A.x[out] = (double)(HONLY ? rh * ip : rh / rP);
      if (A.var) A.var[out] = (double)(HONLY ? ip : T(1) / rP);
      if (A.agg_out[0] && !HONLY) {
        ((V2*)A.agg_out[T1 % 3])[row] = V2{o1P, o1h};
        if (T1 >= 1) ((V2*)A.agg_out[(T1 - 1) % 3])[row] = V2{o2P, o2h};
      }
    }
    if (A.cin_out && !HONLY) {
      const int s0 = own ? A.off_ptr[row] + pos * K : 0;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (k < cnt) {
          ((V2*)A.cin_out)[s0 + k] = V2{mP0[k], mH0[k]};
          ((V2*)A.cin_out)[(size_t)A.E + s0 + k] = V2{mP1[k], mH1[k]};
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
      DevStatus st{};
      st.done = 1;
      st.conv_round = conv;
      st.error = err;
      st.last_rel = last_rel;
      st.last_round = last_round;
      st.prev_rel = prev_rel;
      st.prev_round = prev_round;
      *A.st = st;
    }
  } else {
    // ---- the outer loop: x <- x + d, d an inner solve on r = b - A x --------
    const RecBuf bufx = rec_buf<double>(A.xbuf, n);
    double x = 0.0;      // the row's iterate
    double rnorm = bnorm;
    bool frozen = MODE == kResOuter && A.frozen;  // else false throughout
    bool froze = false;
    int outer = 0, sweeps = 0, oconv = -1, ierr = 0, oerr = 0;
    // step 0 (x = 0, r = b): its residual is relative to itself
    double orel = bnorm > 0.0 ? 1.0 : bnorm;
    if (orel <= A.tol) oconv = 0;
    else if (!(orel <= kDivergeLimit)) oerr = kErrDiverged;
    while (oconv < 0 && !oerr && !err && outer < A.max_outer && sweeps < A.max_iter) {
      const int M = max(0, min(A.inner_max, A.max_iter - sweeps));
      const bool will_freeze = MODE == kResOuter && A.want_freeze && !frozen;
      if constexpr (MODE == kResOuter) {
        if (frozen) run(std::true_type{}, A.inner_tol, M, rnorm);
        else run(std::false_type{}, A.inner_tol, M, rnorm);
      } else if constexpr (SERIAL) {
        run_serial(A.inner_tol, M, rnorm);
      } else {
        run(std::false_type{}, A.inner_tol, M, rnorm);
      }
      if (err) {
        ierr = err;
        break;
      }
      const int ret = conv >= 0 ? conv : M;
      const int T1 = min(ret + (conv >= 0 ? 1 : 0), M);
      sweeps += ret;
      const T rP = ret == T1 ? o1P : o2P, rh = ret == T1 ? o1h : o2h;
      x += (double)(frozen ? rh * ip : rh / rP);
      // the frozen coefficients of the messages of round T1 replace the P
      // messages: g_in = -a / (P~_c - P_out), g_out = -a / (P~_own - P_in)
      if (MODE == kResOuter && will_freeze && conv >= 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const T av = (T)slot_a(k);
          const bool odd = (T1 & 1) != 0;
          const int c = REG ? cc[k] : s_c[k * LANES + tid];
          V2 g = s_agg[(T1 & 1) * cap + (c < 0 ? ~c : 0)];  // round T1 of the neighbour
          if (c >= 0) g = ld_rec<V2>(odd ? buf1 : buf0, (uint32_t)c);
          const T Pin = odd ? mP1[k] : mP0[k], Pold = odd ? mP0[k] : mP1[k];
          T Pout = 0;
          if (T1 > 0) {
            const T inv_o = T(1) / (o2P - Pold);
            Pout = -av * av * inv_o;
          }
          const T inv_in = T(1) / (g.x - Pout);
          const T inv_out = T(1) / (o1P - Pin);
          mP0[k] = k < cnt ? -av * inv_in : T(0);
          mP1[k] = k < cnt ? -av * inv_out : T(0);
          if (!REG) __builtin_amdgcn_sched_barrier(0);
        }
        ip = T(1) / o1P;
        frozen = froze = true;
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        mH0[k] = mH1[k] = 0;
        if (!frozen) mP0[k] = mP1[k] = 0;
      }
      if (tail) {
        if (nb > 1) st_rec<double>(bufx, row, x);
        s_xo[lrow] = x;
      }
      grid_barrier(nullptr, nullptr);
      if (err) break;
      // r = b - A x in FP64, the products subtracted in CSR order
      double xg[K];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const int c = REG ? cc[k] : s_c[k * LANES + tid];
        xg[k] = 0.0;
        if (nb > 1)
          xg[k] = ld_rec<double>(bufx, c < 0 ? kNoRec : (uint32_t)c / (uint32_t)(sizeof(V2) / sizeof(double)));
        const double l = s_xo[c < 0 ? ~c : 0];
        if (nb == 1 || c < 0) xg[k] = l;
      }
      double acc = __builtin_fma(-row_d(), x, row_b());
#pragma unroll
      for (int k = 0; k < K; ++k) xg[k] = slot_a(k) * xg[k];
      for (int c = 0; c < wmax; ++c) {
        if (c > 0) {
          const double au = dpp<kWaveShr1, 0xf>(acc, acc);
          if (pos == c) acc = au;
        }
        if (pos == c) {
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (k < cnt) acc -= xg[k];
        }
      }
      for (int c = wmax - 2; c >= 0; --c) {
        const double ad = dpp<kWaveShl1, 0xf>(acc, acc);
        if (pos == c && pos < len - 1) acc = ad;
      }
      {
        const double v = wsum_r(tail ? acc * acc : 0.0);
        if (lane == 0) s_red[2][wave] = v;
      }
      rhs = (T)acc;
      publish_prior(frozen);
      ++seq;
      grid_barrier(s_red[2], nullptr);
      rnorm = uni_r(sqrt(total(s_red[2])));
      if (err) break;
      ++outer;
      orel = bnorm > 0.0 ? rnorm / bnorm : rnorm;
      if (orel <= A.tol) oconv = 0;
      else if (!(orel <= kDivergeLimit)) oerr = kErrDiverged;
    }
    if (give_up()) return;
    if (tail) A.x[A.inv ? A.inv[row] : row] = x;
    if (froze && A.coef_out) {  // later calls start from the frozen precisions
      if (tail) ((T*)A.inv_pt_out)[row] = ip;
      const int s0 = own ? A.off_ptr[row] + pos * K : 0;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (k < cnt) ((V2*)A.coef_out)[s0 + k] = V2{mP0[k], mP1[k]};
    }
    if (blockIdx.x == 0 && tid == 0) {
      DevStatus st{};
      st.done = 1;
      st.conv_round = oconv;
      st.error = oerr;
      st.pad = ierr;
      st.last_rel = orel;
      st.ticket = (uint32_t)sweeps;
      st.last_round = outer;
      st.pad2 = froze ? 1 : 0;
      *A.st = st;
    }
  }
}

// dynamic LDS of a workgroup
template <typename T>
uint32_t res_lds(int rows_cap, int lanes, int K, int mode) {
  size_t b = 2 * (size_t)rows_cap * (sizeof(vec2<T>) + sizeof(T));
  if (res_outer(mode)) b += sizeof(double) * (size_t)rows_cap;
  if (res_late(mode, lanes)) b += sizeof(vec2<T>) * (size_t)rows_cap;
  if (lanes == kRL) b += (size_t)lanes * (K * (sizeof(double) + sizeof(int)) + 2 * sizeof(double));
  return (uint32_t)b;
}

}  // namespace

}  // namespace gabp
