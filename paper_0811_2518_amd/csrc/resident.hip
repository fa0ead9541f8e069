// Host side of the resident solve (resident.h): the plan, its set-up and the
// FP64 kernels.
#include <algorithm>
#include <cstring>

#include "chip_gate.h"
#include "resident.h"

namespace gabp {

static const int2 kIdleLane{-1, 1 << 8};

// The plan: rows dealt to lanes in order, chains inside one wave, workgroups
// of `lanes` lanes (with XCD parts: no workgroup spans two of them, and every
// part gets the same number).  Empty when the system does not fit.
ResPlanHost plan_resident(const std::vector<int32_t>& op, int32_t n, int K, int lanes, int max_blocks,
                          const std::vector<int32_t>& parts) {
  std::vector<uint8_t> len_of(n);  // lanes of a row
  for (int32_t r = 0; r < n; ++r) {
    const int32_t d = op[r + 1] - op[r];
    const int len = d <= K ? 1 : (d + K - 1) / K;
    if (len > 64) return ResPlanHost{};
    len_of[r] = (uint8_t)len;
  }
  const size_t np = parts.size() > 1 ? parts.size() - 1 : 1;
  // a part's lanes in order, a chain padded to the next wave where it would
  // cross a wave's end
  int64_t most = 0;
  for (size_t p = 0; p < np; ++p) {
    int64_t total = 0;
    for (int32_t r = np > 1 ? parts[p] : 0; r < (np > 1 ? parts[p + 1] : n); ++r) {
      const int len = len_of[r];
      if (total % 64 + len > 64) total += 64 - total % 64;
      total += len;
    }
    most = std::max(most, total);
  }
  // workgroups per part.  The smallest size takes as few as hold the rows; a
  // larger one is only asked for when those would be too many, and spreads
  // over all of them.  Waves per workgroup: evenly, more where the cuts
  // between workgroups leave too many
  const int64_t room = max_blocks / (int64_t)np;
  int64_t want = std::max<int64_t>(1, (most + lanes - 1) / lanes);
  if (lanes > 256) want = std::max(want, room);
  if (want > room) return ResPlanHost{};
  for (int64_t per = std::max<int64_t>(1, ((most + 63) / 64 + want - 1) / want); per * 64 <= lanes; ++per) {
    std::vector<std::vector<int2>> blk(np), lane(np);  // {first row, rows} of every workgroup of a part
    for (size_t p = 0; p < np; ++p) {
      const int32_t lo = np > 1 ? parts[p] : 0, hi = np > 1 ? parts[p + 1] : n;
      std::vector<int2>& ll = lane[p];
      size_t base = 0;  // first lane of the workgroup being filled
      int used = 0;
      int2 cur{lo, 0};
      ll.reserve((size_t)room * lanes);  // grown a workgroup at a time
      ll.assign(lanes, kIdleLane);
      for (int32_t r = lo; r < hi; ++r) {
        const int len = len_of[r];
        int at = used;
        if (at % 64 + len > 64) at += 64 - at % 64;
        if (at + len > per * 64) {  // the row starts the next workgroup
          blk[p].push_back(cur);
          cur = int2{r, 0};
          base += lanes;
          ll.resize(base + lanes, kIdleLane);
          at = 0;
        }
        for (int q = 0; q < len; ++q) ll[base + at + q] = int2{r, q | (len << 8)};
        used = at + len;
        ++cur.y;
      }
      blk[p].push_back(cur);
    }
    size_t q = 0;
    for (auto& v : blk) q = std::max(q, v.size());
    if ((int64_t)q > room) continue;
    ResPlanHost pl;
    pl.K = K;
    pl.lanes = lanes;
    for (size_t p = 0; p < np; ++p) {
      for (; blk[p].size() < q;) {  // empty workgroups keep part p on XCD p
        blk[p].push_back(int2{np > 1 ? parts[p + 1] : n, 0});
        lane[p].resize(lane[p].size() + lanes, kIdleLane);
      }
      pl.blk.insert(pl.blk.end(), blk[p].begin(), blk[p].end());
      if (np == 1) pl.lane = std::move(lane[p]);
      else pl.lane.insert(pl.lane.end(), lane[p].begin(), lane[p].end());
    }
    for (const int2& v : pl.blk) pl.rows_cap = std::max(pl.rows_cap, v.y);
    return pl;
  }
  return ResPlanHost{};
}

// The same for colour-serial sweeps, whose workgroups each take a share of
// every class (all of them work on the class being swept): rows in order inside
// a class, so that the shares of a workgroup lie near each other in a grid.
ResPlanHost plan_resident_serial(const std::vector<int32_t>& op, int32_t n, int K, int lanes, int max_blocks,
                                 const std::vector<int32_t>& classes) {
  auto chain = [&](int32_t r) { return std::max(1, (op[r + 1] - op[r] + K - 1) / K); };
  const int ncls = (int)classes.size() - 1;
  std::vector<int64_t> total(ncls, 0);
  int64_t all = 0;
  for (int q = 0; q < ncls; ++q)
    for (int32_t r = classes[q]; r < classes[q + 1]; ++r) {
      if (chain(r) > 64) return ResPlanHost{};
      total[q] += chain(r);
    }
  for (int64_t v : total) all += v;
  int64_t nb = std::max<int64_t>(1, (all + lanes - 1) / lanes);
  if (lanes > 256) nb = std::max<int64_t>(nb, max_blocks);
  for (; nb <= max_blocks; nb += std::max<int64_t>(1, nb / 16)) {
    ResPlanHost pl;
    pl.K = K;
    pl.lanes = lanes;
    std::vector<int32_t> at(classes.begin(), classes.end() - 1);  // next row of every class
    std::vector<int64_t> done(ncls, 0);
    bool fits = true;
    for (int64_t b = 0; fits && b < nb; ++b) {
      std::vector<int2> ll;
      int32_t rows = 0;
      for (int q = 0; q < ncls; ++q) {
        pl.cls_tab.push_back(int2{at[q], rows});
        const int64_t end = total[q] * (b + 1) / nb;
        while (at[q] < classes[q + 1] && (b == nb - 1 || done[q] < end)) {
          const int32_t r = at[q]++;
          const int len = chain(r);
          if (ll.size() % 64 + len > 64) ll.resize((ll.size() + 63) / 64 * 64, kIdleLane);
          for (int k = 0; k < len; ++k) ll.push_back(int2{r, k | (len << 8) | (q << 16)});
          done[q] += len;
          ++rows;
        }
      }
      pl.cls_tab.push_back(int2{n, rows});
      fits = (int64_t)ll.size() <= lanes;
      ll.resize(lanes, kIdleLane);
      pl.lane.insert(pl.lane.end(), ll.begin(), ll.end());
      pl.blk.push_back(int2{0, rows});
      pl.rows_cap = std::max(pl.rows_cap, rows);
    }
    if (fits) return pl;
  }
  return ResPlanHost{};
}

namespace {

template <int LANES, int K>
ResKernel kernel64(int mode) {
  if constexpr (K == 4) {
    if (mode == kResSerial) return k_resident<double, LANES, 4, kResSerial>;
    return mode == kResFrozen ? k_resident<double, LANES, 4, kResFrozen> : k_resident<double, LANES, 4, kResJoint>;
  } else {
    switch (mode) {
      case kResSerial: return k_resident<double, LANES, K, kResSerial>;
      case kResSerialOuter: return k_resident<double, LANES, K, kResSerialOuter>;
      case kResFrozen: return k_resident<double, LANES, K, kResFrozen>;
      case kResOuter: return k_resident<double, LANES, K, kResOuter>;
      case kResLoop: return k_resident<double, LANES, K, kResLoop>;
      default: return k_resident<double, LANES, K, kResJoint>;
    }
  }
}
template <int K>
ResKernel kernel64_l(int lanes, int mode) {
  if (lanes == 256) return kernel64<256, K>(mode);
  if (lanes == 512) return kernel64<512, K>(mode);
  return kernel64<kRL, K>(mode);
}

ResKernel res_kernel(bool fp32, int lanes, int K, int mode) {
  if (fp32) return res_kernel32(lanes, K, mode);
  return K == 4 ? kernel64_l<4>(lanes, mode) : kernel64_l<6>(lanes, mode);
}

uint32_t lds_bytes(const Ctx* c, int rows_cap, int lanes, int K, int mode) {
  return c->opts.precision == GABP_FP32_REFINE ? res_lds<float>(rows_cap, lanes, K, mode)
                                               : res_lds<double>(rows_cap, lanes, K, mode);
}

// The mode of a handle's first solve, or -1 where an option asks for a step
// between the sweeps or for another layout.
int handle_mode(const Ctx* c) {
  const bool serial = c->opts.layout == kLayoutSerial;
  constexpr int32_t kOtherSerial = GABP_FLAG_MULTI_LAUNCH | GABP_FLAG_TIME_SWEEPS;
  constexpr int32_t kOtherSync = GABP_FLAG_POISON_STALE | GABP_FLAG_PREDICT_ALL | GABP_FLAG_AITKEN | GABP_FLAG_STEFFENSEN;
  const int32_t kOther = kOtherSerial | (serial ? 0 : kOtherSync);
  if ((c->opts.flags & kOther) || (c->opts.layout != 0 && c->opts.layout != kLayoutCompact && !serial)) return -1;
  const bool fp32 = c->opts.precision == GABP_FP32_REFINE;
  if (serial) {
    if (c->ncol < 1 || c->ncol > 0x7fff || (c->opts.flags & GABP_FLAG_SINGLE_LOOP) || c->opts.inner_max_iter < 1)
      return -1;
    return !fp32 && c->gamma_used == 0.0 && c->opts.gamma == 0.0 ? kResSerial : kResSerialOuter;
  }
  if (!fp32 && c->gamma_used == 0.0 && c->opts.gamma == 0.0) return kResJoint;
  const bool single = (c->opts.flags & GABP_FLAG_SINGLE_LOOP) != 0;
  if (single && !fp32) return kResLoop;
  if (single && c->gamma_used > 0.0) return kResOuterLoop;
  // no loading and no reuse: the inner solves never run on frozen precisions
  return fp32 && c->gamma_used == 0.0 && !(c->opts.flags & GABP_FLAG_REUSE_PRECISION) ? kResRefine : kResOuter;
}

}  // namespace

// Slots per lane and lanes per workgroup of a handle.  4 or 6 slots are a lane
// of 2-D and 3-D grids, whose rows then need no chain; longer rows take chains
// of 6 (FP64) or 8 (FP32).  Workgroups: one if it holds every row (no grid
// barrier: the 29 x 23 grid's mean-only sweep takes 2.05 us in one workgroup,
// 3.09 us in three); else as small as the CU count allows, since a sweep of few
// waves per CU is bound by the latency of its dependent divisions and exchanges
// (measured at 256 / 512 / 1024 lanes, checked FP64 sweeps whose stop decision
// falls before the update: 181 x 173 grid 4.58
// / 4.93 / 5.65 us, G(n, 4n) with n = 30011 6.94 / 8.27 / 12.5 us).  At 1024 lanes
// the 128 registers do not hold everything: the FP64 loops on frozen precisions
// spill 120 of them (512 lanes: 13), the FP64 single loop 17, the plain FP64 solve
// 2, the FP32 loops 11 (K = 6) and 37 (K = 8).  They are still ahead of a launch per
// sweep: the FP64 double loop on B^T B + 0.1 I with n = 52000 6.4 against 10.7 ms for
// 60 outer steps and the single loop 6.9 against 11.1, the FP32 double loop with n =
// 56000 5.5 against 9.8; with loading 0.1 the 60^3 grid 4.1 against 10.7 ms in FP64
// and 2.6 against 8.2 in FP32; the plain solve of that grid 1.05 against 2.69 ms.
gabp_status setup_resident(Ctx* c) {
  c->res = ResPlan{};
  const int mode = handle_mode(c);
  if (c->n < 1 || c->E < 1 || mode < 0) return GABP_OK;
  const bool fp32 = c->opts.precision == GABP_FP32_REFINE;
  int dev = 0, ncu = 0, khz = 0;
  GABP_HIP(c, hipGetDevice(&dev));
  GABP_HIP(c, hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
  GABP_HIP(c, hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  int K = 6;
  if (mode == kResOuterLoop && fp32) K = 8;
  else if (c->max_degree <= 4 && (fp32 || mode == kResJoint || mode == kResSerial)) K = 4;
  else if (c->max_degree > 6 && fp32) K = 8;
  const int max_blocks = std::min(ncu, kResMaxBlocks);
  // rows whose chains the lanes can hold, before the plan walks them
  if (c->max_degree > kResMaxChain * K || c->n > (int64_t)max_blocks * kRL ||
      c->E > (int64_t)max_blocks * kRL * K)
    return GABP_OK;
  const bool serial = mode == kResSerial || mode == kResSerialOuter;
  const std::vector<int32_t> none;
  ResPlanHost pl;
  for (int blocks : {1, max_blocks})
    for (int lanes : {256, 512, kRL}) {
      if (!pl.blk.empty() || c->E > (int64_t)blocks * lanes * K || c->n > (int64_t)blocks * lanes) continue;
      pl = serial ? plan_resident_serial(c->off_ptr_h, c->n, K, lanes, blocks, c->colour_start)
                  : plan_resident(c->off_ptr_h, c->n, K, lanes, blocks,
                                  blocks == 1 || c->nparts == 0 ? none : c->part_start);
    }
  if (pl.blk.empty()) return GABP_OK;
  int most = INT32_MAX;  // workgroups that a CU holds
  for (int m : {mode, (int)kResFrozen}) {
    if (m == kResFrozen && (mode != kResJoint || !(c->opts.flags & GABP_FLAG_REUSE_PRECISION))) break;
    const void* f = (const void*)res_kernel(fp32, pl.lanes, K, m);
    const uint32_t lds = lds_bytes(c, pl.rows_cap, pl.lanes, K, m);
    GABP_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per = 0;
    GABP_HIP(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, f, pl.lanes, lds));
    if ((int64_t)per * ncu < (int64_t)pl.blk.size()) return GABP_OK;
    most = std::min(most, per);
  }
  // one allocation: control blocks (zero), workgroups, lanes, class tables
  const size_t nblk = pl.blk.size(), o_lane = 2 * sizeof(ResCtl) + sizeof(int2) * nblk;
  const size_t o_tab = o_lane + sizeof(int2) * pl.lane.size(), o_cls = o_tab + sizeof(int2) * pl.cls_tab.size();
  std::vector<unsigned char> img(o_cls + (serial ? sizeof(int32_t) * c->colour_start.size() : 0), 0);
  std::memcpy(img.data() + 2 * sizeof(ResCtl), pl.blk.data(), sizeof(int2) * nblk);
  std::memcpy(img.data() + o_lane, pl.lane.data(), sizeof(int2) * pl.lane.size());
  if (serial) {
    std::memcpy(img.data() + o_tab, pl.cls_tab.data(), sizeof(int2) * pl.cls_tab.size());
    std::memcpy(img.data() + o_cls, c->colour_start.data(), sizeof(int32_t) * c->colour_start.size());
  }
  void* base = nullptr;
  const gabp_status r = dev_alloc(c, &base, img.size());
  if (r != GABP_OK) return r;
  GABP_HIP(c, hipMemcpyAsync(base, img.data(), img.size(), hipMemcpyHostToDevice, c->stream));
  GABP_HIP(c, hipStreamSynchronize(c->stream));
  c->res.K = K;
  c->res.mode = mode;
  c->res.lanes = pl.lanes;
  c->res.nb = (int32_t)pl.blk.size();
  c->res.rows_cap = pl.rows_cap;
  c->res.ctl_d = (ResCtl*)base;
  c->res.blk_d = (int2*)((char*)base + 2 * sizeof(ResCtl));
  c->res.lane_d = (int2*)((char*)base + o_lane);
  c->res.cls_tab_d = (int2*)((char*)base + o_tab);
  c->res.cls_start_d = (int32_t*)((char*)base + o_cls);
  c->res.khz = khz;
  c->res.dev = dev;
  c->res.ncu = ncu;
  c->res.need = (c->res.nb + most - 1) / most;
  return GABP_OK;
}

ChipGate& chip_gate(int dev) {
  constexpr unsigned kDevices = 64;  // devices beyond share a gate
  static ChipGate* gates = new ChipGate[kDevices];  // kept: threads may solve until the process ends
  return gates[(unsigned)dev % kDevices];
}

hipError_t launch_resident(Ctx* c, ResArgs a, bool frozen_plain, hipStream_t s) {
  ResPlan& p = c->res;
  const int mode = frozen_plain ? (int)kResFrozen : p.mode;
  a.n = c->n;
  a.E = (int32_t)c->E;
  a.off_ptr = c->off_ptr_d;
  a.col = c->off_col_d;
  a.a = c->a64_d;
  a.d64 = c->d64_d;
  a.inv = c->perm_d ? c->inv_d : nullptr;
  a.coef = c->gcoef_d;
  a.inv_pt = c->inv_pt_d;
  a.agg[0] = c->agg_d[0];
  a.agg[1] = c->agg_d[1];
  a.check_every = c->opts.check_every;
  a.st = c->st_small_d;
  a.lost = (int32_t*)(c->st_small_d + 1);
  a.blk = p.blk_d;
  a.lane = p.lane_d;
  a.ncls = c->ncol;
  a.cls_start = p.cls_start_d;
  a.cls_tab = p.cls_tab_d;
  a.rows_cap = p.rows_cap;
  // The launch before cleared this one's control block, if it ran: one that was
  // refused, or recorded into a capture, did not, and left counters behind that
  // would let this one's barriers through.
  if (!p.clean) {
    const hipError_t e = launch_fill((double*)p.ctl_d, 2 * sizeof(ResCtl) / sizeof(double), 0.0, s);
    if (e != hipSuccess) return e;
  }
  p.clean = false;  // until solve_resident has seen the launch's status
  p.phase ^= 1;
  a.ctl = p.ctl_d + p.phase;
  a.ctl_next = p.ctl_d + (p.phase ^ 1);
  a.roll_limit = c->aid[kAidRollLimit] ? (uint64_t)c->aid[kAidRollLimit] - 1 : (uint64_t)p.khz * kResRollMs;
  a.wait_limit = c->aid[kAidWaitLimit] ? (uint64_t)c->aid[kAidWaitLimit] - 1 : (uint64_t)p.khz * kResWaitMs;
  const bool fp32 = c->opts.precision == GABP_FP32_REFINE;
  hipLaunchKernelGGL(res_kernel(fp32, p.lanes, p.K, mode), dim3(p.nb), dim3(p.lanes),
                     lds_bytes(c, p.rows_cap, p.lanes, p.K, mode), s, a);
  return hipGetLastError();
}

}  // namespace gabp
