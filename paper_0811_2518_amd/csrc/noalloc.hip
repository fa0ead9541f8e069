// gabp_solve_noalloc: the plain FP64 solve of gabp_create + gabp_solve for a
// small system, allocating nothing.  For callers that cannot allocate device
// memory (code under stream capture, tight serving loops, harnesses that
// forbid allocation).
//
// One launch of one workgroup validates the caller's full CSR, splits it into
// the off-diagonal CSR of Alg. 2's neighbourhoods N(i) (Ch. 3 Sec. 3.3) and the
// diagonal, and runs the sweeps of small.h, all of it in LDS and registers;
// then one copy brings the status back to the host.  No hipMalloc, hipFree or
// allocating library call.  The status and the validation flags are the only
// device memory beyond the caller's inputs and outputs: one file-scope array,
// `scratch`, of which each device holds its own copy; its address is looked up
// once per device with hipGetSymbolAddress and kept.  Calls that overlap on
// one device share that array and race.
//
// What bounds a call is latency: the launch, the round trip for the inputs, the
// sweeps (small.h) and the copy.  As two launches that walked the rows and
// searched the mirror entries in global memory, and sweeps of two divisions a
// slot, a solve of G(600, 1800) to 1e-10 took 191 us; now 116 us (about 40 us of
// it outside the sweeps, before 60).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>
#include <string>

#include "small.h"

#pragma clang fp contract(off)

namespace gabp {

namespace {

constexpr int kNaRows = kSmallLanes;       // largest n
constexpr int kNaSlots = 4 * kSmallLanes;  // largest number of off-diagonal entries

constexpr int kNaArg = 1;
constexpr int kNaZeroDiag = 2;
constexpr int kNaAsym = 4;
constexpr int kNaNonfinite = 8;
constexpr int kNaTooLarge = 16;

struct NaHeader {
  DevStatus st;   // of the sweeps, where the validation passed
  int32_t flags;  // kNa* bits of the validation
  int32_t pad;
};

constexpr size_t kScratchBytes = (sizeof(NaHeader) + 255) / 256 * 256;

// First of the slots lo .. hi - 1 (sorted by column) whose column is not below r.
template <typename Col>
__device__ __forceinline__ int find_slot(int lo, int hi, int r, Col col_of) {
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (col_of(mid) < r) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// Validation of the caller's full CSR (the checks of gabp_create), the split,
// and the solve.  The caller's CSR is staged in LDS (coalesced, one round trip);
// lane r then walks row r there, and the slot lanes look up their mirror slots
// for the symmetry check, which runs only on a sound structure, so every search
// stays inside the split arrays.
__global__ __launch_bounds__(kNaRows) void k_noalloc(int32_t n, const int32_t* __restrict__ row_ptr,
                                                     const int32_t* __restrict__ col,
                                                     const double* __restrict__ vals, SmallArgs A, NaHeader* out) {
  constexpr int K = kNaSlots / kNaRows, S = kNaSlots, N = kNaRows;
  extern __shared__ __align__(16) double sm[];
  __shared__ int s_flags;
  __shared__ unsigned long long s_max;
  __shared__ int s_bad[3];
  const int tid = threadIdx.x, lane = tid & 63;
  // the caller's CSR, in what will hold the messages (S + N entries of 12 bytes in 16 S)
  static_assert(3 * (S + N) <= 4 * S, "the staged CSR fits in the message buffer");
  double* s_val = sm;                       // [S + N]
  int* s_col = (int*)(sm + S + N);          // [S + N]
  // the split, in what will hold the a x terms, the aggregates and the means
  double* s_a = sm + 2 * S;                 // [S]
  uint32_t* s_rc = (uint32_t*)(sm + 3 * S); // [S] row and column, packed
  int* s_ptr = (int*)(s_rc + S);            // [N + 1]
  static_assert(4 * S + 4 * (N + 1) <= 24 * N, "the split fits in the rows' part");
  const int nnz = row_ptr[n];
  // the caller's arrays are read only where their size makes sense
  const int size_flag = row_ptr[0] != 0 || nnz < n ? kNaArg : (int64_t)nnz - n > kNaSlots ? kNaTooLarge : 0;
  if (size_flag) {
    if (tid == 0) out->flags = size_flag;
    return;
  }
  if (tid == 0) {
    s_flags = 0;
    s_max = 0ull;
  }
  if (tid < 3) s_bad[tid] = 0;
  const int E = nnz - n;
  int lo = 0, hi = 0;
  double br = 0.0;
  if (tid < n) {
    lo = row_ptr[tid];
    hi = row_ptr[tid + 1];
    br = A.rhs[tid];
  }
  for (int e = tid; e < nnz; e += kNaRows) {
    s_col[e] = col[e];
    s_val[e] = vals[e];
  }
  __syncthreads();
  int flags = 0;
  double maxabs = 0.0, dv = 0.0;
  if (tid < n) {
    if (lo < 0 || hi > nnz || hi < lo) {  // never read outside col / vals
      flags |= kNaArg;
      lo = hi = 0;
    }
    int prev = -1, ndiag = 0;
    int k = lo - tid;  // off-diagonal slot of the row's next off-diagonal entry
    for (int e = lo; e < hi; ++e) {
      const int c = s_col[e];
      const double v = s_val[e];
      if (c < 0 || c >= n || c <= prev) flags |= kNaArg;
      prev = c;
      if (!isfinite(v)) flags |= kNaNonfinite;
      maxabs = fmax(maxabs, fabs(v));
      if (c == tid) {
        ++ndiag;
        dv = v;
      } else {
        if (k >= 0 && k < kNaSlots) {
          s_rc[k] = pack_slot(tid, c & 1023);
          s_a[k] = v;
        }
        ++k;
      }
    }
    if (ndiag != 1 || dv == 0.0) flags |= kNaZeroDiag;
    s_ptr[tid] = lo - tid;
    if (tid == n - 1) s_ptr[n] = hi - n;
  }
  if (flags) atomicOr(&s_flags, flags);
  if (!isfinite(maxabs)) maxabs = 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) maxabs = fmax(maxabs, __shfl_xor(maxabs, off, 64));
  if (lane == 0 && maxabs > 0.0) atomicMax(&s_max, (unsigned long long)__double_as_longlong(maxabs));
  __syncthreads();
  if (s_flags) {
    if (tid == 0) out->flags = s_flags;
    return;
  }
  // |A_ij - A_ji| <= 1e-12 max|A| and the mirror entry present
  const double tolv = 1e-12 * __longlong_as_double((long long)s_max);
  uint32_t meta[K];
  double aa[K], am[K];
  int asym = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int s = tid + k * kNaRows;
    meta[k] = (uint32_t)s << 20;
    aa[k] = am[k] = 0.0;
    if (s < E) {
      const uint32_t rc = s_rc[s];
      const int r = slot_row(rc), c = slot_col(rc);
      aa[k] = s_a[s];
      const int end = s_ptr[c + 1];
      const int m = find_slot(s_ptr[c], end, r, [&](int q) { return slot_col(s_rc[q]); });
      if (m < end && slot_col(s_rc[m]) == r) {
        am[k] = s_a[m];
        meta[k] = rc | ((uint32_t)m << 20);
        if (fabs(aa[k] - am[k]) > tolv) asym = 1;
      } else {
        asym = 1;
      }
    }
  }
  if (__syncthreads_or(asym)) {
    if (tid == 0) out->flags = kNaAsym;
    return;
  }
  if (tid == 0) out->flags = 0;
  small_loop<K, false>(A, n, E, sm, s_bad, meta, aa, am, lo - tid, hi - tid - 1, tid < n ? dv : 1.0, br);
}

}  // namespace

}  // namespace gabp

// The library's static device buffer of the no-allocation entry point (one
// copy per device, held until the process ends).  Host code never uses this
// name as an address: it takes the device address from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[gabp::kScratchBytes];

namespace gabp {

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up on the first
// call made with that device current.
gabp_status scratch_on_current_device(NaHeader** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(nullptr, GABP_E_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, GABP_E_ARG, "device index beyond the supported range");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(nullptr, GABP_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    }
    g_scratch_ptr[dev] = p;
  }
  *out = (NaHeader*)g_scratch_ptr[dev];
  return GABP_OK;
}

}  // namespace

}  // namespace gabp

extern "C" gabp_status gabp_solve_noalloc(int32_t n, const int32_t* row_ptr, const int32_t* col_idx,
                                          const double* vals, const double* b, double* x, double* var, double tol,
                                          int32_t max_iter, hipStream_t stream, gabp_info* info) {
  using namespace gabp;
  if (info) std::memset(info, 0, sizeof(*info));
  if (n < 0) return fail(nullptr, GABP_E_ARG, "n < 0");
  if (n > kNaRows)
    return fail(nullptr, GABP_E_ARG,
                "n = " + std::to_string(n) + " exceeds the no-allocation limit of " + std::to_string(kNaRows) +
                    " rows");
  if (max_iter < 0) return fail(nullptr, GABP_E_ARG, "max_iter < 0");
  if (std::isnan(tol)) return fail(nullptr, GABP_E_ARG, "tol is NaN");
  if (n == 0) {
    if (info) info->converged = 1;
    return GABP_OK;
  }
  if (!row_ptr || !col_idx || !vals || !b || !x) return fail(nullptr, GABP_E_ARG, "NULL argument");
  NaHeader* sc = nullptr;
  gabp_status r = scratch_on_current_device(&sc);
  if (r != GABP_OK) return r;

  SmallArgs a{};
  a.n = n;
  a.rhs = b;
  a.tol = tol;
  a.max_iter = max_iter;
  a.check_every = 1;
  a.st = &sc->st;
  a.x_direct = x;
  a.var_direct = var;
  // the split needs the LDS of the largest n
  const uint32_t lds = (uint32_t)small_lds(kNaRows, kNaSlots / kNaRows);
  (void)hipFuncSetAttribute((const void*)k_noalloc, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(k_noalloc, dim3(1), dim3(kNaRows), lds, stream, n, row_ptr, col_idx, vals, a, sc);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(nullptr, GABP_E_HIP, std::string("solve launch: ") + hipGetErrorString(e));
  NaHeader h{};
  e = hipMemcpyAsync(&h, sc, sizeof(h), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return fail(nullptr, GABP_E_HIP, std::string("status copy: ") + hipGetErrorString(e));

  gabp_status st;
  if (h.flags & kNaArg)
    st = fail(nullptr, GABP_E_ARG,
              "CSR structure: row_ptr[0] != 0, row pointers decrease, columns unsorted/duplicated or out of range");
  else if (h.flags & kNaTooLarge)
    st = fail(nullptr, GABP_E_ARG,
              "the matrix has more than " + std::to_string(kNaSlots) +
                  " off-diagonal entries, the no-allocation limit (use gabp_create)");
  else if (h.flags & kNaNonfinite)
    st = fail(nullptr, GABP_E_NONFINITE, "non-finite matrix value");
  else if (h.flags & kNaZeroDiag)
    st = fail(nullptr, GABP_E_ZERO_DIAG, "a diagonal entry is missing or zero");
  else if (h.flags & kNaAsym)
    st = fail(nullptr, GABP_E_NOT_SYMMETRIC, "pattern or values of A are not symmetric");
  else if (h.st.error & kErrNonfinite)
    st = fail(nullptr, GABP_E_NONFINITE, "non-finite message (P~_i = P_ji or overflow)");
  else if (tol > 0.0 && (h.st.error & kErrDiverged))
    st = fail(nullptr, GABP_E_DIVERGED, "residual diverged");
  else
    st = (tol <= 0.0 || h.st.conv_round >= 0) ? GABP_OK : GABP_NOT_CONVERGED;
  if (info && h.flags == 0) {
    info->sweeps = h.st.conv_round >= 0 ? h.st.conv_round : max_iter;
    info->converged = h.st.conv_round >= 0 ? 1 : 0;
    info->rel_residual = h.st.last_rel;
  }
  if (info) info->status = st;
  return st;
}
