// k_scan.hip -- exclusive prefix sums (u32, u64) used to size and place the
// tree's nodes and the per-leaf interaction lists.
// Up to kScanOne elements: one launch, a block per array.  Above: two passes,
// tile totals, then the tile scan, each block first adding up the totals of the
// tiles before its own (a few hundred at most for the sizes here, so this costs
// less than a launch of its own).  Bound by launches and latency: arrays of one
// length are scanned together.  Deterministic (integer arithmetic, fixed order).
#include <algorithm>

#include "sfmm_internal.h"

namespace sfmm {
namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = SCAN_THREADS * SCAN_ITEMS;

// exclusive sum over a block of WAVES waves, and its total (sh: WAVES words)
template <int WAVES>
__device__ __forceinline__ uint64_t block_exclusive(uint64_t v, uint64_t* sh, uint64_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint64_t incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t u = __shfl_up((unsigned long long)incl, o, 64);
    if (lane >= o) incl += u;
  }
  if (lane == 63) sh[w] = incl;
  __syncthreads();
  uint64_t pre = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    const uint64_t c = sh[k];
    if (k < w) pre += c;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return pre + incl - v;
}

// N entries from `at` on (0 past n); all loads before any use
template <int N>
__device__ __forceinline__ void job_in(const ScanJob& j, int64_t at, int64_t n, uint64_t* v) {
  if (j.in32) {
    uint32_t x[N];
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = j.in32[at + k < n ? at + k : 0];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = at + k < n ? x[k] : 0u;
  } else {
    uint64_t x[N];
#pragma unroll
    for (int k = 0; k < N; ++k) x[k] = j.in64[at + k < n ? at + k : 0];
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = at + k < n ? x[k] : 0u;
  }
}
template <int N>
__device__ __forceinline__ void job_out(const ScanJob& j, int64_t at, int64_t n, uint64_t run,
                                        const uint64_t* v) {
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if (at + k < n) {
      if (j.out32) j.out32[at + k] = (uint32_t)run;
      else j.out64[at + k] = run;
    }
    run += v[k];
  }
}
__device__ __forceinline__ void job_total(const ScanJob& j, uint64_t v) {
  if (j.total32) *j.total32 = (uint32_t)v;
  else *j.total64 = v;
}

constexpr int ONE_THREADS = 1024, ONE_ITEMS = 2;
__global__ __launch_bounds__(ONE_THREADS) void k_scan_one(ScanJobs jobs, int n) {
  __shared__ uint64_t sh[ONE_THREADS / 64];
  const ScanJob j = jobs.j[blockIdx.x];
  uint64_t carry = 0;
  for (int base = 0; base < n; base += ONE_THREADS * ONE_ITEMS) {
    const int at = base + (int)threadIdx.x * ONE_ITEMS;
    uint64_t v[ONE_ITEMS], s = 0;
    job_in<ONE_ITEMS>(j, at, n, v);
#pragma unroll
    for (int k = 0; k < ONE_ITEMS; ++k) s += v[k];
    uint64_t tot;
    const uint64_t run = carry + block_exclusive<ONE_THREADS / 64>(s, sh, &tot);
    job_out<ONE_ITEMS>(j, at, n, run, v);
    carry += tot;
  }
  if (threadIdx.x == 0) job_total(j, carry);
}

// (blockIdx.y: the job; its tile totals at tmp + tiles * job)
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(ScanJobs jobs, int64_t n,
                                                              uint64_t* tmp) {
  __shared__ uint64_t sh[SCAN_THREADS / 64];
  const ScanJob j = jobs.j[blockIdx.y];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  uint64_t v[SCAN_ITEMS], s = 0;
  job_in<SCAN_ITEMS>(j, base, n, v);
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) s += v[k];
  uint64_t tot;
  block_exclusive<SCAN_THREADS / 64>(s, sh, &tot);
  if (threadIdx.x == 0) tmp[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = tot;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_down(ScanJobs jobs, int64_t n,
                                                            const uint64_t* tmp) {
  __shared__ uint64_t sh[SCAN_THREADS / 64];
  const ScanJob j = jobs.j[blockIdx.y];
  tmp += (int64_t)blockIdx.y * gridDim.x;
  // the totals of the tiles before this one, in a fixed order
  uint64_t pre = 0;
  for (int64_t i = threadIdx.x; i < (int64_t)blockIdx.x; i += SCAN_THREADS) pre += tmp[i];
  uint64_t prefix;
  block_exclusive<SCAN_THREADS / 64>(pre, sh, &prefix);
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
  uint64_t v[SCAN_ITEMS];
  uint64_t s = 0;
  job_in<SCAN_ITEMS>(j, base, n, v);
#pragma unroll
  for (int k = 0; k < SCAN_ITEMS; ++k) s += v[k];
  uint64_t tot;
  const uint64_t run = block_exclusive<SCAN_THREADS / 64>(s, sh, &tot) + prefix;
  job_out<SCAN_ITEMS>(j, base, n, run, v);
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) job_total(j, prefix + tot);
}

// one tile of the second form: below it a launch is saved (3 us of a solve of
// 1e3 particles, whose walk's three scans took 27 us in six launches); from two
// tiles on the two launches are faster (walk of 1e5 particles, 1.5e4 leaves:
// 0.210 ms with two launches, 0.220 with one block an array, 0.228 with two
// launches an array)
constexpr int64_t kScanOne = ONE_THREADS * ONE_ITEMS;

}  // namespace

size_t scan_tmp_elems(int64_t n) { return (size_t)((n + SCAN_TILE - 1) / SCAN_TILE) + 1; }

void scan_jobs(const ScanJobs& jobs, int count, int64_t n, uint64_t* tmp, hipStream_t s) {
  if (n <= kScanOne) {  // (also n == 0: the totals become 0)
    k_scan_one<<<count, ONE_THREADS, 0, s>>>(jobs, (int)std::max<int64_t>(n, 0));
    return;
  }
  const dim3 grid((unsigned)((n + SCAN_TILE - 1) / SCAN_TILE), (unsigned)count);
  k_scan_reduce<<<grid, SCAN_THREADS, 0, s>>>(jobs, n, tmp);
  k_scan_down<<<grid, SCAN_THREADS, 0, s>>>(jobs, n, tmp);
}

void scan_u32(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* total, uint64_t* tmp,
              hipStream_t s) {
  ScanJobs jobs{};
  jobs.j[0].in32 = in;
  jobs.j[0].out32 = out;
  jobs.j[0].total32 = total;
  scan_jobs(jobs, 1, n, tmp, s);
}

void scan_u64(const uint64_t* in, uint64_t* out, int64_t n, uint64_t* total, uint64_t* tmp,
              hipStream_t s) {
  ScanJobs jobs{};
  jobs.j[0].in64 = in;
  jobs.j[0].out64 = out;
  jobs.j[0].total64 = total;
  scan_jobs(jobs, 1, n, tmp, s);
}

}  // namespace sfmm
