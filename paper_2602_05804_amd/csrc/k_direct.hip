// k_direct.hip -- the softened direct sum of Sect. 2, Eq. (softdirectsum),
// over all N sources for a set of targets: the O(N^2) reference the SFMM
// approximates (accuracy sweeps against the opening angle, the paper's
// Plummer and homogeneous-sphere tests).
//
// A wave takes 64 targets and a chunk of the sources: block (b, c) sums chunk
// c for the targets of group b and writes its partial sums to a buffer
// [chunk][target][4]; a second kernel adds each target's partials in a fixed
// order.  Pairs with j == i are skipped; unequal h are averaged as in P2P.
// The summation order is fixed, so the result is reproducible.
//
// Bound by FP64 issue.  The sources are the same for all lanes: they come
// through scalar loads, four at a time, and stay in scalar registers.  A pair
// beyond both kernels costs 24 FP64 operations and one estimate of 1/sqrt; the
// others are queued and evaluated 64 at a time, or, where most pairs lie inside a
// kernel, all in place.  All pairs of 1e5 particles of a Plummer sphere (softening
// lengths over four decades): 8.7 ms; 16.2 with the sources in LDS (six reads a
// pair), a full 1/sqrt, and the softened pair in place, which nearly a tenth of
// the steps took for one lane; 14.6 with only that left.
#include "sfmm_internal.h"
#include "softening.h"

namespace sfmm {
namespace {

constexpr int kDirTile = 64;    // chunks are whole numbers of this many sources
constexpr int kDirGroup = 4;    // sources loaded at a time
constexpr int64_t kDirSimds = 1024;  // of the chip (256 CUs)

// A chunk of which kDirSample sources lie inside a kernel with half of the wave's
// targets is met in place: a queued pair costs about twice one in place.  All of 5e4
// particles inside each other's kernels: 7.3 ms, 17.0 through the queue; a quarter of
// the pairs inside: 5.1 ms through the queue.
constexpr int kDirSample = 4;
constexpr int kDirQueue = 64 * (kDirGroup + 1);

// a wave's pairs that may lie within a kernel, kept until 64 of them fill the
// lanes: (source within the chunk, target lane).  A few targets with a large h
// have a pair there with every source: in place, all lanes would go through
// the softened pair for the sake of one.
struct DirLds {
  SoftCoef coef[3];
  double t[4][64];    // the targets' x, y, z, 1/h
  double acc[4][64];  // their softened sums
  unsigned long long mask[64];
  uint32_t first[64], last[64];
  uint32_t qj[kDirQueue], sj[64];
  uint8_t ql[kDirQueue], sl[64];
};

// lane `lane`'s value (uniform)
__device__ __forceinline__ double wave_lane(double v, int lane) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// one softened pair a lane, the queue's last `count` (<= 64) entries from `at`
// on: put in the order of their targets, evaluated, and summed over runs of
// one target, whose last lane adds the sum to the target's.  The order of the
// sums depends on the queue alone.
__device__ __forceinline__ void direct_flush(DirLds& sh, uint32_t at, uint32_t count, int64_t j0,
                                             int64_t i0, const int64_t* __restrict__ targets,
                                             const double* __restrict__ x,
                                             const double* __restrict__ m,
                                             const double* __restrict__ h) {
  const uint32_t lane = threadIdx.x;
  const bool on = lane < count;
  sh.mask[lane] = 0ull;
  __syncthreads();
  const uint32_t lq = on ? sh.ql[at + lane] : 0u, jq = on ? sh.qj[at + lane] : 0u;
  if (on) atomicOr(&sh.mask[lq], 1ull << lane);
  __syncthreads();
  const uint32_t own = (uint32_t)__popcll(sh.mask[lane]);
  uint32_t incl = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
    if ((int)lane >= o) incl += u;
  }
  sh.first[lane] = incl - own;
  sh.last[lane] = incl - 1u;
  __syncthreads();
  if (on) {
    const uint32_t pos =
        sh.first[lq] + (uint32_t)__popcll(sh.mask[lq] & ((1ull << lane) - 1ull));
    sh.sj[pos] = jq;
    sh.sl[pos] = (uint8_t)lq;
  }
  __syncthreads();
  const uint32_t l = on ? sh.sl[lane] : 0u;
  const int64_t j = j0 + (on ? sh.sj[lane] : 0u);
  const int64_t i = targets ? targets[i0 + l] : i0 + l;
  const uint32_t first = on ? sh.first[l] : lane;
  const double tx = sh.t[0][l], ty = sh.t[1][l], tz = sh.t[2][l], hiinv = sh.t[3][l];
  const double hjinv = 1.0 / h[j];
  const double w = on && j != i ? 0.5 * m[j] : 0.0;
  const double dx = tx - x[3 * j], dy = ty - x[3 * j + 1], dz = tz - x[3 * j + 2];
  const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
  const double rinv = rsqrt_pair(r2), r = r2 * rinv;
  const bool apart = r2 > 0.0;  // (at one place no force, where h^-3 may overflow)
  // (outside both kernels, both pieces are 1/r^3 and 1/r)
  double g1, p1, g2, p2;
  soft_piece(sh.coef, r * hiinv, hiinv, rinv, g1, p1);
  soft_piece(sh.coef, r * hjinv, hjinv, rinv, g2, p2);
  const double mg = apart ? w * (g1 + g2) : 0.0;
  double v[4] = {mg * dx, mg * dy, mg * dz, w * (p1 + p2)};
  for (int o = 1; o < 64 && __ballot((int)own > o); o <<= 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double u = __shfl_up(v[k], o, 64);
      if ((int)lane - o >= (int)first) v[k] += u;
    }
  }
  if (on && lane == sh.last[l]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sh.acc[k][l] += v[k];
  }
  __syncthreads();
}

// Every pair of a chunk as one that may lie inside a kernel, in place, and with
// 1/r = 0 where r^2 overflows: for a chunk most of whose pairs lie inside one, and
// for one whose sums came out as NaN.
__device__ __forceinline__ void direct_all(const DirLds& sh, int64_t j0, int64_t j1, int64_t i,
                                           double xi, double yi, double zi, double hi,
                                           const double* __restrict__ x,
                                           const double* __restrict__ m,
                                           const double* __restrict__ h, double& ax, double& ay,
                                           double& az, double& ph) {
  const uint32_t lane = threadIdx.x;
  const double hiinv = 1.0 / hi;
  for (int64_t b = j0; b < j1; b += 64) {
    const double inv = 1.0 / h[b + lane < j1 ? b + lane : b];  // (a lane's share of 64 sources')
    const int cnt = (int)(j1 - b < 64 ? j1 - b : 64);
    for (int k = 0; k < cnt; ++k) {
      const int64_t j = b + k;
      const double hj = h[j];
      const double hjinv = wave_lane(inv, k);
      const double dx = xi - x[3 * j], dy = yi - x[3 * j + 1], dz = zi - x[3 * j + 2];
      const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
      const double y = rsqrt_refined(r2);
      const bool apart = r2 > 0.0, in_range = r2 < INFINITY;
      const double rinv = apart && in_range ? y : 0.0;
      const double r = r2 * rinv;
      // (one kernel's piece from LDS, the other's selected: both pipes are busy)
      double g1, p1, g2, p2;
      soft_piece(sh.coef, r * hiinv, hiinv, rinv, g1, p1);
      soft_sel(r * hjinv, hjinv, hj * rinv, rinv, rinv * rinv * rinv, g2, p2);
      const double w = 0.5 * m[j];
      const double mg = apart && in_range ? w * (g1 + g2) : 0.0;
      const double mp = in_range && j != i ? w * (p1 + p2) : 0.0;
      ax = fma(mg, dx, ax);
      ay = fma(mg, dy, ay);
      az = fma(mg, dz, az);
      ph += mp;
    }
  }
}

// WAVES a SIMD: five (1e5 particles: 8.7 ms, with four 9.0, with three 9.9), four
// where no SIMD gets a fifth, whose registers need no spill (1e3 particles: 75 us
// with four, 78 with five)
template <int WAVES>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_direct_part(
    int64_t n, const double* __restrict__ x, const double* __restrict__ m,
    const double* __restrict__ h, int64_t nt, const int64_t* __restrict__ targets, int64_t chunk,
    double* __restrict__ part, int* status) {
  __shared__ DirLds sh;
  const uint32_t lane = threadIdx.x;
  if (lane < sizeof(kSoftCoef) / sizeof(double))
    reinterpret_cast<double*>(sh.coef)[lane] = reinterpret_cast<const double*>(kSoftCoef)[lane];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int64_t t = i0 + lane;
  const int64_t it = t < nt ? (targets ? targets[t] : t) : 0;
  const bool valid = it >= 0 && it < n;  // a bad index is reported, never read
  if (t < nt && !valid && blockIdx.y == 0) atomicOr(status, ST_OVERFLOW);
  const int64_t i = valid ? it : 0;
  const bool on = t < nt && valid;
  const double xi = x[3 * i], yi = x[3 * i + 1], zi = x[3 * i + 2], hi = h[i];
  const double h4 = 4.0 * hi * hi;
  sh.t[0][lane] = xi;
  sh.t[1][lane] = yi;
  sh.t[2][lane] = zi;
  sh.t[3][lane] = 1.0 / hi;
#pragma unroll
  for (int k = 0; k < 4; ++k) sh.acc[k][lane] = 0.0;
  __syncthreads();
  double ax = 0.0, ay = 0.0, az = 0.0, ph = 0.0;
  uint32_t nq = 0;  // (uniform)
  const uint64_t on_mask = __ballot(on);
  const int64_t j0 = (int64_t)blockIdx.y * chunk;
  const int64_t j1 = j0 + chunk < n ? j0 + chunk : n;

  // one source (j, sx .. sm the same for all lanes); r^2 beyond far2 lies
  // outside both kernels
  auto source = [&](int64_t j, double far2, double sx, double sy, double sz, double sm) {
    const double dx = xi - sx, dy = yi - sy, dz = zi - sz;
    const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
    const bool near = !(r2 > far2);  // (also when the comparison fails for a NaN)
    const double y = rsqrt_refined(r2);
    double mr = sm * y;
    double mg = mr * (y * y);
    const uint64_t nb = __ballot(near) & on_mask;
    if (nb != 0) {
      const uint32_t k = nq + __builtin_amdgcn_mbcnt_hi(
                                  (uint32_t)(nb >> 32),
                                  __builtin_amdgcn_mbcnt_lo((uint32_t)nb, 0u));
      mr = near ? 0.0 : mr;
      mg = near ? 0.0 : mg;
      if ((nb >> lane) & 1u) {
        sh.qj[k] = (uint32_t)(j - j0);
        sh.ql[k] = (uint8_t)lane;
      }
      nq += (uint32_t)__popcll(nb);
    }
    ax = fma(mg, dx, ax);
    ay = fma(mg, dy, ay);
    az = fma(mg, dz, az);
    ph += mr;
    // (sums made here, not kept for later: twice the registers otherwise)
    asm volatile("" : "+v"(ax), "+v"(ay), "+v"(az), "+v"(ph));
  };

  // some of the sources: do half of their pairs lie inside a kernel?
  uint32_t met = 0;
  const int64_t every = (j1 - j0) / kDirSample;
#pragma unroll
  for (int k = 0; k < kDirSample; ++k) {
    const int64_t j = j0 + k * every;
    const double dx = xi - x[3 * j], dy = yi - x[3 * j + 1], dz = zi - x[3 * j + 2];
    const double r2 = fma(dz, dz, fma(dy, dy, dx * dx));
    met += (uint32_t)__popcll(__ballot(!(r2 > fmax(h4, 4.0 * h[j] * h[j]))));
  }
  bool all = met >= kDirSample * 32;
  if (!all) {
    for (int64_t j = j0; j < j1; j += kDirGroup) {
      if (j + kDirGroup <= j1) {
        double s[3 * kDirGroup], sm[kDirGroup], sj[kDirGroup];
#pragma unroll
        for (int k = 0; k < 3 * kDirGroup; ++k) s[k] = x[3 * j + k];
#pragma unroll
        for (int k = 0; k < kDirGroup; ++k) sm[k] = m[j + k];
#pragma unroll
        for (int k = 0; k < kDirGroup; ++k) sj[k] = h[j + k];
#pragma unroll
        for (int k = 0; k < kDirGroup; ++k)
          source(j + k, fmax(h4, 4.0 * sj[k] * sj[k]), s[3 * k], s[3 * k + 1], s[3 * k + 2], sm[k]);
      } else {
        for (int64_t k = j; k < j1; ++k)
          source(k, fmax(h4, 4.0 * h[k] * h[k]), x[3 * k], x[3 * k + 1], x[3 * k + 2], m[k]);
      }
      const bool last = j + kDirGroup >= j1;
      while (nq >= 64 || (last && nq > 0)) {
        const uint32_t c = nq < 64 ? nq : 64;
        nq -= c;
        __syncthreads();
        direct_flush(sh, nq, c, j0, i0, targets, x, m, h);
      }
    }
    // (the refined 1/sqrt of an r^2 that overflows is NaN, where 1/r is 0)
    all = __ballot(on && !(fabs(ph + sh.acc[3][lane]) < INFINITY)) != 0;
  }
  if (all) {
    ax = ay = az = ph = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) sh.acc[k][lane] = 0.0;
    direct_all(sh, j0, j1, on ? i : -1, xi, yi, zi, hi, x, m, h, ax, ay, az, ph);
  }
  if (t >= nt) return;
  double* o = part + ((int64_t)blockIdx.y * nt + t) * 4;
  o[0] = ax + sh.acc[0][lane];
  o[1] = ay + sh.acc[1][lane];
  o[2] = az + sh.acc[2][lane];
  o[3] = ph + sh.acc[3][lane];
}

// Above kDirWide chunks, which few targets have, a wave per target (the chain of
// loads of one thread set the time: 2e5 sources and 1, 1000, 5000 targets 67, 273,
// 995 us; with a thread per target 483, 750, 1160).
constexpr int kDirWide = 256;

// per target: the chunks' partial sums in chunk order, the self term, -G
__global__ void k_direct_final(int64_t n, const double* __restrict__ m,
                               const double* __restrict__ h, int64_t nt,
                               const int64_t* __restrict__ targets, int nchunk,
                               const double* __restrict__ part, double G, int include_self,
                               double* __restrict__ acc, double* __restrict__ pot) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nt) return;
  const int64_t it = targets ? targets[t] : t;
  if (it < 0 || it >= n) return;  // reported by the first kernel
  double ax = 0.0, ay = 0.0, az = 0.0, ph = 0.0;
  // eight partials' loads at a time, added one after the other
  for (int c = 0; c < nchunk; c += 8) {
    double v[8][4];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double* q = part + ((int64_t)min(c + u, nchunk - 1) * nt + t) * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[u][k] = q[k];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (c + u >= nchunk) break;
      ax += v[u][0]; ay += v[u][1]; az += v[u][2]; ph += v[u][3];
    }
  }
  if (include_self) ph = fma(m[it], 1.4 * (1.0 / h[it]), ph);
  acc[3 * t] = -G * ax;
  acc[3 * t + 1] = -G * ay;
  acc[3 * t + 2] = -G * az;
  pot[t] = -G * ph;
}

// the same with a wave per target, for many chunks
__global__ __launch_bounds__(64) void k_direct_final_wide(
    int64_t n, const double* __restrict__ m, const double* __restrict__ h, int64_t nt,
    const int64_t* __restrict__ targets, int nchunk, const double* __restrict__ part, double G,
    int include_self, double* __restrict__ acc, double* __restrict__ pot) {
  const int64_t t = blockIdx.x;
  const int64_t it = targets ? targets[t] : t;
  if (it < 0 || it >= n) return;
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c = threadIdx.x; c < nchunk; c += 256) {
    double u[4][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double* p = part + ((int64_t)min(c + 64 * q, nchunk - 1) * nt + t) * 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) u[q][k] = p[k];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (c + 64 * q >= nchunk) break;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] += u[q][k];
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += __shfl_xor(v[k], o, 64);
  }
  if (threadIdx.x != 0) return;
  if (include_self) v[3] = fma(m[it], 1.4 * (1.0 / h[it]), v[3]);
  acc[3 * t] = -G * v[0];
  acc[3 * t + 1] = -G * v[1];
  acc[3 * t + 2] = -G * v[2];
  pot[t] = -G * v[3];
}

__global__ void k_clear_int(int* p) { *p = 0; }

}  // namespace

int direct_chunks(int64_t n, int64_t nt, uint64_t max_part_bytes) {
  if (n <= 0 || nt <= 0) return 1;
  const int64_t nb = (nt + 63) / 64;
  int64_t c = (49152 + nb - 1) / nb;                     // about 49152 waves in all: waves
  // with a far-reaching target take longer (1e5 targets: 10.1 ms with 16384, 9.2
  // with 32768, 8.9 with 49152 and with 65536)
  const int64_t tiles = (n + kDirTile - 1) / kDirTile;   // at least one tile per chunk
  if (c > tiles) c = tiles;
  const int64_t fit = (int64_t)(max_part_bytes / ((uint64_t)nt * 4 * sizeof(double)));
  if (c > fit) c = fit;
  if (c > 65535) c = 65535;  // (grid y)
  return (int)c;             // 0: not even one chunk fits
}

void launch_direct(int64_t n, const double* x, const double* m, const double* h, int64_t nt,
                   const int64_t* targets, double G, int include_self, double* acc, double* pot,
                   int* status, double* part, int nchunk, hipStream_t s) {
  k_clear_int<<<1, 1, 0, s>>>(status);
  if (nt <= 0 || n <= 0 || nchunk < 1) return;
  // chunks of whole tiles
  const int64_t tiles = (n + kDirTile - 1) / kDirTile;
  const int64_t chunk = ((tiles + nchunk - 1) / nchunk) * kDirTile;
  const int nc = (int)((n + chunk - 1) / chunk);
  const dim3 grid((unsigned)((nt + 63) / 64), (unsigned)nc);
  if ((int64_t)grid.x * grid.y <= 4 * kDirSimds)
    k_direct_part<4><<<grid, 64, 0, s>>>(n, x, m, h, nt, targets, chunk, part, status);
  else
    k_direct_part<5><<<grid, 64, 0, s>>>(n, x, m, h, nt, targets, chunk, part, status);
  if (nc > kDirWide)
    k_direct_final_wide<<<(unsigned)nt, 64, 0, s>>>(n, m, h, nt, targets, nc, part, G,
                                                    include_self, acc, pot);
  else
    k_direct_final<<<(unsigned)((nt + 255) / 256), 256, 0, s>>>(n, m, h, nt, targets, nc, part, G,
                                                                 include_self, acc, pot);
}

}  // namespace sfmm
