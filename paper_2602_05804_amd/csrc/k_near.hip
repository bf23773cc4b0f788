// k_near.hip -- near field (P2P) and the output in the caller's order, plus
// the FP64 momentum diagnostics.
//
// P2P is the softened direct sum of Sect. 2, Eq. (softdirectsum), over the
// source leaves the walk cached for the particle's leaf (the self leaf
// included, j != i).  Softening: cubic spline with support 2h; for a pair
// with unequal h the two kernels are averaged, which keeps the pair force
// antisymmetric (Newton's third law).  Kernel shapes, with q = r/h:
//   force  f(q)/q:  4/3 - 6/5 q^2 + 1/2 q^3                       (q < 1)
//                   8/3 - 3 q + 6/5 q^2 - 1/6 q^3 - 1/(15 q^3)     (1 <= q < 2)
//                   1/q^3                                          (q >= 2)
//   potential:      7/5 - 2/3 q^2 + 3/10 q^4 - 1/10 q^5            (q < 1)
//                   8/5 - 4/3 q^2 + q^3 - 3/10 q^4 + 1/30 q^5 - 1/(15 q)
//                   1/q                                            (q >= 2)
// (force per unit separation = shape / h^3, potential = shape / h).
#include "sfmm_internal.h"
#include "p2p_wave.h"
#include "softening.h"

namespace sfmm {
namespace {

template <bool NODE>
__global__ __launch_bounds__(256) void k_near(NearArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.n) return;
  const double xi = a.xs[i], yi = a.ys[i], zi = a.zs[i], hi = a.hs[i];
  const double hinv_i = 1.0 / hi;
  const int leaf = a.p_leaf[i];
  uint64_t e0, e1;
  const int32_t* list;
  if (NODE) {
    const int node = a.leaf_node[leaf];
    e0 = a.node_p2p_off[node];
    e1 = e0 + a.node_p2p_cnt[node];
    list = reinterpret_cast<const int32_t*>(a.node_p2p_pool);
  } else {
    e0 = a.p2p_off[leaf];
    e1 = a.p2p_off[leaf + 1];
    list = a.p2p_list;
  }
  double fx = 0.0, fy = 0.0, fz = 0.0, ph = 0.0;
  for (uint64_t e = e0; e < e1; ++e) {
    const NodeInfo si = a.info[list[e]];
    for (int j = si.lo; j < si.lo + si.cnt; ++j) {
      if (j == i) continue;
      const double dx = xi - a.xs[j], dy = yi - a.ys[j], dz = zi - a.zs[j];
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double hj = a.hs[j], mj = a.ms[j];
      const double hm = fmax(hi, hj);
      double gs, ps;
      if (r2 >= 4.0 * hm * hm) {
        const double rinv = rsqrt(r2);
        gs = rinv * rinv * rinv;
        ps = rinv;
      } else {
        const double r = sqrt(r2);
        double g1, p1, g2, p2;
        if (r >= 2.0 * hi) {
          const double rinv = 1.0 / r;
          g1 = rinv * rinv * rinv; p1 = rinv;
        } else {
          soft(r, hinv_i, g1, p1);
        }
        if (r >= 2.0 * hj) {
          const double rinv = 1.0 / r;
          g2 = rinv * rinv * rinv; p2 = rinv;
        } else {
          soft(r, 1.0 / hj, g2, p2);
        }
        gs = 0.5 * (g1 + g2);
        ps = 0.5 * (p1 + p2);
      }
      const double mg = mj * gs;
      fx = fma(mg, dx, fx);
      fy = fma(mg, dy, fy);
      fz = fma(mg, dz, fz);
      ph = fma(mj, ps, ph);
    }
  }
  if (a.include_self) ph = fma(a.ms[i], 1.4 * hinv_i, ph);
  // far[] holds the L2P field F and potential polynomial (acc = -G F); the
  // near sums above use the same convention: acc = -G (F + f), pot = -G (P + ph).
  const double* fr = a.far + 4 * (int64_t)i;
  const double G = a.G;
  const int64_t o = a.perm[i];
  a.acc[3 * o] = -G * (fr[0] + fx);
  a.acc[3 * o + 1] = -G * (fr[1] + fy);
  a.acc[3 * o + 2] = -G * (fr[2] + fz);
  a.pot[o] = -G * (fr[3] + ph);
}

// inclusive sum over the wave's lanes
__device__ __forceinline__ int wave_incl_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ---- wave per work item, targets in LDS -----------------------------------------
// The lanes walk the item's flattened source particles, 64 at a time, and each
// accumulates the field of its source on every target; a butterfly reduction
// then gives each target its total.  In passes of TG targets each, fully unrolled
// (static accumulator indices; nt is the same on every lane, so the guard is a
// scalar branch); the sources are read once per pass.  Pairs inside a kernel are not
// evaluated in the wave's pass over the sources (where most lanes would idle
// through the softening branch) but queued in LDS as (target, source); every
// 64 queued pairs are evaluated together, one per lane, and added to the same
// per-target accumulators.
template <int LS, bool NODE, int TG>
__global__ __launch_bounds__(64) void k_p2p_leaf(NearArgs a) {
  constexpr int NA = TG;  // accumulators per pass
  const int lane = threadIdx.x;
  const uint32_t item = blockIdx.x;
  if (item >= a.item_off[a.nleaves]) return;  // the grid is an upper bound
  const P2PItem it0 = a.item[item];
  const int tlo = it0.lo, nt = it0.cnt();
  // targets in LDS (read back as broadcasts): x, y, z, 1/h, h
  __shared__ double tg[LS][5];
  if (lane < nt) {
    const int j = tlo + lane;
    tg[lane][0] = a.xs[j]; tg[lane][1] = a.ys[j]; tg[lane][2] = a.zs[j];
    tg[lane][3] = a.his[j]; tg[lane][4] = a.hs[j];
  }
  __syncthreads();
  // this item's run [f_lo, f_hi) of the leaf's flattened sources, from the
  // list entry that holds its first source
  const uint64_t e0 = it0.e0, e1 = e0 + it0.ne;
  const int32_t* list = p2p_list<NODE>(a);
  const uint32_t f_lo = it0.f0, f_hi = it0.f1, carry0 = it0.c0;
  __shared__ int qj[128];
  __shared__ int qi[128];
  uint32_t qn = 0;     // queued softened pairs (the same on every lane)
  uint32_t nsoft = 0;  // softened pairs of this item
  for (int t0 = 0; t0 < nt; t0 += NA) {
    double fx[NA], fy[NA], fz[NA], ph[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) { fx[i] = 0.0; fy[i] = 0.0; fz[i] = 0.0; ph[i] = 0.0; }
    // the softened pairs of queue slots [0, count), one per lane, into the
    // accumulators of their targets; the rest of the queue moves to the front
    auto flush = [&](uint32_t count) {
      __syncthreads();
      const bool act = (uint32_t)lane < count;
      const int j2 = act ? qj[lane] : tlo;
      const int i2 = act ? qi[lane] : 0;
      const double thi = tg[i2][3];
      const double dx = tg[i2][0] - a.xs[j2], dy = tg[i2][1] - a.ys[j2], dz = tg[i2][2] - a.zs[j2];
      const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
      const double rinv = rsqrt_pair(r2);
      const double rinv3 = rinv * rinv * rinv;
      const double r = r2 * rinv;
      const double hj = a.hs[j2], hjinv = a.his[j2];
      double g1, p1, g2, p2;
      soft_sel(r * thi, thi, tg[i2][4] * rinv, rinv, rinv3, g1, p1);
      soft_sel(r * hjinv, hjinv, hj * rinv, rinv, rinv3, g2, p2);
      const double w = act ? a.ms[j2] : 0.0;
      const double mg = w * (0.5 * (g1 + g2));
      const double cx = mg * dx, cy = mg * dy, cz = mg * dz, cp = w * (0.5 * (p1 + p2));
#pragma unroll
      for (int ii = 0; ii < NA; ++ii) {
        if (act && i2 == t0 + ii) {
          fx[ii] += cx; fy[ii] += cy; fz[ii] += cz; ph[ii] += cp;
        }
      }
      const uint32_t rem = qn - count;
      int tj = 0, tq = 0;
      if ((uint32_t)lane < rem) { tj = qj[count + lane]; tq = qi[count + lane]; }
      __syncthreads();
      if ((uint32_t)lane < rem) { qj[lane] = tj; qi[lane] = tq; }
      qn = rem;
      __syncthreads();
    };
    uint32_t carry = carry0;  // sources of the list entries before c0
    for (uint64_t c0 = e0; c0 < e1; c0 += 64) {
      // 64 list entries: their particle ranges [fb, fe) in the flattened
      // order, then clipped to the run
      int cnt = 0, lo = 0;
      uint32_t fb = 0xffffffffu;
      NodeInfo si{};
      if (c0 + lane < e1) si = a.info[list[c0 + lane]];
      const int sincl = wave_incl_scan(c0 + lane < e1 ? si.cnt : 0);
      if (c0 + lane < e1) {
        const uint32_t fe = carry + (uint32_t)sincl;
        fb = fe - (uint32_t)si.cnt;
        const uint32_t b = fb > f_lo ? fb : f_lo;
        const uint32_t en = fe < f_hi ? fe : f_hi;
        if (en > b) { cnt = (int)(en - b); lo = si.lo + (int)(b - fb); }
      }
      carry += (uint32_t)__shfl(sincl, 63, 64);
      if (__shfl((int)fb, 0, 64) >= (int)f_hi) break;  // the run is done (uniform)
      const int incl = wave_incl_scan(cnt);
      const int pre = incl - cnt;
      const int total = __shfl(incl, 63, 64);
      for (int f0 = 0; f0 < total; f0 += 64) {
        const int f = f0 + lane;
        // owner lane k: the last lane with pre <= f (binary search over lanes)
        int k = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) {
          const int pk = __shfl(pre, k + step, 64);
          if (pk <= f) k += step;
        }
        const int jj = __shfl(lo, k, 64) + (f - __shfl(pre, k, 64));
        // lanes past the window's end stay in step with the others (the queue
        // count and its barriers are per wave) and contribute nothing
        const bool fv = f < total;
        const int j = fv ? jj : tlo;
        const double xj = a.xs[j], yj = a.ys[j], zj = a.zs[j], mj = a.ms[j];
        const double hjinv = a.his[j];
        const double hj2inv = hjinv * hjinv;
#pragma unroll
        for (int ii = 0; ii < NA; ++ii) {
          const int i = t0 + ii;
          if (i >= nt) continue;
          const double w = (!fv || j == tlo + i) ? 0.0 : mj;  // the pair (i, i) is skipped
          const double thi = tg[i][3];
          const double dx = tg[i][0] - xj, dy = tg[i][1] - yj, dz = tg[i][2] - zj;
          const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
          const double rinv = rsqrt_pair(r2);
          const double rinv3 = rinv * rinv * rinv;
          const bool inside = fv && ((r2 * (thi * thi) < 4.0) || (r2 * hj2inv < 4.0));
          const bool push = inside && w != 0.0;
          const uint64_t bal = __ballot(push);
          if (bal) {
            const uint32_t below =
                __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (push) { qj[qn + below] = j; qi[qn + below] = i; }
            qn += (uint32_t)__popcll(bal);
            nsoft += (uint32_t)__popcll(bal);
          }
          // both kernels at q >= 2 outside; a pair inside went to the queue
          const double wq = inside ? 0.0 : w;
          const double mg = wq * rinv3;
          fx[ii] = fma(mg, dx, fx[ii]);
          fy[ii] = fma(mg, dy, fy[ii]);
          fz[ii] = fma(mg, dz, fz[ii]);
          ph[ii] = fma(wq, rinv, ph[ii]);
          if (qn >= 64) flush(64);
        }
      }
    }
    if (qn > 0) flush(qn);
#pragma unroll
    for (int ii = 0; ii < NA; ++ii) {
      const int i = t0 + ii;
      if (i >= nt) break;
      const double sx = wave_sum(fx[ii]), sy = wave_sum(fy[ii]), sz = wave_sum(fz[ii]);
      const double sp = wave_sum(ph[ii]);
      if (lane == i) {
        double* o = a.part + ((int64_t)item * LS + i) * 4;
        o[0] = sx; o[1] = sy; o[2] = sz; o[3] = sp;
      }
    }
  }
  if (lane == 0) a.soft_pairs[item] = nsoft;
}

// ---- wave per work item, targets in scalar registers ------------------------------
// The same sums as k_p2p_leaf with less work per pair: the loop control is
// wave-uniform (scalar), the targets of a pass are wave-uniform values, a pair is
// inside a kernel when r^2 < 4 h_i^2 or r^2 < 4 h_j^2, and the field of a pair
// beyond both kernels is m/r^3 (dx, dy, dz) and m/r, with the refined 1/r replaced
// by 0 for pairs inside a kernel (the self pair and coincident particles included:
// r^2 = 0 is always inside).  Pairs inside a kernel, other than the self pair, go
// to a queue per target in LDS.  When a queue might overflow, and at the end, the
// queued pairs of all targets of the pass are shared out over the lanes
// (p2p_wave_queued).  A leaf's targets are taken in as few passes of at most TG as
// they need, of equal size within one, each with a fixed target count (no
// per-target exits inside the unrolled loop).
//
// The item's sources (at most kP2PItem) are flattened once into LDS, as byte
// offsets into the 16-byte particle arrays (so n < 2^28), padded to whole
// groups of 64; every pass then only streams over them.  The records of the
// next group load while the current one is evaluated.
//
// Bound: FP64 issue.  A pair takes 21 FP64-rate instructions of 4 cycles a
// wave and one v_rsq_f64 of 16 (100 cycles for 64 pairs), so 1.76e9 pairs need
// 1.3 ms at the 2.05 GHz the chip holds under this load.  Measured (Plummer
// sphere of 1e6, 1.76e9 pairs, 3.5 % softened): 2.73 ms, before 3.84 ms; of
// 9.95e8 VALU instructions (40 per 64 pairs) 23 are the pair's, the others the
// queues, the softened pairs, list scans and reductions, and the VALU is busy
// 77 % of the time.  Polytrope of 1e6 at leaf size 16: 1.87 ms, before 2.50.

// the queued pairs of a pass, a lane's run of one target's
template <int K, int TG>
__device__ __forceinline__ double p2p_wave_soft(const NearArgs& a, int t0p, WaveLds<TG>& sh,
                                                uint32_t lens, uint32_t total) {
  return p2p_wave_queued<K, TG>(sh, lens, total, [&](int t, uint32_t at, uint32_t mylen,
                                                     uint32_t run, double* sum) {
    const int it = t0p + t;
    const double2 txy = a.pxy[it], tzm = a.pzm[it];
    const double hiinv = a.his[it];
    const uint16_t* qt = sh.q + t * kTQ;
    double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
    // (the next source's record loads while the current pair is evaluated)
    struct Src {
      double2 xy, zm;
      double hinv;
    };
    auto load = [&](uint32_t b) {
      const int j = at + b < mylen ? (int)(sh.off[qt[at + b]] >> 4) : it;
      return Src{a.pxy[j], a.pzm[j], a.his[j]};
    };
    Src next = load(0);
    for (uint32_t b = 0; b < run; ++b) {
      const bool act = at + b < mylen;
      const double2 sxy = next.xy, szm = next.zm;
      const double hjinv = next.hinv;
      if (b + 1 < run) next = load(b + 1);
      const double dx = txy.x - sxy.x, dy = txy.y - sxy.y, dz = tzm.x - szm.x;
      const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
      const double rinv = rsqrt_pair(r2), r = r2 * rinv;
      // (at one place no force, where h^-3 may overflow; lanes past the end hold the
      // target itself)
      const bool apart = r2 > 0.0;
      double g1, p1, g2, p2;
      soft_piece(sh.coef, r * hiinv, hiinv, rinv, g1, p1);
      soft_piece(sh.coef, r * hjinv, hjinv, rinv, g2, p2);
      const double wm = act ? 0.5 * szm.y : 0.0;
      const double mg = apart ? wm * (g1 + g2) : 0.0;
      sx = fma(mg, dx, sx);
      sy = fma(mg, dy, sy);
      sz = fma(mg, dz, sz);
      sp = fma(wm, p1 + p2, sp);
    }
    sum[0] = sx; sum[1] = sy; sum[2] = sz; sum[3] = sp;
  });
}

template <int K, int LS, int TG>
__device__ __forceinline__ void p2p_wave_pass(const NearArgs& a, const WaveItem& w, int t0,
                                              WaveLds<TG>& sh, uint32_t& nsoft) {
  const int lane = threadIdx.x;
  const int t0p = w.tlo + t0;
  double tx[K], ty[K], tz[K], t4[K];
  double fx[K], fy[K], fz[K], ph[K];
  uint32_t qn[K];  // per-target queue length (wave-uniform)
#pragma unroll
  for (int ii = 0; ii < K; ++ii) {
    const double2 xy = a.pxy[t0p + ii], zm = a.pzm[t0p + ii];
    tx[ii] = wave_uniform(xy.x);
    ty[ii] = wave_uniform(xy.y);
    tz[ii] = wave_uniform(zm.x);
    t4[ii] = wave_uniform(a.h4[t0p + ii]);
    fx[ii] = 0.0; fy[ii] = 0.0; fz[ii] = 0.0; ph[ii] = 0.0;
    qn[ii] = 0;
  }
  double soft = 0.0;  // sums over queued pairs, by lane as p2p_wave_soft returns them
  const char* bxy = reinterpret_cast<const char*>(a.pxy);
  const char* bzm = reinterpret_cast<const char*>(a.pzm);
  const char* bh4 = reinterpret_cast<const char*>(a.h4);
  auto load_src = [&](int u0, uint32_t& off, double2& xy, double2& zm, double& h4) {
    off = sh.off[u0 + lane];
    xy = *reinterpret_cast<const double2*>(bxy + off);
    zm = *reinterpret_cast<const double2*>(bzm + off);
    h4 = *reinterpret_cast<const double*>(bh4 + (off >> 1));
  };
  uint32_t off;
  double2 xy, zm;
  double h4;
  load_src(0, off, xy, zm, h4);
  for (int u0 = 0; u0 < w.total; u0 += 64) {
    const uint32_t offc = off;
    const double xj = xy.x, yj = xy.y, zj = zm.x;
    double mj = zm.y;
    const uint64_t h4b = (uint64_t)__double_as_longlong(h4);
    const bool end = u0 + 64 >= w.total;
    uint64_t valid = ~0ull;
    if (!end) {
      load_src(u0 + 64, off, xy, zm, h4);
    } else if (w.total - u0 < 64) {
      // lanes past the end contribute nothing
      valid = (1ull << (w.total - u0)) - 1ull;
      mj = __builtin_amdgcn_inverse_ballot_w64(valid) ? mj : 0.0;
    }
    uint64_t im[K], met = 0;  // the lanes whose pair lies inside a kernel
#pragma unroll
    for (int ii = 0; ii < K; ++ii) {
      const double dx = tx[ii] - xj, dy = ty[ii] - yj, dz = tz[ii] - zj;
      const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
      // (r^2 >= 0 orders like its bits: with one compare of each kind the
      // compiler keeps two of them, where it would fold two of a kind into
      // one against the larger bound, whose maximum costs three more)
      im[ii] = __builtin_amdgcn_ballot_w64(r2 < t4[ii]) |
               __builtin_amdgcn_ballot_w64((uint64_t)__double_as_longlong(r2) < h4b);
      const bool inside = __builtin_amdgcn_inverse_ballot_w64(im[ii]);
      // (inside: the high word alone is cleared, which leaves a number below
      // 2^-1022, 0 to every sum that holds a softened pair)
      const double ri = rsqrt_refined(r2);
      const double rinv = make_double(lo32(ri), inside ? 0u : hi32(ri));
      const double mr = mj * rinv;
      const double mg = mr * (rinv * rinv);
      fx[ii] = fma(mg, dx, fx[ii]);
      fy[ii] = fma(mg, dy, fy[ii]);
      fz[ii] = fma(mg, dz, fz[ii]);
      ph[ii] += mr;
      met |= im[ii];
      // (an empty statement that reads the sums: keeps this arithmetic ahead
      // of the queue branch below, so that the compiler does not move it past
      // that branch and hold every target's separation vector at once)
      asm volatile("" ::"v"(fx[ii]), "v"(fy[ii]), "v"(fz[ii]), "v"(ph[ii]));
    }
    if (__builtin_expect_with_probability((met & valid) != 0 || end, 1, 0.1)) {
      uint32_t lens = 0, most = 0, sum = 0;
#pragma unroll
      for (int ii = 0; ii < K; ++ii) {
        // (the self pair has r^2 = 0 and is always inside)
        const uint64_t bal =
            im[ii] & valid & ~__builtin_amdgcn_ballot_w64(offc == 16u * (uint32_t)(t0p + ii));
        if (__builtin_amdgcn_inverse_ballot_w64(bal)) {
          const uint32_t below = __builtin_amdgcn_mbcnt_hi(
              (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
          sh.q[ii * kTQ + (int)(qn[ii] + below)] = (uint16_t)(u0 + lane);
        }
        qn[ii] = __builtin_amdgcn_readfirstlane(qn[ii] + (uint32_t)__popcll(bal));
        most = qn[ii] > most ? qn[ii] : most;
        sum += qn[ii];
        lens = lane == ii ? qn[ii] : lens;
      }
      // queues that might overflow in the next group, at the end all of them
      if (__builtin_expect_with_probability(most > (end ? 0u : (uint32_t)(kTQ - 64)), 1, 0.05)) {
        nsoft += sum;
        __syncthreads();
        soft += p2p_wave_soft<K, TG>(a, t0p, sh, lens, sum);
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < K; ++ii) qn[ii] = 0;
      }
    }
  }
  p2p_wave_store<K, LS>(a, w, t0, fx, fy, fz, ph, soft);
  __syncthreads();  // (the queues are reused by the next pass)
}

template <int LS, bool NODE, int TG, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE))) void k_p2p_wave(
    NearArgs a) {
  const int lane = threadIdx.x;
  const uint32_t item = xcd_block(blockIdx.x, gridDim.x);
  if (item >= a.item_off[a.nleaves]) return;  // the grid is an upper bound
  const P2PItem it0 = a.item[item];
  __shared__ WaveLds<TG> sh;
  if (lane < (int)(sizeof(kSoftCoef) / sizeof(double)))
    reinterpret_cast<double*>(sh.coef)[lane] = reinterpret_cast<const double*>(kSoftCoef)[lane];
  const WaveItem w = p2p_wave_sources<NODE>(a, it0, item, sh.off);
  uint32_t nsoft = 0;
  const int npass = (w.nt + TG - 1) / TG;
  int t0 = 0;
  for (int p = 0; p < npass; ++p) {
    const int k = (w.nt - t0 + (npass - p) - 1) / (npass - p);
    // a pass with a fixed target count (uniform branches)
    static_for<TG>([&](auto rc) {
      constexpr int r = decltype(rc)::value + 1;
      if (k == r) p2p_wave_pass<r, LS, TG>(a, w, t0, sh, nsoft);
    });
    t0 += k;
  }
  if (lane == 0) a.soft_pairs[item] = nsoft;
}

// per leaf, the particles over its P2P list entries and its work items:
// max(1, ceil(sources / the rule's run length)).  One wave per leaf.  (The
// level walk computes both in its leaf pass.)
template <bool NODE>
__global__ __launch_bounds__(64) void k_p2p_items_count(NearArgs a, uint32_t* __restrict__ src_total,
                                                        uint32_t* __restrict__ cnt) {
  const int l = blockIdx.x;
  const int lane = threadIdx.x;
  uint64_t e0, e1;
  const int32_t* list;
  if (NODE) {
    const int node = a.leaf_node[l];
    e0 = a.node_p2p_off[node];
    e1 = e0 + a.node_p2p_cnt[node];
    list = reinterpret_cast<const int32_t*>(a.node_p2p_pool);
  } else {
    e0 = a.p2p_off[l];
    e1 = a.p2p_off[l + 1];
    list = a.p2p_list;
  }
  uint32_t carry = 0;
  for (uint64_t c0 = e0; c0 < e1; c0 += 64) {
    const bool in = c0 + lane < e1;
    const int c = in ? a.info[list[c0 + lane]].cnt : 0;
    const int incl = wave_incl_scan(c);
    carry += (uint32_t)__shfl(incl, 63, 64);
  }
  if (lane == 0) {
    src_total[l] = carry;
    const uint32_t len = a.rule.len(a.info[a.leaf_node[l]].lo);
    const uint32_t k = (carry + len - 1) / len;
    cnt[l] = k > 0 ? k : 1u;
  }
}

// the work items.  A block of kFillLeaves waves per kFillLeaves leaves, a wave
// per leaf: it writes the leaf's items and, when there are several, scans the
// leaf's list for the entries that hold their first sources.  (One wave for
// all 16 leaves took 441 us on a Plummer sphere of 1e6, whose halo leaves all
// have lists of thousands of entries and sit together in the leaf order.)
constexpr int kFillLeaves = 16;
constexpr int kFillGroups = 8;
template <bool NODE>
__global__ __launch_bounds__(64 * kFillLeaves) void k_p2p_items_fill(NearArgs a,
                                                                     P2PItem* __restrict__ item) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  {
    const int l = blockIdx.x * kFillLeaves + wv;
    if (l >= a.nleaves) return;
    const uint32_t b = a.item_off[l], e = a.item_off[l + 1];
    const int node = a.leaf_node[l];
    const NodeInfo ti = a.info[node];
    uint64_t e0, e1;
    if (NODE) {
      e0 = a.node_p2p_off[node];
      e1 = e0 + a.node_p2p_cnt[node];
    } else {
      e0 = a.p2p_off[l];
      e1 = a.p2p_off[l + 1];
    }
    const uint32_t len = a.rule.len(ti.lo), ftot = a.src_total[l];
    P2PItem q{};
    q.e0 = e0;
    q.ne = (uint32_t)(e1 - e0);
    q.lo = ti.lo;
    q.nd = (uint32_t)node | ((uint32_t)ti.cnt << kSrcBits);
    for (uint32_t t = b + lane; t < e; t += 64) {
      q.f0 = (t - b) * len;
      q.f1 = q.f0 + len < ftot ? q.f0 + len : ftot;
      if (t == b) item[t] = q;
      else { item[t].f0 = q.f0; item[t].f1 = q.f1; item[t].lo = q.lo; item[t].nd = q.nd; }
    }
    if (e - b <= 1) return;
    const int32_t* list = p2p_list<NODE>(a);
    // kFillGroups groups of 64 entries per step, their loads issued together
    // (the longest lists, a few thousand entries, set this kernel's time)
    uint32_t carry = 0;
    for (uint64_t c0 = e0; c0 < e1; c0 += 64 * kFillGroups) {
      int src[kFillGroups];
#pragma unroll
      for (int u = 0; u < kFillGroups; ++u) src[u] = c0 + 64 * u + lane < e1 ? list[c0 + 64 * u + lane] : -1;
      uint32_t cu[kFillGroups];
#pragma unroll
      for (int u = 0; u < kFillGroups; ++u) cu[u] = src[u] >= 0 ? (uint32_t)a.info[src[u]].cnt : 0u;
#pragma unroll
      for (int u = 0; u < kFillGroups; ++u) {
        const uint64_t g0 = c0 + 64 * u;
        if (g0 >= e1) break;  // (uniform)
        const bool in = g0 + lane < e1;
        const uint32_t c = cu[u];
        const int incl = wave_incl_scan((int)c);
        const uint32_t fe = carry + (uint32_t)incl, fb = fe - c;
        if (in && c > 0) {
          uint32_t k = (fb + len - 1) / len;
          if (k == 0) k = 1;
          for (; k * len < fe && b + k < e; ++k) {
            item[b + k].e0 = g0 + lane;
            item[b + k].ne = (uint32_t)(e1 - g0 - lane);
            item[b + k].c0 = fb;
          }
        }
        carry += (uint32_t)__shfl(incl, 63, 64);
      }
    }
  }
}

__global__ __launch_bounds__(1024) void k_soft_total(int64_t items,
                                                     const uint32_t* __restrict__ soft_pairs,
                                                     uint64_t* __restrict__ total) {
  __shared__ uint64_t sh[16];
  uint64_t s = 0;
  for (int64_t i = threadIdx.x; i < items; i += 1024) s += soft_pairs[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 16; ++k) s += sh[k];
    *total = s;
  }
}

// one thread per sorted particle: its items' partial sums in item order,
// the far field and the self term, in the caller's order
__global__ void k_p2p_reduce(NearArgs a, int ls) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= a.n) return;
  const int l = a.p_leaf[j];
  const uint32_t t0 = a.item_off[l], t1 = a.item_off[l + 1];
  const int i = j - a.info[a.leaf_node[l]].lo;
  double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
  // eight items' loads in flight: a particle of a Plummer sphere's halo has
  // hundreds of items, and its lane summed them one load latency at a time
  // (309 us at 1e6)
  uint32_t t = t0;
  for (; t + 8 <= t1; t += 8) {
    double2 u[8], v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const double2* q = reinterpret_cast<const double2*>(a.part + ((int64_t)(t + k) * ls + i) * 4);
      u[k] = q[0];
      v[k] = q[1];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) { sx += u[k].x; sy += u[k].y; sz += v[k].x; sp += v[k].y; }
  }
  for (; t < t1; ++t) {
    const double* q = a.part + ((int64_t)t * ls + i) * 4;
    sx += q[0]; sy += q[1]; sz += q[2]; sp += q[3];
  }
  if (a.include_self) sp = fma(a.ms[j], 1.4 * a.his[j], sp);
  const double* fr = a.far + 4 * (int64_t)j;
  const int64_t o = a.perm[j];
  const double G = a.G;
  a.acc[3 * o] = -G * (fr[0] + sx);
  a.acc[3 * o + 1] = -G * (fr[1] + sy);
  a.acc[3 * o + 2] = -G * (fr[2] + sz);
  a.pot[o] = -G * (fr[3] + sp);
}

constexpr int MOM_THREADS = 256;

__global__ __launch_bounds__(MOM_THREADS) void k_momentum_partial(int n, const double* __restrict__ m,
                                                                  const double* __restrict__ acc,
                                                                  double* __restrict__ part) {
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int i = blockIdx.x * MOM_THREADS + threadIdx.x; i < n; i += gridDim.x * MOM_THREADS) {
    const double F0 = m[i] * acc[3 * (int64_t)i], F1 = m[i] * acc[3 * (int64_t)i + 1],
                 F2 = m[i] * acc[3 * (int64_t)i + 2];
    s[0] += F0; s[1] += F1; s[2] += F2;
    s[3] += sqrt(F0 * F0 + F1 * F1 + F2 * F2);
  }
  __shared__ double sh[4][MOM_THREADS];
  for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] = s[c];
  __syncthreads();
  for (int w = MOM_THREADS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int c = 0; c < 4; ++c) sh[c][threadIdx.x] += sh[c][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) part[4 * blockIdx.x + threadIdx.x] = sh[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_momentum_final(int nb, const double* __restrict__ part,
                                                        double* __restrict__ out) {
  // fixed summation tree: thread t sums partials t, t+64, ... of component
  // t / 64, then a fixed pairwise reduction
  __shared__ double sh[256];
  const int c = threadIdx.x >> 6, t = threadIdx.x & 63;
  double s = 0.0;
  for (int b = t; b < nb; b += 64) s += part[4 * b + c];
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int w = 32; w > 0; w >>= 1) {
    if (t < w) sh[threadIdx.x] += sh[threadIdx.x + w];
    __syncthreads();
  }
  if (t == 0) out[c] = sh[threadIdx.x];
}

}  // namespace

#define WAVE_LAUNCH(LS, TG, WPE)                                           \
  do {                                                                     \
    if (node_lists) k_p2p_wave<LS, true, TG, WPE><<<nbl, 64, 0, s>>>(a); \
    else k_p2p_wave<LS, false, TG, WPE><<<nbl, 64, 0, s>>>(a);          \
    record_mark(km.end, s);                                                \
    if (!km.skip_reduce) launch_p2p_reduce(a, LS, s);                      \
  } while (0)

#define NEAR_LAUNCH(LS, TG)                                                \
  do {                                                                     \
    if (node_lists) k_p2p_leaf<LS, true, TG><<<nbl, 64, 0, s>>>(a);        \
    else k_p2p_leaf<LS, false, TG><<<nbl, 64, 0, s>>>(a);                  \
    record_mark(km.end, s);                                                \
    if (!km.skip_reduce) launch_p2p_reduce(a, LS, s);                      \
  } while (0)

void launch_p2p_items_count(bool node_lists, const NearArgs& a, uint32_t* src_total,
                            uint32_t* item_cnt, hipStream_t s) {
  if (a.nleaves <= 0) return;
  if (node_lists) k_p2p_items_count<true><<<a.nleaves, 64, 0, s>>>(a, src_total, item_cnt);
  else k_p2p_items_count<false><<<a.nleaves, 64, 0, s>>>(a, src_total, item_cnt);
}

void launch_p2p_items_fill(bool node_lists, const NearArgs& a, P2PItem* item, hipStream_t s) {
  if (a.nleaves <= 0) return;
  const unsigned nb = (unsigned)((a.nleaves + kFillLeaves - 1) / kFillLeaves);
  if (node_lists) k_p2p_items_fill<true><<<nb, 64 * kFillLeaves, 0, s>>>(a, item);
  else k_p2p_items_fill<false><<<nb, 64 * kFillLeaves, 0, s>>>(a, item);
}

void launch_soft_total(int64_t items, const uint32_t* soft_pairs, uint64_t* total, hipStream_t s) {
  k_soft_total<<<1, 1024, 0, s>>>(items, soft_pairs, total);
}

void launch_p2p_reduce(const NearArgs& a, int ls, hipStream_t s) {
  if (a.n <= 0) return;
  k_p2p_reduce<<<blocks_for(a.n, 256), 256, 0, s>>>(a, ls);
}

void launch_near(bool node_lists, int leaf_size, int variant, const NearArgs& a, int64_t items,
                 hipStream_t s, KernelMarks km) {
  if (a.n <= 0) return;
  const unsigned nbl = (unsigned)items;
  record_mark(km.begin, s);
  if (variant == 1) leaf_size = 1 << 20;  // particle per thread
  // variant (the shapes are listed with sfmm_config.near_kernel)
  // The wave shape (numbers 0 and 13; 13 was one with the targets in lane stripes
  // and the sources staged in LDS, which it beats on every system tried, e.g. at
  // leaf size 16 on a polytrope of 1e6 1.87 against 1.97 ms, on a Plummer sphere
  // at leaf size 10 2.73 against 3.51): eight targets per pass at three waves per SIMD (at leaf
  // size 10 on the Plummer sphere and the polytrope of 1e6: 2.86 ms, with six
  // at three 2.97, five or six at four, which spill, 2.95).  It addresses the
  // particles by 32-bit byte offsets of 16 bytes each, so from 2^28 particles
  // on shape 6 takes its place.
  if (a.n >= (1 << 28) && variant != 6) variant = 6;
  if (leaf_size <= 10) {
    if (variant == 6) NEAR_LAUNCH(10, 5);
    else WAVE_LAUNCH(10, 8, 3);
  } else if (leaf_size <= 16) {
    if (variant == 6) NEAR_LAUNCH(16, 8);
    else WAVE_LAUNCH(16, 8, 3);
  } else if (leaf_size <= 32) {
    if (variant == 6) NEAR_LAUNCH(32, 8);
    else WAVE_LAUNCH(32, 8, 3);
  } else {
    if (node_lists) k_near<true><<<(a.n + 255) / 256, 256, 0, s>>>(a);
    else k_near<false><<<(a.n + 255) / 256, 256, 0, s>>>(a);
    record_mark(km.end, s);
  }
}

// leapfrog update of one system: v += kick * acc; x += drift * v
__global__ void k_leapfrog(int64_t n3, double* __restrict__ x, double* __restrict__ v,
                           const double* __restrict__ acc, double kick, double drift) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n3) return;
  // separate multiply and add (no contraction), as the update is written
  const double vi = v[i] + kick * acc[i];
  v[i] = vi;
  x[i] = x[i] + drift * vi;
}

void launch_leapfrog(int64_t n, double* x, double* v, const double* acc, double kick, double drift,
                     hipStream_t s) {
  if (n <= 0) return;
  const int64_t n3 = 3 * n;
  k_leapfrog<<<(unsigned)((n3 + 255) / 256), 256, 0, s>>>(n3, x, v, acc, kick, drift);
}

int momentum_blocks(int64_t n) {
  int64_t b = (n + MOM_THREADS * 8 - 1) / (MOM_THREADS * 8);
  if (b < 1) b = 1;
  if (b > 512) b = 512;
  return (int)b;
}

void launch_momentum(int n, const double* m, const double* acc, double* part, double* out,
                     hipStream_t s) {
  const int nb = momentum_blocks(n);
  k_momentum_partial<<<nb, MOM_THREADS, 0, s>>>(n, m, acc, part);
  k_momentum_final<<<1, 256, 0, s>>>(nb, part, out);
}

}  // namespace sfmm
