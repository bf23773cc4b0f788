// k_f32c.hip -- the FP32-compensated form (SFMM_FP32C) of the far field and
// of P2P.
//
// Geometry, moments, the L2L chain and L2P stay in FP64.  The bulk terms run
// in FP32 and every term is added into an FP64 accumulator, which bounds the
// summation error below that of an FP32 hi/lo (TwoSum) pair at a lower cost
// here (an FP64 add issues at the FP32 rate).
//   M2L  targets at depth < top: FP64 as in k_far; deeper targets: the
//        separation of the two centres is formed in FP64 and rounded, the
//        moments are an FP32 copy, the derivatives and the contraction are
//        FP32 (Exp<P>::m2l_add_f32).
//   P2P  each particle carries its FP32 offset from its leaf's centre; a pair
//        (i in A, j in B) uses d = fl32(c_A - c_B) + (o_i - o_j), which is
//        exactly minus the separation seen from j, so each pair force is
//        antisymmetric.
#include "p2p_wave.h"
#include "sfmm_internal.h"

namespace sfmm {
namespace {

template <int P>
__global__ void k_prep_nodes32(int nn, const double* __restrict__ rec,
                               float* __restrict__ rec32) {
  constexpr int NQ = Exp<P>::NQ;
  constexpr int RS = rec_stride(P), RS32 = rec32_stride(P);
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nn) return;
  const double* r = rec + (int64_t)v * RS;
  float* o = rec32 + (int64_t)v * RS32;
  double* c = reinterpret_cast<double*>(o);
  c[0] = r[0]; c[1] = r[1]; c[2] = r[2];
#pragma unroll
  for (int k = 0; k < NQ; ++k) o[6 + k] = (float)r[8 + k];
}

// (a thread per particle: one per leaf took 123 us at 2e6 particles)
template <int RS>
__global__ void k_prep_particles32(int n, const int32_t* __restrict__ p_leaf,
                                   const int32_t* __restrict__ leaf_node,
                                   const double* __restrict__ rec, const double* __restrict__ xs,
                                   const double* __restrict__ ys, const double* __restrict__ zs,
                                   const double* __restrict__ ms, const double* __restrict__ hs,
                                   Part32 p) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const double* r = rec + (int64_t)leaf_node[p_leaf[j]] * RS;
  const double c0 = r[0], c1 = r[1], c2 = r[2];
  p.off[j] = make_float4((float)(xs[j] - c0), (float)(ys[j] - c1), (float)(zs[j] - c2),
                         (float)ms[j]);
  p.cxy[j] = make_double2(c0, c1);
  p.czh[j] = Part32Z{c2, (float)hs[j], (float)(1.0 / hs[j])};
}

// ---- far field -----------------------------------------------------------------
template <int P, bool NODE, int SPLIT>
__global__ __launch_bounds__(64) void k_far32(FarArgs a, const float* __restrict__ rec32, int top) {
  using E = Exp<P>;
  constexpr int NQ = E::NQ;
  constexpr int NL = E::NL;
  constexpr int RS = rec_stride(P), RS32 = rec32_stride(P);
  const int lane = threadIdx.x;
  const int sub = lane % SPLIT;
  const int l = blockIdx.x * (64 / SPLIT) + lane / SPLIT;
  const bool active = l < a.nleaves;
  const NodeInfo* __restrict__ info = a.info;
  const double* __restrict__ rec = a.rec;
  const int leaf = active ? a.leaf_node[l] : 0;
  const int d = active ? a.leaf_depth[l] : -1;
  const int lo = info[leaf].lo;
  const int cnt = active ? info[leaf].cnt : 0;

  double L[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) L[q] = 0.0;
  bool have = false;
  const uint32_t* list = NODE ? a.node_m2l_pool : a.m2l_list;
  const uint32_t* dc = NODE ? nullptr : a.depth_cnt + (active ? a.leaf_doff[l] : 0);
  uint64_t seg = NODE ? 0 : (active ? a.m2l_off[l] : 0);
  uint64_t e = 0, ne = 0;
  int v = 0, k = 0;
  double sv[3] = {rec[0], rec[1], rec[2]};
  if (d >= 0) {
    if (NODE) { e = a.node_m2l_off[0]; ne = e + a.node_m2l_cnt[0]; }
    else { e = seg; ne = seg + dc[0]; }
    e += sub;
  }
  // FP32 entries: source centre (FP64) and FP32 moments of the current entry,
  // with the next entry prefetched
  double cs[3] = {0.0, 0.0, 0.0};
  float cq[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) cq[q] = 0.f;
  uint32_t idx_next = 0;
  auto load32 = [&](uint32_t ent, double* sd, float* qd) {
    const uint32_t s = ent & kSrcMask;
    const double* rs = rec + (int64_t)s * RS;
    sd[0] = rs[0]; sd[1] = rs[1]; sd[2] = rs[2];
    const float* r32 = rec32 + (int64_t)s * RS32 + 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) qd[q] = r32[q];
  };
  auto start_depth = [&]() {
    if (k >= top && e < ne) {
      load32(list[e], cs, cq);
      idx_next = list[e + SPLIT < ne ? e + SPLIT : ne - 1];
    }
  };
  start_depth();
  for (;;) {
    if (e < ne) {
      if (k < top) {
        const double* rs = rec + (int64_t)(list[e] & kSrcMask) * RS;
        const double r[3] = {rs[0] - sv[0], rs[1] - sv[1], rs[2] - sv[2]};
        double Q[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) Q[q] = rs[8 + q];
        E::m2l_add(r, Q, L);
        e += SPLIT;
      } else {
        const uint64_t en = e + SPLIT;
        double ns[3];
        float nq[NQ];
        load32(idx_next, ns, nq);
        idx_next = list[en + SPLIT < ne ? en + SPLIT : ne - 1];
        const float r[3] = {(float)(cs[0] - sv[0]), (float)(cs[1] - sv[1]), (float)(cs[2] - sv[2])};
        E::m2l_add_f32(r, cq, L);
        e = en;
        cs[0] = ns[0]; cs[1] = ns[1]; cs[2] = ns[2];
#pragma unroll
        for (int q = 0; q < NQ; ++q) cq[q] = nq[q];
      }
      have = true;
    } else if (k < d) {
      const int c = info[v].child;
      const int nv = (lo < info[c + 1].lo) ? c : c + 1;
      const double* rn = rec + (int64_t)nv * RS;
      const double sn[3] = {rn[0], rn[1], rn[2]};
      if (have) {
        const double hv[3] = {sn[0] - sv[0], sn[1] - sv[1], sn[2] - sv[2]};
        E::l2l(hv, L);
      }
      v = nv;
      sv[0] = sn[0]; sv[1] = sn[1]; sv[2] = sn[2];
      ++k;
      if (NODE) {
        e = a.node_m2l_off[v];
        ne = e + a.node_m2l_cnt[v];
      } else {
        seg += dc[k - 1];
        e = seg;
        ne = seg + dc[k];
      }
      e += sub;
      start_depth();
    } else {
      break;
    }
  }
#pragma unroll
  for (int o = SPLIT / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int q = 0; q < NL; ++q) L[q] += __shfl_xor(L[q], o, 64);
    const int other = __shfl_xor((int)have, o, 64);
    have = have || other != 0;
  }
  for (int j = lo + sub; j < lo + cnt; j += SPLIT) {
    const double off[3] = {a.xs[j] - sv[0], a.ys[j] - sv[1], a.zs[j] - sv[2]};
    double f[3] = {0.0, 0.0, 0.0}, phi = 0.0;
    if (have) E::l2p(off, L, f, phi);
    double* o = a.far + 4 * (int64_t)j;
    o[0] = f[0]; o[1] = f[1]; o[2] = f[2]; o[3] = phi;
  }
}

// ---- P2P ------------------------------------------------------------------------
__device__ __forceinline__ void soft32(float q, float hinv, float qi, float rinv, float rinv3,
                                       float& g, float& psi) {
  const float q2 = q * q;
  const float h3 = hinv * hinv * hinv;
  const float gA = h3 * fmaf(q2, fmaf(0.5f, q, -1.2f), 4.0f / 3.0f);
  const float pA = hinv * fmaf(q2, fmaf(q2, fmaf(-0.1f, q, 0.3f), -2.0f / 3.0f), 1.4f);
  const float qi3 = qi * qi * qi;
  const float gB = h3 * (fmaf(q, fmaf(q, fmaf(q, -1.0f / 6.0f, 1.2f), -3.0f), 8.0f / 3.0f) -
                         qi3 * (1.0f / 15.0f));
  const float pB = hinv * (fmaf(q2, fmaf(q, fmaf(q, fmaf(q, 1.0f / 30.0f, -0.3f), 1.0f), -4.0f / 3.0f), 1.6f) -
                           qi * (1.0f / 15.0f));
  g = q >= 2.0f ? rinv3 : (q < 1.0f ? gA : gB);
  psi = q >= 2.0f ? rinv : (q < 1.0f ? pA : pB);
}

__device__ __forceinline__ int wave_incl_scan32(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  return v;
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// targets in passes of TG, each pass unrolled (static accumulator indices);
// the sources are read once per pass
template <int LS, bool NODE, int TG>
__global__ __launch_bounds__(64) void k_p2p_leaf32(NearArgs a, Part32 p) {
  const float4* __restrict__ pf = p.off;
  const Part32Z* __restrict__ phh = p.czh;
  const int RS = a.rec_stride;
  const int lane = threadIdx.x;
  const uint32_t item = blockIdx.x;
  if (item >= a.item_off[a.nleaves]) return;  // the grid is an upper bound
  const P2PItem it0 = a.item[item];
  const int node = it0.node(), tlo = it0.lo, nt = it0.cnt();
  const double* rt = a.rec + (int64_t)node * RS;
  const double ct0 = rt[0], ct1 = rt[1], ct2 = rt[2];
  __shared__ float tg[LS][5];  // offset x, y, z, 1/h, h
  if (lane < nt) {
    const float4 o = pf[tlo + lane];
    const Part32Z hh = phh[tlo + lane];
    tg[lane][0] = o.x; tg[lane][1] = o.y; tg[lane][2] = o.z;
    tg[lane][3] = hh.hinv; tg[lane][4] = hh.h;
  }
  __syncthreads();
  // this item's run [f_lo, f_hi) of the leaf's flattened sources, from the
  // list entry that holds its first source
  const uint64_t e0 = it0.e0, e1 = e0 + it0.ne;
  const int32_t* list = NODE ? reinterpret_cast<const int32_t*>(a.node_p2p_pool) : a.p2p_list;
  const uint32_t f_lo = it0.f0, f_hi = it0.f1, carry0 = it0.c0;
  uint32_t nsoft = 0;  // pairs inside a kernel (complete on lane 0)
  for (int t0 = 0; t0 < nt; t0 += TG) {
    double fx[TG], fy[TG], fz[TG], ph[TG];
#pragma unroll
    for (int i = 0; i < TG; ++i) { fx[i] = 0.0; fy[i] = 0.0; fz[i] = 0.0; ph[i] = 0.0; }
    uint32_t carry = carry0;  // sources of the list entries before c0
    for (uint64_t c0 = e0; c0 < e1; c0 += 64) {
      int cnt = 0, lo = 0, sub = 0;
      uint32_t fb = 0xffffffffu;
      float dcx = 0.f, dcy = 0.f, dcz = 0.f;
      const bool in = c0 + lane < e1;
      const int src = in ? list[c0 + lane] : 0;
      NodeInfo si{};
      if (in) si = a.info[src];
      const int sincl = wave_incl_scan32(in ? si.cnt : 0);
      if (in) {
        const uint32_t fe = carry + (uint32_t)sincl;
        fb = fe - (uint32_t)si.cnt;
        const uint32_t b = fb > f_lo ? fb : f_lo;
        const uint32_t en = fe < f_hi ? fe : f_hi;
        if (en > b) { cnt = (int)(en - b); lo = si.lo + (int)(b - fb); }
        // a whole subtree: its particles' offsets are relative to their own
        // leaves, whose centres are looked up per particle
        sub = si.child >= 0 ? 1 : 0;
        const double* rs = a.rec + (int64_t)src * RS;
        dcx = (float)(ct0 - rs[0]);
        dcy = (float)(ct1 - rs[1]);
        dcz = (float)(ct2 - rs[2]);
      }
      carry += (uint32_t)__shfl(sincl, 63, 64);
      if (__shfl((int)fb, 0, 64) >= (int)f_hi) break;  // the run is done (uniform)
      const int incl = wave_incl_scan32(cnt);
      const int pre = incl - cnt;
      const int total = __shfl(incl, 63, 64);
      for (int f0 = 0; f0 < total; f0 += 64) {
        const int f = f0 + lane;
        int k = 0;
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) {
          const int pk = __shfl(pre, k + step, 64);
          if (pk <= f) k += step;
        }
        const int j = __shfl(lo, k, 64) + (f - __shfl(pre, k, 64));
        float cx = __shfl(dcx, k, 64), cy = __shfl(dcy, k, 64), cz = __shfl(dcz, k, 64);
        const int jsub = __shfl(sub, k, 64);
        if (f >= total) continue;
        if (jsub) {
          const double* rl = a.rec + (int64_t)a.leaf_node[a.p_leaf[j]] * RS;
          cx = (float)(ct0 - rl[0]);
          cy = (float)(ct1 - rl[1]);
          cz = (float)(ct2 - rl[2]);
        }
        const float4 oj = pf[j];
        const Part32Z hj = phh[j];
        const float hj2inv = hj.hinv * hj.hinv;
#pragma unroll
        for (int ii = 0; ii < TG; ++ii) {
          const int i = t0 + ii;
          if (i >= nt) continue;
          const bool self = j == tlo + i;  // (whose g may be infinite)
          const float w = self ? 0.f : oj.w;
          const float thi = tg[i][3];
          const float dx = cx + (tg[i][0] - oj.x);
          const float dy = cy + (tg[i][1] - oj.y);
          const float dz = cz + (tg[i][2] - oj.z);
          const float r2 = dx * dx + dy * dy + dz * dz;
          const float rinv = r2 > 0.f ? __frsqrt_rn(r2) : 0.f;
          const float rinv3 = rinv * rinv * rinv;
          float gs = rinv3, ps = rinv;
          const bool inside = (r2 * (thi * thi) < 4.0f) || (r2 * hj2inv < 4.0f);
          nsoft += (uint32_t)__popcll(__ballot(inside && w != 0.f));  // lane 0 is always active
          if (__ballot(inside)) {
            const float r = r2 * rinv;
            float g1, p1, g2, p2;
            soft32(r * thi, thi, tg[i][4] * rinv, rinv, rinv3, g1, p1);
            soft32(r * hj.hinv, hj.hinv, hj.h * rinv, rinv, rinv3, g2, p2);
            if (inside) {
              gs = self ? 0.f : 0.5f * (g1 + g2);
              ps = self ? 0.f : 0.5f * (p1 + p2);
            }
          }
          const float mg = w * gs;
          fx[ii] += (double)(mg * dx);
          fy[ii] += (double)(mg * dy);
          fz[ii] += (double)(mg * dz);
          ph[ii] += (double)(w * ps);
        }
      }
    }
#pragma unroll
    for (int ii = 0; ii < TG; ++ii) {
      const int i = t0 + ii;
      if (i >= nt) break;
      const double sx = wave_sum64(fx[ii]), sy = wave_sum64(fy[ii]), sz = wave_sum64(fz[ii]);
      const double sp = wave_sum64(ph[ii]);
      if (lane == i) {
        double* o = a.part + ((int64_t)item * LS + i) * 4;
        o[0] = sx; o[1] = sy; o[2] = sz; o[3] = sp;
      }
    }
  }
  if (lane == 0) a.soft_pairs[item] = nsoft;
}

// ---- P2P, wave per item with the targets in scalar registers -------------------
// The FP32 form of k_p2p_wave (k_near.hip), with its flattened sources, passes
// and queues: the targets of a pass (FP32 offsets and 4 h^2) as wave-uniform
// values, the field of a pair beyond both kernels as m/r^3 (dx, dy, dz) and m/r
// with 1/r replaced by 0 inside a kernel.  A source brings its own leaf's
// centre (FP64; the difference to the target leaf's is rounded once a pass), so
// entries need no table.  Every term is added into FP64 sums.
//
// Bound by issue: a pair takes 22 FP32 instructions, an FP32 1/sqrt, and four
// conversions and additions in FP64.  2e6 particles of a binary (1.45e9 pairs,
// 8.4 % softened): 2.61 ms, a cloud of 8e6 (6.0e9 pairs) 11.0 ms; with the
// sources searched anew for every pass of five targets 3.33 and 13.8 ms.

// Sums of FP32 pair terms: each term added to an FP64 accumulator (AccD, the
// default), or compensated in FP32 (AccT: Knuth's TwoSum keeps the rounding
// error of every addition, hi + lo is rounded to FP64 once at the end).
struct AccD {
  double v = 0.0;
  __device__ __forceinline__ void add(float x) { v += (double)x; }
  __device__ __forceinline__ double get() const { return v; }
  __device__ __forceinline__ void keep() { asm volatile("" ::"v"(v)); }
};
struct AccT {
  float hi = 0.f, lo = 0.f;
  __device__ __forceinline__ void add(float x) {
    const float s = hi + x;
    const float bb = s - hi;
    const float e = (hi - (s - bb)) + (x - bb);
    hi = s;
    lo += e;
  }
  __device__ __forceinline__ double get() const { return (double)hi + (double)lo; }
  __device__ __forceinline__ void keep() { asm volatile("" ::"v"(hi), "v"(lo)); }
};

__device__ __forceinline__ float wave_uniform_f(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// the target leaf's centre (wave-uniform)
struct Centre32 {
  double x, y, z;
};

// one source's record, and its leaf's centre as seen from the target leaf
struct Src32 {
  float4 o;
  double2 cxy;
  Part32Z czh;
};
__device__ __forceinline__ Src32 load_src32(const Part32& p, uint32_t off) {
  return Src32{*reinterpret_cast<const float4*>(reinterpret_cast<const char*>(p.off) + off),
               *reinterpret_cast<const double2*>(reinterpret_cast<const char*>(p.cxy) + off),
               *reinterpret_cast<const Part32Z*>(reinterpret_cast<const char*>(p.czh) + off)};
}

template <int K, int TG>
__device__ __forceinline__ double p2p_wave32_soft(const Part32& p, const Centre32& ct, int t0p,
                                                  WaveLds<TG>& sh, uint32_t lens, uint32_t total) {
  return p2p_wave_queued<K, TG>(sh, lens, total, [&](int t, uint32_t at, uint32_t mylen,
                                                     uint32_t run, double* sum) {
    const uint32_t self = 16u * (uint32_t)(t0p + t);
    const Src32 tg = load_src32(p, self);
    const float hi = tg.czh.h, hiinv = tg.czh.hinv;
    const uint16_t* qt = sh.q + t * kTQ;
    double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
    auto load = [&](uint32_t b) {
      return load_src32(p, at + b < mylen ? sh.off[qt[at + b]] : self);
    };
    Src32 next = load(0);
    for (uint32_t b = 0; b < run; ++b) {
      const bool act = at + b < mylen;
      const Src32 s = next;
      if (b + 1 < run) next = load(b + 1);
      const float cx = (float)(ct.x - s.cxy.x), cy = (float)(ct.y - s.cxy.y),
                  cz = (float)(ct.z - s.czh.cz);
      const float dx = cx + (tg.o.x - s.o.x), dy = cy + (tg.o.y - s.o.y),
                  dz = cz + (tg.o.z - s.o.z);
      const float r2 = dx * dx + dy * dy + dz * dz;
      const float rinv = r2 > 0.f ? __frsqrt_rn(r2) : 0.f;
      const float rinv3 = rinv * rinv * rinv;
      const float r = r2 * rinv;
      float g1, p1, g2, p2;
      soft32(r * hiinv, hiinv, hi * rinv, rinv, rinv3, g1, p1);
      soft32(r * s.czh.hinv, s.czh.hinv, s.czh.h * rinv, rinv, rinv3, g2, p2);
      // (an idle lane meets its target itself, whose g may be infinite)
      const float mg = act ? s.o.w * (0.5f * (g1 + g2)) : 0.f;
      const float mp = act ? s.o.w * (0.5f * (p1 + p2)) : 0.f;
      sx += (double)(mg * dx);
      sy += (double)(mg * dy);
      sz += (double)(mg * dz);
      sp += (double)mp;
    }
    sum[0] = sx; sum[1] = sy; sum[2] = sz; sum[3] = sp;
  });
}

template <int K, int LS, int TG, typename Acc>
__device__ __forceinline__ void p2p_wave32_pass(const NearArgs& a, const Part32& p,
                                                const Centre32& ct, const WaveItem& w, int t0,
                                                WaveLds<TG>& sh, uint32_t& nsoft) {
  const int lane = threadIdx.x;
  const int t0p = w.tlo + t0;
  float tx[K], ty[K], tz[K], t4[K];
  Acc fx[K], fy[K], fz[K], ph[K];
  uint32_t qn[K];  // per-target queue length (wave-uniform)
#pragma unroll
  for (int ii = 0; ii < K; ++ii) {
    const float4 o = p.off[t0p + ii];
    tx[ii] = wave_uniform_f(o.x);
    ty[ii] = wave_uniform_f(o.y);
    tz[ii] = wave_uniform_f(o.z);
    const float hu = wave_uniform_f(p.czh[t0p + ii].h);
    t4[ii] = fmaxf(4.0f * hu * hu, 0x1p-126f);  // (above 0: the self pair is inside)
    fx[ii] = Acc(); fy[ii] = Acc(); fz[ii] = Acc(); ph[ii] = Acc();
    qn[ii] = 0;
  }
  double soft = 0.0;  // sums over queued pairs, by lane as p2p_wave32_soft returns them
  uint32_t off = sh.off[lane];
  Src32 s = load_src32(p, off);
  for (int u0 = 0; u0 < w.total; u0 += 64) {
    const uint32_t offc = off;
    const float cx = (float)(ct.x - s.cxy.x), cy = (float)(ct.y - s.cxy.y),
                cz = (float)(ct.z - s.czh.cz);
    const float xj = s.o.x, yj = s.o.y, zj = s.o.z;
    float mj = s.o.w;
    const float h4j = 4.0f * s.czh.h * s.czh.h;
    const bool end = u0 + 64 >= w.total;
    uint64_t valid = ~0ull;
    if (!end) {
      off = sh.off[u0 + 64 + lane];
      s = load_src32(p, off);
    } else if (w.total - u0 < 64) {
      // lanes past the end contribute nothing
      valid = (1ull << (w.total - u0)) - 1ull;
      mj = __builtin_amdgcn_inverse_ballot_w64(valid) ? mj : 0.f;
    }
    uint64_t im[K], met = 0;  // the lanes whose pair lies inside a kernel
#pragma unroll
    for (int ii = 0; ii < K; ++ii) {
      const float dx = cx + (tx[ii] - xj), dy = cy + (ty[ii] - yj), dz = cz + (tz[ii] - zj);
      const float r2 = dx * dx + dy * dy + dz * dz;
      const bool inside = r2 < fmaxf(t4[ii], h4j);
      im[ii] = __builtin_amdgcn_ballot_w64(inside);
      const float rinv = inside ? 0.f : __builtin_amdgcn_rsqf(r2);
      const float mr = mj * rinv;
      const float mg = mr * (rinv * rinv);
      fx[ii].add(mg * dx);
      fy[ii].add(mg * dy);
      fz[ii].add(mg * dz);
      ph[ii].add(mr);
      met |= im[ii];
      // (keeps this target's arithmetic ahead of the queue branch)
      fx[ii].keep(); fy[ii].keep(); fz[ii].keep(); ph[ii].keep();
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
        soft += p2p_wave32_soft<K, TG>(p, ct, t0p, sh, lens, sum);
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < K; ++ii) qn[ii] = 0;
      }
    }
  }
  double gx[K], gy[K], gz[K], gp[K];
#pragma unroll
  for (int ii = 0; ii < K; ++ii) {
    gx[ii] = fx[ii].get();
    gy[ii] = fy[ii].get();
    gz[ii] = fz[ii].get();
    gp[ii] = ph[ii].get();
  }
  p2p_wave_store<K, LS>(a, w, t0, gx, gy, gz, gp, soft);
  __syncthreads();  // (the queues are reused by the next pass)
}

template <int LS, bool NODE, int TG, int WPE, typename Acc>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE))) void k_p2p_wave32(
    NearArgs a, Part32 p) {
  const int lane = threadIdx.x;
  const uint32_t item = xcd_block(blockIdx.x, gridDim.x);
  if (item >= a.item_off[a.nleaves]) return;  // the grid is an upper bound
  const P2PItem it0 = a.item[item];
  __shared__ WaveLds<TG> sh;
  const WaveItem w = p2p_wave_sources<NODE>(a, it0, item, sh.off);
  const double2 cxy = p.cxy[w.tlo];
  const Centre32 ct{wave_uniform(cxy.x), wave_uniform(cxy.y), wave_uniform(p.czh[w.tlo].cz)};
  uint32_t nsoft = 0;
  const int npass = (w.nt + TG - 1) / TG;
  int t0 = 0;
  for (int q = 0; q < npass; ++q) {
    const int k = (w.nt - t0 + (npass - q) - 1) / (npass - q);
    // a pass with a fixed target count (uniform branches)
    static_for<TG>([&](auto rc) {
      constexpr int r = decltype(rc)::value + 1;
      if (k == r) p2p_wave32_pass<r, LS, TG, Acc>(a, p, ct, w, t0, sh, nsoft);
    });
    t0 += k;
  }
  if (lane == 0) a.soft_pairs[item] = nsoft;
}

constexpr int kFarSplit32 = 2;

template <int P>
void far32_order(bool node_lists, const FarArgs& a, const float* rec32, int top, hipStream_t s) {
  const unsigned nb = (unsigned)((a.nleaves + 64 / kFarSplit32 - 1) / (64 / kFarSplit32));
  if (node_lists) k_far32<P, true, kFarSplit32><<<nb, 64, 0, s>>>(a, rec32, top);
  else k_far32<P, false, kFarSplit32><<<nb, 64, 0, s>>>(a, rec32, top);
}

// variant 0: the wave kernel with scalar-register targets; 7: the same with
// TwoSum-compensated FP32 sums instead of FP64 ones; 6: the earlier shape
// (targets in LDS, the softened branch taken in the pass)
template <int LS>
void p2p32(bool node_lists, int variant, const NearArgs& a, const Part32& p, int64_t items, hipStream_t s, KernelMarks km) {
  // eight targets a pass at three waves a SIMD: 2.61 ms for 2e6 particles of a
  // binary, 11.0 for a cloud of 8e6 (five at four: 2.65 and 10.8; six at four
  // spill: 2.91 and 11.7)
  constexpr int TG = 8, WPE = 3;
  const unsigned nb = (unsigned)items;
  // (16-byte offsets in 32 bits)
  if (a.n >= (1 << 28)) variant = 6;
  record_mark(km.begin, s);
  if (variant == 6) {
    if (node_lists) k_p2p_leaf32<LS, true, LS <= 10 ? 5 : 8><<<nb, 64, 0, s>>>(a, p);
    else k_p2p_leaf32<LS, false, LS <= 10 ? 5 : 8><<<nb, 64, 0, s>>>(a, p);
  } else if (variant == 7) {
    if (node_lists) k_p2p_wave32<LS, true, TG, WPE, AccT><<<nb, 64, 0, s>>>(a, p);
    else k_p2p_wave32<LS, false, TG, WPE, AccT><<<nb, 64, 0, s>>>(a, p);
  } else {
    if (node_lists) k_p2p_wave32<LS, true, TG, WPE, AccD><<<nb, 64, 0, s>>>(a, p);
    else k_p2p_wave32<LS, false, TG, WPE, AccD><<<nb, 64, 0, s>>>(a, p);
  }
  record_mark(km.end, s);
  if (!km.skip_reduce) launch_p2p_reduce(a, LS, s);
}

}  // namespace

void launch_prep32(int order, int nn, int n, const int32_t* p_leaf, const int32_t* leaf_node,
                   const double* rec, const double* xs, const double* ys, const double* zs,
                   const double* ms, const double* hs, float* rec32, const Part32& p, hipStream_t s) {
  const unsigned nb = (unsigned)((nn + 255) / 256);
  switch (order) {
    case 0: k_prep_nodes32<0><<<nb, 256, 0, s>>>(nn, rec, rec32); break;
    case 1: k_prep_nodes32<1><<<nb, 256, 0, s>>>(nn, rec, rec32); break;
    case 2: k_prep_nodes32<2><<<nb, 256, 0, s>>>(nn, rec, rec32); break;
    case 3: k_prep_nodes32<3><<<nb, 256, 0, s>>>(nn, rec, rec32); break;
    case 4: k_prep_nodes32<4><<<nb, 256, 0, s>>>(nn, rec, rec32); break;
  }
  const unsigned np = (unsigned)((n + 255) / 256);
  switch (rec_stride(order)) {
    case 16: k_prep_particles32<16><<<np, 256, 0, s>>>(n, p_leaf, leaf_node, rec, xs, ys, zs, ms, hs, p); break;
    case 24: k_prep_particles32<24><<<np, 256, 0, s>>>(n, p_leaf, leaf_node, rec, xs, ys, zs, ms, hs, p); break;
    case 32: k_prep_particles32<32><<<np, 256, 0, s>>>(n, p_leaf, leaf_node, rec, xs, ys, zs, ms, hs, p); break;
    case 48: k_prep_particles32<48><<<np, 256, 0, s>>>(n, p_leaf, leaf_node, rec, xs, ys, zs, ms, hs, p); break;
  }
}

void launch_far32(int order, bool node_lists, const FarArgs& a, const float* rec32, int top,
                  hipStream_t s) {
  if (a.nleaves <= 0) return;
  switch (order) {
    case 0: far32_order<0>(node_lists, a, rec32, top, s); break;
    case 1: far32_order<1>(node_lists, a, rec32, top, s); break;
    case 2: far32_order<2>(node_lists, a, rec32, top, s); break;
    case 3: far32_order<3>(node_lists, a, rec32, top, s); break;
    case 4: far32_order<4>(node_lists, a, rec32, top, s); break;
  }
}

bool launch_near32(int order, bool node_lists, int leaf_size, int variant, const NearArgs& a,
                   const Part32& p, int64_t items, hipStream_t s, KernelMarks km) {
  if (a.n <= 0) return true;
  if (leaf_size > 16) return false;
  (void)order;
  if (leaf_size <= 10) p2p32<10>(node_lists, variant, a, p, items, s, km);
  else p2p32<16>(node_lists, variant, a, p, items, s, km);
  return true;
}

}  // namespace sfmm
