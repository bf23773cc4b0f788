// p2p_wave.h -- what the wave kernels of P2P share (FP64 in k_near.hip, FP32 in
// k_f32c.hip): an item's sources flattened in LDS, the queues of pairs inside a
// kernel shared out over the lanes, and the sums over the wave.
#pragma once
#include "sfmm_internal.h"
#include "softening.h"

namespace sfmm {
namespace {

template <bool NODE>
__device__ __forceinline__ const int32_t* p2p_list(const NearArgs& a) {
  return NODE ? reinterpret_cast<const int32_t*>(a.node_p2p_pool) : a.p2p_list;
}

// inclusive sum over the wave's lanes (data-parallel moves, no LDS)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t add_dpp(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_incl_sum(uint32_t v) {
  v = add_dpp<0x111, 0xf>(v);  // rows of 16: shifted by 1, 2, 4, 8
  v = add_dpp<0x112, 0xf>(v);
  v = add_dpp<0x114, 0xf>(v);
  v = add_dpp<0x118, 0xf>(v);
  v = add_dpp<0x142, 0xa>(v);  // lane 15 (47) to row 1 (3)
  v = add_dpp<0x143, 0xc>(v);  // lane 31 to rows 2 and 3
  return v;
}

struct WaveItem {
  int tlo, nt;
  int total;  // flattened sources of the item
  int64_t item;
};

constexpr int kTQ = 256;  // queue slots per target

template <int TG>
struct alignas(16) WaveLds {
  uint32_t off[kP2PItem];  // 16 x particle index of each source
  union {
    uint16_t q[TG * kTQ];  // queued sources (places in off)
    double red[4][64];     // a soft pass's sums by component (x, z, y, p) and lane
  };
  SoftCoef coef[3];        // the spline pieces (kSoftCoef)
};

__device__ __forceinline__ double make_double(uint32_t lo, uint32_t hi) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ uint32_t lo32(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t hi32(double v) {
  return (uint32_t)((unsigned long long)__double_as_longlong(v) >> 32);
}

// lanes 0..31: a summed over the wave's two halves, lanes 32..63: b
__device__ __forceinline__ double fold32(double a, double b) {
  auto l = __builtin_amdgcn_permlane32_swap(lo32(a), lo32(b), false, false);
  auto h = __builtin_amdgcn_permlane32_swap(hi32(a), hi32(b), false, false);
  return make_double(l[0], h[0]) + make_double(l[1], h[1]);
}
// within each half: its even row of 16 lanes gets a summed over the half's
// two rows, its odd row b
__device__ __forceinline__ double fold16(double a, double b) {
  auto l = __builtin_amdgcn_permlane16_swap(lo32(a), lo32(b), false, false);
  auto h = __builtin_amdgcn_permlane16_swap(hi32(a), hi32(b), false, false);
  return make_double(l[0], h[0]) + make_double(l[1], h[1]);
}
// v plus v of the lane N places on in the row of 16 (rotated)
template <int N>
__device__ __forceinline__ double add_ror(double v) {
  const int l = __builtin_amdgcn_mov_dpp((int)lo32(v), 0x120 + N, 0xf, 0xf, true);
  const int h = __builtin_amdgcn_mov_dpp((int)hi32(v), 0x120 + N, 0xf, 0xf, true);
  return v + make_double((uint32_t)l, (uint32_t)h);
}
// the wave's sums of four values, one per row of 16 lanes: x, z, y, p
__device__ __forceinline__ double wave_sum4(double x, double y, double z, double p) {
  double v = fold16(fold32(x, y), fold32(z, p));
  v = add_ror<8>(v);
  v = add_ror<4>(v);
  v = add_ror<2>(v);
  return add_ror<1>(v);
}

// The queued pairs of a pass of K targets (lane t of lens: the length of
// target t's queue, total their sum).  A lane takes `run` consecutive entries
// of one target, each target as many lanes as its queue needs:
// sum_t ceil(len_t / run) <= total / run + K <= 64 for run >= total / (64 - K).
// pairs(t, at, mylen, run, sum) sums entries at .. at + run - 1 of target t's
// mylen into sum (x, y, z, p).  The lanes' sums are added per target in lane
// order, into the component that lane (row, t) holds (rows of 16 lanes: x, z,
// y, p).
template <int K, int TG, typename Pairs>
__device__ __forceinline__ double p2p_wave_queued(WaveLds<TG>& sh, uint32_t lens, uint32_t total,
                                                  Pairs pairs) {
  const int lane = threadIdx.x;
  const uint32_t run = (total + (64 - K) - 1) / (64 - K);
  const uint32_t len = lane < K ? lens : 0u;
  // (small whole numbers: the quotient's floor is exact)
  const uint32_t nl = (uint32_t)(((float)(len + run - 1) + 0.5f) / (float)run);
  const uint32_t end = wave_incl_sum(lane < K ? nl : 0u);  // (lanes K.. repeat the last end)
  int t = 0;
  uint32_t first = 0;
#pragma unroll
  for (int k = 0; k + 1 < K; ++k) {
    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)end, k);
    const bool past = (uint32_t)lane >= e;
    t = past ? k + 1 : t;
    first = past ? e : first;
  }
  const uint32_t at = ((uint32_t)lane - first) * run;  // this lane's first entry
  const uint32_t mylen = (uint32_t)__shfl((int)len, t, 64);
  double s[4];
  pairs(t, at, mylen, run, s);
  __syncthreads();  // (the sums take the place of the queues)
  sh.red[0][lane] = s[0];
  sh.red[1][lane] = s[2];
  sh.red[2][lane] = s[1];
  sh.red[3][lane] = s[3];
  __syncthreads();
  const int tk = lane & 15;
  const uint32_t e1 = (uint32_t)__shfl((int)end, tk, 64);
  uint32_t e0 = (uint32_t)__shfl((int)end, tk > 0 ? tk - 1 : 0, 64);
  if (tk == 0) e0 = 0;
  double sum = 0.0;
  if (tk < K)
    for (uint32_t e = e0; e < e1; ++e) sum += sh.red[lane >> 4][e];
  return sum;
}

// the sums of a pass over the wave, with those of its queued pairs (soft, by
// lane as p2p_wave_queued returns them): row r of 16 lanes gets component
// {x, z, y, p}[r], lane ii of the row keeps target ii's
template <int K, int LS>
__device__ __forceinline__ void p2p_wave_store(const NearArgs& a, const WaveItem& w, int t0,
                                               const double (&fx)[K], const double (&fy)[K],
                                               const double (&fz)[K], const double (&ph)[K],
                                               double soft) {
  const int lane = threadIdx.x;
  double mine = 0.0;
#pragma unroll
  for (int ii = 0; ii < K; ++ii) {
    const double v = wave_sum4(fx[ii], fy[ii], fz[ii], ph[ii]);
    mine = (lane & 15) == ii ? v : mine;
  }
  const int row = lane >> 4, tk = lane & 15;
  if (tk < K) {
    const int comp = row == 1 ? 2 : row == 2 ? 1 : row;
    a.part[(w.item * LS + t0 + tk) * 4 + comp] = mine + soft;
  }
}

// an item's run [f_lo, f_hi) of its leaf's flattened sources, from the list
// entry that holds its first source, as places in off
template <bool NODE>
__device__ __forceinline__ WaveItem p2p_wave_sources(const NearArgs& a, const P2PItem& it0,
                                                     uint32_t item, uint32_t* off) {
  const int lane = threadIdx.x;
  const uint64_t e0 = it0.e0, e1 = e0 + it0.ne;
  const int32_t* list = p2p_list<NODE>(a);
  const uint32_t f_lo = it0.f0, f_hi = it0.f1;
  uint32_t carry = it0.c0;  // the flattened start of the entries of a step
  // 64 list entries per step: entry [fb, fe) of the flattened order, clipped
  // to the run, goes to its place in LDS; entries of at most 16 sources one
  // source per iteration, larger ones by the whole wave
  for (uint64_t c0 = e0; c0 < e1 && carry < f_hi; c0 += 64) {
    NodeInfo si{};
    if (c0 + lane < e1) si = a.info[list[c0 + lane]];
    const uint32_t fe = carry + wave_incl_sum((uint32_t)si.cnt);
    const uint32_t fb = fe - (uint32_t)si.cnt;
    carry = (uint32_t)__builtin_amdgcn_readlane((int)fe, 63);
    const uint32_t b = fb > f_lo ? fb : f_lo, en = fe < f_hi ? fe : f_hi;
    const int nw = en > b ? (int)(en - b) : 0;
    const int at = (int)(b - f_lo);
    const uint32_t from = 16u * (uint32_t)(si.lo + (int)(b - fb));
    const bool big = nw > 16;
    const int nsm = big ? 0 : nw;
    for (int k = 0; k < 16; ++k) {
      if (!__builtin_amdgcn_ballot_w64(k < nsm)) break;
      if (k < nsm) off[at + k] = from + 16u * (uint32_t)k;
    }
    uint64_t bigm = __builtin_amdgcn_ballot_w64(big);
    while (bigm) {
      const int k = __builtin_ctzll(bigm);
      bigm &= bigm - 1;
      const int kat = __builtin_amdgcn_readlane(at, k), kn = __builtin_amdgcn_readlane(nw, k);
      const uint32_t kfrom = (uint32_t)__builtin_amdgcn_readlane((int)from, k);
      for (int q = lane; q < kn; q += 64) off[kat + q] = kfrom + 16u * (uint32_t)q;
    }
  }
  WaveItem w;
  w.tlo = __builtin_amdgcn_readfirstlane(it0.lo);
  w.nt = __builtin_amdgcn_readfirstlane(it0.cnt());
  const uint32_t f_end = carry < f_hi ? carry : f_hi;
  w.total = __builtin_amdgcn_readfirstlane(f_end > f_lo ? (int)(f_end - f_lo) : 0);
  w.item = item;
  // (lanes past the last source read a valid record)
  if (w.total == 0 || w.total + lane < (w.total + 63) / 64 * 64)
    off[w.total + lane] = 16u * (uint32_t)w.tlo;
  __syncthreads();
  return w;
}

}  // namespace
}  // namespace sfmm
