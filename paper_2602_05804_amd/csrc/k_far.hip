// k_far.hip -- far field of each leaf: M2L on every ancestor, the L2L chain
// down the branch and L2P at the leaf's particles (Sect. 2.2, Algorithm 1,
// Appendix A.2).
//
// A group of SPLIT lanes per leaf.  The leaf's M2L list is grouped by the
// depth of the target ancestor; the lanes of the group take every SPLIT-th
// entry of each depth and keep a partial local expansion in registers: at
// depth k it is re-centred from p_{k-1} to p_k (exact for the polynomial)
// and the lane's M2L terms for p_k are added.  Re-centring is linear, so the
// group's partial expansions are summed at the leaf and evaluated at its
// particles.  Every leaf still evaluates all M2L interactions of all of its
// ancestors.  Neighbouring leaves (Morton order) share their upper
// ancestors, so lanes mostly read the same source records.
#include <algorithm>

#include "sfmm_internal.h"

namespace sfmm {
namespace {

template <int P, bool NODE, int SPLIT, int WAVES>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_far(FarArgs a) {
  using E = Exp<P>;
  constexpr int NQ = E::NQ;
  constexpr int NL = E::NL;
  constexpr int RS = rec_stride(P);
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
  // list range of depth k for this lane: entries base + sub, base + sub + SPLIT, ...
  const uint32_t* list = NODE ? a.node_m2l_pool : a.m2l_list;
  const uint32_t* dc = NODE ? nullptr : a.depth_cnt + (active ? a.leaf_doff[l] : 0);
  uint64_t seg = NODE ? 0 : (active ? a.m2l_off[l] : 0);  // per-leaf lists: start of depth k
  uint64_t e = 0, ne = 0;
  int v = 0, k = 0;
  double sv[3] = {rec[0], rec[1], rec[2]};
  if (d >= 0) {
    if (NODE) { e = a.node_m2l_off[0]; ne = e + a.node_m2l_cnt[0]; }
    else { e = seg; ne = seg + dc[0]; }
    e += sub;
  }
  // one loop per lane: an M2L while the current depth has entries left,
  // else a step down the branch (L2L), until the leaf's list is done.  The
  // source record of the next entry and the list index of the one after it
  // are loaded while the current M2L is computed.
  double cs[3], cq[NQ];
  uint32_t idx_next = 0;
  auto load_rec = [&](uint32_t ent, double* sd, double* qd) {
    const double* rs = rec + (int64_t)(ent & kSrcMask) * RS;
    sd[0] = rs[0]; sd[1] = rs[1]; sd[2] = rs[2];
#pragma unroll
    for (int q = 0; q < NQ; ++q) qd[q] = rs[8 + q];
  };
  // at the top of the loop, when e < ne: (cs, cq) hold entry e's source and
  // idx_next the list index of the following entry (the last one repeated
  // when there is none)
  auto start_depth = [&]() {
    if (e < ne) {
      load_rec(list[e], cs, cq);
      idx_next = list[e + SPLIT < ne ? e + SPLIT : ne - 1];
    }
  };
  start_depth();
  for (;;) {
    if (e < ne) {
      const uint64_t en = e + SPLIT;
      double ns[3], nq[NQ];
      load_rec(idx_next, ns, nq);
      idx_next = list[en + SPLIT < ne ? en + SPLIT : ne - 1];
      const double r[3] = {cs[0] - sv[0], cs[1] - sv[1], cs[2] - sv[2]};
      E::m2l_add(r, cq, L);
      have = true;
      e = en;
      cs[0] = ns[0]; cs[1] = ns[1]; cs[2] = ns[2];
#pragma unroll
      for (int q = 0; q < NQ; ++q) cq[q] = nq[q];
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
  // the SPLIT lanes of a leaf hold partial expansions about the same centre
#pragma unroll
  for (int o = SPLIT / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int q = 0; q < NL; ++q) L[q] += __shfl_xor(L[q], o, 64);
    // every lane must take part in the shuffle (no short-circuit around it)
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

// ---- shared far field -------------------------------------------------------
// The caching of shared interactions of Sect. 5: the M2L list of node v (the
// pairs the level walk accepted with v as target) is evaluated once into
// LN[v]; a leaf's far field is then the root-to-leaf chain
//   L <- L2L(L, s_v - s_parent) (when L is non-zero), L <- L + LN[v],
// and L2P at its particles -- the same terms as the per-leaf form, whose
// replicated evaluation of every ancestor's list is what this removes.
//
// k_m2l: 8 lanes per node, 8 nodes per wave; each lane sums every 8th entry
// of its node's list, the group's sums are added with row moves, and lane q of
// the group stores the coefficients q, q + 8, ...  FP64 targets use the
// reduced components (Exp<P>::m2l_h, 388 flops a pair at P = 3 where all
// components take 660), FP32 targets (FP32C, depth >= top) all of them with
// FP32 terms and FP64 sums.
//
// The order of the nodes (launch_m2l_order): a wave takes nodes of lists of
// like length, or its lanes idle until the longest ends; the longest lists of
// all come first, or they run on alone at the end; and the other nodes stay in
// windows that follow each other in level order, one XCD taking a whole window,
// so that the sources its nodes share are met in one L2.  (All nodes sorted by
// length alone fetched 3.0 GB a launch at 1e6 particles where this fetches
// 0.4 GB.)
//
// Bound: FP64 (FP32C: all) VALU issue, then L2 to L1.  Polytrope of 1e6 at leaf
// size 16 (2.7e7 pairs): 0.76 -> 0.47 ms, 5.8e10 pairs/s at 54 % VALU busy;
// binary of 2e6 in FP32C (8.5e7 pairs): 2.9 -> 1.67 ms at 95 %.
//
// The eight source records of a group's step go straight to LDS
// (global_load_lds, no registers): the group's lanes load them together, 16
// bytes a lane and 128 contiguous bytes an instruction, where a lane loading
// its own record makes every instruction touch 64 lines, one a clock.
// The 16-byte chunks of a record are taken in a block of eight (a lane each)
// and a rest of at most eight, padded to R = 2, 4 or 8 lanes a record.
// Instruction k of a block of R lanes a record loads, in lane sub, slot
// (sub % R) ^ k of record sub / R + (8 / R) k, and LDS receives the lanes in
// order; the exclusive-or keeps the reads (one chunk of eight records) free of
// bank conflicts.
template <int NC>
struct M2LStage {
  static constexpr int REST = NC % 8;
  static constexpr int R = REST == 0 ? 0 : REST <= 2 ? 2 : REST <= 4 ? 4 : 8;
  static constexpr int NB = NC / 8 * 8;  // chunks in the block of eight (0 or 8)
  double2 c[NB + R][64];                 // [instruction][lane]
};

// the value of lane (group, I) of a group of 8
template <int I>
__device__ __forceinline__ uint32_t group_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (I << 5) | 0x18);
}

// (the low word of a shared pointer is its LDS address)
__device__ __forceinline__ void load_to_lds(const char* from, double2* to) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)from,
      (__attribute__((address_space(3))) void*)(uint32_t)(uintptr_t)to, 16, 0, 0);
}

// f(k, address) for every instruction k that loads the records of the wave's
// 64 entries (src: this lane's source node)
template <int NC, typename F>
__device__ __forceinline__ void m2l_addresses(const char* __restrict__ recs, uint32_t src, F&& f) {
  using S = M2LStage<NC>;
  constexpr uint32_t BYTES = NC * 16;
  const uint32_t lane = threadIdx.x;
  uint32_t sub = lane & 7;
  asm volatile("" : "+v"(sub));  // (addresses are formed here, not held over the loop)
  if constexpr (S::NB > 0)
    static_for<8>([&](auto ic) {
      constexpr uint32_t k = decltype(ic)::value;
      f(ic, recs + (uint64_t)group_lane<k>(src) * BYTES + ((sub ^ k) * 16));
    });
  if constexpr (S::R > 0)
    static_for<S::R>([&](auto kc) {
      constexpr uint32_t k = decltype(kc)::value, R = S::R;
      const uint32_t slot = (sub % R) ^ k;
      const uint32_t chunk = S::NB + (slot < S::REST ? slot : S::REST - 1);
      uint32_t s;
      if constexpr (R == 8) s = group_lane<k>(src);
      else s = (uint32_t)__shfl((int)src, (int)((lane & ~7u) + sub / R + (8 / R) * k), 64);
      f(std::integral_constant<int, S::NB + (int)k>{}, recs + (uint64_t)s * BYTES + chunk * 16);
    });
}

// straight to LDS, and waited for
template <int NC>
__device__ __forceinline__ void m2l_stage(const char* __restrict__ recs, uint32_t src,
                                          M2LStage<NC>& sh) {
  // (the reads of the last step's records are done)
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  m2l_addresses<NC>(recs, src, [&](auto k, const char* p) { load_to_lds(p, sh.c[k.value]); });
  // (the compiler's own waits for such loads do not cover every read of them)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// into registers, and from there to LDS
template <int NC>
struct M2LRegs {
  static constexpr int N = M2LStage<NC>::NB + M2LStage<NC>::R;
  double x[N], y[N];
};
template <int NC>
__device__ __forceinline__ void m2l_load(const char* __restrict__ recs, uint32_t src,
                                         M2LRegs<NC>& r) {
  constexpr int N = M2LStage<NC>::NB + M2LStage<NC>::R;
  const char* p[N];
  m2l_addresses<NC>(recs, src, [&](auto k, const char* q) { p[k.value] = q; });
#pragma unroll
  for (int k = 0; k < N; ++k) {
    const double2 v = *reinterpret_cast<const double2*>(p[k]);
    r.x[k] = v.x;
    r.y[k] = v.y;
  }
}
template <int NC>
__device__ __forceinline__ void m2l_put(const M2LRegs<NC>& r, M2LStage<NC>& sh) {
#pragma unroll
  for (int k = 0; k < M2LRegs<NC>::N; ++k) sh.c[k][threadIdx.x] = make_double2(r.x[k], r.y[k]);
}

// chunk I of this lane's record
template <int NC, int I>
__device__ __forceinline__ double2 m2l_chunk(const M2LStage<NC>& sh) {
  using S = M2LStage<NC>;
  const uint32_t lane = threadIdx.x, sub = lane & 7, g8 = lane & ~7u;
  if constexpr (I < S::NB) {
    return sh.c[sub][g8 + (I ^ sub)];
  } else {
    constexpr uint32_t R = S::R, J = I - S::NB;
    const uint32_t k = sub / (8 / R);  // the instruction that loaded this record
    return sh.c[S::NB + k][g8 + (sub % (8 / R)) * R + (J ^ k)];
  }
}

// the sum of v over the 8 lanes of a group
__device__ __forceinline__ double group_sum8(double v) {
  auto mv = [](double x, auto ctrl) {
    constexpr int CTRL = decltype(ctrl)::value;
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
  };
  v += mv(v, std::integral_constant<int, 0xb1>{});   // lanes 1 0 3 2 of each four
  v += mv(v, std::integral_constant<int, 0x4e>{});   // lanes 2 3 0 1
  v += mv(v, std::integral_constant<int, 0x141>{});  // each eight mirrored
  return v;
}

// the node that group grp of block b takes; -1 for none
__device__ __forceinline__ int m2l_node(const SharedFarArgs& a, unsigned b, int grp) {
  // (blocks of 8 nodes: the FP64 targets, the long lists, the windows)
  const unsigned b64 = ((unsigned)a.n64 + 7) / 8;
  if (b < b64) {
    const int g = (int)b * 8 + grp;
    return g < a.n64 ? a.level_nodes[g] : -1;
  }
  b -= b64;
  const unsigned nlong = a.nlong ? *a.nlong - (unsigned)a.n64 : 0u, bl = (nlong + 7) / 8;
  if (b < bl) {
    const unsigned g = b * 8 + grp;
    return g < nlong ? a.level_nodes[a.n64 + g] : -1;
  }
  b -= bl;
  // (consecutive blocks are dealt to the XCDs in turn)
  const unsigned wb = (unsigned)a.window / 8, x = b % kXcds, k = b / kXcds;
  const uint64_t g = (uint64_t)a.n64 + nlong +
                     (uint64_t)((k / wb) * kXcds + x) * (unsigned)a.window + (k % wb) * 8 + grp;
  return g < (uint64_t)a.nn ? a.level_nodes[g] : -1;
}

template <int P, bool F32>
struct M2LShape {
  static constexpr int NC = F32 ? rec32_stride(P) / 4 : recq_stride(P) / 2;
};

template <int P, bool F32>
__device__ __forceinline__ void m2l_wave(const SharedFarArgs& a,
                                         M2LStage<M2LShape<P, F32>::NC>& sh) {
  using E = Exp<P>;
  constexpr int NL = E::NL;
  constexpr int NS = F32 ? NL : E::NLR;  // sums
  constexpr int RS = rec_stride(P);
  constexpr int NC = M2LShape<P, F32>::NC;
  const int lane = threadIdx.x, sub = lane & 7, grp = lane >> 3;
  const int node = m2l_node(a, blockIdx.x, grp);
  const bool active = node >= 0;
  const int v = active ? node : 0;
  const uint32_t cnt = active ? a.m2l_cnt[v] : 0u;
  const uint32_t* list = a.pool + (active ? a.m2l_off[v] : 0u);
  const char* __restrict__ recs =
      F32 ? reinterpret_cast<const char*>(a.rec32) : reinterpret_cast<const char*>(a.recq);
  const double* rv = a.rec + (int64_t)v * RS;
  const double sv[3] = {rv[0], rv[1], rv[2]};
  double L[NS];
#pragma unroll
  for (int q = 0; q < NS; ++q) L[q] = 0.0;
  // (a lane past the end of its list repeats the first entry and adds nothing)
  const uint32_t first = cnt > 0 ? list[0] & kSrcMask : 0u;
  auto entry = [&](uint32_t e) { return e + sub < cnt ? list[e + sub] & kSrcMask : first; };
  uint32_t src = entry(0);
  uint32_t most = cnt;  // the wave's longest list
#pragma unroll
  for (int o = 32; o > 4; o >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, o, 64));
  most = __builtin_amdgcn_readfirstlane(most);
  // FP64 terms (half the registers) load the next step's records into
  // registers while a step is computed; with FP32 terms, whose sums leave no
  // room for that, the other wave of the SIMD computes meanwhile
  M2LRegs<NC> regs = {};
  if (!F32 && most > 0) {
    m2l_load<NC>(recs, src, regs);
    src = entry(8);
  }
  for (uint32_t e = 0; e < most; e += 8) {
    const bool ok = e + sub < cnt;
    if constexpr (F32) {
      m2l_stage<NC>(recs, src, sh);
      src = entry(e + 8);
    } else {
      m2l_put<NC>(regs, sh);
      if (e + 8 < most) m2l_load<NC>(recs, src, regs);
      src = entry(e + 16);
    }
    __syncthreads();
    double2 c[NC];
    static_for<NC>([&](auto ic) { c[ic.value] = m2l_chunk<NC, ic.value>(sh); });
    const double d[3] = {c[0].x - sv[0], c[0].y - sv[1], c[1].x - sv[2]};
    if constexpr (F32) {
      const float r[3] = {(float)d[0], (float)d[1], (float)d[2]};
      float w[4 * NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        const unsigned long long x = (unsigned long long)__double_as_longlong(c[i].x);
        const unsigned long long y = (unsigned long long)__double_as_longlong(c[i].y);
        w[4 * i] = __uint_as_float((uint32_t)x);
        w[4 * i + 1] = __uint_as_float((uint32_t)(x >> 32));
        w[4 * i + 2] = __uint_as_float((uint32_t)y);
        w[4 * i + 3] = __uint_as_float((uint32_t)(y >> 32));
      }
      E::m2l_add_f32(r, w + 6, L, ok);
    } else {
      double w[2 * NC];
#pragma unroll
      for (int i = 0; i < NC; ++i) { w[2 * i] = c[i].x; w[2 * i + 1] = c[i].y; }
      E::m2l_h(d, w + 3, L, ok);
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NS; ++q) L[q] = group_sum8(L[q]);
  if (active && cnt > 0) {
    double* out = a.ln + (int64_t)v * NL;
    if constexpr (F32) {
#pragma unroll
      for (int q = 0; q < NL; ++q)
        if (q % 8 == sub) out[q] = L[q];
    } else {
      double full[NL];
      E::expand(L, full);
#pragma unroll
      for (int q = 0; q < NL; ++q)
        if (q % 8 == sub) out[q] = full[q];
    }
  }
}

// F32: the blocks of FP64 targets (the first ones) and those of FP32 targets
// in one launch, so that the few FP64 ones do not run alone
template <int P, bool F32, int WAVES>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_m2l(
    SharedFarArgs a) {
  __shared__ union {
    M2LStage<M2LShape<P, false>::NC> q;
    M2LStage<M2LShape<P, true>::NC> f;
  } sh;
  if constexpr (F32) {
    if (blockIdx.x >= ((unsigned)a.n64 + 7) / 8) {
      m2l_wave<P, true>(a, sh.f);
      return;
    }
  }
  m2l_wave<P, false>(a, sh.q);
}

// The one-sided symmetric M2L (Sect. 5 notes that an interaction can be
// applied to both nodes of a pair): every unordered pair of the interaction
// set -- node v's M2L list holds s exactly when s's holds v -- is evaluated
// once, by the node with the smaller id, with one derivative tensor D(r) for
// both directions (Exp<P>::m2l_pair): the owner's side is summed in
// registers as in k_m2l, the partner's side is added to the partner's
// local coefficients with FP64 atomic adds, and the owner adds its own sum
// last, also atomically.  ln must hold zeros before.  The order of the
// atomic additions is not fixed, so results agree with the directed form to
// rounding, not bit for bit.
template <int P, int SPLIT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1))) void k_m2l_mutual(
    SharedFarArgs a) {
  using E = Exp<P>;
  constexpr int NQ = E::NQ;
  constexpr int NL = E::NL;
  constexpr int RS = rec_stride(P);
  const int lane = threadIdx.x;
  const int sub = lane % SPLIT;
  const int g = blockIdx.x * (64 / SPLIT) + lane / SPLIT;
  const bool active = g < a.nn;
  const int v = active ? a.level_nodes[g] : 0;
  const uint32_t cnt = active ? a.m2l_cnt[v] : 0u;
  const uint32_t off = active ? a.m2l_off[v] : 0u;
  const double* __restrict__ rec = a.rec;
  const double* rv = rec + (int64_t)v * RS;
  const double sv[3] = {rv[0], rv[1], rv[2]};
  // the owner's moments with odd degrees negated (its side of D(-r))
  double QTs[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) QTs[q] = rv[8 + q];
  {
    int k = 0;
#pragma unroll
    for (int n = 0; n <= P; ++n)
#pragma unroll
      for (int c = 0; c < (n + 1) * (n + 2) / 2; ++c, ++k)
        if (n & 1) QTs[k] = -QTs[k];
  }
  double L[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) L[q] = 0.0;
  for (uint32_t e = off + sub; e < off + cnt; e += SPLIT) {
    const uint32_t src = a.pool[e] & kSrcMask;
    if ((int)src <= v) continue;  // the partner owns this pair
    const double* rs = rec + (int64_t)src * RS;
    const double r[3] = {rs[0] - sv[0], rs[1] - sv[1], rs[2] - sv[2]};
    double QS[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) QS[q] = rs[8 + q];
    E::m2l_pair(r, QS, QTs, L, a.ln + (int64_t)src * NL);
  }
#pragma unroll
  for (int o = SPLIT / 2; o > 0; o >>= 1) {
#pragma unroll
    for (int q = 0; q < NL; ++q) L[q] += __shfl_xor(L[q], o, 64);
  }
  if (active && cnt > 0) {
    double* out = a.ln + (int64_t)v * NL;
#pragma unroll
    for (int q = 0; q < NL; ++q)
      if (q % SPLIT == sub) unsafeAtomicAdd(&out[q], L[q]);
  }
}

// Sort key of the node at level position g: FP64 targets of FP32C by steps of
// 8 entries, longest first (0..31), other nodes of more than `longer` steps
// likewise (32..62), and all others together (63, in level order: the pass is
// stable)
__global__ void k_m2l_order_keys(int nn, const int32_t* __restrict__ level_nodes,
                                 const uint32_t* __restrict__ cnt,
                                 const int32_t* __restrict__ depth, int top, int f32,
                                 uint32_t longer, uint64_t* __restrict__ key,
                                 uint32_t* __restrict__ ids) {
  const int g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= nn) return;
  const int v = level_nodes[g];
  const uint32_t steps = (cnt[v] + 7u) / 8u;
  uint32_t k = 63;
  if (f32 && depth[v] < top) k = 31u - min(steps / 8u, 31u);
  else if (steps > longer) k = 62u - min((steps - longer) / 8u, 30u);
  key[g] = k;
  ids[g] = (uint32_t)v;
}

// each window of the nodes after the long lists, sorted by steps, longest
// first (nodes of like length in any order: every node's sum is its own).
// Bound: a few latencies; 1024 threads a window of at most 1024 nodes.
constexpr int kWindowMax = 1024;
__global__ __launch_bounds__(kWindowMax) void k_m2l_windows(SharedFarArgs a,
                                                            const uint32_t* __restrict__ in,
                                                            uint32_t* __restrict__ out) {
  __shared__ uint32_t at[256];
  const uint32_t t = threadIdx.x, lead = a.nlong ? *a.nlong : (uint32_t)a.n64;
  const uint64_t beg = lead + (uint64_t)blockIdx.x * (unsigned)a.window;
  if (blockIdx.x == 0)  // (those before the windows stay where they are)
    for (uint32_t g = t; g < lead; g += blockDim.x) out[g] = in[g];
  if (beg >= (uint64_t)a.nn) return;
  const bool ok = t < (uint32_t)a.window && beg + t < (uint64_t)a.nn;
  if (t < 256) at[t] = 0;
  __syncthreads();
  uint32_t v = 0, b = 0;
  if (ok) {
    v = in[beg + t];
    b = 255u - min((a.m2l_cnt[v] + 7u) / 8u, 255u);
    atomicAdd(&at[b], 1u);
  }
  __syncthreads();
  // exclusive sums of the 256 counters: a wave, four counters a lane
  if (t < 64) {
    uint32_t c[4], s = 0;
    for (int k = 0; k < 4; ++k) { c[k] = at[4 * t + k]; s += c[k]; }
    uint32_t incl = s;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
      if ((int)t >= o) incl += u;
    }
    uint32_t run = incl - s;
    for (int k = 0; k < 4; ++k) { at[4 * t + k] = run; run += c[k]; }
  }
  __syncthreads();
  if (ok) out[beg + atomicAdd(&at[b], 1u)] = v;
}

__global__ void k_zero_f64(int64_t n, double* __restrict__ p) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// k_far_shared: one lane per leaf goes down its branch from the root.  Bound by
// the chain of loads of a branch: the branch is noted in LDS first (one load a
// level, up the parents), so that on the way down a node's record is read while
// its parent's is used.  20 us at 1e3 particles, 24 at 1e5, 70 at 1e6; finding
// each child from its parent on the way down 34, 46, 95.
template <int P>
__global__ __launch_bounds__(64) void k_far_shared(FarArgs a, const double* __restrict__ ln) {
  using E = Exp<P>;
  constexpr int NL = E::NL;
  constexpr int RS = rec_stride(P);
  extern __shared__ int path[];  // [depth][64]: the leaf's ancestors, the leaf last
  const int lane = threadIdx.x;
  const int l = xcd_block(blockIdx.x, gridDim.x) * 64 + lane;
  if (l >= a.nleaves) return;
  const NodeInfo* __restrict__ info = a.info;
  const double* __restrict__ rec = a.rec;
  const int leaf = a.leaf_node[l];
  const int d = a.leaf_depth[l];
  const NodeInfo li = info[leaf];
  const int lo = li.lo, cnt = li.cnt;
  path[d * 64 + lane] = leaf;
  for (int k = d - 1, u = li.parent; k >= 0; --k, u = info[u].parent) path[k * 64 + lane] = u;
  double L[NL];
#pragma unroll
  for (int q = 0; q < NL; ++q) L[q] = 0.0;
  bool have = false;
  double sv[3] = {0.0, 0.0, 0.0};
  // (the next node's centre and list length load while this one's are used)
  struct Next {
    int v;
    uint32_t m2l;
    double s[3];
  };
  auto load = [&](int k) {
    const int v = path[k * 64 + lane];
    const double* r = rec + (int64_t)v * RS;
    return Next{v, a.node_m2l_cnt[v], {r[0], r[1], r[2]}};
  };
  Next next = load(0);
  for (int k = 0; k <= d; ++k) {
    const Next n = next;
    if (k < d) next = load(k + 1);
    const double* lu = ln + (int64_t)n.v * NL;
    if (have) {
      const double hv[3] = {n.s[0] - sv[0], n.s[1] - sv[1], n.s[2] - sv[2]};
      E::l2l(hv, L);
    }
    if (n.m2l != 0) {
#pragma unroll
      for (int q = 0; q < NL; ++q) L[q] += lu[q];
      have = true;
    }
    sv[0] = n.s[0]; sv[1] = n.s[1]; sv[2] = n.s[2];
  }
  for (int j = lo; j < lo + cnt; ++j) {
    const double off[3] = {a.xs[j] - sv[0], a.ys[j] - sv[1], a.zs[j] - sv[2]};
    double f[3] = {0.0, 0.0, 0.0}, phi = 0.0;
    if (have) E::l2p(off, L, f, phi);
    double* o = a.far + 4 * (int64_t)j;
    o[0] = f[0]; o[1] = f[1]; o[2] = f[2]; o[3] = phi;
  }
}

template <int P>
void shared_order(const FarArgs& f, const SharedFarArgs& a, bool f32, hipStream_t s) {
  if (a.nn > 0) {
    // blocks: FP64 targets, long lists (at most one partial block each), and
    // whole windows for every XCD
    const int64_t per = (int64_t)a.window * kXcds;
    const unsigned nb = (unsigned)((a.n64 + 7) / 8 + (a.maxlong + 7) / 8 +
                                   (a.nn + per - 1) / per * per / 8);
    // two waves a SIMD; at order 4 the sums alone leave no room for a second (FP64,
    // 1e6 particles: 4.6 ms a solve, with two waves and 82 spilled registers 6.9)
    constexpr int WAVES = P < 4 ? 2 : 1;
    if (f32) k_m2l<P, true, WAVES><<<nb, 64, 0, s>>>(a);
    else k_m2l<P, false, WAVES><<<nb, 64, 0, s>>>(a);
  }
  if (f.nleaves > 0) k_far_shared<P><<<(unsigned)((f.nleaves + 63) / 64), 64, 64 * sizeof(int) * (f.maxdepth + 1), s>>>(f, a.ln);
}

template <int P>
void mutual_order(const FarArgs& f, const SharedFarArgs& a, hipStream_t s) {
  if (a.nn > 0) {
    const int64_t nz = (int64_t)a.nn * Exp<P>::NL;
    k_zero_f64<<<(unsigned)std::min<int64_t>((nz + 255) / 256, 4096), 256, 0, s>>>(nz, a.ln);
    constexpr int SPLIT = 8;
    k_m2l_mutual<P, SPLIT><<<(unsigned)((a.nn + 64 / SPLIT - 1) / (64 / SPLIT)), 64, 0, s>>>(a);
  }
  if (f.nleaves > 0) k_far_shared<P><<<(unsigned)((f.nleaves + 63) / 64), 64, 64 * sizeof(int) * (f.maxdepth + 1), s>>>(f, a.ln);
}

}  // namespace

void launch_far_shared(int order, const FarArgs& f, const SharedFarArgs& a, bool f32,
                       hipStream_t s) {
  switch (order) {
    case 0: shared_order<0>(f, a, f32, s); break;
    case 1: shared_order<1>(f, a, f32, s); break;
    case 2: shared_order<2>(f, a, f32, s); break;
    case 3: shared_order<3>(f, a, f32, s); break;
    case 4: shared_order<4>(f, a, f32, s); break;
  }
}

void m2l_windows(SharedFarArgs& a, uint64_t m2l_total) {
  // windows: four and more for each XCD, so that their costs even out, of 64 to
  // kWindowMax nodes
  int w = 64;
  while (w < kWindowMax && (int64_t)2 * w * kXcds * 4 <= a.nn) w *= 2;
  a.window = w;
  // long lists: four times the mean and more
  const uint64_t mean = a.nn > 0 ? m2l_total / (8 * (uint64_t)a.nn) : 0;
  a.steps = m2l_total / 8 + (uint64_t)a.nn;
  a.longer = (uint32_t)std::max<uint64_t>(16, 4 * mean);
  a.nlong = nullptr;
  a.maxlong = 0;
}

void launch_m2l_order(SharedFarArgs& a, bool f32, const M2LOrderBufs& b, hipStream_t s) {
  if (a.nn <= 0) return;
  const uint32_t* in = reinterpret_cast<const uint32_t*>(a.level_nodes);
  // (a small tree has no room for long tails, and the key sort is four launches)
  if (a.nn > 8192 || a.n64 > 0) {
    k_m2l_order_keys<<<(unsigned)((a.nn + 255) / 256), 256, 0, s>>>(
        a.nn, a.level_nodes, a.m2l_cnt, a.depth, a.top, f32 ? 1 : 0, a.longer, b.key0, b.ids0);
    radix_pass(a.nn, false, b.key0, b.ids0, b.key1, b.ids2, b.base, b.words, s);
    a.maxlong = (int)std::min<uint64_t>(a.nn, a.steps / (a.longer + 1));
    a.nlong = b.base + 63;  // the first place of key 63
    in = b.ids2;
  }
  k_m2l_windows<<<(unsigned)((a.nn + a.window - 1) / a.window), kWindowMax, 0, s>>>(a, in, b.ids1);
}

void launch_far_mutual(int order, const FarArgs& f, const SharedFarArgs& a, hipStream_t s) {
  switch (order) {
    case 0: mutual_order<0>(f, a, s); break;
    case 1: mutual_order<1>(f, a, s); break;
    case 2: mutual_order<2>(f, a, s); break;
    case 3: mutual_order<3>(f, a, s); break;
    case 4: mutual_order<4>(f, a, s); break;
  }
}

template <bool NODE, int SPLIT, int WAVES>
void far_dispatch(int order, const FarArgs& a, hipStream_t s) {
  const unsigned nb = (unsigned)((a.nleaves + 64 / SPLIT - 1) / (64 / SPLIT));
  switch (order) {
    case 0: k_far<0, NODE, SPLIT, WAVES><<<nb, 64, 0, s>>>(a); break;
    case 1: k_far<1, NODE, SPLIT, WAVES><<<nb, 64, 0, s>>>(a); break;
    case 2: k_far<2, NODE, SPLIT, WAVES><<<nb, 64, 0, s>>>(a); break;
    case 3: k_far<3, NODE, SPLIT, WAVES><<<nb, 64, 0, s>>>(a); break;
    case 4: k_far<4, NODE, SPLIT, WAVES><<<nb, 64, 0, s>>>(a); break;
  }
}

void launch_far(int order, bool node_lists, const FarArgs& a, hipStream_t s) {
  if (a.nleaves <= 0) return;
  // 4 lanes per leaf, one wave per SIMD
  if (node_lists) far_dispatch<true, 4, 1>(order, a, s);
  else far_dispatch<false, 4, 1>(order, a, s);
}

}  // namespace sfmm
