// k_nodewalk.hip -- level-synchronous form of the dual tree walk.
//
// In Algorithm 1 (Sect. 3) every leaf walks from (root, root) down its own
// branch; the pairs a leaf tests against its ancestor p_k, and their outcome,
// depend only on p_k, so all leaves below p_k repeat them.  Here each node
// is visited once, level by level from the root:
//   tested(v) = expand(opened(parent(v)))   (a leaf source stays, an
//               internal source is replaced by its two children; for the
//               root, tested = {root})
// and each tested source is, as in Algorithm 2,
//   the node itself            -> opened
//   accepted (MAC + softening) -> M2L entry of v
//   otherwise                  -> opened
// An internal v hands its opened list to its children.  A leaf v lowers
// its opened sources in place: a leaf source becomes a P2P entry, an
// internal one is replaced by its children and tested against v again.
// The list of leaf L in Algorithm 1 is exactly the concatenation of the
// M2L lists of p_0 .. p_d plus L's P2P list (same pairs; the order inside a
// depth differs).
//
// Bound by the traffic between L1 and L2 and by latency.  The sources' fields
// are in one record of 64 bytes, a pair of children in one line, and the
// lists name the pair (an expansion record and the node's topology apart,
// looked up per source, took 4.5 lines a pair: 2.24 ms for the walk of a 1e6
// Plummer sphere, now 1.48; 2.29 and 1.58 ms for 2e6 particles of a binary).
//
// One wave (a 64-thread block) per node; lanes take 64 sources at a time,
// and entries are written in lane order.  An internal node's M2L and opened
// lists together are its tested list, whose size its parent records while
// walking (opened leaves once, opened internal nodes twice).  So one region
// of the M2L pool holds both lists, M2L entries from the front and opened
// entries from the back, and its size is known before the node is walked:
// the region is the node's fixed slot, or a piece of an arena when larger.
// Each level is then one launch, or a few small levels together.  The leaves come after all levels, in one
// pass that writes each leaf's lists into fixed per-leaf slots (or a few
// large slots).  A second pass, at exact offsets, takes only the leaves that
// fit neither.
#include "sfmm_internal.h"

namespace sfmm {
namespace {

// an opened internal node is listed as its first child with this bit: the
// walks of its lists read the two children at once, without a lookup
constexpr uint32_t kOpenInternal = 0x80000000u;

// centre, size and largest h, first child, particles of a node
struct Src {
  double x, y, z, l, h;
  int child, cnt;
};
__device__ __forceinline__ Src load_src(const NodeWalkArgs& a, uint32_t s) {
  const double2* p = reinterpret_cast<const double2*>(a.wrec + s);
  const double2 u = p[0], v = p[1], w = p[2];
  const uint64_t b = (uint64_t)__double_as_longlong(w.y);
  return {u.x, u.y, v.x, v.y, w.x, (int)(uint32_t)b, (int)(uint32_t)(b >> 32)};
}

__device__ __forceinline__ bool accept(const Src& t, const Src& s, double theta2, double r_kern) {
  const double dx = s.x - t.x;
  const double dy = s.y - t.y;
  const double dz = s.z - t.z;
  const double d2 = dx * dx + dy * dy + dz * dz;
  const double lsum = t.l + s.l;
  const double hm = fmax(t.h, s.h);
  const double rsum = lsum + r_kern * hm;
  return (lsum * lsum < theta2 * d2) && (d2 >= rsum * rsum);
}

// set bits of m below this lane, added to acc
__device__ __forceinline__ uint32_t below(uint64_t m, uint32_t acc) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)m, acc));
}

// appends, in lane order, v0 of the lanes with c0 and v1 of those with c1 (a
// lane's v0 before its v1) to a list of `run` entries with room for lim
__device__ __forceinline__ void append(uint32_t* list, uint32_t lim, uint32_t& run, bool c0,
                                       uint32_t v0, bool c1, uint32_t v1) {
  const uint64_t b0 = __ballot(c0), b1 = __ballot(c1);
  if ((b0 | b1) == 0) return;  // (uniform)
  const uint32_t k0 = run + below(b1, below(b0, 0u)), k1 = k0 + (c0 ? 1u : 0u);
  if (c0 && k0 < lim) list[k0] = v0;
  if (c1 && k1 < lim) list[k1] = v1;
  run += (uint32_t)__popcll(b0) + (uint32_t)__popcll(b1);
}
// the same from the end of a range of `size` entries backwards
__device__ __forceinline__ void append_back(uint32_t* list, uint32_t size, uint32_t lim,
                                            uint32_t& run, bool c0, uint32_t v0, bool c1,
                                            uint32_t v1) {
  const uint64_t b0 = __ballot(c0), b1 = __ballot(c1);
  if ((b0 | b1) == 0) return;
  const uint32_t r0 = run + below(b1, below(b0, 0u)), r1 = r0 + (c0 ? 1u : 0u);
  if (c0 && r0 < size && size - 1u - r0 < lim) list[size - 1u - r0] = v0;
  if (c1 && r1 < size && size - 1u - r1 < lim) list[size - 1u - r1] = v1;
  run += (uint32_t)__popcll(b0) + (uint32_t)__popcll(b1);
}

// entries of a pool that may be written from `base` on, at most `want`
__device__ __forceinline__ uint32_t pool_room(uint64_t base, uint64_t cap, uint32_t want) {
  const uint64_t room = base < cap ? cap - base : 0;
  return room < want ? (uint32_t)room : want;
}

// ---- the lists of one leaf ------------------------------------------------------
struct Emit {
  uint32_t m2l_run;
  // P2P entries that may fall inside a kernel from the front of the list, those beyond both kernels (plain_run of them so far) from the back
  uint32_t p2p_run, plain_run;
  uint32_t src_lane;  // this lane's share of the particles of the P2P entries
  uint64_t m2l_base, p2p_base;  // places in the pools, entries
  uint32_t *m2l, *p2p;          // the same as addresses
  uint32_t room_m, room_p;      // entries that may be written there
  // exact pass: P2P entries of the leaf.  Slot pass: the sizes of the slots,
  // and the entries beyond both kernels staged in LDS (in rank order) until
  // the leaf's P2P count is known, or in global memory (plain_g) once the
  // leaf has a large slot
  uint32_t p2p_total;
  uint32_t slot_m, slot_p;
  uint32_t* plain;
  uint32_t* plain_g;
  bool big_m, big_p;  // a large slot was asked for (M2L, P2P)
};

__device__ __forceinline__ void place_m2l(const NodeWalkArgs& a, Emit& e, uint64_t base,
                                          uint32_t want) {
  e.m2l_base = base;
  e.m2l = a.m2l_pool + base;
  e.room_m = pool_room(base, a.m2l_cap, want);
}
__device__ __forceinline__ void place_p2p(const NodeWalkArgs& a, Emit& e, uint64_t base,
                                          uint32_t want) {
  e.p2p_base = base;
  e.p2p = a.p2p_pool + base;
  e.room_p = pool_room(base, a.p2p_cap, want);
}

// A leaf's lists: M2L entries, P2P entries that may need softening, and P2P
// entries beyond both kernels, which are written from the end of the leaf's
// range, so the P2P kernel meets the softened pairs first and the rest in
// whole chunks without them.
// W = kLeafExact writes at the leaf's exact offsets (its P2P count known);
// W = kLeafSlot writes the M2L and softening entries into the leaf's fixed
// slots as far as they fit and stages the others in LDS
constexpr int kLeafExact = 1;
constexpr int kLeafSlot = 2;

// slot mode: a leaf whose M2L list outgrows its slot moves it to one of the
// large slots (a.nbig of a.big_m entries after all slots), in one piece; with
// none left it keeps its slot (and is walked again afterwards)
__device__ __forceinline__ void promote_m2l(const NodeWalkArgs& a, Emit& e) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t b = 0;
  if (lane == 0) b = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(a.run + 8), 1ull);
  b = __builtin_amdgcn_readfirstlane(b);
  e.big_m = true;
  if (b >= a.nbig) return;
  const uint32_t* from = e.m2l;
  const uint32_t have = e.m2l_run < e.room_m ? e.m2l_run : e.room_m;
  place_m2l(a, e, a.leaf_base + (uint64_t)a.nleaves * a.slot_m + (uint64_t)b * a.big_m, a.big_m);
  e.slot_m = a.big_m;
  __threadfence();  // the wave's own slot entries, read back below
  for (uint32_t i = lane; i < have; i += 64)
    if (i < e.room_m) e.m2l[i] = from[i];
}

// the same for the P2P list: its entries that may need softening move to a
// large P2P slot, the staged ones to that slot's global staging area
__device__ __forceinline__ void promote_p2p(const NodeWalkArgs& a, Emit& e) {
  const uint32_t lane = threadIdx.x & 63;
  uint32_t b = 0;
  if (lane == 0) b = (uint32_t)atomicAdd(reinterpret_cast<unsigned long long*>(a.run + 9), 1ull);
  b = __builtin_amdgcn_readfirstlane(b);
  e.big_p = true;
  if (b >= a.nbig) return;
  const uint32_t* from = e.p2p;
  const uint32_t have = e.p2p_run < e.room_p ? e.p2p_run : e.room_p;
  place_p2p(a, e, (uint64_t)a.nleaves * a.slot_p + (uint64_t)b * a.big_p, a.big_p);
  e.slot_p = a.big_p;
  uint32_t* g = a.big_plain + (uint64_t)b * a.big_p;
  __syncthreads();  // the staged entries (LDS)
  __threadfence();  // the wave's own slot entries
  for (uint32_t i = lane; i < have; i += 64)
    if (i < e.room_p) e.p2p[i] = from[i];
  for (uint32_t i = lane; i < e.plain_run; i += 64) g[i] = e.plain[i];
  e.plain_g = g;
}

// the test of a leaf target, from one evaluation of d^2.  m2l:
// accepted; beyond: d beyond both kernels (a P2P pair of leaves then needs no
// softening); whole: every node below s would fail the softening test against
// v too: s lies inside v's own kernel reach, d + l_s < l_v + R_kern h_max(v)
// (any node below s has its centre within l_s of s's and h_max >= 0), so the
// lowering would end with all of s's leaves as P2P sources; the margin keeps
// rounding in the tests the lowering would make from deciding otherwise
struct LeafTest {
  bool m2l, beyond, whole;
};
__device__ __forceinline__ LeafTest leaf_test(const NodeWalkArgs& a, int v, const Src& rv,
                                              uint32_t s, const Src& rs) {
  const double dx = rs.x - rv.x;
  const double dy = rs.y - rv.y;
  const double dz = rs.z - rv.z;
  const double d2 = dx * dx + dy * dy + dz * dz;
  const double lsum = rv.l + rs.l;
  const double rsum = lsum + a.r_kern * fmax(rv.h, rs.h);
  const double reach = rv.l + a.r_kern * rv.h - rs.l;
  const bool other = (int)s != v;
  LeafTest k;
  k.beyond = other && d2 >= rsum * rsum;
  k.m2l = k.beyond && lsum * lsum < a.theta2 * d2;
  k.whole = other && !k.beyond && reach > 0.0 && d2 < reach * reach * (1.0 - 1e-9);
  return k;
}

// internal target: the opened list of its parent, 64 * kWalkBatch entries at a
// time; every load of a batch (entries, then the records of the nodes they
// stand for) is issued before the classification, so a node waits for one
// chain of two loads per batch; entries are emitted in the order of the list
// (a batch of one group, 50 registers: 0.62 ms for the walk at 1e6 particles of a
// polytrope; two groups took 0.65, three 0.68: the waves in flight matter more)
constexpr int kWalkBatch = 1;

// entries of an internal node's lists so far: M2L entries from the front of its
// region, opened entries from the back; exp_lane sums this lane's opened entries,
// an internal one counted twice
struct NodeRuns {
  uint32_t m2l = 0, open = 0, exp_lane = 0;
};

__device__ __forceinline__ void walk_internal(const NodeWalkArgs& a, int v, const Src& rv, const uint32_t* src,
                              uint32_t nsrc, uint32_t region, uint32_t room, uint32_t* list,
                              NodeRuns& e) {
  const uint32_t lane = threadIdx.x & 63;
  for (uint32_t base = 0; base < nsrc; base += 64 * kWalkBatch) {
    uint32_t sb[kWalkBatch];
#pragma unroll
    for (int u = 0; u < kWalkBatch; ++u) {
      const uint32_t i = base + 64u * u + lane;
      sb[u] = i < nsrc ? src[i] : 0xffffffffu;
    }
    // invalid slots read node v (a valid index) and are masked afterwards,
    // so the loads and tests need no branches
    Src r0[kWalkBatch], r1[kWalkBatch];
    uint32_t t0[kWalkBatch], t1[kWalkBatch];
#pragma unroll
    for (int u = 0; u < kWalkBatch; ++u) {
      const bool ok = sb[u] != 0xffffffffu;
      t0[u] = ok ? sb[u] & ~kOpenInternal : (uint32_t)v;
      t1[u] = ok && (sb[u] & kOpenInternal) ? t0[u] + 1u : (uint32_t)v;
      r0[u] = load_src(a, t0[u]);
      r1[u] = load_src(a, t1[u]);
    }
#pragma unroll
    for (int u = 0; u < kWalkBatch; ++u) {
      if (base + 64u * u >= nsrc) break;  // uniform
      const bool ok = sb[u] != 0xffffffffu, two = ok && (sb[u] & kOpenInternal);
      const bool m0 = (int)t0[u] != v && accept(rv, r0[u], a.theta2, a.r_kern);
      const bool m1 = (int)t1[u] != v && accept(rv, r1[u], a.theta2, a.r_kern);
      const bool i0 = r0[u].child >= 0, i1 = r1[u].child >= 0;
      const bool p0 = ok && !m0, p1 = two && !m1;
      append(list, room, e.m2l, ok && m0, t0[u], two && m1, t1[u]);
      append_back(list, region, room, e.open, p0,
                  i0 ? (uint32_t)r0[u].child | kOpenInternal : t0[u], p1,
                  i1 ? (uint32_t)r1[u].child | kOpenInternal : t1[u]);
      // the children's tested list: an opened leaf once, an internal node twice
      e.exp_lane += (p0 ? (i0 ? 2u : 1u) : 0u) + (p1 ? (i1 ? 2u : 1u) : 0u);
    }
  }
}

// leaf target: U groups of 64 entries per step (all their loads issued before
// the tests), an entry being a leaf or the pair of children of an opened
// node; opened internal sources push their pair on the lowering stack (in
// LDS).  Returns false when the stack would overflow (the walk is then rerun
// with a larger stack).
template <int W, int U>
__device__ __forceinline__ bool leaf_step(const NodeWalkArgs& a, int v, const Src& rv,
                                          const uint32_t (&t0)[U], const int (&nt)[U], Emit& e,
                                          uint32_t* stk, uint32_t& sp) {
  Src r[U][2];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int q = 0; q < 2; ++q) r[u][q] = load_src(a, q < nt[u] ? t0[u] + q : (uint32_t)v);
  bool ok = true;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bool cm[2], cp[2], cq[2], open[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const bool valid = q < nt[u];
      const LeafTest k = leaf_test(a, v, rv, t0[u] + q, r[u][q]);
      // P2P: a leaf, or a whole subtree of P2P sources kept as one entry
      const bool direct = valid && !k.m2l && (r[u][q].child < 0 || k.whole);
      cm[q] = valid && k.m2l;
      cq[q] = direct && k.beyond;
      cp[q] = direct && !k.beyond;
      open[q] = valid && !k.m2l && !direct;
      e.src_lane += direct ? (uint32_t)r[u][q].cnt : 0u;
    }
    const uint32_t s0 = t0[u], s1 = t0[u] + 1u;
    if (W == kLeafSlot) {
      const uint32_t tm = (uint32_t)__popcll(__ballot(cm[0])) + (uint32_t)__popcll(__ballot(cm[1]));
      const bool d0 = cp[0] || cq[0], d1 = cp[1] || cq[1];
      const uint32_t td = (uint32_t)__popcll(__ballot(d0)) + (uint32_t)__popcll(__ballot(d1));
      // (uniform tests: the wave's totals)
      if (!e.big_m && e.m2l_run + tm > e.slot_m) promote_m2l(a, e);
      if (!e.big_p && e.p2p_run + e.plain_run + td > e.slot_p) promote_p2p(a, e);
    }
    append(e.m2l, e.room_m, e.m2l_run, cm[0], s0, cm[1], s1);
    append(e.p2p, e.room_p, e.p2p_run, cp[0], s0, cp[1], s1);
    if (W == kLeafSlot) {
      if (e.plain_g) append(e.plain_g, e.slot_p, e.plain_run, cq[0], s0, cq[1], s1);
      else append(e.plain, e.slot_p, e.plain_run, cq[0], s0, cq[1], s1);
    } else {
      append_back(e.p2p, e.p2p_total, e.room_p, e.plain_run, cq[0], s0, cq[1], s1);
    }
    const uint64_t b0 = __ballot(open[0]), b1 = __ballot(open[1]);
    const uint32_t tpush = (uint32_t)__popcll(b0) + (uint32_t)__popcll(b1);
    if (!ok || sp + tpush > a.stack_cap) { ok = false; continue; }  // uniform
    uint32_t w = sp + below(b1, below(b0, 0u));
    if (open[0]) stk[w++] = (uint32_t)r[u][0].child;
    if (open[1]) stk[w] = (uint32_t)r[u][1].child;
    sp += tpush;
  }
  __syncthreads();
  return ok;
}

// The stack is drained in steps of U groups while it holds as many entries
// and has room for what they may push (2 each), one group at a time while it
// lacks the room, and by what is left once the opened list is at its end: the
// lanes of a step are used, and the stack stays within a few groups per level.
template <int W>
__device__ void walk_leaf(const NodeWalkArgs& a, int v, const Src& rv, const uint32_t* src,
                          uint32_t nsrc, bool root, Emit& e, uint32_t* stk, int* status) {
  // two groups a step: 1.48 ms for the walk of a 1e6 Plummer sphere (one 1.55,
  // three 1.56)
  constexpr int U = 2;
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t n0 = root ? 1u : nsrc;
  uint32_t sp = 0;
  bool ok = true;
  for (uint32_t base = 0; base < n0 && ok; base += 64 * U) {
    uint32_t t0[U];
    int nt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = base + 64u * u + lane;
      const uint32_t sb = i < n0 ? (root ? (uint32_t)v : src[i]) : 0u;
      t0[u] = sb & ~kOpenInternal;
      nt[u] = i < n0 ? ((sb & kOpenInternal) ? 2 : 1) : 0;
    }
    ok = leaf_step<W, U>(a, v, rv, t0, nt, e, stk, sp);
    const bool last = base + 64 * U >= n0;
    while (ok && (last ? sp > 0 : sp >= 64u * U)) {
      const uint32_t kw = sp < 64u * U ? sp : 64u * U;
      if (sp > 64u && sp + kw <= a.stack_cap) {  // (uniform)
        uint32_t d0[U];
        int dn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          dn[u] = 64u * u + lane < kw ? 2 : 0;
          d0[u] = dn[u] ? stk[sp - kw + 64u * u + lane] : 0u;
        }
        __syncthreads();
        sp -= kw;
        ok = leaf_step<W, U>(a, v, rv, d0, dn, e, stk, sp);
      } else {
        const uint32_t k = sp < 64u ? sp : 64u;
        uint32_t d0[1] = {0};
        int dn[1] = {lane < k ? 2 : 0};
        if (dn[0]) d0[0] = stk[sp - k + lane];
        __syncthreads();
        sp -= k;
        ok = leaf_step<W, 1>(a, v, rv, d0, dn, e, stk, sp);
      }
    }
  }
  if (!ok && lane == 0) atomicOr(status, ST_OVERFLOW);
}

// ---- internal nodes, level by level ---------------------------------------
// The M2L pool region of an internal node is its tested list (1 for a root,
// else exp[parent]), known before the node is walked: the node's fixed slot
// of int_slot entries (by its rank among the internal nodes), or for a
// larger region a piece of the arena of int_big entries after all slots
// (run[0] entries of it taken, by run[10] nodes).  Leaves take no room at
// their level (they are walked after all levels); a node over two systems
// gets empty lists.
// a node's opened list, and the tested-list size of its children
struct Opened {
  uint32_t off, cnt, exp;
};

// one wave walks node v (internal), given its parent's opened list.  flag 0: a
// node over two systems (several systems solved together) is never walked; the
// walk of each system starts at its own root (flag 1)
__device__ __forceinline__ Opened walk_node(const NodeWalkArgs& a, int v, const NodeInfo& vi,
                                            int flag, Opened up) {
  const uint32_t lane = threadIdx.x & 63;
  const Src rv = load_src(a, (uint32_t)v);
  const bool root = flag == 1;
  const uint32_t region = flag == 0 ? 0u : root ? 1u : up.exp;
  bool fits = true;
  uint64_t at;
  if (region <= a.int_slot) {
    // (the internal nodes are numbered by their children: 1 + 2c, 2 + 2c)
    at = (uint64_t)((uint32_t)(vi.child - 1) / 2u) * a.int_slot;
  } else {
    uint64_t t = 0;
    if (lane == 0) {
      t = atomicAdd(reinterpret_cast<unsigned long long*>(a.run), (unsigned long long)region);
      atomicAdd(reinterpret_cast<unsigned long long*>(a.run + 10), 1ull);
    }
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)t);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(t >> 32));
    t = ((uint64_t)hi << 32) | lo;
    at = (uint64_t)a.int_nodes * a.int_slot + t;
    fits = t + region <= a.int_big;
  }
  // a region that does not fit gets no offset (the walk goes on counting,
  // the host grows the pool and walks again)
  fits = fits && at + region <= a.m2l_cap;
  NodeRuns e;
  // (root, root) is opened: both root children meet both root children
  if (root && lane == 0 && fits) a.open_pool[at] = (uint32_t)vi.child | kOpenInternal;
  uint32_t nsrc = flag == 2 ? up.cnt : 0u;
  if ((uint64_t)up.off + nsrc > a.open_cap) nsrc = 0;  // pool too small: the walk is rerun
  walk_internal(a, v, rv, a.open_pool + up.off, nsrc, region, fits ? region : 0u,
                a.m2l_pool + at, e);
  uint32_t ex = e.exp_lane;
#pragma unroll
  for (int k = 32; k > 0; k >>= 1) ex += (uint32_t)__shfl_xor((int)ex, k, 64);
  const uint32_t open = root ? 1u : e.open;
  const Opened o{fits ? (uint32_t)(at + region - open) : kNoList, open, root ? 2u : ex};
  if (lane == 0) {
    a.m2l_off[v] = fits ? (uint32_t)at : kNoList;
    a.m2l_cnt[v] = e.m2l;
    a.open_off[v] = o.off;
    a.open_cnt[v] = o.cnt;
    a.exp[v] = o.exp;
    a.p2p_cnt[v] = 0;
    a.p2p_off[v] = 0;
  }
  return o;
}

__device__ __forceinline__ int walk_flag(const NodeWalkArgs& a, int v, const NodeInfo& vi) {
  return a.node_flag ? (int)a.node_flag[v] : (vi.parent < 0 ? 1 : 2);
}
__device__ __forceinline__ Opened parent_opened(const NodeWalkArgs& a, const NodeInfo& vi) {
  if (vi.parent < 0) return {0u, 0u, 0u};
  return {a.open_off[vi.parent], a.open_cnt[vi.parent], a.exp[vi.parent]};
}

// one level, a wave per node
__global__ __launch_bounds__(64) void k_nodewalk_internal(NodeWalkArgs a, int level) {
  const uint32_t idx = a.level_base[2 * level] + xcd_block(blockIdx.x, gridDim.x);
  if (idx >= a.level_base[2 * level + 1]) return;
  const int v = a.level_nodes[idx];
  const NodeInfo vi = a.info[v];
  walk_node(a, v, vi, walk_flag(a, v, vi), parent_opened(a, vi));
}

// kWalkRun levels from `level` on, a block per node of the first: 1, 2, .. of
// its waves take the node, its internal children, theirs.  Bound by the chain
// of loads of a level; a launch a level adds the lookups of the node and of its
// parent's list, which the block passes on in LDS.  Walk phase of 1e3 particles
// 0.093 ms (0.122 with a launch a level), of 1e4 0.167 (0.214).
constexpr int kWalkRun = 3;
constexpr int kRunWaves = 1 << (kWalkRun - 1);
__global__ __launch_bounds__(64 * kRunWaves) void k_nodewalk_run(NodeWalkArgs a, int level) {
  __shared__ int node[kRunWaves];
  __shared__ Opened up[kRunWaves];
  const uint32_t idx = a.level_base[2 * level] + xcd_block(blockIdx.x, gridDim.x);
  if (idx >= a.level_base[2 * level + 1]) return;
  const int w = threadIdx.x >> 6;
  int v = w == 0 ? a.level_nodes[idx] : -1;
  Opened mine{0u, 0u, 0u};
  if (w == 0) mine = parent_opened(a, a.info[v]);
  for (int r = 0;; ++r) {
    NodeInfo vi{0, 0, -1, -1};
    if (v >= 0) {
      vi = a.info[v];
      mine = walk_node(a, v, vi, walk_flag(a, v, vi), mine);
    }
    if (r == kWalkRun - 1) break;
    // the internal children of the round's nodes, and their parent's list
    if (w < (1 << r) && (threadIdx.x & 63) == 0) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        node[2 * w + q] = v >= 0 && a.info[vi.child + q].child >= 0 ? vi.child + q : -1;
        up[2 * w + q] = mine;
      }
    }
    __syncthreads();  // (the lists written by a wave are read by others)
    v = w < (2 << r) ? node[w] : -1;
    mine = up[w];
    v = __builtin_amdgcn_readfirstlane(v);
    __syncthreads();
  }
}

// ---- leaves, all levels at once ---------------------------------------------
// A leaf's lists depend only on its parent's opened list, so the leaves are
// walked after every level's internal nodes, in leaf order (one wave per
// leaf).  One pass writes each leaf's lists into fixed slots (slot_m M2L
// entries per leaf after the internal nodes' regions in the M2L pool, slot_p
// P2P entries per leaf at the front of the P2P pool).  A leaf whose lists do
// not fit its slots is listed (in one of kXcds lists by its leaf range,
// run[11 + range] of them) and walked again by a second
// pass, which writes its lists after all slots, at offsets from scans of
// such leaves' counts.
template <bool OVF>
__device__ __forceinline__ void leaf_lists(const NodeWalkArgs& a, int l, uint32_t* stk) {
  const int v = a.leaf_node[l];
  const NodeInfo vi = a.info[v];
  const int flag = a.node_flag ? (int)a.node_flag[v] : (vi.parent < 0 ? 1 : 2);
  const uint32_t lane = threadIdx.x & 63;
  if (flag == 0) {  // (a leaf never spans two systems; kept for safety)
    if (lane == 0) {
      a.m2l_cnt[v] = 0; a.open_cnt[v] = 0; a.p2p_cnt[v] = 0;
      a.m2l_off[v] = 0; a.open_off[v] = 0; a.p2p_off[v] = 0;
      a.leaf_m2l_cnt[l] = 0; a.leaf_p2p_cnt[l] = 0;
      a.src_total[l] = 0; a.item_cnt[l] = 1;
    }
    return;
  }
  const bool root = flag == 1;
  const Src rv = load_src(a, (uint32_t)v);
  const uint32_t* src = nullptr;
  uint32_t nsrc = 0;
  if (!root) {
    const uint32_t po = a.open_off[vi.parent];
    nsrc = a.open_cnt[vi.parent];
    src = a.open_pool + po;
    if ((uint64_t)po + nsrc > a.open_cap) nsrc = 0;  // pool too small: the walk is rerun
  }
  const uint64_t nl = (uint64_t)a.nleaves;
  Emit e{};
  if (OVF) {
    place_m2l(a, e, a.leaf_base + nl * a.slot_m + (uint64_t)a.nbig * a.big_m + a.leaf_m2l_off[l],
              0xffffffffu);
    place_p2p(a, e, nl * a.slot_p + (uint64_t)a.nbig * a.big_p + a.leaf_p2p_off[l], 0xffffffffu);
    e.p2p_total = a.p2p_cnt[v];  // from the first pass
    if (lane == 0) {
      const bool fm = e.m2l_base + a.m2l_cnt[v] <= a.m2l_cap;
      const bool fp = e.p2p_base + e.p2p_total <= a.p2p_cap;
      a.m2l_off[v] = fm ? (uint32_t)e.m2l_base : kNoList;
      a.p2p_off[v] = fp ? (uint32_t)e.p2p_base : kNoList;
    }
    walk_leaf<kLeafExact>(a, v, rv, src, nsrc, root, e, stk, a.status);
    __syncthreads();  // (the stack is reused by the wave's next leaf)
    return;
  }
  place_m2l(a, e, a.leaf_base + (uint64_t)l * a.slot_m, a.slot_m);
  place_p2p(a, e, (uint64_t)l * a.slot_p, a.slot_p);
  e.slot_m = a.slot_m;
  e.slot_p = a.slot_p;
  e.plain = stk + a.stack_cap;
  walk_leaf<kLeafSlot>(a, v, rv, src, nsrc, root, e, stk, a.status);
  uint32_t ns = e.src_lane;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ns += (uint32_t)__shfl_xor((int)ns, o, 64);
  const uint32_t nm = e.m2l_run, np = e.p2p_run, nq = e.plain_run;
  const bool fits = nm <= e.slot_m && np + nq <= e.slot_p;  // uniform
  __syncthreads();  // the staged entries are complete
  if (e.plain_g) __threadfence();  // (staged in global memory by this wave)
  if (fits) {
    // the entries beyond both kernels after the others, in reverse rank
    // order (as the exact pass writes them)
    const uint32_t* pl = e.plain_g ? e.plain_g : e.plain;
    for (uint32_t i = lane; i < nq; i += 64)
      if (np + i < e.room_p) e.p2p[np + i] = pl[nq - 1u - i];
  }
  if (lane == 0) {
    a.m2l_cnt[v] = nm;
    a.p2p_cnt[v] = np + nq;
    a.open_cnt[v] = 0;
    a.open_off[v] = 0;
    if (fits) {
      a.m2l_off[v] = e.m2l_base + nm <= a.m2l_cap ? (uint32_t)e.m2l_base : kNoList;
      a.p2p_off[v] = e.p2p_base + np + nq <= a.p2p_cap ? (uint32_t)e.p2p_base : kNoList;
    } else {
      // (the list of its range of leaves, the range this XCD walks here and
      // walks again in the second pass: its lists' sources stay in its L2)
      const uint32_t seg = ((uint32_t)a.nleaves + kXcds - 1) / kXcds;
      const uint32_t part = (uint32_t)l / seg;
      const unsigned long long k =
          atomicAdd(reinterpret_cast<unsigned long long*>(a.run + 11 + part), 1ull);
      a.ovf_leaf[(uint64_t)part * seg + k] = (uint32_t)l;
    }
    // lists left for the second pass (none when they fit)
    a.leaf_m2l_cnt[l] = fits ? 0u : nm;
    a.leaf_p2p_cnt[l] = fits ? 0u : np + nq;
    // P2P work items of the leaf
    a.src_total[l] = ns;
    const uint32_t len = a.rule.len(vi.lo);
    const uint32_t k = (ns + len - 1) / len;
    a.item_cnt[l] = k > 0 ? k : 1u;
  }
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_nodewalk_leaves(NodeWalkArgs a) {
  extern __shared__ uint32_t stk[];
  const int l = (int)xcd_block(blockIdx.x, gridDim.x);
  if (l < a.nleaves) leaf_lists<false>(a, l, stk);
}

// the second pass: a fixed grid of waves takes the listed leaves in turn
constexpr unsigned kOvfWaves = 4096;

__global__ __launch_bounds__(64) void k_nodewalk_leaves_ovf(NodeWalkArgs a) {
  extern __shared__ uint32_t stk[];
  // block b runs on XCD b % kXcds (the hardware's round-robin) and takes
  // that range's list
  const uint32_t part = blockIdx.x % kXcds, stride = gridDim.x / kXcds;
  const uint32_t seg = ((uint32_t)a.nleaves + kXcds - 1) / kXcds;
  const uint64_t nov = a.run[11 + part];
  for (uint64_t i = blockIdx.x / kXcds; i < nov; i += stride)
    leaf_lists<true>(a, (int)a.ovf_leaf[(uint64_t)part * seg + i], stk);
}

__global__ void k_leaf_stats(LeafStatArgs a) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l >= a.nleaves) return;
  const int leaf = a.leaf_node[l];
  const int d = a.leaf_depth[l];
  const NodeInfo li = a.info[leaf];
  int v = 0;
  uint64_t m2l = a.m2l_cnt[0];
  int kfirst = m2l > 0 ? 0 : -1;
  for (int k = 1; k <= d; ++k) {
    const int c = a.info[v].child;
    v = (li.lo < a.info[c + 1].lo) ? c : c + 1;
    const uint32_t mc = a.m2l_cnt[v];
    if (mc > 0 && kfirst < 0) kfirst = k;
    m2l += mc;
  }
  uint64_t src = 0;
  const uint32_t off = a.p2p_off[leaf], cnt = a.p2p_cnt[leaf];
  for (uint32_t q = 0; q < cnt; ++q) src += (uint64_t)a.info[a.p2p_pool[off + q]].cnt;
  a.m2l[l] = m2l;
  a.l2l[l] = kfirst < 0 ? 0u : (uint64_t)(d - kfirst);
  a.pairs[l] = src * (uint64_t)li.cnt - (uint64_t)li.cnt;
}

// one thread per node: the lists a consumer reads (M2L of every node, P2P
// of every leaf) must lie inside the part of the pools this walk wrote, and
// (check_entries) hold only node ids below nn.  Also the walk's totals:
// run[1] += M2L entries, run[4] += P2P entries, run[6] / run[7] = max with
// the longest M2L / P2P list of a leaf.
template <bool ENTRIES>
__global__ __launch_bounds__(256) void k_check_lists(NodeWalkArgs a, int nn) {
  __shared__ uint64_t red[4][4];
  if (blockIdx.x == 0 && threadIdx.x == 0) *a.items_total = a.item_off[a.nleaves];
  const uint64_t nl = (uint64_t)a.nleaves;
  const uint64_t used_m = a.leaf_base + nl * a.slot_m + (uint64_t)a.nbig * a.big_m + a.run[3];
  const uint64_t used_p = nl * a.slot_p + (uint64_t)a.nbig * a.big_p + a.run[2];
  const uint64_t lim_m = used_m < a.m2l_cap ? used_m : a.m2l_cap;
  const uint64_t lim_p = used_p < a.p2p_cap ? used_p : a.p2p_cap;
  bool bad = false;
  uint64_t sm = 0, sp = 0, xm = 0, xp = 0;
  // (a grid of a few blocks, so that few atomics meet at the totals)
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < nn; v += gridDim.x * blockDim.x) {
    const uint32_t mc = a.m2l_cnt[v];
    sm += mc;
    if (mc > 0) {
      const uint64_t off = a.m2l_off[v];
      if (off + mc > lim_m) bad = true;
      else if (ENTRIES)
        for (uint32_t k = 0; k < mc; ++k) bad |= (a.m2l_pool[off + k] & kSrcMask) >= (uint32_t)nn;
    }
    if (a.info[v].child < 0) {
      const uint32_t pc = a.p2p_cnt[v];
      sp += pc;
      xm = max(xm, (uint64_t)mc);
      xp = max(xp, (uint64_t)pc);
      if (pc > 0) {
        const uint64_t off = a.p2p_off[v];
        if (off + pc > lim_p) bad = true;
        else if (ENTRIES)
          for (uint32_t k = 0; k < pc; ++k) bad |= a.p2p_pool[off + k] >= (uint32_t)nn;
      }
    }
  }
  if (bad) atomicOr(a.status, ST_BADLIST);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sm += __shfl_xor(sm, o, 64);
    sp += __shfl_xor(sp, o, 64);
    xm = max(xm, (uint64_t)__shfl_xor(xm, o, 64));
    xp = max(xp, (uint64_t)__shfl_xor(xp, o, 64));
  }
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { red[0][w] = sm; red[1][w] = sp; red[2][w] = xm; red[3][w] = xp; }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t[4] = {red[0][0], red[1][0], red[2][0], red[3][0]};
    for (int k = 1; k < 4; ++k) {
      t[0] += red[0][k]; t[1] += red[1][k];
      t[2] = max(t[2], red[2][k]); t[3] = max(t[3], red[3][k]);
    }
    auto* run = reinterpret_cast<unsigned long long*>(a.run);
    if (t[0]) atomicAdd(run + 1, (unsigned long long)t[0]);
    if (t[1]) atomicAdd(run + 4, (unsigned long long)t[1]);
    if (t[2]) atomicMax(run + 6, (unsigned long long)t[2]);
    if (t[3]) atomicMax(run + 7, (unsigned long long)t[3]);
  }
}

}  // namespace

void launch_check_lists(const NodeWalkArgs& a, int nn, bool check_entries, hipStream_t s) {
  if (nn <= 0) return;
  const unsigned nb = std::min<unsigned>(128, blocks_for(nn, 256));
  if (check_entries) k_check_lists<true><<<nb, 256, 0, s>>>(a, nn);
  else k_check_lists<false><<<nb, 256, 0, s>>>(a, nn);
}

void launch_leaf_stats(const LeafStatArgs& a, hipStream_t s) {
  if (a.nleaves <= 0) return;
  k_leaf_stats<<<(a.nleaves + 127) / 128, 128, 0, s>>>(a);
}

// levels of at most this many nodes are walked kWalkRun at a time (walk phase at
// 1e5 particles 0.191 ms, with every level by itself 0.210, runs up to 512 nodes
// 0.193; a batch of 24 systems 1.152, 1.175 and 1.154, up to 8192 1.28: idle waves
// then take the place of busy ones; runs of four levels gain nothing more)
constexpr uint32_t kRunMax = 2048;

void launch_nodewalk_levels(const NodeWalkArgs& a, const uint32_t* level_base, int maxdepth,
                            hipStream_t s) {
  auto nodes = [&](int k) {
    return k <= maxdepth ? level_base[2 * k + 1] - level_base[2 * k] : 0u;  // the internal ones
  };
  for (int k = 0; k <= maxdepth && nodes(k) > 0;) {
    uint32_t most = 0;
    for (int r = 0; r < kWalkRun; ++r) most = std::max(most, nodes(k + r));
    if (most <= kRunMax && nodes(k + 1) > 0) {
      k_nodewalk_run<<<nodes(k), 64 * kRunWaves, 0, s>>>(a, k);
      k += kWalkRun;
    } else {
      k_nodewalk_internal<<<nodes(k), 64, 0, s>>>(a, k);
      ++k;
    }
  }
}

void launch_nodewalk_leaves(const NodeWalkArgs& a, uint64_t* scan_tmp, hipStream_t s) {
  if (a.nleaves <= 0) return;
  const size_t lds = a.stack_cap * sizeof(uint32_t);
  k_nodewalk_leaves<<<a.nleaves, 64, lds + a.slot_p * sizeof(uint32_t), s>>>(a);
  ScanJobs jobs{};
  jobs.j[0].in32 = a.leaf_m2l_cnt;
  jobs.j[0].out64 = a.leaf_m2l_off;
  jobs.j[0].total64 = a.run + 3;
  jobs.j[1].in32 = a.leaf_p2p_cnt;
  jobs.j[1].out64 = a.leaf_p2p_off;
  jobs.j[1].total64 = a.run + 2;
  // P2P work items: item_off[nleaves] = their total (read back with the walk's)
  jobs.j[2].in32 = a.item_cnt;
  jobs.j[2].out32 = a.item_off;
  jobs.j[2].total32 = a.item_off + a.nleaves;
  scan_jobs(jobs, 3, a.nleaves, scan_tmp, s);
  const unsigned ng = std::min<unsigned>(kOvfWaves, ((unsigned)a.nleaves + kXcds - 1) / kXcds * kXcds);
  k_nodewalk_leaves_ovf<<<ng, 64, lds, s>>>(a);
}

}  // namespace sfmm
