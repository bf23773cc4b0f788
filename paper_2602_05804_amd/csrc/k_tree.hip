// k_tree.hip -- tree construction on the GPU.
//
//   bbox                corners of the cubic box (keys: 21-bit cells per axis,
//                       x > y > z interleave)
//   (the radix sorts are in k_sort.hip)
//   binary radix tree   Karras-style parallel build on the sorted keys; equal
//                       keys split on the bits of their sorted positions
//   leaf collapse       a node with <= leaf_size particles is a leaf
//   geometry + moments  leaves sum their particles; internal nodes combine
//                       their two children bottom-up (M2M, Appendix A.1)
//   node size l         largest distance from the centre of mass to a
//                       particle of the node (read of Sect. 3's l_tgt/l_src)
//
// The whole library is compiled with -ffp-contract=off: the centres of mass,
// sizes and the acceptance test below round exactly as written, so every
// node-pair decision matches a CPU evaluation of the same formulas.
#include <algorithm>

#include "morton.h"
#include "sfmm_internal.h"

namespace sfmm {
namespace {

constexpr int BBOX_THREADS = 256;

__device__ __forceinline__ double wave_min(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// per-block min/max of each axis; input validation on the side
__global__ __launch_bounds__(BBOX_THREADS) void k_bbox_partial(int n, const double* __restrict__ x,
                                                               const double* __restrict__ m,
                                                               const double* __restrict__ h,
                                                               double* __restrict__ part,
                                                               int* status, int check) {
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  int bad = 0;
  for (int i = blockIdx.x * BBOX_THREADS + threadIdx.x; i < n; i += gridDim.x * BBOX_THREADS) {
    for (int d = 0; d < 3; ++d) {
      double v = x[3 * (int64_t)i + d];
      mn[d] = fmin(mn[d], v);
      mx[d] = fmax(mx[d], v);
      if (check && !isfinite(v)) bad = 1;
    }
    if (check && !(m[i] > 0.0 && h[i] > 0.0 && isfinite(m[i]) && isfinite(h[i]))) bad = 1;
  }
  if (bad) atomicOr(status, ST_NONFINITE);
  __shared__ double sh[6][BBOX_THREADS / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int d = 0; d < 3; ++d) {
    double a = wave_min(mn[d]), b = wave_max(mx[d]);
    if (lane == 0) { sh[d][w] = a; sh[3 + d][w] = b; }
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    double v = sh[threadIdx.x][0];
    for (int k = 1; k < BBOX_THREADS / 64; ++k)
      v = threadIdx.x < 3 ? fmin(v, sh[threadIdx.x][k]) : fmax(v, sh[threadIdx.x][k]);
    part[6 * blockIdx.x + threadIdx.x] = v;
  }
}

// ---- several systems (forest) -----------------------------------------------
// box of system s: its particles in parts (one block a system took 327 us for
// 24 systems of up to 2e5 particles: a chain of loads), then one wave joins them.
// box[0..2] = min corner, box[3] = cube extent, box[4] = 2^21 / extent (0 if flat)
__global__ __launch_bounds__(256) void k_bbox_sys(const int64_t* __restrict__ off, int parts,
                                                  const double* __restrict__ x,
                                                  const double* __restrict__ m,
                                                  const double* __restrict__ h,
                                                  double* __restrict__ part, int* status,
                                                  int check) {
  const int sidx = blockIdx.x / parts, q = blockIdx.x % parts;
  const int64_t e = off[sidx + 1];
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  int bad = 0;
  for (int64_t i = off[sidx] + q * 256 + threadIdx.x; i < e; i += 256 * parts) {
    for (int d = 0; d < 3; ++d) {
      const double v = x[3 * i + d];
      mn[d] = fmin(mn[d], v);
      mx[d] = fmax(mx[d], v);
      if (check && !isfinite(v)) bad = 1;
    }
    if (check && !(m[i] > 0.0 && h[i] > 0.0 && isfinite(m[i]) && isfinite(h[i]))) bad = 1;
  }
  if (bad) atomicOr(status, ST_NONFINITE);
  __shared__ double sh[6][4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int d = 0; d < 3; ++d) {
    const double a = wave_min(mn[d]), c = wave_max(mx[d]);
    if (lane == 0) { sh[d][w] = a; sh[3 + d][w] = c; }
  }
  __syncthreads();
  const int d = threadIdx.x;
  if (d < 3) part[6 * (int64_t)blockIdx.x + d] = fmin(fmin(sh[d][0], sh[d][1]), fmin(sh[d][2], sh[d][3]));
  else if (d < 6) part[6 * (int64_t)blockIdx.x + d] = fmax(fmax(sh[d][0], sh[d][1]), fmax(sh[d][2], sh[d][3]));
}

__global__ __launch_bounds__(256) void k_bbox_sys_join(int nsys, int parts,
                                                       const double* __restrict__ part,
                                                       double* __restrict__ boxes) {
  const int sidx = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (sidx >= nsys) return;
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int q = lane; q < parts; q += 64)
    for (int d = 0; d < 3; ++d) {
      mn[d] = fmin(mn[d], part[6 * ((int64_t)sidx * parts + q) + d]);
      mx[d] = fmax(mx[d], part[6 * ((int64_t)sidx * parts + q) + 3 + d]);
    }
  double ext = 0.0;
  double* box = boxes + 8 * sidx;
  for (int d = 0; d < 3; ++d) {
    const double lo = wave_min(mn[d]), hi = wave_max(mx[d]);
    if (lane == 0) box[d] = lo;
    if (hi - lo > ext) ext = hi - lo;
  }
  if (lane != 0) return;
  box[3] = ext;
  box[4] = ext > 0.0 ? 2097152.0 / ext : 0.0;
}

__global__ void k_keys_sys(int n, int nsys, const int64_t* __restrict__ off,
                           const double* __restrict__ x, const double* __restrict__ boxes,
                           uint64_t* __restrict__ key, uint32_t* __restrict__ sys) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int lo = 0, hi = nsys - 1;  // last s with off[s] <= i
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  key[i] = morton(x + 3 * (int64_t)i, boxes + 8 * lo);
  sys[i] = (uint32_t)lo;
}

// after the key sort: the system of each key-sorted position, as a sort key
__global__ void k_sys_sortkey(int n, const uint32_t* __restrict__ perm1,
                              const uint32_t* __restrict__ sys, uint64_t* __restrict__ skey) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  skey[i] = sys[perm1[i]];
}

// final order = (system, key, caller index): gather permutation, keys, systems
__global__ void k_sys_final(int n, const uint32_t* __restrict__ q, const uint32_t* __restrict__ perm1,
                            const uint64_t* __restrict__ key1, const uint32_t* __restrict__ sys,
                            uint32_t* __restrict__ perm, uint64_t* __restrict__ key,
                            uint32_t* __restrict__ sys_sorted) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t p = q[i];
  const uint32_t o = perm1[p];
  perm[i] = o;
  key[i] = key1[p];
  sys_sorted[i] = sys[o];
}

__global__ void k_sys_start(int nsys, const int64_t* __restrict__ off, int32_t* __restrict__ start) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < nsys) start[s] = (int32_t)off[s];
}

// 0: the node spans two systems (never walked); 1: the root of a system; 2: other
__global__ void k_node_flags(int nn, const NodeInfo* __restrict__ info,
                             const uint32_t* __restrict__ sys, uint8_t* __restrict__ flag) {
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nn) return;
  const NodeInfo ni = info[v];
  const bool within = !sys || sys[ni.lo] == sys[ni.lo + ni.cnt - 1];
  bool root = ni.parent < 0;
  if (!root && sys) {
    const NodeInfo pi = info[ni.parent];
    root = sys[pi.lo] != sys[pi.lo + pi.cnt - 1];
  }
  flag[v] = !within ? 0 : (root ? 1 : 2);
}

__global__ void k_gather(int n, const uint32_t* __restrict__ perm, const double* __restrict__ x,
                         const double* __restrict__ m, const double* __restrict__ h,
                         double* __restrict__ xs, double* __restrict__ ys,
                         double* __restrict__ zs, double* __restrict__ ms,
                         double* __restrict__ hs, double* __restrict__ his,
                         double* __restrict__ h4, double2* __restrict__ pxy,
                         double2* __restrict__ pzm) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int64_t j = perm[i];
  const double px = x[3 * j], py = x[3 * j + 1], pz = x[3 * j + 2], pm = m[j], ph = h[j];
  const double phi = 1.0 / ph;
  xs[i] = px;
  ys[i] = py;
  zs[i] = pz;
  ms[i] = pm;
  hs[i] = ph;
  his[i] = phi;
  // (at least the smallest normal number: r^2 = 0, a particle with itself, is then
  // below it for every h; pairs that close are evaluated one by one anyway)
  h4[i] = fmax(4.0 * ph * ph, 0x1p-1022);
  pxy[i] = make_double2(px, py);
  pzm[i] = make_double2(pz, pm);
}

// ---- binary radix tree (Karras 2012) ----------------------------------------
// delta = length of the common prefix of the augmented keys
// (system, key, position within the system); sys == nullptr: one system
__device__ __forceinline__ int delta(const uint64_t* __restrict__ k, const uint32_t* __restrict__ sys,
                                     const int32_t* __restrict__ sys_start, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  uint32_t si = 0, sj = 0;
  if (sys) {
    si = sys[i];
    sj = sys[j];
    if (si != sj) return __clz((int)(si ^ sj));
  }
  const uint64_t a = k[i], b = k[j];
  if (a != b) return 32 + __clzll((long long)(a ^ b));
  const int s0 = sys ? sys_start[si] : 0;
  return 96 + __clz((int)((uint32_t)(i - s0) ^ (uint32_t)(j - s0)));
}

// internal node i (0..n-2); child codes: >= 0 internal node, < 0 leaf -(pos+1)
__global__ void k_karras(int n, const uint64_t* __restrict__ key, const uint32_t* __restrict__ sys,
                         const int32_t* __restrict__ sys_start, int leaf_size,
                         int32_t* __restrict__ kfirst, int32_t* __restrict__ klast,
                         int32_t* __restrict__ kleft, int32_t* __restrict__ kright,
                         int32_t* __restrict__ kpar, int32_t* __restrict__ kside,
                         uint32_t* __restrict__ kept) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n - 1) return;
  const int d = (delta(key, sys, sys_start, n, i, i + 1) - delta(key, sys, sys_start, n, i, i - 1)) >= 0 ? 1 : -1;
  const int dmin = delta(key, sys, sys_start, n, i, i - d);
  int lmax = 2;
  while (delta(key, sys, sys_start, n, i, i + lmax * d) > dmin) lmax *= 2;
  int l = 0;
  for (int t = lmax / 2; t >= 1; t /= 2)
    if (delta(key, sys, sys_start, n, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  const int dnode = delta(key, sys, sys_start, n, i, j);
  int s = 0;
  for (int div = 2;; div *= 2) {
    int t = (l + div - 1) / div;
    if (delta(key, sys, sys_start, n, i, i + (s + t) * d) > dnode) s += t;
    if (t <= 1) break;
  }
  const int gamma = i + s * d + (d < 0 ? -1 : 0);
  const int first = min(i, j), last = max(i, j);
  const int left = (first == gamma) ? -(gamma + 1) : gamma;
  const int right = (last == gamma + 1) ? -(gamma + 2) : gamma + 1;
  kfirst[i] = first;
  klast[i] = last;
  kleft[i] = left;
  kright[i] = right;
  if (left >= 0) { kpar[left] = i; kside[left] = 0; }
  if (right >= 0) { kpar[right] = i; kside[right] = 1; }
  // a node over particles of two systems never becomes a leaf
  const bool spans = sys && sys[first] != sys[last];
  kept[i] = ((last - first + 1) > leaf_size || spans) ? 1u : 0u;
  if (i == 0) kpar[0] = -1;
}

// final node ids: root 0; the children of the kept internal node with
// compact index c sit at 1 + 2c (left) and 2 + 2c (right)
__device__ __forceinline__ int final_id(int i, const int32_t* kpar, const int32_t* kside,
                                        const uint32_t* cidx) {
  return i == 0 ? 0 : 1 + 2 * (int)cidx[kpar[i]] + kside[i];
}

__global__ void k_assign(int n, int leaf_size, const uint32_t* __restrict__ sys,
                         const int32_t* __restrict__ kfirst,
                         const int32_t* __restrict__ klast, const int32_t* __restrict__ kleft,
                         const int32_t* __restrict__ kright, const int32_t* __restrict__ kpar,
                         const int32_t* __restrict__ kside, const uint32_t* __restrict__ cidx,
                         NodeInfo* __restrict__ info, uint32_t* __restrict__ leaf_flag,
                         int32_t* __restrict__ leaf_at) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n - 1) return;
  const int first = kfirst[i], last = klast[i];
  const bool spans = sys && sys[first] != sys[last];
  if (last - first + 1 <= leaf_size && !spans) return;  // not a kept internal node
  const int me = final_id(i, kpar, kside, cidx);
  const int par = i == 0 ? -1 : final_id(kpar[i], kpar, kside, cidx);
  const int base = 1 + 2 * (int)cidx[i];
  NodeInfo ni;
  ni.lo = first; ni.cnt = last - first + 1; ni.child = base; ni.parent = par;
  info[me] = ni;
  const int ch[2] = {kleft[i], kright[i]};
  for (int side = 0; side < 2; ++side) {
    int c = ch[side], lo, cnt;
    if (c < 0) { lo = -c - 1; cnt = 1; }
    else { lo = kfirst[c]; cnt = klast[c] - kfirst[c] + 1; }
    const bool child_spans = sys && sys[lo] != sys[lo + cnt - 1];
    if (cnt <= leaf_size && !child_spans) {
      NodeInfo li;
      li.lo = lo; li.cnt = cnt; li.child = -1; li.parent = me;
      info[base + side] = li;
      leaf_flag[lo] = 1u;
      leaf_at[lo] = base + side;
    }
  }
}

// leaves in order, and the leaf of every particle (a leaf begins at each flag)
__global__ void k_leaf_fill(int n, const uint32_t* __restrict__ leaf_flag,
                            const uint32_t* __restrict__ leaf_scan,
                            const int32_t* __restrict__ leaf_at, int32_t* __restrict__ leaf_node,
                            int32_t* __restrict__ p_leaf) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  const uint32_t f = leaf_flag[p], k = leaf_scan[p];
  if (f) leaf_node[k] = leaf_at[p];
  p_leaf[p] = (int32_t)(k + f) - 1;
}

__global__ void k_single_leaf(int n, NodeInfo* info, int32_t* leaf_node, int32_t* p_leaf) {
  NodeInfo ni;
  ni.lo = 0; ni.cnt = n; ni.child = -1; ni.parent = -1;
  info[0] = ni;
  leaf_node[0] = 0;
  for (int p = 0; p < n; ++p) p_leaf[p] = 0;
}

// ---- per node, once the tree's shape is known -----------------------------------
// Depths, the keys of the grouping by depth and their counts; the subtrees and
// the nodes above them for the moments; the chunks of the node sizes.
// (One launch of 8 us at 1e5 particles instead of seven of 34 us: these tables
// are small, the launches were the cost.)

// kept internal nodes in the subtree of an internal node: their numbers follow
// the particles' order, so besides the node itself they are those of the
// binary tree's internal nodes strictly inside its range
__device__ __forceinline__ uint32_t kept_before(const NodeSetupArgs& a, int i) {
  return i < a.n - 1 ? a.kept_scan[i] : a.nkept;
}
__device__ __forceinline__ uint32_t kept_below(const NodeSetupArgs& a, const NodeInfo& ni) {
  return 1u + kept_before(a, ni.lo + ni.cnt - 1) - kept_before(a, ni.lo + 1);
}

constexpr int kSetupThreads = 512;
__global__ __launch_bounds__(kSetupThreads) void k_node_setup(NodeSetupArgs a) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t wsum[2][kSetupThreads / 64];
  __shared__ uint32_t sbase[2];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t < 256) hist[t] = 0;
  __syncthreads();
  const int v = blockIdx.x * kSetupThreads + t;
  NodeInfo ni{0, 0, -1, -1};
  uint32_t nch = 0;
  bool few = false;
  if (v < a.nn) {
    ni = a.info[v];
    int d = 0;
    for (int u = ni.parent; u >= 0; u = a.info[u].parent) ++d;
    a.depth[v] = d;
    // grouped by depth, and within a depth the internal nodes first
    const int k = min(2 * d + (ni.child < 0 ? 1 : 0), 255);
    a.key[v] = (uint64_t)k;
    atomicAdd(&hist[k], 1u);
    if (d > kMaxDepthCap) atomicMax(a.too_deep, d);
    a.l2bits[v] = 0ull;
    if (ni.child < 0) {
      a.leaf_depth[a.p_leaf[ni.lo]] = d;
    } else {
      few = ni.cnt <= kExtentFew;
      nch = few ? 0u : (uint32_t)((ni.cnt + kExtentChunk - 1) / kExtentChunk);
      if (kept_below(a, ni) > a.kmax)
        a.top[atomicAdd(a.ntop, 1u)] = (uint32_t)v | ((uint32_t)d << kSrcBits);
      else if (ni.parent < 0 || kept_below(a, a.info[ni.parent]) > a.kmax)
        a.roots[atomicAdd(a.nroots, 1u)] = (uint32_t)v;
    }
  }
  // places of the chunks and of the nodes of few particles: one addition to
  // each common total per block
  const uint64_t fm = __ballot(few);
  uint32_t incl = nch;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += u;
  }
  if (lane == 63) {
    wsum[0][w] = incl;
    wsum[1][w] = (uint32_t)__popcll(fm);
  }
  __syncthreads();
  if (t < 2) {
    uint32_t tot = 0;
    for (int k = 0; k < kSetupThreads / 64; ++k) {
      const uint32_t c = wsum[t][k];
      wsum[t][k] = tot;
      tot += c;
    }
    sbase[t] = tot ? atomicAdd(t == 0 ? a.nitems : a.nfew, tot) : 0u;
  }
  if (t < 256 && hist[t]) atomicAdd(&a.hist[t], hist[t]);
  __syncthreads();
  if (few)
    a.few[sbase[1] + wsum[1][w] +
          __builtin_amdgcn_mbcnt_hi((uint32_t)(fm >> 32),
                                    __builtin_amdgcn_mbcnt_lo((uint32_t)fm, 0u))] = (uint32_t)v;
  const uint32_t at = sbase[0] + wsum[0][w] + incl - nch;
  if (nch > 0 && nch <= 4)
    for (uint32_t c = 0; c < nch; ++c) a.items[at + c] = make_uint2((uint32_t)v, c);
  // (the chunks of a large node by the whole wave)
  uint64_t big = __ballot(nch > 4);
  while (big) {
    const int l = __ffsll((unsigned long long)big) - 1;
    big &= big - 1;
    const uint32_t bv = (uint32_t)__shfl(v, l, 64), bn = (uint32_t)__shfl((int)nch, l, 64);
    const uint32_t ba = (uint32_t)__shfl((int)at, l, 64);
    for (uint32_t c = lane; c < bn; c += 64) a.items[ba + c] = make_uint2(bv, c);
  }
}

// ---- geometry, moments (bottom-up, one level after the other) --------------
// A leaf sums its particles in sorted order; an internal node combines its
// two children, deeper nodes first.  Three launches: all leaves; subtrees of at
// most kmax internal nodes, a block each, level by level with a barrier
// between levels; the nodes above them in one block, the same way.  Bound by
// the chain of levels (loads of the children's records, a division, the
// shifts of the moments).
// 41 us at 1e3 particles, 51 at 1e5, 153 at 1e6; with a launch for each of the
// larger levels and a run of the smaller ones in one block it was 92, 197, 324.
// a node's moments, and its M2L source record (recq, may be null)
template <int P>
__device__ __forceinline__ void store_moments(int v, const double* r, const double* Q, double* rec,
                                              double* recq) {
  using E = Exp<P>;
  double* o = rec + (int64_t)v * rec_stride(P) + 8;
#pragma unroll
  for (int k = 0; k < E::NQ; ++k) o[k] = Q[k];
  if (recq) {
    double* q = recq + (int64_t)v * recq_stride(P);
    double Qr[E::NQR];
    E::reduce(Q, Qr);
    q[0] = r[0]; q[1] = r[1]; q[2] = r[2];
#pragma unroll
    for (int k = 0; k < E::NQR; ++k) q[3 + k] = Qr[k];
  }
}

// (kGeomLoads particles' loads at a time; the sums in the particles' order)
constexpr int kGeomLoads = 4;
template <int P>
__global__ __launch_bounds__(64) void k_geom_leaves(
    int nleaves, const int32_t* __restrict__ leaf_node, const NodeInfo* __restrict__ info,
    const double* __restrict__ xs, const double* __restrict__ ys, const double* __restrict__ zs,
    const double* __restrict__ ms, const double* __restrict__ hs, double* __restrict__ rec,
    double* __restrict__ recq) {
  using E = Exp<P>;
  const int l = blockIdx.x * 64 + threadIdx.x;
  if (l >= nleaves) return;
  const int v = leaf_node[l];
  const NodeInfo ni = info[v];
  double Q[E::NQ];
#pragma unroll
  for (int k = 0; k < E::NQ; ++k) Q[k] = 0.0;
  const int end = ni.lo + ni.cnt;
  double M = 0.0, S0 = 0.0, S1 = 0.0, S2 = 0.0, hm = 0.0;
  for (int j = ni.lo; j < end; j += kGeomLoads) {
    double m[kGeomLoads], x[kGeomLoads], y[kGeomLoads], z[kGeomLoads], h[kGeomLoads];
#pragma unroll
    for (int u = 0; u < kGeomLoads; ++u) {
      const int i = min(j + u, end - 1);
      m[u] = ms[i]; x[u] = xs[i]; y[u] = ys[i]; z[u] = zs[i]; h[u] = hs[i];
    }
#pragma unroll
    for (int u = 0; u < kGeomLoads; ++u) {
      if (j + u >= end) break;
      M += m[u];
      S0 += m[u] * x[u];
      S1 += m[u] * y[u];
      S2 += m[u] * z[u];
      hm = fmax(hm, h[u]);
    }
  }
  const double s0 = S0 / M, s1 = S1 / M, s2 = S2 / M;
  double d2max = 0.0;
  for (int j = ni.lo; j < end; j += kGeomLoads) {
    double m[kGeomLoads], x[kGeomLoads], y[kGeomLoads], z[kGeomLoads];
#pragma unroll
    for (int u = 0; u < kGeomLoads; ++u) {
      const int i = min(j + u, end - 1);
      m[u] = ms[i]; x[u] = xs[i]; y[u] = ys[i]; z[u] = zs[i];
    }
#pragma unroll
    for (int u = 0; u < kGeomLoads; ++u) {
      if (j + u >= end) break;
      const double b[3] = {x[u] - s0, y[u] - s1, z[u] - s2};
      const double d2 = b[0] * b[0] + b[1] * b[1] + b[2] * b[2];
      d2max = fmax(d2max, d2);
      E::p2m_add(b, m[u], Q);
    }
  }
  double* r = rec + (int64_t)v * rec_stride(P);
  r[0] = s0; r[1] = s1; r[2] = s2; r[3] = sqrt(d2max); r[4] = hm; r[5] = M;
  const double c[3] = {s0, s1, s2};
  store_moments<P>(v, c, Q, rec, recq);
}

template <int P>
__device__ __forceinline__ void geom_internal(int v, int child, double* rec, double* recq) {
  using E = Exp<P>;
  constexpr int NQ = E::NQ;
  constexpr int RS = rec_stride(P);
  double* r = rec + (int64_t)v * RS;
  double Q[NQ];
#pragma unroll
  for (int k = 0; k < NQ; ++k) Q[k] = 0.0;
  const double* rl = rec + (int64_t)child * RS;
  const double* rr = rl + RS;
  const double ML = rl[5], MR = rr[5];
  const double M = ML + MR;
  double s[3];
  for (int d = 0; d < 3; ++d) s[d] = (ML * rl[d] + MR * rr[d]) / M;
  const double hm = fmax(rl[4], rr[4]);
  double Qc[NQ];
  {
    const double g[3] = {rl[0] - s[0], rl[1] - s[1], rl[2] - s[2]};
#pragma unroll
    for (int k = 0; k < NQ; ++k) Qc[k] = rl[8 + k];
    E::m2m_add(g, Qc, Q);
  }
  {
    const double g[3] = {rr[0] - s[0], rr[1] - s[1], rr[2] - s[2]};
#pragma unroll
    for (int k = 0; k < NQ; ++k) Qc[k] = rr[8 + k];
    E::m2m_add(g, Qc, Q);
  }
  r[0] = s[0]; r[1] = s[1]; r[2] = s[2]; r[4] = hm; r[5] = M;
  store_moments<P>(v, s, Q, rec, recq);
}

// the nodes of a list sorted by depth (off[d]: the first of depth d), deepest
// level first; the barrier makes a level's records visible to the block.  A
// thread's next node is read before the barrier
template <int P>
__device__ __forceinline__ void geom_levels(const uint32_t* lst, const uint32_t* off, int dmin,
                                            int dmax, const NodeInfo* __restrict__ info,
                                            double* rec, double* recq) {
  uint32_t idx = off[dmax] + threadIdx.x;
  int v = 0, child = 0;
  if (idx < off[dmax + 1]) {
    v = (int)lst[idx];
    child = info[v].child;
  }
  for (int d = dmax; d >= dmin; --d) {
    const uint32_t end = off[d + 1];
    while (idx < end) {
      geom_internal<P>(v, child, rec, recq);
      idx += blockDim.x;
      if (idx < end) {
        v = (int)lst[idx];
        child = info[v].child;
      }
    }
    if (d > dmin) {
      idx = off[d - 1] + threadIdx.x;
      if (idx < off[d]) {
        v = (int)lst[idx];
        child = info[v].child;
      }
    }
    __syncthreads();
  }
}

// a list of packed nodes (id, depth above it) sorted by depth: lst gets the
// ids, off[0 .. 128] the first of each depth; hist and off: 129 words of LDS
template <typename Raw>
__device__ __forceinline__ void sort_by_depth(uint32_t count, Raw raw, uint32_t* lst,
                                              uint32_t* hist, uint32_t* off, int& dmin,
                                              int& dmax) {
  const uint32_t t = threadIdx.x;
  for (uint32_t q = t; q < 129; q += blockDim.x) hist[q] = 0;
  __syncthreads();
  for (uint32_t q = t; q < count; q += blockDim.x) atomicAdd(&hist[raw(q) >> kSrcBits], 1u);
  __syncthreads();
  if (t < 64) {
    const uint32_t a = hist[2 * t], b = hist[2 * t + 1];
    uint32_t incl = a + b;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
      if ((int)t >= o) incl += u;
    }
    const uint32_t ex = incl - a - b;
    off[2 * t] = ex;
    off[2 * t + 1] = ex + a;
    if (t == 63) off[128] = incl;
    hist[2 * t] = ex;  // the places handed out below
    hist[2 * t + 1] = ex + a;
  }
  __syncthreads();
  for (uint32_t q = t; q < count; q += blockDim.x) {
    const uint32_t p = raw(q);
    lst[atomicAdd(&hist[p >> kSrcBits], 1u)] = p & kSrcMask;
  }
  __syncthreads();
  dmin = 0;
  while (off[dmin + 1] == 0) ++dmin;  // (count > 0)
  dmax = dmin;
  while (dmax < 127 && off[dmax + 1] < count) ++dmax;
}

constexpr int kSubThreads = 256, kTopThreads = 512;
template <int P>
__global__ __launch_bounds__(kSubThreads) void k_geom_subtrees(NodeSetupArgs a, double* rec,
                                                               double* recq) {
  __shared__ uint32_t raw[kGeomMax], lst[kGeomMax];
  __shared__ uint32_t hist[129], off[129];
  const uint32_t nroots = *a.nroots;
  for (uint32_t r = blockIdx.x; r < nroots; r += gridDim.x) {
    const NodeInfo ni = a.info[a.roots[r]];
    const uint32_t c0 = kept_before(a, ni.lo + 1);
    const uint32_t count = min(kept_below(a, ni), (uint32_t)kGeomMax);
    for (uint32_t q = threadIdx.x; q < count; q += kSubThreads) {
      // number c: the children of that internal node are 1 + 2c and 2 + 2c
      const uint32_t child = q == 0 ? (uint32_t)ni.child : 1u + 2u * (c0 + q - 1u);
      const uint32_t v = (uint32_t)a.info[child].parent;
      raw[q] = v | ((uint32_t)a.depth[v] << kSrcBits);
    }
    __syncthreads();
    int dmin, dmax;
    sort_by_depth(count, [&](uint32_t q) { return raw[q]; }, lst, hist, off, dmin, dmax);
    geom_levels<P>(lst, off, dmin, dmax, a.info, rec, recq);
  }
}

template <int P>
__global__ __launch_bounds__(kTopThreads) void k_geom_top(NodeSetupArgs a, double* rec,
                                                          double* recq) {
  __shared__ uint32_t hist[129], off[129];
  const uint32_t count = *a.ntop;
  if (count == 0) return;
  int dmin, dmax;
  sort_by_depth(count, [&](uint32_t q) { return a.top[q]; }, a.top_sorted, hist, off, dmin, dmax);
  geom_levels<P>(a.top_sorted, off, dmin, dmax, a.info, rec, recq);
}

// The largest squared distance of a node's particles to its centre of mass:
// chunks of the larger nodes by a wave each, folded with an integer max on the
// FP64 bits (non-negative doubles order like their bit patterns), then the
// nodes of few particles by 16 lanes each (at 1e6 particles a wave for every
// node took 67 us, 16 lanes for every chunk 100: lanes that wait for the others)
template <int RS>
__global__ __launch_bounds__(256) void k_extent(NodeSetupArgs a, const double* __restrict__ xs,
                                                const double* __restrict__ ys,
                                                const double* __restrict__ zs,
                                                const double* __restrict__ rec) {
  const uint32_t nitems = *a.nitems, nfew = *a.nfew;
  for (uint32_t i = blockIdx.x * 4 + (threadIdx.x >> 6); i < nitems; i += gridDim.x * 4) {
    const int lane = threadIdx.x & 63;
    const uint2 it = a.items[i];
    const NodeInfo ni = a.info[it.x];
    const int beg = ni.lo + (int)it.y * kExtentChunk;
    const int end = min(ni.lo + ni.cnt, beg + kExtentChunk);
    const double* r = rec + (int64_t)it.x * RS;
    const double s0 = r[0], s1 = r[1], s2 = r[2];
    double d2max = 0.0;
    // four loads in flight (the last particle again past the end)
    for (int j = beg; j < end; j += 256) {
      double x[4], y[4], z[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = min(j + 64 * u + lane, end - 1);
        x[u] = xs[k]; y[u] = ys[k]; z[u] = zs[k];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double dx = x[u] - s0, dy = y[u] - s1, dz = z[u] - s2;
        d2max = fmax(d2max, dx * dx + dy * dy + dz * dz);
      }
    }
    d2max = wave_max(d2max);
    if (lane == 0) {
      const auto bits = (unsigned long long)__double_as_longlong(d2max);
      auto* to = reinterpret_cast<unsigned long long*>(a.l2bits) + it.x;
      if (ni.cnt <= kExtentChunk) *to = bits;
      else atomicMax(to, bits);
    }
  }
  for (uint32_t i = blockIdx.x * 16 + (threadIdx.x >> 4); i < nfew; i += gridDim.x * 16) {
    const int lane = threadIdx.x & 15;
    const uint32_t v = a.few[i];
    const NodeInfo ni = a.info[v];
    const int end = ni.lo + ni.cnt;
    const double* r = rec + (int64_t)v * RS;
    const double s0 = r[0], s1 = r[1], s2 = r[2];
    double d2max = 0.0;
#pragma unroll
    for (int u = 0; u < kExtentFew / 16; ++u) {
      const int k = min(ni.lo + 16 * u + lane, end - 1);
      const double dx = xs[k] - s0, dy = ys[k] - s1, dz = zs[k] - s2;
      d2max = fmax(d2max, dx * dx + dy * dy + dz * dz);
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) d2max = fmax(d2max, __shfl_xor(d2max, o, 16));
    if (lane == 0) a.l2bits[v] = (uint64_t)__double_as_longlong(d2max);
  }
}

// sizes of the internal nodes, and what the level walk reads of every node
template <int RS>
__global__ void k_extent_final(int nn, const NodeInfo* __restrict__ info,
                               const unsigned long long* __restrict__ l2bits, double* rec,
                               WalkRec* __restrict__ wrec) {
  int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= nn) return;
  double* r = rec + (int64_t)v * RS;
  const NodeInfo ni = info[v];
  WalkRec w{};
  w.x = r[0]; w.y = r[1]; w.z = r[2]; w.h = r[4];
  if (ni.child < 0) {
    w.l = r[3];
  } else {
    w.l = sqrt(__longlong_as_double((long long)l2bits[v]));
    r[3] = w.l;
  }
  w.child = ni.child;
  w.cnt = ni.cnt;
  wrec[v] = w;
}

}  // namespace

int bbox_blocks(int64_t n) {
  int64_t b = (n + BBOX_THREADS * 8 - 1) / (BBOX_THREADS * 8);
  if (b < 1) b = 1;
  if (b > 512) b = 512;  // (every block of the key kernel reads them all)
  return (int)b;
}

void launch_bbox(int n, const double* x, const double* m, const double* h, double* part,
                 int* status, int check, hipStream_t s) {
  k_bbox_partial<<<bbox_blocks(n), BBOX_THREADS, 0, s>>>(n, x, m, h, part, status, check);
}

// two loads of a thread in the largest system, within 2048 blocks
int bbox_sys_parts(int nsys, const int64_t* off_host) {
  int64_t most = 0;
  for (int k = 0; k < nsys; ++k) most = std::max(most, off_host[k + 1] - off_host[k]);
  return (int)std::max<int64_t>(1, std::min<int64_t>((most + 511) / 512, 2048 / nsys));
}

void launch_sys_keys(int n, int nsys, const int64_t* off, int parts, const double* x,
                     const double* m, const double* h, double* part, double* boxes, int* status,
                     int check, uint64_t* key, uint32_t* sys, int32_t* sys_start, hipStream_t s) {
  k_bbox_sys<<<(unsigned)nsys * parts, 256, 0, s>>>(off, parts, x, m, h, part, status, check);
  k_bbox_sys_join<<<blocks_for(nsys, 4), 256, 0, s>>>(nsys, parts, part, boxes);
  k_keys_sys<<<blocks_for(n, 256), 256, 0, s>>>(n, nsys, off, x, boxes, key, sys);
  k_sys_start<<<blocks_for(nsys, 256), 256, 0, s>>>(nsys, off, sys_start);
}

void launch_sys_sortkey(int n, const uint32_t* perm1, const uint32_t* sys, uint64_t* skey,
                        hipStream_t s) {
  k_sys_sortkey<<<blocks_for(n, 256), 256, 0, s>>>(n, perm1, sys, skey);
}

void launch_sys_final(int n, const uint32_t* q, const uint32_t* perm1, const uint64_t* key1,
                      const uint32_t* sys, uint32_t* perm, uint64_t* key, uint32_t* sys_sorted,
                      hipStream_t s) {
  k_sys_final<<<blocks_for(n, 256), 256, 0, s>>>(n, q, perm1, key1, sys, perm, key, sys_sorted);
}

void launch_node_flags(int nn, const NodeInfo* info, const uint32_t* sys, uint8_t* flag,
                       hipStream_t s) {
  k_node_flags<<<blocks_for(nn, 256), 256, 0, s>>>(nn, info, sys, flag);
}

void launch_gather(int n, const uint32_t* perm, const double* x, const double* m,
                   const double* h, double* xs, double* ys, double* zs, double* ms,
                   double* hs, double* his, double* h4, double2* pxy, double2* pzm,
                   hipStream_t s) {
  k_gather<<<blocks_for(n, 256), 256, 0, s>>>(n, perm, x, m, h, xs, ys, zs, ms, hs, his, h4, pxy,
                                             pzm);
}

void launch_karras(int n, const uint64_t* key, const uint32_t* sys, const int32_t* sys_start,
                   int leaf_size, int32_t* kfirst, int32_t* klast, int32_t* kleft,
                   int32_t* kright, int32_t* kpar, int32_t* kside, uint32_t* kept, hipStream_t s) {
  k_karras<<<blocks_for(n - 1, 256), 256, 0, s>>>(n, key, sys, sys_start, leaf_size, kfirst, klast,
                                                  kleft, kright, kpar, kside, kept);
}

void launch_assign(int n, int leaf_size, const uint32_t* sys, const int32_t* kfirst,
                   const int32_t* klast, const int32_t* kleft, const int32_t* kright,
                   const int32_t* kpar, const int32_t* kside, const uint32_t* cidx, NodeInfo* info,
                   uint32_t* leaf_flag, int32_t* leaf_at, hipStream_t s) {
  k_assign<<<blocks_for(n - 1, 256), 256, 0, s>>>(n, leaf_size, sys, kfirst, klast, kleft, kright,
                                                  kpar, kside, cidx, info, leaf_flag, leaf_at);
}

void launch_leaf_fill(int n, const uint32_t* leaf_flag, const uint32_t* leaf_scan,
                      const int32_t* leaf_at, int32_t* leaf_node, int32_t* p_leaf,
                      hipStream_t s) {
  k_leaf_fill<<<blocks_for(n, 256), 256, 0, s>>>(n, leaf_flag, leaf_scan, leaf_at, leaf_node,
                                                 p_leaf);
}

void launch_single_leaf(int n, NodeInfo* info, int32_t* leaf_node, int32_t* p_leaf,
                        hipStream_t s) {
  k_single_leaf<<<1, 1, 0, s>>>(n, info, leaf_node, p_leaf);
}

// a block's share: 512 nodes (10 levels, two rounds of its threads on the
// deepest), or more so that a level has at most 256 nodes above the subtrees,
// which are one block's work
uint32_t geom_kmax(uint32_t nkept) {
  return std::min<uint32_t>(kGeomMax, std::max<uint32_t>(512, (nkept + 255) / 256));
}

size_t extent_items(int n, uint32_t nkept) {
  return (size_t)nkept + (size_t)n * (kMaxDepthCap + 1) / kExtentChunk + 1;
}

void launch_node_setup(const NodeSetupArgs& a, hipStream_t s) {
  k_node_setup<<<blocks_for(a.nn, kSetupThreads), kSetupThreads, 0, s>>>(a);
}

void launch_geometry(int order, const NodeSetupArgs& a, int nleaves, const int32_t* leaf_node,
                     const double* xs, const double* ys, const double* zs, const double* ms,
                     const double* hs, double* rec, double* recq, hipStream_t s) {
  // (the numbers of subtrees and chunks are known on the device only: grids
  // that fill the chip take them in turn)
  const unsigned nsub = std::min<unsigned>(a.nkept, 1024);
  const unsigned next = (unsigned)std::min<uint32_t>((a.nkept + 3) / 4, 4096);
  switch (order) {
#define GEOM_CASE(P)                                                                             \
  case P:                                                                                        \
    k_geom_leaves<P><<<blocks_for(nleaves, 64), 64, 0, s>>>(nleaves, leaf_node, a.info, xs, ys,  \
                                                            zs, ms, hs, rec, recq);              \
    if (a.nkept > 0) {                                                                           \
      k_geom_subtrees<P><<<nsub, kSubThreads, 0, s>>>(a, rec, recq);                             \
      if (a.nkept > a.kmax) k_geom_top<P><<<1, kTopThreads, 0, s>>>(a, rec, recq);               \
      k_extent<rec_stride(P)><<<next, 256, 0, s>>>(a, xs, ys, zs, rec);                          \
    }                                                                                            \
    break;
    GEOM_CASE(0) GEOM_CASE(1) GEOM_CASE(2) GEOM_CASE(3) GEOM_CASE(4)
#undef GEOM_CASE
  }
}

void launch_extent_final(int order, int nn, const NodeInfo* info,
                         const unsigned long long* l2bits, double* rec, WalkRec* wrec,
                         hipStream_t s) {
  const unsigned nb = blocks_for(nn, 256);
  switch (rec_stride(order)) {
    case 16: k_extent_final<16><<<nb, 256, 0, s>>>(nn, info, l2bits, rec, wrec); break;
    case 24: k_extent_final<24><<<nb, 256, 0, s>>>(nn, info, l2bits, rec, wrec); break;
    case 32: k_extent_final<32><<<nb, 256, 0, s>>>(nn, info, l2bits, rec, wrec); break;
    case 48: k_extent_final<48><<<nb, 256, 0, s>>>(nn, info, l2bits, rec, wrec); break;
  }
}

}  // namespace sfmm
