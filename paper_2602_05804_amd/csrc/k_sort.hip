// k_sort.hip -- stable LSD radix sorts of (64-bit key, 32-bit value) by 8-bit
// digits: the particles by Morton key, the nodes by depth and by list length.
//
// Small inputs (at most kSortSmall): one block keeps keys and values in LDS
// over all passes, and for a single system computes the box and the keys as
// well: one launch for the whole ordering.
//
// Otherwise one launch a pass, with decoupled look-back (Merrill and Garland
// 2016).  The counts of every digit are known before (digits do not change from
// pass to pass), so a block only lacks the counts of the tiles before its own,
// which it takes from the words those publish: a block takes its tile by ticket,
// publishes the tile's digit counts, then walks back over the earlier tiles,
// adding counts until it meets one whose inclusive sums are known, and publishes
// its own.  A tile's block has started before any later tile's (the tickets), and
// it publishes its counts before it waits, so every wait ends.  A word holds flag
// and count together; words are read and written whole, with relaxed atomic
// accesses of agent scope, and nothing else passes between blocks of a launch.
//
// Bound by latency: of the look-back in tiles of 1024 (9 us a pass at 1e5
// particles), of the scattered writes in tiles of 4096 (20 us at 1e6, where 24 B
// a particle in and out take 5 us).  A pass of four launches (counts, a scan in
// two, scatter) took 34 us and 39 us.  The whole ordering of 1e3 particles, keys
// included, takes 25 us in one block (187 us in 36 launches).
#include <algorithm>

#include "morton.h"
#include "sfmm_internal.h"

namespace sfmm {
namespace {

constexpr int ST = 256;  // threads of a pass block
constexpr uint32_t kAgg = 1u << 30, kIncl = 2u << 30, kCount = kAgg - 1u;

__device__ __forceinline__ double wave_min(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// the cube of a block's corners (sh: [6][waves] doubles), the same on every thread
template <int WAVES>
__device__ __forceinline__ void block_box(const double* mn, const double* mx, double (*sh)[WAVES],
                                          double* box) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double a = wave_min(mn[d]), b = wave_max(mx[d]);
    if (lane == 0) { sh[d][w] = a; sh[3 + d][w] = b; }
  }
  __syncthreads();
  double ext = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double lo = sh[d][0], hi = sh[3 + d][0];
    for (int k = 1; k < WAVES; ++k) { lo = fmin(lo, sh[d][k]); hi = fmax(hi, sh[3 + d][k]); }
    box[d] = lo;
    if (hi - lo > ext) ext = hi - lo;
  }
  box[3] = ext;
  box[4] = ext > 0.0 ? 2097152.0 / ext : 0.0;
}

// exclusive sum over the first 256 threads of a block (sh: 4 words); the
// other threads must call it too
__device__ __forceinline__ uint32_t scan256(uint32_t v, uint32_t* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)incl, o, 64);
    if (lane >= o) incl += u;
  }
  if (w < 4 && lane == 63) sh[w] = incl;
  __syncthreads();
  uint32_t pre = 0;
  for (int k = 0; k < 4; ++k)
    if (k < w) pre += sh[k];
  __syncthreads();
  return pre + incl - v;
}

// rank of this lane's element among the wave's valid elements of its digit
// (in lane order) and their number; every lane must take part
__device__ __forceinline__ uint32_t wave_rank(uint32_t d, bool valid, uint32_t& same) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const uint64_t m = __ballot((d >> b) & 1u);
    peers &= ((d >> b) & 1u) ? m : ~m;
  }
  same = (uint32_t)__popcll(peers);
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
}

// adds a wave's elements of one round to its counters; returns each element's
// place among the wave's elements of its digit
__device__ __forceinline__ uint32_t wave_count(uint32_t* cnt, uint32_t d, bool valid) {
  uint32_t same;
  const uint32_t below = wave_rank(d, valid, same);
  const uint32_t old = valid ? cnt[d] : 0u;
  __builtin_amdgcn_wave_barrier();
  if (valid && below == 0) cnt[d] = old + same;
  __builtin_amdgcn_wave_barrier();
  return old + below;
}

// ---- small inputs: one block --------------------------------------------------
constexpr int SB = 1024;                    // threads
constexpr int SI = kSortSmall / SB;         // elements a thread

// BOX: a single system's particles, box and keys computed here (m, h checked
// when check is set); else the keys are read.  The values are the positions.
template <bool BOX>
__global__ __launch_bounds__(SB) void k_sort_small(int n, const double* __restrict__ x,
                                                   const double* __restrict__ m,
                                                   const double* __restrict__ h, int check,
                                                   int* status, const uint64_t* __restrict__ kin,
                                                   int bits, uint64_t* __restrict__ kout,
                                                   uint32_t* __restrict__ vout,
                                                   uint32_t* __restrict__ base) {
  __shared__ uint64_t sk[kSortSmall];
  __shared__ uint16_t sv[kSortSmall];
  __shared__ alignas(8) uint32_t cnt[SB / 64][256];
  __shared__ uint32_t sh4[4];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // a wave takes a run of elements, in rounds of 64
  const int rounds = (n + SB - 1) / SB;
  const int beg = w * rounds * 64 + lane;
  uint64_t k[SI];
  uint32_t v[SI], r[SI];
  if constexpr (BOX) {
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    int bad = 0;
    for (int i = t; i < n; i += SB) {
      for (int d = 0; d < 3; ++d) {
        const double c = x[3 * i + d];
        mn[d] = fmin(mn[d], c);
        mx[d] = fmax(mx[d], c);
        if (check && !isfinite(c)) bad = 1;
      }
      if (check && !(m[i] > 0.0 && h[i] > 0.0 && isfinite(m[i]) && isfinite(h[i]))) bad = 1;
    }
    if (bad) atomicOr(status, ST_NONFINITE);
    double box[5];
    block_box<SB / 64>(mn, mx, reinterpret_cast<double(*)[SB / 64]>(&cnt[0][0]), box);
    for (int i = t; i < n; i += SB) sk[i] = morton(x + 3 * i, box);
  } else {
    for (int i = t; i < n; i += SB) sk[i] = kin[i];
  }
  for (int i = t; i < n; i += SB) sv[i] = (uint16_t)i;
  for (int shift = 0; shift < bits; shift += 8) {
    __syncthreads();
    for (int q = t; q < (SB / 64) * 256; q += SB) (&cnt[0][0])[q] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SI; ++q) {
      if (q >= rounds) break;
      const int i = beg + q * 64;
      const bool ok = i < n;
      k[q] = ok ? sk[i] : 0ull;
      v[q] = ok ? sv[i] : 0u;
      r[q] = wave_count(cnt[w], (uint32_t)(k[q] >> shift) & 255u, ok);
    }
    __syncthreads();
    // each digit's waves in order, then the digits
    uint32_t tot = 0;
    if (t < 256)
      for (int q = 0; q < SB / 64; ++q) {
        const uint32_t c = cnt[q][t];
        cnt[q][t] = tot;
        tot += c;
      }
    const uint32_t pre = scan256(t < 256 ? tot : 0u, sh4);
    if (t < 256) {
      for (int q = 0; q < SB / 64; ++q) cnt[q][t] += pre;
      if (base && shift == 0) base[t] = pre;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SI; ++q) {
      if (q >= rounds) break;
      if (beg + q * 64 < n) {
        const uint32_t p = cnt[w][(uint32_t)(k[q] >> shift) & 255u] + r[q];
        sk[p] = k[q];
        sv[p] = (uint16_t)v[q];
      }
    }
  }
  __syncthreads();
  for (int i = t; i < n; i += SB) {
    kout[i] = sk[i];
    vout[i] = sv[i];
  }
}

// ---- larger inputs --------------------------------------------------------------
__global__ void k_clear_words(size_t n, uint32_t* __restrict__ p, size_t n2,
                              uint32_t* __restrict__ p2) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n + n2;
       i += (size_t)gridDim.x * blockDim.x) {
    if (i < n) p[i] = 0u;
    else p2[i - n] = 0u;
  }
}

// digit counts of NP passes from the first 8 NP bits of the keys
template <int NP>
struct DigitCounts {
  uint32_t c[NP][256];
  __device__ __forceinline__ void clear() {
    for (int q = threadIdx.x; q < NP * 256; q += blockDim.x) (&c[0][0])[q] = 0;
    __syncthreads();
  }
  __device__ __forceinline__ void add(uint64_t k) {
#pragma unroll
    for (int p = 0; p < NP; ++p) atomicAdd(&c[p][(uint32_t)(k >> (8 * p)) & 255u], 1u);
  }
  __device__ __forceinline__ void flush(uint32_t* hist) {
    __syncthreads();
    for (int q = threadIdx.x; q < NP * 256; q += blockDim.x)
      if ((&c[0][0])[q]) atomicAdd(&hist[q], (&c[0][0])[q]);
  }
};

// the box from the blocks' corners, the keys and their digit counts
__global__ __launch_bounds__(ST) void k_keys(int n, const double* __restrict__ x, int nb,
                                             const double* __restrict__ part,
                                             uint64_t* __restrict__ key,
                                             uint32_t* __restrict__ hist) {
  __shared__ DigitCounts<8> dc;
  __shared__ double sh[6][ST / 64];
  double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int b = threadIdx.x; b < nb; b += ST)
    for (int d = 0; d < 3; ++d) {
      mn[d] = fmin(mn[d], part[6 * b + d]);
      mx[d] = fmax(mx[d], part[6 * b + 3 + d]);
    }
  double box[5];
  block_box<ST / 64>(mn, mx, sh, box);
  dc.clear();
  for (int i = blockIdx.x * ST + threadIdx.x; i < n; i += gridDim.x * ST) {
    const double p[3] = {x[3 * (int64_t)i], x[3 * (int64_t)i + 1], x[3 * (int64_t)i + 2]};
    const uint64_t k = morton(p, box);
    key[i] = k;
    dc.add(k);
  }
  dc.flush(hist);
}

template <int NP>
__global__ __launch_bounds__(ST) void k_digit_counts(int n, const uint64_t* __restrict__ key,
                                                     uint32_t* __restrict__ hist) {
  __shared__ DigitCounts<NP> dc;
  dc.clear();
  for (int i = blockIdx.x * ST + threadIdx.x; i < n; i += gridDim.x * ST) dc.add(key[i]);
  dc.flush(hist);
}

// one pass.  vin == nullptr: the values are the positions; base: the digits'
// first places ([256], may be null)
template <int ITEMS>
__global__ __launch_bounds__(ST) void k_sort_pass(int n, const uint64_t* __restrict__ kin,
                                                  const uint32_t* __restrict__ vin,
                                                  uint64_t* __restrict__ kout,
                                                  uint32_t* __restrict__ vout, int shift,
                                                  const uint32_t* __restrict__ hist,
                                                  uint32_t* __restrict__ base,
                                                  uint32_t* ticket, uint32_t* state) {
  constexpr int TILE = ST * ITEMS;
  __shared__ uint64_t sk[TILE];
  __shared__ uint32_t sv[TILE];
  __shared__ uint32_t cnt[ST / 64][256];
  __shared__ uint32_t dbase[256];
  __shared__ uint32_t sh4[4];
  __shared__ uint32_t stile;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t == 0) stile = atomicAdd(ticket, 1u);
#pragma unroll
  for (int q = 0; q < ST / 64; ++q) cnt[q][t] = 0;
  __syncthreads();
  const uint32_t tile = stile;
  const int64_t first = (int64_t)tile * TILE;
  const int here = n - first < TILE ? (int)(n - first) : TILE;  // >= 1
  const int beg = w * ITEMS * 64 + lane;
  uint64_t k[ITEMS];
  uint32_t v[ITEMS], r[ITEMS];
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const int i = beg + q * 64;
    k[q] = i < here ? kin[first + i] : 0ull;
    v[q] = i < here ? (vin ? vin[first + i] : (uint32_t)(first + i)) : 0u;
  }
#pragma unroll
  for (int q = 0; q < ITEMS; ++q)
    r[q] = wave_count(cnt[w], (uint32_t)(k[q] >> shift) & 255u, beg + q * 64 < here);
  __syncthreads();
  // thread t: digit t
  uint32_t tot = 0;
#pragma unroll
  for (int q = 0; q < ST / 64; ++q) {
    const uint32_t c = cnt[q][t];
    cnt[q][t] = tot;
    tot += c;
  }
  uint32_t* mine = state + (size_t)tile * 256 + t;
  __hip_atomic_store(mine, (tile == 0 ? kIncl : kAgg) | tot, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t te = scan256(tot, sh4);          // the tile's elements of smaller digits
  const uint32_t gb = scan256(hist[t], sh4);      // all elements of smaller digits
  if (base && tile == 0) base[t] = gb;
  uint32_t pre = 0;
  if (tile > 0) {
    // eight earlier tiles' words at a time, nearest first
    int p = (int)tile - 1;
    bool done = false;
    while (!done) {
      uint32_t s[8];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        s[q] = p - q >= 0 ? __hip_atomic_load(state + (size_t)(p - q) * 256 + t, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT)
                          : kIncl;
      int adv = 0;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        if (done || adv < q || s[q] < kAgg) continue;  // (a word not yet written ends the batch)
        pre += s[q] & kCount;
        adv = q + 1;
        done = s[q] >= kIncl;
      }
      p -= adv;
    }
    __hip_atomic_store(mine, kIncl | (pre + tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  dbase[t] = gb + pre - te;
#pragma unroll
  for (int q = 0; q < ST / 64; ++q) cnt[q][t] += te;
  __syncthreads();
  // in digit order through LDS, so that a digit's run is written in one piece
#pragma unroll
  for (int q = 0; q < ITEMS; ++q)
    if (beg + q * 64 < here) {
      const uint32_t at = cnt[w][(uint32_t)(k[q] >> shift) & 255u] + r[q];
      sk[at] = k[q];
      sv[at] = v[q];
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    const int i = q * ST + t;
    if (i < here) {
      const uint64_t key = sk[i];
      const uint32_t at = dbase[(uint32_t)(key >> shift) & 255u] + (uint32_t)i;
      kout[at] = key;
      vout[at] = sv[i];
    }
  }
}

// tiles of 1024 elements while they give every CU one at most, else of 4096
// (fewer tiles to look back over, longer runs of a digit to write).  So the
// number of tiles falls by a factor of four past kSmallTiles elements.
constexpr int64_t kSmallTiles = 1 << 18;
int sort_items(int64_t n) { return n <= kSmallTiles ? 4 : 16; }
int64_t sort_tiles(int64_t n) { return (n + ST * sort_items(n) - 1) / (ST * sort_items(n)); }

void pass(int n, const uint64_t* kin, const uint32_t* vin, uint64_t* kout, uint32_t* vout,
          int shift, const uint32_t* hist, uint32_t* base, uint32_t* ticket, uint32_t* state,
          hipStream_t s) {
  const unsigned nb = (unsigned)sort_tiles(n);
  if (sort_items(n) == 4)
    k_sort_pass<4><<<nb, ST, 0, s>>>(n, kin, vin, kout, vout, shift, hist, base, ticket, state);
  else
    k_sort_pass<16><<<nb, ST, 0, s>>>(n, kin, vin, kout, vout, shift, hist, base, ticket, state);
}

unsigned count_blocks(int64_t n) { return (unsigned)std::min<int64_t>((n + 1023) / 1024, 512); }

}  // namespace

// per pass: 256 digit counts, a ticket (padded), the tiles' words
static size_t words_of_tiles(int64_t tiles, int passes) {
  return (size_t)passes * (256 + 64 + 256 * (size_t)tiles);
}
size_t sort_words(int64_t n, int passes) { return words_of_tiles(sort_tiles(n), passes); }
size_t sort_room(int64_t n, int passes) {
  return words_of_tiles(std::max(sort_tiles(n), sort_tiles(std::min(n, kSmallTiles))), passes);
}

void launch_clear_words(uint32_t* p, size_t n, uint32_t* p2, size_t n2, hipStream_t s) {
  if (n + n2 == 0) return;
  k_clear_words<<<(unsigned)std::min<size_t>((n + n2 + 1023) / 1024, 2048), 256, 0, s>>>(n, p, n2,
                                                                                        p2);
}

void launch_keys(int n, const double* x, int nb, const double* part, uint64_t* key,
                 uint32_t* words, hipStream_t s) {
  k_keys<<<count_blocks(n), ST, 0, s>>>(n, x, nb, part, key, words);
}

void launch_small_sort(int n, const double* x, const double* m, const double* h, int check,
                       int* status, uint64_t* key, uint32_t* val, hipStream_t s) {
  k_sort_small<true><<<1, SB, 0, s>>>(n, x, m, h, check, status, nullptr, 64, key, val, nullptr);
}

void radix_sort(int n, int passes, bool counted, uint64_t* key0, uint32_t* val0, uint64_t* key1,
                uint32_t* val1, uint32_t* words, hipStream_t s) {
  if (!counted) {
    if (passes == 8) k_digit_counts<8><<<count_blocks(n), ST, 0, s>>>(n, key0, words);
    else if (passes == 1) k_digit_counts<1><<<count_blocks(n), ST, 0, s>>>(n, key0, words);
    else if (passes == 2) k_digit_counts<2><<<count_blocks(n), ST, 0, s>>>(n, key0, words);
    else if (passes == 3) k_digit_counts<3><<<count_blocks(n), ST, 0, s>>>(n, key0, words);
    else k_digit_counts<4><<<count_blocks(n), ST, 0, s>>>(n, key0, words);
  }
  uint32_t* ticket = words + (size_t)passes * 256;
  uint32_t* state = ticket + (size_t)passes * 64;
  uint64_t *kin = key0, *kout = key1;
  uint32_t *vin = val0, *vout = val1;
  for (int p = 0; p < passes; ++p) {
    pass(n, kin, p == 0 ? nullptr : vin, kout, vout, 8 * p, words + 256 * p, nullptr,
         ticket + 64 * p, state + (size_t)p * 256 * sort_tiles(n), s);
    std::swap(kin, kout);
    std::swap(vin, vout);
  }
}

void radix_pass(int n, bool counted, const uint64_t* kin, const uint32_t* vin, uint64_t* kout,
                uint32_t* vout, uint32_t* base, uint32_t* words, hipStream_t s) {
  if (n <= kSortSmall && !vin) {
    k_sort_small<false><<<1, SB, 0, s>>>(n, nullptr, nullptr, nullptr, 0, nullptr, kin, 8, kout,
                                         vout, base);
    return;
  }
  if (!counted) k_digit_counts<1><<<count_blocks(n), ST, 0, s>>>(n, kin, words);
  pass(n, kin, vin, kout, vout, 0, words, base, words + 256, words + 320, s);
}

}  // namespace sfmm
