// k_stack.hip - one pass that serves every LRU capacity at once.
//
// Under LRU a block is resident in a cache of capacity C exactly when its
// stack distance D_i <= C, where D_i is the weight of the block itself plus
// the weight of the distinct other blocks touched since its previous access
// (Mattson et al., "Evaluation techniques for storage hierarchies", IBM
// Systems Journal 1970; with unit weights D_i counts distinct blocks).  The
// paper's tiers use LRU (Section 2.1) and its simulator models the tier
// hierarchy by replay (Section 3.2); the inclusion property lets one pass
// over the trace answer every tier capacity of every configuration.
//
// With p = prev(i) and key_j = prev(j) + 1 (0 for a first access):
//   D_i = w_i + sum_{p < j < i} w_j [key_j <= p]
// (a block touched in (p, i) is counted at its first touch there, the one
// whose own previous access lies before p).  Positions are cut into blocks of
// B (1,024 to 8,192 by the length of the trace); with P = block(p),
// I = block(i):
//   P == I:  D_i = w_i + A(i) - Wloc(p)
//   P <  I:  D_i = w_i + A(i) + E(p) + RQ[I-1][P]
// where, inside one block,
//   A(i)    = sum_{j in block(i), j < i} w_j [key_j < key_i]     (dominance count)
//   Wloc(p) = sum_{j in block(p), j <= p} w_j
//   E(p)    = Cnt_P(p) - Wloc(p) + C(p)
//   Cnt_P(p)= sum_{j in block P} w_j [key_j <= p]
//   C(p)    = sum_{q in block P, q < p} w_q [P < block(next(q)) < block(next(p))]
// A key at most p is either below the block or the link of a q < p of the
// block, so with S(p) = sum_{q in block P, q < p} w_q [block(next(q)) = P]:
//   Cnt_P(p) = (weight of block P - S(end of P)) + S(p),  and
//   C(p) + S(p) = N(p) = sum_{q in block P, q < p} w_q [block(next(q)) < block(next(p))]:
//   E(p)    = (weight of block P - S(end of P)) - Wloc(p) + N(p).
// Across blocks RQ[X][Y] = sum_{X'=Y+1..X} Q[X'][Y] with
//   Q[X][Y] = sum_{j in block X} w_j [key_j <= Y * B]
// stored as a lower triangle.  The two in-block dominance counts come from
// an LDS merge sort that accumulates, for every element of a right-hand run,
// the weight of smaller keys in the left-hand run.
//
// Outputs per (group, bin): the count / weight of accesses whose D falls in
// the bin (bins cut at the batch's capacity values), and the count / weight
// of blocks whose final stack depth (the weight of distinct blocks accessed
// at or after their last access) falls in the bin; cumulative over bins on
// return, so hits(C) is one lookup.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "kv_device.h"
#include "kv_internal.h"

namespace kv {
namespace {

constexpr int kLocItems = 8;            // positions per thread of the in-block sorts
constexpr uint32_t kSentinel = 0xFFFFFFFFu;
constexpr uint32_t kRowChunk = 16384;   // LDS histogram bins per row chunk
constexpr int kRowNT = 1024;            // threads per row of the block matrix
constexpr int kAsmNT = 1024;            // threads per workgroup of the distance binning kernels
constexpr uint32_t kSubs = kAsmNT / 64; // parts of a block, one per wavefront of the assembly
constexpr uint32_t kThrLds = 6144;      // thresholds kept in LDS for binning

__host__ __device__ __forceinline__ uint64_t tri_off(uint64_t x) { return x * (x - 1) / 2; }

// What the pass adds to with atomics, cleared by its first kernel where that
// pays (rows_clear).
struct Zero {
  uint64_t* p[3];
  uint32_t n[3];
};

// ---------------------------------------------------------------------------
// Q rows: Q[X][Y] for Y < X, inclusive prefix over ceil(key / B); the weight of
// the last occurrences in each sixteenth of a block.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kRowNT) void k_sd_rowhist(const uint32_t* __restrict__ key,
                                                    const uint32_t* __restrict__ nxt,
                                                    const uint8_t* __restrict__ w8, uint32_t w0,
                                                    uint64_t n, uint32_t logb, uint32_t row_chunk,
                                                    uint32_t* __restrict__ Q,
                                                    uint32_t* __restrict__ lsum, Zero z) {
  // bin j lives at hp(j), one padding word after every 64: the scan below
  // gives each thread a run of up to kRowChunk / kRowNT bins, which would
  // otherwise put the lanes of a wavefront on a few banks
  __shared__ uint32_t h[kRowChunk + kRowChunk / 64];
  __shared__ uint32_t sh[kRowNT / 64 + 1];
  const auto hp = [](uint32_t j) { return j + (j >> 6); };
  const uint32_t X = blockIdx.x;
  for (int q = 0; q < 3; ++q)
    for (uint32_t j = X * kRowNT + threadIdx.x; j < z.n[q]; j += gridDim.x * kRowNT) z.p[q][j] = 0;
  const uint64_t base = (uint64_t)X << logb;
  const uint32_t nb = (uint32_t)min<uint64_t>(1ull << logb, n - base);
  // a wavefront's 64 positions lie in one sixteenth of the block
  if (threadIdx.x < kSubs) sh[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t j = threadIdx.x; j < (1u << logb); j += kRowNT) {
    uint32_t v = 0;
    if (j < nb && nxt[base + j] == kNone) v = w0 ? w0 : (uint32_t)w8[base + j];
    v = wave_add_dpp(v);
    if (v && lane_id() == 0) atomicAdd(&sh[(j * kSubs) >> logb], v);
  }
  __syncthreads();
  if (threadIdx.x < kSubs) lsum[X * kSubs + threadIdx.x] = sh[threadIdx.x];
  __syncthreads();
  const uint64_t row = tri_off(X);
  for (uint32_t c0 = 0; c0 < X; c0 += row_chunk) {
    const uint32_t width = min(row_chunk, X - c0);
    for (uint32_t j = threadIdx.x; j < width; j += kRowNT) h[hp(j)] = 0;
    __syncthreads();
    uint32_t carry = 0;
    for (uint32_t j = threadIdx.x; j < nb; j += kRowNT) {
      const uint32_t c = (key[base + j] + ((1u << logb) - 1u)) >> logb;
      const uint32_t w = w0 ? w0 : (uint32_t)w8[base + j];
      if (c < c0) carry += w;
      else if (c < c0 + width) atomicAdd(&h[hp(c - c0)], w);
    }
    carry = block_sum<kRowNT>(carry, sh);
    // inclusive scan of h[0, width) in LDS, each thread a contiguous run
    const uint32_t per = (width + kRowNT - 1) / kRowNT;
    const uint32_t a = min(width, threadIdx.x * per), b = min(width, a + per);
    uint32_t run = 0;
    for (uint32_t j = a; j < b; ++j) run += h[hp(j)];
    uint32_t tot;
    uint32_t pre = block_excl_scan<kRowNT>(run, sh, &tot) + carry;
    for (uint32_t j = a; j < b; ++j) {
      pre += h[hp(j)];
      h[hp(j)] = pre;
    }
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < width; j += kRowNT) Q[row + c0 + j] = h[hp(j)];
    __syncthreads();
  }
}

struct SegArgs {
  uint64_t seg[KV_MAX_GROUPS + 1];
  uint32_t partitioned;
};

// Column prefix sums of Q (rows X > Y count), kCols columns per workgroup: each
// row of kCols threads sums a range of rows, then writes the running sums from
// the ranges above (three kernels over chunks of 64 rows left most of the
// chip idle and cost two more launches: 2,256 blocks 35 -> 21 us, 13,277
// blocks 370 -> 410 us, before the launches).  The last workgroup sums
// up the last occurrences instead: lpre[q] before the q-th sixteenth of a
// block, and per segment their weight up to its end (of the whole order when
// shared).
template <uint32_t kCols>
__global__ __launch_bounds__(kRowNT) void k_sd_cols(uint32_t* __restrict__ Q, uint32_t G,
                                                    const uint32_t* __restrict__ lsum,
                                                    uint32_t* __restrict__ lpre,
                                                    uint32_t* __restrict__ segend,
                                                    const uint32_t* __restrict__ nxt,
                                                    const uint8_t* __restrict__ w8, uint64_t n,
                                                    uint32_t logb, SegArgs sa) {
  constexpr uint32_t kW = kRowNT / 64, kRanges = kRowNT / kCols;
  __shared__ uint32_t part[kRanges][kCols];
  const uint32_t lane = lane_id(), w = (uint32_t)wave_id();
  if (blockIdx.x + 1 == gridDim.x) {
    uint32_t run = 0;
    const uint32_t m = G * kSubs;
    for (uint32_t b = 0; b < m; b += kRowNT * 4) {  // four per thread (m is a multiple of four)
      const uint32_t q = b + threadIdx.x * 4;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (q < m) v = *reinterpret_cast<const uint4*>(lsum + q);
      uint32_t tot;
      const uint32_t pre =
          run + block_excl_scan_u32<kRowNT>(v.x + v.y + v.z + v.w, &part[0][0], tot);
      if (q < m)
        *reinterpret_cast<uint4*>(lpre + q) =
            make_uint4(pre, pre + v.x, pre + v.x + v.y, pre + v.x + v.y + v.z);
      run += tot;
    }
    __syncthreads();
    static_assert(kW >= KV_MAX_GROUPS, "a wavefront per segment");
    if (w < KV_MAX_GROUPS) {
      const uint64_t e = sa.partitioned ? sa.seg[w + 1] : n, s0 = sa.partitioned ? sa.seg[w] : 0;
      uint32_t v = 0;
      if (e > s0) {
        const uint64_t X = (e - 1) >> logb;
        for (uint64_t i = (X << logb) + lane; i < e; i += 64)
          if (nxt[i] == kNone) v += w8[i];
        v = wave_sum(v) + lpre[X * kSubs];
      }
      if (lane == 0) segend[w] = v;
    }
    return;
  }
  const uint32_t c = threadIdx.x % kCols, r = threadIdx.x / kCols;
  const uint32_t Y0 = blockIdx.x * kCols, Y = Y0 + c;
  const uint32_t per = (G - 1 - Y0 + kRanges - 1) / kRanges;  // rows Y0 + 1 .. G - 1
  const uint32_t x0 = Y0 + 1 + r * per, x1 = min(G, x0 + per);
  constexpr int kU = 8;  // loads in flight
  uint32_t s = 0;
  for (uint32_t X = x0; X < x1; X += kU) {
    uint32_t v[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) v[q] = X + q < x1 && X + q > Y ? Q[tri_off(X + q) + Y] : 0u;
#pragma unroll
    for (int q = 0; q < kU; ++q) s += v[q];
  }
  part[r][c] = s;
  __syncthreads();
  // exclusive sums over the ranges: a wavefront per column
  static_assert(kRanges <= 64, "a wavefront scans a column");
  for (uint32_t q = w; q < kCols; q += kW) {
    const uint32_t v = lane < kRanges ? part[lane][q] : 0u;
    const uint32_t inc = wave_incl_scan_u32(v);
    if (lane < kRanges) part[lane][q] = inc - v;
  }
  __syncthreads();
  uint32_t run = part[r][c];
  for (uint32_t X = x0; X < x1; X += kU) {
    uint32_t v[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) v[q] = X + q < x1 && X + q > Y ? Q[tri_off(X + q) + Y] : 0u;
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      run += v[q];
      if (X + q < x1 && X + q > Y) Q[tri_off(X + q) + Y] = run;
    }
  }
}

// ---------------------------------------------------------------------------
// In-block dominance by LDS merge sort.
// ---------------------------------------------------------------------------
// Element i of a block-wide LDS array lives at pd(i): one padding word after
// every 16, so that the 8-element runs of the threads of a wavefront (and
// the merge positions inside them) fall into different banks.
__host__ __device__ constexpr uint32_t pd(uint32_t i) { return i + (i >> 4); }

// The sorts' LDS.  Per element its key and
//   one weight (kUni):  tag = count of smaller keys at earlier positions << 13 | position
//   mixed weights:      tag = position, acc = weight of smaller keys at earlier positions,
//                       pw  = inclusive prefix weight inside the element's run
// With one weight a run's prefix weight is the index in the run, so half the
// words move per merge and two workgroups of 8,192 fit a compute unit.
template <int kLogB, bool kUni>
struct SortLds {
  using Tag = std::conditional_t<kUni, uint32_t, uint16_t>;
  static constexpr uint32_t kPad = pd(1u << kLogB);
  uint32_t v[kPad];
  Tag tag[kPad];
  uint32_t acc[kUni ? 1 : kPad];
  uint32_t pw[kUni ? 1 : kPad];
};

template <int N, bool kUni>
__device__ __forceinline__ void cswap(uint32_t (&v)[N], uint32_t (&w)[N], uint32_t (&a)[N],
                                      uint32_t (&x)[N], int i, int l, bool up) {
  const bool sw = (v[i] > v[l]) == up;
  if (sw) {
    uint32_t t;
    t = v[i]; v[i] = v[l]; v[l] = t;
    t = x[i]; x[i] = x[l]; x[l] = t;
    if (!kUni) {
      t = w[i]; w[i] = w[l]; w[l] = t;
      t = a[i]; a[i] = a[l]; a[l] = t;
    }
  }
}

// LDS exchange among the lanes of one wavefront: its LDS operations execute
// in issue order, so a compiler fence at wavefront scope suffices.
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// On return S holds the block's elements sorted by v, each with its position
// and the weight (kUni: number) of smaller keys at earlier positions - exact
// whenever v is unique in the block, i.e. for every element that uses it.
template <int kLogB, bool kUni>
__device__ void block_sort_dominance(SortLds<kLogB, kUni>& S, const uint32_t (&vin)[kLocItems],
                                     const uint32_t (&win)[kLocItems]) {
  constexpr uint32_t kB = 1u << kLogB;
  const uint32_t t = threadIdx.x;
  uint32_t v[kLocItems], w[kLocItems], a[kLocItems], x[kLocItems];
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    v[e] = vin[e];
    w[e] = win[e];
    uint32_t s = 0;
#pragma unroll
    for (int f = 0; f < e; ++f) s += (vin[f] < vin[e]) ? (kUni ? 1u : win[f]) : 0u;
    a[e] = s;
    x[e] = t * kLocItems + e;
    if (kUni) x[e] |= s << 13;
  }
  // bitonic network on the thread's register-resident elements
#pragma unroll
  for (int k = 2; k <= kLocItems; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
#pragma unroll
      for (int i = 0; i < kLocItems; ++i) {
        const int l = i ^ j;
        if (l > i) cswap<kLocItems, kUni>(v, w, a, x, i, l, (i & k) == 0);
      }
    }
  }
  uint32_t run = 0;
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    const uint32_t s = pd(t * kLocItems + e);
    S.v[s] = v[e];
    S.tag[s] = (typename SortLds<kLogB, kUni>::Tag)x[e];
    if (!kUni) {
      run += w[e];
      S.pw[s] = run;
      S.acc[s] = a[e];
    }
  }
  uint32_t pw[kLocItems];
  for (uint32_t s = kLocItems; s < kB; s <<= 1) {
    // a pair of runs of s spans 2s / kLocItems threads: up to 64, one wavefront
    const bool in_wave = 2 * s <= 64u * kLocItems;
    if (in_wave) wave_sync_lds(); else __syncthreads();
    const uint32_t o0 = t * kLocItems;
    const uint32_t pair = o0 & ~(2 * s - 1);
    const uint32_t d0 = o0 - pair;
    const uint32_t Lb = pair, Rb = pair + s;
    uint32_t lo = d0 > s ? d0 - s : 0u, hi = min(d0, s);
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (S.v[pd(Lb + mid)] <= S.v[pd(Rb + d0 - mid - 1)]) lo = mid + 1; else hi = mid;
    }
    uint32_t ia = lo, ib = d0 - lo;
    if constexpr (kUni) {
      uint32_t vl = S.v[pd(Lb + min(ia, s - 1))], vr = S.v[pd(Rb + min(ib, s - 1))];
#pragma unroll
      for (int e = 0; e < kLocItems; ++e) {
        const bool takeL = (ib >= s) || (ia < s && vl <= vr);
        v[e] = takeL ? vl : vr;
        x[e] = S.tag[pd(takeL ? Lb + ia : Rb + ib)] + (takeL ? 0u : ia << 13);
        ia += takeL ? 1u : 0u;
        ib += takeL ? 0u : 1u;
        const uint32_t nv = S.v[pd(takeL ? Lb + min(ia, s - 1) : Rb + min(ib, s - 1))];
        vl = takeL ? nv : vl;
        vr = takeL ? vr : nv;
      }
    } else {
#pragma unroll
      for (int e = 0; e < kLocItems; ++e) {
        const uint32_t li = pd(Lb + ia), ri = pd(Rb + ib);
        const bool takeL = (ib >= s) || (ia < s && S.v[li] <= S.v[ri]);
        if (takeL) {
          v[e] = S.v[li];
          a[e] = S.acc[li];
          x[e] = S.tag[li];
          pw[e] = S.pw[li] + (ib ? S.pw[pd(Rb + ib - 1)] : 0u);
          ++ia;
        } else {
          const uint32_t pl = ia ? S.pw[pd(Lb + ia - 1)] : 0u;
          v[e] = S.v[ri];
          a[e] = S.acc[ri] + pl;
          x[e] = S.tag[ri];
          pw[e] = pl + S.pw[ri];
          ++ib;
        }
      }
    }
    if (in_wave) wave_sync_lds(); else __syncthreads();
#pragma unroll
    for (int e = 0; e < kLocItems; ++e) {
      const uint32_t o = pd(o0 + e);
      S.v[o] = v[e];
      S.tag[o] = (typename SortLds<kLogB, kUni>::Tag)x[e];
      if (!kUni) {
        S.acc[o] = a[e];
        S.pw[o] = pw[e];
      }
    }
  }
  __syncthreads();
}

// Per position block: A(i) and same-block distances -> partial[i]; E(p) for
// positions whose next access lies in a later block.  Bound by the LDS
// traffic and latency of the two merge sorts: with one weight an element
// moves two words per merge level instead of four, and two workgroups of
// 8,192 share a compute unit (1.09e8 accesses, blocks of 8,192: 6.7 -> 2.7
// ms; E(p) needs no search, see the top of the file).
// w0: the weight of every access (kUni).
template <int kLogB, bool kUni>
__global__ __launch_bounds__((1 << kLogB) / kLocItems, kUni ? 8 : 1) void k_sd_local(
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ nxt,
    const uint8_t* __restrict__ w8, uint32_t w0, uint64_t n, uint32_t G,
    uint32_t* __restrict__ partial, uint32_t* __restrict__ E) {
  constexpr uint32_t kB = 1u << kLogB;
  constexpr int kNT = kB / kLocItems;
  __shared__ SortLds<kLogB, kUni> S;
  __shared__ uint32_t P[kUni ? 1 : pd(kB)];  // Wloc, position order (kUni: (position + 1) w0)
  __shared__ uint32_t sh[kNT / 64 + 1];
  const uint32_t X = blockIdx.x;
  const uint64_t base = (uint64_t)X << kLogB;
  const uint32_t nb = (uint32_t)min<uint64_t>(kB, n - base);
  const uint32_t t = threadIdx.x;
  uint32_t* nextw;  // the next links, staged before the sorts
  if constexpr (kUni) nextw = S.tag;
  else nextw = S.acc;
  for (uint32_t j = t; j < kB; j += kNT) {
    const bool in = j < nb;
    S.v[pd(j)] = in ? key[base + j] : kSentinel;
    nextw[pd(j)] = in ? nxt[base + j] : kNone;
    if (!kUni) S.pw[pd(j)] = in ? (uint32_t)w8[base + j] : 0u;
  }
  __syncthreads();
  uint32_t k[kLocItems], nx[kLocItems], w[kLocItems];
  uint32_t run = 0, same = 0;  // weight (kUni: number) of positions, and of those with next here
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    const uint32_t j = pd(t * kLocItems + e);
    k[e] = S.v[j];
    nx[e] = nextw[j];
    w[e] = kUni ? (t * kLocItems + e < nb ? 1u : 0u) : S.pw[j];
    run += w[e];
    same += nx[e] != kNone && (nx[e] >> kLogB) == X ? w[e] : 0u;
  }
  const uint32_t below = block_sum<kNT>(run - same, sh);  // weight of keys below the block
  if constexpr (!kUni) {
    uint32_t tot;
    uint32_t wl = block_excl_scan<kNT>(run, sh, &tot);
#pragma unroll
    for (int e = 0; e < kLocItems; ++e) {
      wl += w[e];
      P[pd(t * kLocItems + e)] = wl;
    }
  }
  __syncthreads();
  // The result of sorted element s goes back to its position's slot, so that
  // it leaves the block in position order; `mine` says which slots hold one.
  uint32_t out[kLocItems], at[kLocItems];
  const auto put = [&](uint32_t* __restrict__ dst, const bool (&mine)[kLocItems]) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kLocItems; ++e) S.v[pd(at[e])] = out[e];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kLocItems; ++e) out[e] = S.v[pd(t * kLocItems + e)];
    const uint64_t p = base + t * kLocItems;
    if (mine[0] && mine[1] && mine[2] && mine[3])
      *reinterpret_cast<uint4*>(dst + p) = make_uint4(out[0], out[1], out[2], out[3]);
    else
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (mine[e]) dst[p + e] = out[e];
    if (mine[4] && mine[5] && mine[6] && mine[7])
      *reinterpret_cast<uint4*>(dst + p + 4) = make_uint4(out[4], out[5], out[6], out[7]);
    else
#pragma unroll
      for (int e = 4; e < kLocItems; ++e)
        if (mine[e]) dst[p + e] = out[e];
    __syncthreads();
  };
  // ---- sort 1: keys -> A(i)
  block_sort_dominance<kLogB, kUni>(S, k, w);
  bool mine[kLocItems];
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    const uint32_t s = t * kLocItems + e, sp = pd(s);
    const uint32_t kk = S.v[sp], tag = S.tag[sp];
    const uint32_t i = tag & (kB - 1);
    at[e] = i;
    mine[e] = s < nb && k[e] != 0u;
    uint32_t d = 0;
    if (kk != 0u) {
      const bool here = (uint64_t)kk > base && kk != kSentinel;  // p = kk - 1 lies in the block
      if (kUni) {
        d = (1u + (tag >> 13) - (here ? (uint32_t)(kk - base) : 0u)) * w0;
      } else {
        d = S.pw[sp] - (s ? S.pw[pd(s - 1)] : 0u) + S.acc[sp];
        if (here) d -= P[pd((uint32_t)(kk - 1 - base))];
      }
    }
    out[e] = d;
  }
  put(partial, mine);
  // ---- sort 2: (block of next access, reversed position) -> N(p)
  uint32_t v2[kLocItems];
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    const uint32_t lp = t * kLocItems + e;
    const uint32_t nbk = (nx[e] == kNone) ? G : (nx[e] >> kLogB);
    v2[e] = (lp < nb) ? ((nbk << kLogB) | (kB - 1u - lp)) : kSentinel;
    mine[e] = lp < nb && nx[e] != kNone && (nx[e] >> kLogB) > X;
  }
  block_sort_dominance<kLogB, kUni>(S, v2, w);
#pragma unroll
  for (int e = 0; e < kLocItems; ++e) {
    const uint32_t sp = pd(t * kLocItems + e), tag = S.tag[sp];
    const uint32_t i = tag & (kB - 1);
    at[e] = i;
    out[e] = kUni ? (below - (i + 1) + (tag >> 13)) * w0 : below - P[pd(i)] + S.acc[sp];
  }
  put(E, mine);
}

// ---------------------------------------------------------------------------
// Assembly of cross-block distances and binning.
// ---------------------------------------------------------------------------
struct BinArgs {
  const uint32_t* thr;   // thresholds of all groups, concatenated
  const uint32_t* off;   // [n_groups + 1]
  uint32_t n_thr, n_groups;
  uint64_t* hist;        // u64[bins][4]
};

// Disk TTL tiers.  A bounded TTL tier (capacity C, TTL t, least recently
// accessed block displaced first) holds a block at access i iff D_i <= C and
// its gap delta_i <= t: the blocks it holds are the top of the LRU stack up
// to C, minus those not accessed for t, and with one TTL the latter are a
// bottom part of the stack (ages grow with depth).  An unbounded one is
// C = infinity.  So per group one joint histogram of (D bin, gap bin) serves
// every (capacity, TTL), and one of (final depth bin, end-age bin) gives the
// blocks held at the last request.
constexpr uint64_t kAsmLds = 150 * 1024;  // most LDS of the assembly's tables

struct AsmArgs {
  const uint32_t *key, *nxt;
  const uint8_t *w8, *g8, *real;
  uint64_t n;
  uint32_t w0;          // every access's weight, or 0
  uint32_t logb, G;
  const uint32_t *partial, *E, *RQ;
  uint32_t* dout;       // distances, or null
  const uint32_t *lpre, *segend;
  uint32_t partitioned;
  const uint32_t* req;  // joint histograms
  const double* rt;
};

// Number of values below x in sorted a[lo, lo + len), the same steps for every
// lane: several searches of a thread run side by side.
template <int R, class T>
__device__ __forceinline__ void count_below(const T* a, const uint32_t (&lo)[R],
                                            const uint32_t (&len)[R], uint32_t longest,
                                            const T (&x)[R], uint32_t (&at)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) at[r] = 0;
  uint32_t h = 1;
  while (h <= longest / 2) h *= 2;  // largest power of two <= longest (1 if none)
  for (; h; h >>= 1) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t t = at[r] + h;
      if (t <= len[r] && a[lo[r] + t - 1] < x[r]) at[r] = t;
    }
  }
}

// Assembles the distances and bins them, and the final depths of the blocks
// (the weight of distinct blocks whose last access is at or after their own,
// inside their segment) at their last accesses; with kJoint both also by gap
// and by age.  One pass over the positions: a thread takes R = B / 1,024 of
// them, whose chains of gathers and threshold searches run side by side.
// The histograms add up in LDS (kLds; the joint ones kJoint = 1; else, and
// kJoint = 2, in device memory), each flushed once per workgroup.  Bound by
// the latency of the gathers.  Against separate kernels for the assembly, the
// last-occurrence weights, their scan and the final depths: 4.6e6 accesses
// 102 -> 45 us, 3.9e8 of mixed weights 9.6 -> 8.5 ms.
template <int R, bool kLds, int kJoint>
__global__ __launch_bounds__(kAsmNT) void k_sd_assemble(AsmArgs a, BinArgs ba, JointArgs ja) {
  extern __shared__ double lds[];
  __shared__ uint32_t soff[KV_MAX_GROUPS + 1], stoff[KV_MAX_GROUPS + 1], sjb[KV_MAX_GROUPS + 1];
  __shared__ uint32_t send[KV_MAX_GROUPS];
  const uint32_t ng = ba.n_groups, nbins = ba.n_thr + ng;
  const uint32_t ntb = kJoint ? ja.n_tthr + ng : 0u;
  // doubles first: TTL values, weighted gaps; then thresholds and histograms
  double* stt = lds;
  double* swd = stt + (kJoint == 1 ? ja.n_tthr : 0u);
  uint32_t* sthr = reinterpret_cast<uint32_t*>(swd + (kJoint == 1 ? ntb : 0u));
  uint32_t* hist = sthr + (kLds ? ba.n_thr : 0u);  // [4][nbins], then [4][n_joint]
  uint32_t* joint = hist + (kLds ? 4 * nbins : 0u);
  if (threadIdx.x <= ng) {
    soff[threadIdx.x] = ba.off[threadIdx.x];
    stoff[threadIdx.x] = kJoint ? ja.toff[threadIdx.x] : 0u;
    sjb[threadIdx.x] = kJoint ? ja.jbase[threadIdx.x] : 0u;
  }
  if (threadIdx.x < KV_MAX_GROUPS) send[threadIdx.x] = a.segend[a.partitioned ? threadIdx.x : 0u];
  if (kLds) {
    for (uint32_t j = threadIdx.x; j < ba.n_thr; j += kAsmNT) sthr[j] = ba.thr[j];
    for (uint32_t j = threadIdx.x; j < 4 * nbins; j += kAsmNT) hist[j] = 0;
    if (kJoint == 1) {
      for (uint32_t j = threadIdx.x; j < ja.n_tthr; j += kAsmNT) stt[j] = ja.tthr[j];
      for (uint32_t j = threadIdx.x; j < ntb; j += kAsmNT) swd[j] = 0.0;
      for (uint32_t j = threadIdx.x; j < 4 * ja.n_joint; j += kAsmNT) joint[j] = 0;
    }
  }
  __syncthreads();
  const uint32_t* thr = kLds ? sthr : ba.thr;
  const double* tthr = kJoint == 1 ? stt : ja.tthr;
  uint32_t longest = 0, tlongest = 0;
  for (uint32_t g = 0; g < ng; ++g) {
    longest = max(longest, soff[g + 1] - soff[g]);
    tlongest = max(tlongest, stoff[g + 1] - stoff[g]);
  }
  const double t_end = kJoint ? a.rt[a.req[a.n - 1]] : 0.0;  // the last access's request
  // field f (0 / 1: accesses, their weight; 2 / 3: blocks, theirs) of a bin
  const auto add = [&](uint32_t bin, uint32_t f, uint32_t w) {
    if (kLds) {
      atomicAdd(&hist[f * nbins + bin], 1u);
      if (!a.w0) atomicAdd(&hist[(f + 1) * nbins + bin], w);
    } else {
      atomicAdd((unsigned long long*)&ba.hist[bin * 4 + f], 1ull);
      atomicAdd((unsigned long long*)&ba.hist[bin * 4 + f + 1], (unsigned long long)w);
    }
  };
  const auto add_joint = [&](uint32_t bin, uint32_t f, uint32_t w) {
    if (kJoint == 1) {
      atomicAdd(&joint[f * ja.n_joint + bin], 1u);
      if (!a.w0) atomicAdd(&joint[(f + 1) * ja.n_joint + bin], w);
    } else {
      uint64_t* h = f ? ja.fh : ja.jh;
      atomicAdd((unsigned long long*)&h[2 * (uint64_t)bin], 1ull);
      atomicAdd((unsigned long long*)&h[2 * (uint64_t)bin + 1], (unsigned long long)w);
    }
  };
  const uint32_t wv = (uint32_t)wave_id(), lane = lane_id();
  for (uint32_t X = blockIdx.x; X < a.G; X += gridDim.x) {
    const uint64_t i0 = ((uint64_t)X << a.logb) + wv * (64 * R) + lane;
    const uint64_t end = min<uint64_t>(a.n, (uint64_t)(X + 1) << a.logb);
    uint32_t k[R], w[R], g[R], lo[R], len[R], dep[R], d[R], at[R];
    bool in[R], fin[R], hit[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint64_t i = i0 + r * 64;
      in[r] = i < end;
      const uint64_t q = in[r] ? i : 0;
      k[r] = a.key[q];
      fin[r] = in[r] && a.nxt[q] == kNone;
      w[r] = a.w0 ? a.w0 : (uint32_t)a.w8[q];
      g[r] = ng > 1 ? (uint32_t)a.g8[q] : 0u;
      hit[r] = in[r] && k[r] != 0u && !(a.real && !a.real[q]);  // a re-touch is not binned
      d[r] = hit[r] ? a.partial[q] : 0u;
    }
    // the rest of the distances
    const uint64_t row = X >= 2 ? tri_off(X - 1) : 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t p = k[r] - 1u, Pb = p >> a.logb;
      if (hit[r] && Pb < X) {
        d[r] += a.E[p];
        if (Pb + 1 < X) d[r] += a.RQ[row + Pb];
      }
    }
    // weight of the last occurrences before each position
    uint32_t tot = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t v = fin[r] ? w[r] : 0u, inc = wave_incl_scan_u32(v);
      dep[r] = tot + inc - v;
      tot += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    const uint32_t below = a.lpre[X * kSubs + wv];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      dep[r] = send[a.partitioned ? g[r] : 0u] - (below + dep[r]);
      lo[r] = soff[g[r]];
      len[r] = soff[g[r] + 1] - lo[r];
      if (a.dout && in[r]) a.dout[i0 + r * 64] = k[r] ? d[r] : kNone;
    }
    uint32_t db[R], fb[R];
    count_below<R>(thr, lo, len, longest, d, db);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (hit[r]) add(lo[r] + g[r] + db[r], 0, w[r]);
    bool any = false;
#pragma unroll
    for (int r = 0; r < R; ++r) any |= fin[r];
    any = __ballot(any) != 0ull;
    if (any) {
      count_below<R>(thr, lo, len, longest, dep, fb);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (fin[r]) add(lo[r] + g[r] + fb[r], 2, w[r]);
    }
    if constexpr (kJoint != 0) {
      double gap[R], age[R];
      uint32_t tlo[R], tlen[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint64_t q = in[r] ? i0 + r * 64 : 0;
        const double t = a.rt[a.req[q]];
        gap[r] = hit[r] ? t - a.rt[a.req[k[r] - 1u]] : 0.0;
        age[r] = t_end - t;
        tlo[r] = stoff[g[r]];
        tlen[r] = stoff[g[r] + 1] - tlo[r];
      }
      count_below<R>(tthr, tlo, tlen, tlongest, gap, at);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (!in[r]) continue;
        // a first access: past every threshold and every TTL
        const uint32_t b = hit[r] ? db[r] : len[r], t = hit[r] ? at[r] : tlen[r];
        add_joint(sjb[g[r]] + b * (tlen[r] + 1) + t, 0, w[r]);
        if (hit[r])
          atomicAdd((kJoint == 1 ? swd : ja.wd) + tlo[r] + g[r] + t, (double)w[r] * gap[r]);
      }
      if (any) {
        count_below<R>(tthr, tlo, tlen, tlongest, age, at);
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (fin[r]) add_joint(sjb[g[r]] + fb[r] * (tlen[r] + 1) + at[r], 2, w[r]);
      }
    }
  }
  if (!kLds) return;
  __syncthreads();
  // with one weight the counts give the weights
  for (uint32_t j = threadIdx.x; j < 2 * nbins; j += kAsmNT) {
    const uint32_t f = j < nbins ? 0u : 2u, b = j < nbins ? j : j - nbins;
    const uint32_t c = hist[f * nbins + b];
    if (!c) continue;
    const unsigned long long cw = a.w0 ? (unsigned long long)c * a.w0 : hist[(f + 1) * nbins + b];
    atomicAdd((unsigned long long*)&ba.hist[b * 4 + f], (unsigned long long)c);
    atomicAdd((unsigned long long*)&ba.hist[b * 4 + f + 1], cw);
  }
  if constexpr (kJoint == 1) {
    for (uint32_t j = threadIdx.x; j < 2 * ja.n_joint; j += kAsmNT) {
      const uint32_t f = j < ja.n_joint ? 0u : 2u, b = j < ja.n_joint ? j : j - ja.n_joint;
      const uint32_t c = joint[f * ja.n_joint + b];
      if (!c) continue;
      const unsigned long long cw =
          a.w0 ? (unsigned long long)c * a.w0 : joint[(f + 1) * ja.n_joint + b];
      uint64_t* h = f ? ja.fh : ja.jh;
      atomicAdd((unsigned long long*)&h[2 * (uint64_t)b], (unsigned long long)c);
      atomicAdd((unsigned long long*)&h[2 * (uint64_t)b + 1], cw);
    }
    for (uint32_t j = threadIdx.x; j < ntb; j += kAsmNT)
      if (swd[j] != 0.0) atomicAdd(&ja.wd[j], swd[j]);
  }
}

// First position of every request r (rstart[r], r <= n_req; an empty
// request starts where the next one does): request indices are
// non-decreasing over the positions.
__global__ __launch_bounds__(256) void k_sd_rstart(const uint32_t* __restrict__ req, uint64_t n,
                                                   uint32_t n_req, uint32_t* __restrict__ rstart) {
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p <= n;
       p += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t lo = p == 0 ? 0u : req[p - 1] + 1u;  // requests that start here
    const uint32_t hi = p == n ? n_req : req[p];
    for (uint32_t r = lo; r <= hi && r <= n_req; ++r) rstart[r] = (uint32_t)p;
  }
}

// Prefix reuse: a block is reused from a cache of capacity C only if every
// block of its request up to it is (radix-tree caches reuse a request's
// longest cached prefix), i.e. the running maximum of the stack distances
// over the request, D'_i = max(D_j : j <= i in i's request), is at most C.
// One wavefront per request scans its distances 64 at a time, up to a first
// access (nothing behind it is reused), and bins D' into fields 0 and 1 of
// `ba.hist`.  D' only grows along a request, so neighbouring lanes share a
// bin: the last lane of each run of equal bins adds for the run.  Workgroups
// add their bins to the same words one after another, so they are few (two to
// a compute unit), large, and take no more LDS than the bins need: 4.6e6
// accesses in 1.2e5 requests, 36 us; 123 with 4096 workgroups of 256.
constexpr int kPfNT = 1024;
template <bool kLds>
__global__ __launch_bounds__(kPfNT) void k_sd_prefix(const uint32_t* __restrict__ D,
                                                   const uint32_t* __restrict__ rstart,
                                                   uint32_t n_req, const uint8_t* __restrict__ w8,
                                                   const uint8_t* __restrict__ g8, BinArgs ba) {
  extern __shared__ uint32_t sm[];  // kLds: thresholds, counts, weights
  __shared__ uint32_t soff[KV_MAX_GROUPS + 1];
  const uint32_t nbins = ba.n_thr + ba.n_groups;
  uint32_t *sthr = sm, *scnt = sm + ba.n_thr, *sw = scnt + nbins;
  if (threadIdx.x <= ba.n_groups) soff[threadIdx.x] = ba.off[threadIdx.x];
  if (kLds) {
    for (uint32_t j = threadIdx.x; j < ba.n_thr; j += kPfNT) sthr[j] = ba.thr[j];
    for (uint32_t j = threadIdx.x; j < nbins; j += kPfNT) {
      scnt[j] = 0;
      sw[j] = 0;
    }
  }
  __syncthreads();
  const uint32_t lane = lane_id();
  const uint32_t waves = gridDim.x * (kPfNT / 64);
  for (uint32_t r = blockIdx.x * (kPfNT / 64) + threadIdx.x / 64; r < n_req; r += waves) {
    const uint32_t b = rstart[r], e = rstart[r + 1];
    uint32_t carry = 0;
    for (uint32_t c = b; c < e && carry != kNone; c += 64) {
      const uint32_t i = c + lane;
      const uint32_t q = min(i, e - 1);
      uint32_t m = i < e ? D[q] : 0u;
      const uint32_t g = g8[q], w = w8[q];
      m = max(wave_incl_max_u32(m), carry);
      carry = (uint32_t)__builtin_amdgcn_readlane((int)m, 63);
      const bool in = i < e && m != kNone;  // not past the request, nor behind a first access
      uint32_t bin = kNone;
      if (in) {
        const uint32_t lo = soff[g], hi = soff[g + 1];
        bin = lo + g + (lower_bound(kLds ? (const uint32_t*)sthr : ba.thr, lo, hi, m) - lo);
      }
      // `in` holds for the low lanes: a run is `in` in all its lanes or in none
      const uint32_t before = (uint32_t)__shfl_up((int)bin, 1, 64);
      const uint64_t heads = __ballot(lane == 0 || bin != before);
      const uint32_t sum = wave_incl_scan_u32(in ? w : 0u);
      const uint32_t head = 63u - (uint32_t)__builtin_clzll(heads & (~0ull >> (63u - lane)));
      const uint32_t sum0 = (uint32_t)__shfl((int)sum, (int)head - 1, 64);
      const bool last = lane == 63 || ((heads >> (lane + 1)) & 1ull);
      if (in && last) {
        const uint32_t cn = lane - head + 1, cw = sum - (head ? sum0 : 0u);
        if (kLds) {
          atomicAdd(&scnt[bin], cn);
          atomicAdd(&sw[bin], cw);
        } else {
          atomicAdd((unsigned long long*)&ba.hist[bin * 4 + 0], (unsigned long long)cn);
          atomicAdd((unsigned long long*)&ba.hist[bin * 4 + 1], (unsigned long long)cw);
        }
      }
    }
  }
  if (kLds) {
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < nbins; j += kPfNT) {
      if (scnt[j]) {
        atomicAdd((unsigned long long*)&ba.hist[j * 4 + 0], (unsigned long long)scnt[j]);
        atomicAdd((unsigned long long*)&ba.hist[j * 4 + 1], (unsigned long long)sw[j]);
      }
    }
  }
}

// Histograms made cumulative, one workgroup per group and kind (blockIdx.y:
// 0 the capacity bins, 1 the prefix-reuse ones, 2 the joint ones).
constexpr uint32_t kCumLds = 8192;  // joint words of one group staged in LDS
__global__ __launch_bounds__(256) void k_sd_cum(uint64_t* hist, uint64_t* phist,
                                                const uint32_t* __restrict__ off, JointArgs ja) {
  __shared__ uint64_t sj[kCumLds];
  __shared__ double swd[256];
  const uint32_t g = blockIdx.x, lane = lane_id(), w = (uint32_t)wave_id();
  const uint32_t nd = off[g + 1] - off[g] + 1;
  if (blockIdx.y == 1 && !phist) return;
  if (blockIdx.y < 2) {
    // a wavefront per field, 64 bins at a time
    uint64_t* h = (blockIdx.y ? phist : hist) + (uint64_t)(off[g] + g) * 4 + w;
    uint64_t run = 0;
    for (uint32_t b = 0; b < nd; b += 64) {
      const uint32_t i = b + lane;
      const uint64_t v = wave_incl_scan<uint64_t>(i < nd ? h[(uint64_t)i * 4] : 0ull) + run;
      if (i < nd) h[(uint64_t)i * 4] = v;
      run = (uint64_t)__shfl((unsigned long long)v, 63, 64);
    }
    return;
  }
  // both bin dimensions, in LDS where they fit
  const uint32_t nt = ja.toff[g + 1] - ja.toff[g] + 1, nw = 2 * nd * nt;
  for (int f = 0; f < 2; ++f) {
    uint64_t* src = (f ? ja.fh : ja.jh) + 2ull * ja.jbase[g];
    const bool lds = nw <= kCumLds;
    uint64_t* h = lds ? sj : src;
    if (lds)
      for (uint32_t j = threadIdx.x; j < nw; j += 256) sj[j] = src[j];
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < 2 * nd; q += 256) {  // along gap bins
      uint64_t* x = h + (uint64_t)(q >> 1) * nt * 2 + (q & 1);
      uint64_t run = 0;
      for (uint32_t t = 0; t < nt; ++t) {
        run += x[2 * t];
        x[2 * t] = run;
      }
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < 2 * nt; q += 256) {  // along distance bins
      uint64_t run = 0;
      for (uint32_t d = 0; d < nd; ++d) {
        uint64_t& x = h[(uint64_t)d * nt * 2 + q];
        run += x;
        x = run;
      }
    }
    __syncthreads();
    if (lds)
      for (uint32_t j = threadIdx.x; j < nw; j += 256) src[j] = sj[j];
    __syncthreads();
  }
  double run = 0.0;  // weighted gaps over gap bins
  double* wd = ja.wd + ja.toff[g] + g;
  for (uint32_t b = 0; b < nt; b += 256) {
    const uint32_t m = min(256u, nt - b);
    if (threadIdx.x < m) swd[threadIdx.x] = wd[b + threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0)
      for (uint32_t t = 0; t < m; ++t) {
        run += swd[t];
        swd[t] = run;
      }
    __syncthreads();
    if (threadIdx.x < m) wd[b + threadIdx.x] = swd[threadIdx.x];
    __syncthreads();
  }
}

// Test hooks, read at every call: KVCFG_TEST_ROW_CHUNK narrows the LDS
// histogram of a block-matrix row (so that short traces take the
// column-chunk path of long ones); KVCFG_TEST_BLOCK_LOG sets the size of the
// position blocks; KVCFG_TEST_THR_LDS lowers the number of
// thresholds binned in LDS (so that few thresholds take the global-atomic
// path of very many).  Both only select among paths of the same result.
uint32_t env_limit(const char* name, uint32_t dflt, uint32_t lo) {
  const char* e = std::getenv(name);
  if (!e) return dflt;
  const unsigned long v = std::strtoul(e, nullptr, 10);
  return (uint32_t)std::max<unsigned long>(lo, std::min<unsigned long>(v, dflt));
}

uint32_t grid_of(uint64_t m, uint32_t cap = 32768) {
  uint64_t g = (m + 255) / 256;
  if (g > cap) g = cap;
  return (uint32_t)(g ? g : 1);
}

// log2 of the position block.  Small blocks sort in fewer merge levels, and
// more of them fit a compute unit and run at once; the block matrix grows
// with the square of their number.  Matrix and in-block kernels, us, for
// blocks of 1,024 / 2,048 / 4,096 / 8,192: 238,313 accesses 43 / 47 / 57 / 84;
// 4.6e6: 216 / 173 / 171 / 246; 1.09e8: 46,230 / 11,080 / 4,950 / 3,730.
uint32_t block_log(uint64_t n) {
  if (const char* e = std::getenv("KVCFG_TEST_BLOCK_LOG"))
    return (uint32_t)std::min(13ul, std::max(10ul, std::strtoul(e, nullptr, 10)));
  return n <= (1ull << 18) ? 10 : n <= (1ull << 23) ? 11 : n <= (1ull << 25) ? 12 : 13;
}

}  // namespace

kv_status stack_pass(Trace& t, Order& o, bool partitioned, const ThresholdSet& ts,
                     const uint32_t* thr_dev, const uint32_t* off_dev, uint64_t* hist,
                     uint64_t* phist, const JointArgs* ja, const uint8_t* real, hipStream_t s) {
  const uint64_t n = o.n ? o.n : t.n;
  const uint32_t logb = block_log(n);
  const uint32_t G = div_up(n, 1u << logb);
  const bool uni = t.st.w_min == t.st.w_max;
  kv_status st;
  const uint64_t tri = G >= 2 ? tri_off(G) : 1;
  DevBuf& b_partial = t.ws[0];
  DevBuf& b_E = t.ws[1];
  DevBuf& b_Q = t.ws[2];
  DevBuf& b_last = t.ws[3];  // per part of a block: weight of its last occurrences, and before
  if ((st = b_partial.reserve(n * 4)) != KV_OK) return st;
  if ((st = b_E.reserve(n * 4)) != KV_OK) return st;
  if ((st = b_Q.reserve(tri * 4)) != KV_OK) return st;
  if ((st = b_last.reserve((2ull * kSubs * G + KV_MAX_GROUPS) * 4)) != KV_OK) return st;
  if ((phist || ja) && partitioned) return fail(KV_ERR_UNSUPPORTED, "this mode needs the trace order");
  // prefix reuse: every access's distance; request starts
  uint32_t* dist = nullptr;
  uint32_t* rstart = nullptr;
  if (phist) {
    if ((st = t.ws[25].reserve(n * 4)) != KV_OK) return st;
    dist = t.ws[25].as<uint32_t>();
    if ((st = t.ws[26].reserve(((uint64_t)t.st.n_req + 1) * 4)) != KV_OK) return st;
    rstart = t.ws[26].as<uint32_t>();
  }
  const uint32_t* key = o.key.as<uint32_t>();
  const uint32_t* nxt = o.nxt.as<uint32_t>();
  const uint8_t* w8 = o.w.as<uint8_t>();
  const uint8_t* g8 = o.g.as<uint8_t>();
  uint32_t* Q = b_Q.as<uint32_t>();
  uint32_t* lsum = b_last.as<uint32_t>();
  uint32_t* lpre = lsum + G * kSubs;
  uint32_t* segend = lpre + G * kSubs;
  SegArgs sa{};
  for (int g = 0; g <= KV_MAX_GROUPS; ++g) sa.seg[g] = o.seg[g];
  sa.partitioned = partitioned ? 1u : 0u;
  {
    StageTimer tm(kStStackMatrix, s);
    const uint32_t row_chunk = env_limit("KVCFG_TEST_ROW_CHUNK", kRowChunk, 1);
    Zero z{};
    const auto clear = [&](int q, uint64_t* p, uint64_t words) -> kv_status {
      if (!rows_clear(words, G)) return fill_u64(p, 0, words, s);
      z.p[q] = p;
      z.n[q] = (uint32_t)words;
      return KV_OK;
    };
    if ((st = clear(0, hist, 4ull * ts.total_bins())) != KV_OK) return st;
    if (phist && (st = clear(1, phist, 4ull * ts.total_bins())) != KV_OK) return st;
    // jh, fh and wd lie together
    if (ja && (st = clear(2, ja->jh, joint_words(ja->n_joint, ja->n_tthr, ts.n_groups))) != KV_OK)
      return st;
    hipLaunchKernelGGL(k_sd_rowhist, dim3(G), dim3(kRowNT), 0, s, key, nxt, w8,
                       uni ? t.st.w_max : 0u, n, logb, row_chunk,
                       Q, lsum, z);
    KV_HIP(hipGetLastError());
    // 16 columns per workgroup, more of them, for a few thousand blocks; 32
    // (whole cache lines) where the matrix does not stay in the caches
    const auto cols = [&](auto kernel, uint32_t c) {
      hipLaunchKernelGGL(kernel, dim3(div_up(G - 1, c) + 1), dim3(kRowNT), 0, s, Q, G, lsum, lpre,
                         segend, nxt, w8, n, logb, sa);
    };
    if (G <= 4096) cols(k_sd_cols<16>, 16);
    else cols(k_sd_cols<32>, 32);
    KV_HIP(hipGetLastError());
  }
  {
    StageTimer tm(kStStackLocal, s);
    const auto local = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(G), dim3((1u << logb) / kLocItems), 0, s, key, nxt, w8,
                         t.st.w_max, n, G, b_partial.as<uint32_t>(), b_E.as<uint32_t>());
    };
    switch (logb) {
      case 10: uni ? local(k_sd_local<10, true>) : local(k_sd_local<10, false>); break;
      case 11: uni ? local(k_sd_local<11, true>) : local(k_sd_local<11, false>); break;
      case 12: uni ? local(k_sd_local<12, true>) : local(k_sd_local<12, false>); break;
      default: uni ? local(k_sd_local<13, true>) : local(k_sd_local<13, false>);
    }
    KV_HIP(hipGetLastError());
  }
  BinArgs ba{thr_dev, off_dev, (uint32_t)ts.values.size(), ts.n_groups, hist};
  const uint32_t lds_limit = env_limit("KVCFG_TEST_THR_LDS", kThrLds, 0);
  const bool lds = ts.values.size() + ts.n_groups <= lds_limit;
  uint64_t bytes = lds ? (ts.values.size() + 4ull * ts.total_bins()) * 4 : 0;
  const uint64_t jbytes = ja ? (2ull * ja->n_tthr + ts.n_groups) * 8 + 16ull * ja->n_joint : 0;
  const bool jlds = ja && lds && lds_limit > 0 && bytes + jbytes <= kAsmLds;
  if (jlds) bytes += jbytes;
  {
    StageTimer tm(kStStackAssemble, s);
    AsmArgs aa{key, nxt, w8, g8, real, n, uni ? t.st.w_max : 0u, logb, G,
               b_partial.as<uint32_t>(), b_E.as<uint32_t>(), Q, dist, lpre, segend,
               sa.partitioned, t.req.as<uint32_t>(), t.req_time.as<double>()};
    // two workgroups per compute unit where their LDS allows: each flushes
    // its histograms once, so fewer and larger ones flush less
    const uint32_t ga = std::min<uint32_t>(G, 512);
    const JointArgs none{};
    const auto assemble = [&](auto kernel) {
      if (bytes > 64 * 1024 &&  // has to be asked for
          hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) != hipSuccess)
        (void)hipGetLastError();
      hipLaunchKernelGGL(kernel, dim3(ga), dim3(kAsmNT), (uint32_t)bytes, s, aa, ba, ja ? *ja : none);
    };
    const auto by_rows = [&](auto r) {
      constexpr int R = decltype(r)::value;
      if (jlds) assemble(k_sd_assemble<R, true, 1>);
      else if (ja) lds ? assemble(k_sd_assemble<R, true, 2>) : assemble(k_sd_assemble<R, false, 2>);
      else lds ? assemble(k_sd_assemble<R, true, 0>) : assemble(k_sd_assemble<R, false, 0>);
    };
    switch (logb) {
      case 10: by_rows(std::integral_constant<int, 1>{}); break;
      case 11: by_rows(std::integral_constant<int, 2>{}); break;
      case 12: by_rows(std::integral_constant<int, 4>{}); break;
      default: by_rows(std::integral_constant<int, 8>{});
    }
    KV_HIP(hipGetLastError());
    if (phist) {
      const uint32_t nr = t.st.n_req;
      hipLaunchKernelGGL(k_sd_rstart, dim3(grid_of(n + 1)), dim3(256), 0, s,
                         t.req.as<uint32_t>(), n, nr, rstart);
      KV_HIP(hipGetLastError());
      BinArgs bp{thr_dev, off_dev, (uint32_t)ts.values.size(), ts.n_groups, phist};
      // two workgroups to a compute unit: each adds its bins to the same words
      const uint32_t gp = std::min<uint32_t>(div_up(nr, kPfNT / 64), 512);
      if (lds) {
        const uint32_t pbytes = (bp.n_thr + 2 * (bp.n_thr + bp.n_groups)) * 4;
        if (pbytes > 64 * 1024 &&  // has to be asked for
            hipFuncSetAttribute(reinterpret_cast<const void*>(k_sd_prefix<true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)pbytes) != hipSuccess)
          (void)hipGetLastError();
        hipLaunchKernelGGL(k_sd_prefix<true>, dim3(gp), dim3(kPfNT), pbytes, s, (const uint32_t*)dist,
                           (const uint32_t*)rstart, nr, w8, g8, bp);
      } else {
        hipLaunchKernelGGL(k_sd_prefix<false>, dim3(gp), dim3(kPfNT), 0, s, (const uint32_t*)dist,
                           (const uint32_t*)rstart, nr, w8, g8, bp);
      }
      KV_HIP(hipGetLastError());
    }
  }
  StageTimer tm(kStStackFinal, s);
  hipLaunchKernelGGL(k_sd_cum, dim3(ts.n_groups, ja ? 3 : phist ? 2 : 1), dim3(256), 0, s, hist,
                     phist, off_dev, ja ? *ja : JointArgs{});
  KV_HIP(hipGetLastError());
  return KV_OK;
}

}  // namespace kv
