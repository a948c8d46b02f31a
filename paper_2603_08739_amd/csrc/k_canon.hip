// k_canon.hip - trace canonicalisation.
//
// The paper's simulator consumes traces of salted KV-block hashes, 16 tokens
// per block (Section 3.3, trace description; Section 4.1, simulator).  Every
// later step needs, per access, the position of the previous and of the next
// access to the same block, and a dense id per distinct block.
//
// Equal hashes only have to meet, in trace order; they need not be sorted.
// The accesses are partitioned, stably, by 1 to 20 bits of their mixed hash
// (one or two passes), so that a few hundred consecutive ones share all the
// accesses of their blocks.  A wavefront then takes such a stretch in order,
// 64 accesses at a time, through a hash table in LDS that holds each block's
// first and latest position; a stretch that a much-read block makes long is cut
// into parts, which are joined afterwards.  Each pass also records where every element
// went, so the results come back to trace order by gathers whose sources are
// runs of a tile, not by scattering records to random positions.  Links to the
// next access and dense ids follow in trace order, where consecutive accesses
// mostly have consecutive previous and first accesses.  A load of 1.09e8
// accesses moves about 165 B per access in 7.5 ms; the radix sort over the
// high hash bits, the second sort of its mixed runs and the 16-byte link
// scatter that this replaced took 15.2 ms (4.6e6 accesses: 0.43 and 1.03 ms;
// 238,313 accesses, 24 launches fewer than eight sort passes: 0.13 and 0.45).
//
// A stretch with more distinct blocks than the table holds sends the load to
// a stable LSD radix sort of (hash, position) pairs instead, where neighbours
// are the previous / next occurrences.  Up to 2^29 accesses that takes hashes
// made to collide: with 20 bits a stretch of distinct blocks has at most 512
// on average.  (With at most 18 bits, loads of more than 2.2e8 distinct blocks
// came to the sort: 3e8 of them took 133 ms, now 24; 5e8 230 ms, now 44.)
#include <cstdlib>

#include "kv_device.h"
#include "kv_internal.h"

namespace kv {
namespace {

constexpr int kRsNT = 1024;
constexpr int kRsItems = 8;
constexpr uint32_t kRsTile = kRsNT * kRsItems;  // 8192
constexpr int kRsDigits = 256;                   // 8-bit digits
constexpr int kRsWaves = kRsNT / 64;

constexpr int kPtBits = 10;                      // most bits of a partition digit
constexpr uint32_t kPtDigits = 1u << kPtBits;
constexpr int kLkBits = 10;                      // slots of the linking table
constexpr uint32_t kLkSlots = 1u << kLkBits;
// A table with more blocks is emptied at the next stretch (one that starts
// inside a row may add the row's blocks first: a quarter at most is in use)
constexpr uint32_t kLkClear = kLkSlots / 4 - 64;
constexpr uint32_t kPiece = 8192;                // a long stretch is cut at multiples of this
constexpr uint32_t kJoinCuts = 16;               // such multiples a joining wavefront looks at
constexpr uint32_t kCutFrom = 1u << 14;          // traces of more accesses have stretches cut

enum : uint32_t {
  kErrGroup = 1u,
  kErrWeight = 2u,
  kErrReq = 4u,
  kErrInconsistent = 8u,
  kErrTime = 16u,
};

struct DevStats {
  unsigned long long n_g[KV_MAX_GROUPS];
  unsigned long long n_w_g[KV_MAX_GROUPS];
  unsigned long long u_g[KV_MAX_GROUPS];
  unsigned long long u_w_g[KV_MAX_GROUPS];
  unsigned long long mult;
  double t0, t1;             // first and last request time
  uint32_t w_min, w_max, err;
  uint32_t u;                // distinct blocks
  uint32_t full;             // a stretch had more distinct blocks than its table holds
  uint32_t pad;
};

// A bijection of the hashes whose top bits depend on all of them (Murmur3's
// 64-bit finaliser, by its author in the public domain): equal hashes stay
// equal, others spread over the partitions whatever their pattern.
__device__ __forceinline__ uint64_t mixed_hash(uint64_t h) {
  h ^= h >> 33;
  h *= 0xFF51AFD7ED558CCDull;
  h ^= h >> 33;
  h *= 0xC4CEB9FE1A85EC53ull;
  return h ^ (h >> 33);
}

// Per access: check group / weight / request index, copy request, group and
// weight into the trace, count the first pass's digits of each tile
// (counts[digit * ntiles + tile]), accumulate per-group totals.  The request
// times are checked and copied along the way, by workgroups beyond the tiles'
// too where requests outnumber accesses (1,000 accesses of 5e7 requests: 0.34
// ms, 47 ms with a workgroup per tile only).  Workgroups take several tiles, so
// that few global atomics queue on each statistic.
__global__ __launch_bounds__(kRsNT) void k_load_tiles(
    const uint64_t* __restrict__ hash, const uint32_t* __restrict__ req,
    const uint8_t* __restrict__ group, const uint8_t* __restrict__ weight, uint64_t n,
    const double* __restrict__ req_time, uint32_t n_req, uint32_t n_groups,
    uint32_t* __restrict__ req_out, double* __restrict__ time_out, uint8_t* __restrict__ g8,
    uint8_t* __restrict__ w8, int shift, uint32_t digits, uint32_t* __restrict__ counts,
    uint32_t ntiles, DevStats* st) {
  __shared__ unsigned long long sn[KV_MAX_GROUPS], sw[KV_MAX_GROUPS];
  __shared__ uint32_t smin, smax, serr;
  __shared__ uint32_t h[kPtDigits];
  if (threadIdx.x < KV_MAX_GROUPS) {
    sn[threadIdx.x] = 0;
    sw[threadIdx.x] = 0;
  }
  if (threadIdx.x == 0) {
    smin = 0xFFFFFFFFu;
    smax = 0;
    serr = 0;
  }
  uint32_t err = 0, wmin = 0xFFFFFFFFu, wmax = 0;
  for (uint64_t i = blockIdx.x * kRsNT + threadIdx.x; i < n_req; i += gridDim.x * kRsNT) {
    const double t = req_time[i];
    time_out[i] = t;
    if (i + 1 < n_req ? !(t <= req_time[i + 1]) : t != t) err |= kErrTime;
    if (i == 0) st->t0 = t;
    if (i + 1 == n_req) st->t1 = t;
  }
  // per-group totals add up in registers while the thread's group stays
  // the same (always, with one group) and go to LDS when it changes: LDS
  // atomics of a wavefront on one address are taken one lane at a time
  uint32_t cg = 0xFFFFFFFFu;
  unsigned long long cn = 0, cw = 0;
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    if (threadIdx.x < digits) h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)tile * kRsTile;
    uint64_t k[kRsItems];
    uint32_t r[kRsItems], rn[kRsItems], g[kRsItems], w[kRsItems];
#pragma unroll
    for (int e = 0; e < kRsItems; ++e) {
      const uint64_t i = base + (uint64_t)e * kRsNT + threadIdx.x, j = min(i, n - 1);
      k[e] = hash[j];
      r[e] = req[j];
      rn[e] = req[min(i + 1, n - 1)];
      g[e] = group ? group[j] : 0u;
      w[e] = weight ? weight[j] : 1u;
    }
#pragma unroll
    for (int e = 0; e < kRsItems; ++e) {
      const uint64_t i = base + (uint64_t)e * kRsNT + threadIdx.x;
      if (i >= n) continue;
      if (g[e] >= n_groups) { err |= kErrGroup; g[e] = 0; }
      if (w[e] == 0) err |= kErrWeight;
      if (r[e] >= n_req || rn[e] < r[e]) err |= kErrReq;
      req_out[i] = r[e];
      g8[i] = (uint8_t)g[e];
      w8[i] = (uint8_t)w[e];
      atomicAdd(&h[(uint32_t)(mixed_hash(k[e]) >> shift) & (digits - 1)], 1u);
      if (g[e] != cg) {
        if (cn) {
          atomicAdd(&sn[cg], cn);
          atomicAdd(&sw[cg], cw);
        }
        cg = g[e];
        cn = 0;
        cw = 0;
      }
      ++cn;
      cw += w[e];
      wmin = min(wmin, w[e]);
      wmax = max(wmax, w[e]);
    }
    __syncthreads();
    if (threadIdx.x < digits) counts[(uint64_t)threadIdx.x * ntiles + tile] = h[threadIdx.x];
    __syncthreads();
  }
  if (n_groups == 1) {
    // one group: a wavefront's totals add up before its atomics
    cn = wave_sum(cn);
    cw = wave_sum(cw);
    if (lane_id() != 0) cn = 0;
    cg = 0;
  }
  if (cn) {
    atomicAdd(&sn[cg], cn);
    atomicAdd(&sw[cg], cw);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    wmin = min(wmin, (uint32_t)__shfl_xor((int)wmin, d, 64));
    wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, d, 64));
    err |= (uint32_t)__shfl_xor((int)err, d, 64);
  }
  if (lane_id() == 0) {
    atomicMin(&smin, wmin);
    atomicMax(&smax, wmax);
    if (err) atomicOr(&serr, err);
  }
  __syncthreads();
  if (threadIdx.x < n_groups) {
    if (sn[threadIdx.x]) atomicAdd(&st->n_g[threadIdx.x], sn[threadIdx.x]);
    if (sw[threadIdx.x]) atomicAdd(&st->n_w_g[threadIdx.x], sw[threadIdx.x]);
  }
  if (threadIdx.x == 0) {
    atomicMin(&st->w_min, smin);
    atomicMax(&st->w_max, smax);
    if (serr) atomicOr(&st->err, serr);
  }
}

__global__ void k_load_init(DevStats* st, uint32_t* err) {
  uint32_t* p = reinterpret_cast<uint32_t*>(st);
  for (uint32_t i = threadIdx.x; i < sizeof(DevStats) / 4; i += blockDim.x) p[i] = 0;
  if (threadIdx.x < 2) err[threadIdx.x] = 0;  // the replays' error record
  __syncthreads();
  if (threadIdx.x == 0) st->w_min = 0xFFFFFFFFu;
}

// (hash, position) pairs for the radix sort of the fallback.
__global__ __launch_bounds__(256) void k_sort_pairs(const uint64_t* __restrict__ hash, uint64_t n,
                                                    uint64_t* __restrict__ keys,
                                                    uint32_t* __restrict__ vals) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    keys[i] = hash[i];
    vals[i] = (uint32_t)i;
  }
}

// Digits of the second partition pass, per tile.
__global__ __launch_bounds__(kRsNT) void k_pt_count(const uint64_t* __restrict__ keys, uint64_t n,
                                                    int shift, uint32_t digits,
                                                    uint32_t* __restrict__ counts,
                                                    uint32_t ntiles) {
  __shared__ uint32_t h[kPtDigits];
  if (threadIdx.x < digits) h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = (uint64_t)blockIdx.x * kRsTile;
#pragma unroll
  for (int e = 0; e < kRsItems; ++e) {
    const uint64_t i = base + (uint64_t)e * kRsNT + threadIdx.x;
    if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & (digits - 1)], 1u);
  }
  __syncthreads();
  if (threadIdx.x < digits)
    counts[(uint64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Stable partition of one tile by a digit of up to kBits bits, given the
// exclusive digit offsets (as k_rs_scatter; each 64-lane wavefront ranks 64
// consecutive items per round by matching digits with ballots).  dst[i]: where
// element i went.  kFirst: the input is the caller's hashes in trace order.
template <bool kFirst, int kBits>
__global__ __launch_bounds__(kRsNT) void k_pt_scatter(const uint64_t* __restrict__ kin,
                                                      const uint32_t* __restrict__ vin,
                                                      uint64_t* __restrict__ kout,
                                                      uint32_t* __restrict__ vout,
                                                      uint32_t* __restrict__ dst, uint64_t n,
                                                      int shift, uint32_t digits,
                                                      const uint32_t* __restrict__ offsets,
                                                      uint32_t ntiles) {
  constexpr uint32_t kDigits = 1u << kBits;
  static_assert(kDigits <= kRsNT, "a thread per digit");
  __shared__ uint16_t wcnt[kRsWaves][kDigits];
  __shared__ uint32_t gbase[kDigits];   // the digit's first output position, less its tile start
  __shared__ uint32_t red[kRsWaves];
  __shared__ uint64_t sk[kRsTile];
  __shared__ uint32_t sv[kRsTile];
  const int w = threadIdx.x / 64;
  const uint32_t lane = lane_id();
  for (int d = threadIdx.x; d < kRsWaves * (int)kDigits / 2; d += kRsNT)
    reinterpret_cast<uint32_t*>(&wcnt[0][0])[d] = 0;
  const uint32_t g0 =
      threadIdx.x < digits ? offsets[(uint64_t)threadIdx.x * ntiles + blockIdx.x] : 0u;
  __syncthreads();
  const uint64_t t0 = (uint64_t)blockIdx.x * kRsTile;
  const uint64_t base = t0 + (uint64_t)w * (kRsItems * 64);
  uint64_t k[kRsItems];
  uint32_t v[kRsItems], d[kRsItems], rk[kRsItems];
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < kRsItems; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    const bool valid = i < n;
    k[r] = valid ? kin[i] : 0ull;
    v[r] = kFirst ? (uint32_t)i : valid ? vin[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kRsItems; ++r) {
    const bool valid = base + (uint64_t)r * 64 + lane < n;
    if (kFirst) k[r] = mixed_hash(k[r]);
    d[r] = (uint32_t)(k[r] >> shift) & (digits - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
      const bool bit = (d[r] >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t before = (uint32_t)__popcll(peers & lt);
    const uint32_t cur = wcnt[w][d[r]];
    rk[r] = cur + before;
    const bool leader = valid && ((peers >> lane) == 1ull);
    if (leader) wcnt[w][d[r]] = (uint16_t)(cur + (uint32_t)__popcll(peers));
  }
  __syncthreads();
  {
    const uint32_t dg = threadIdx.x;
    const bool has = dg < digits;
    uint32_t tot = 0;
    if (has) {
#pragma unroll
      for (int ww = 0; ww < kRsWaves; ++ww) tot += wcnt[ww][dg];
    }
    uint32_t all;
    const uint32_t ls = block_excl_scan_u32<kRsNT, false>(tot, red, all);
    if (has) {
      uint32_t run = ls;
#pragma unroll
      for (int ww = 0; ww < kRsWaves; ++ww) {
        const uint32_t c = wcnt[ww][dg];
        wcnt[ww][dg] = (uint16_t)run;
        run += c;
      }
      gbase[dg] = g0 - ls;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRsItems; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    if (i < n) {
      const uint32_t lp = wcnt[w][d[r]] + rk[r];
      sk[lp] = k[r];
      sv[lp] = v[r];
      dst[i] = gbase[d[r]] + lp;
    }
  }
  __syncthreads();
  const uint32_t m = (uint32_t)min<uint64_t>(kRsTile, n - t0);
  for (uint32_t p = threadIdx.x; p < m; p += kRsNT) {
    const uint64_t key = sk[p];
    const uint32_t at = gbase[(uint32_t)(key >> shift) & (digits - 1)] + p;
    kout[at] = key;
    vout[at] = sv[p];
  }
}

// What the blocks of each part of a cut stretch leave to the joining pass: one
// entry per block at [part * kPiece ..], their number in count[part].
struct PtLists {
  uint32_t *elem, *last, *cnt;  // its first element there, its latest position, its accesses
  uint32_t* count;
};

// Whether a stretch is cut at m, a multiple of kPiece: it reaches back a whole
// piece and more (equal top bits are consecutive).  n: 0 if none is cut.
__device__ __forceinline__ bool pt_cut(const uint64_t* __restrict__ K, uint32_t n, int dshift,
                                       uint32_t m) {
  return m >= kPiece && m < n && (K[m - kPiece] >> dshift) == (K[m] >> dshift);
}

// The linking table of a wavefront: 20,480 bytes, an eighth of a compute
// unit's LDS.  A free slot's key is 0, so the block whose hash mixes to 0 is
// kept beside it, in registers that all lanes hold alike.  (With a slot of its
// own, 20,520 bytes, seven fit: k_pt_link over 1e8 accesses 1.44 ms, now 1.34.)
struct PtTable {
  unsigned long long key[kLkSlots];
  uint32_t last[kLkSlots], first[kLkSlots], cnt[kLkSlots];
};
static_assert(sizeof(PtTable) * 8 == 160 * 1024, "eight wavefronts to a compute unit");

struct PtZero {
  uint32_t last = kNone, first = 0, cnt = 0;
};

__device__ __forceinline__ void pt_clear(PtTable& T) {
  __syncthreads();
  for (uint32_t i = lane_id(); i < kLkSlots; i += 64) {
    T.key[i] = 0;
    T.last[i] = kNone;
  }
  __syncthreads();
}

// The slot of the lane's block (`in`), inserted where it is new (kLkSlots for
// the one that is kept beside the table); the number of new ones.  The caller
// has checked that the table has room.
__device__ __forceinline__ uint32_t pt_slot(PtTable& T, uint64_t k, bool in, int sshift,
                                            uint32_t& fresh_n) {
  uint32_t s = k == 0ull ? kLkSlots : (uint32_t)(k >> sshift) & (kLkSlots - 1);
  bool todo = in && k != 0ull, fresh = false;
  while (__ballot(todo)) {
    if (todo) {
      const unsigned long long old = atomicCAS(&T.key[s], 0ull, (unsigned long long)k);
      fresh = old == 0ull;
      if (fresh || old == k) todo = false;
      else s = (s + 1) & (kLkSlots - 1);
    }
  }
  fresh_n = (uint32_t)__popcll(__ballot(fresh));
  return s;
}

// Atomics on one address are taken one at a time: only those that may count.
__device__ __forceinline__ void pt_most(uint32_t most, DevStats* st) {
  most = wave_max_u32(most);
  if (lane_id() == 0 &&
      most > __hip_atomic_load(&st->mult, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(&st->mult, (unsigned long long)most);
}

// Links of the partitioned accesses.  A wavefront takes the stretches (equal
// top `bits` bits) that start in its `chunk` elements, in order, 64 elements
// at a time: each finds its block's slot in an LDS hash table, its previous
// access is the latest lower lane of that slot or the slot's latest position.
// out[k] = (previous position + 1 or 0, position of the block's first access).
// The table is emptied between stretches once it fills up; bound by the chain
// of LDS operations per 64 elements, with eight wavefronts to a compute unit.
// Rows were cut where a stretch ended, and the next one loaded
// from there; they are now taken whole and loaded two ahead (1.09e8 accesses:
// 2.03 -> 1.67 ms, 4.6e6: 114 -> 79 us).
//
// A block that many requests share makes its stretch as long as its accesses
// are many, so a stretch is cut at the multiples of kPiece that lie a whole
// piece and more inside it (a chunk lies between two such multiples).  The
// wavefront that comes to the first cut ends there; the workgroups from
// `chunks` on take one piece each, if the stretch is cut at its start.  A part
// links its own accesses and lists its blocks for k_pt_join.  (One wavefront
// for a whole stretch: 1e7 accesses, every second one of one block, loaded in
// 58 ms, now 1.4; 1e8 accesses, one in 75 of one block, 26.7 ms, now 12.6.  Pieces
// of 4,096 serve the second of these alike, the first in 1.75 ms: more parts to
// join one after another.)
__global__ __launch_bounds__(64) void k_pt_link(const uint64_t* __restrict__ K,
                                                const uint32_t* __restrict__ V, uint32_t n,
                                                uint32_t cut_n, int bits, uint32_t chunk,
                                                uint32_t chunks, uint2* __restrict__ out,
                                                PtLists pl, DevStats* st) {
  __shared__ PtTable T;
  const uint32_t lane = lane_id();
  const uint64_t lt = lanemask_lt();
  const int dshift = 64 - bits, sshift = 64 - bits - kLkBits;
  // the elements [at, stop), less those from the first stretch on that starts
  // at c1 or later; `part` is the list to write if `stop` is reached, or in any case
  uint32_t at, c1, stop, part = kNone;
  const bool piece = blockIdx.x >= chunks;
  if (piece) {
    at = (blockIdx.x - chunks + 1) * kPiece;
    if (!pt_cut(K, cut_n, dshift, at)) return;
    c1 = at + 1;
    stop = min(n, at + kPiece);
    part = at / kPiece;
  } else {
    at = blockIdx.x * chunk;
    c1 = min(n, at + chunk);
    if (at) {  // the first stretch that starts in the chunk
      const uint64_t before = K[at - 1] >> dshift;
      if ((K[c1 - 1] >> dshift) == before) return;
      for (;;) {
        const uint32_t i = at + lane;
        const uint64_t dg = (i < c1 ? K[i] : 0ull) >> dshift;
        const uint64_t m = __ballot(i < c1 && dg != before);
        if (m) {
          at += (uint32_t)__builtin_ctzll(m);
          break;
        }
        at += 64;
      }
    }
    // the first cut that the last of them may come to
    stop = (c1 + kPiece - 1) / kPiece * kPiece;
    if (!pt_cut(K, cut_n, dshift, stop)) {
      stop += kPiece;
      if (!pt_cut(K, cut_n, dshift, stop)) stop = n;
    }
    if (stop < n) part = stop / kPiece - 1;
  }
  pt_clear(T);
  PtZero z;
  // rows of 64, two loaded ahead.  A row is taken whole, whatever stretches it
  // spans; it is cut only where the table is emptied and at the end.
  uint32_t occ = 0, most = 0;
  const auto ldk = [&](uint32_t i) { return K[min(i, n - 1)]; };
  const auto ldv = [&](uint32_t i) { return V[min(i, n - 1)]; };
  uint64_t k = ldk(at + lane), k1 = ldk(at + 64 + lane);
  uint32_t v = ldv(at + lane), v1 = ldv(at + 64 + lane);
  uint64_t prev = ~0ull;  // the digit before the row (none yet: no digit has 64 bits)
  uint32_t from = at, to = stop;  // the stretch in hand, and the end
  bool full = false;
  for (; at < stop; at += 64) {
    const uint32_t i = at + lane;
    const uint64_t k2 = ldk(i + 128);
    const uint32_t v2 = ldv(i + 128);
    const uint64_t dg = k >> dshift;
    // lanes at which a stretch starts
    const uint32_t up = (uint32_t)max((int)lane - 1, 0);
    uint64_t db = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(dg >> 32), (int)up, 64) << 32) |
                  (uint32_t)__shfl((int)(uint32_t)dg, (int)up, 64);
    if (lane == 0) db = prev;
    const uint64_t starts = __ballot(i < stop && dg != db);
    prev = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(dg >> 32), 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)dg, 63);
    uint64_t row = __ballot(i < stop);  // still to be taken
    bool end = false;
    if (at + 64 > c1) {
      const uint64_t out_of = at >= c1 ? starts : starts & (~0ull << (c1 - at));
      if (out_of) {
        to = at + (uint32_t)__builtin_ctzll(out_of);
        row &= (1ull << __builtin_ctzll(out_of)) - 1;
        end = true;
      }
    }
    if (starts & row) from = at + 63 - (uint32_t)__builtin_clzll(starts & row);
    while (row) {
      uint64_t mine = row;
      if (occ > kLkClear) {
        const uint64_t b = starts & row;
        if (b) {
          mine = row & ((1ull << __builtin_ctzll(b)) - 1);
          if (!mine) {  // the stretch starts here
            pt_clear(T);
            occ = 0;
            mine = row;
          }
        }
      }
      row &= ~mine;
      const bool in = (mine >> lane) & 1ull;
      if (occ + 64 > kLkSlots) {  // too many distinct blocks: the load is redone by sorting
        full = true;
        break;
      }
      uint32_t fresh;
      const uint32_t s = pt_slot(T, k, in, sshift, fresh);
      occ += fresh;
      uint64_t peers = mine;
#pragma unroll
      for (int b = 0; b <= kLkBits; ++b) {
        const bool bit = (s >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
      }
      const uint64_t lower = peers & lt;
      const bool tab = in && s < kLkSlots;
      const uint32_t l = tab ? T.last[s] : z.last, f = tab ? T.first[s] : z.first;
      const uint32_t c = tab ? T.cnt[s] : z.cnt;
      const int pl = lower ? 63 - __builtin_clzll(lower) : 0;
      const int ll = peers ? __builtin_ctzll(peers) : 0;
      const uint32_t vp = (uint32_t)__shfl((int)v, pl, 64), v0 = (uint32_t)__shfl((int)v, ll, 64);
      const uint32_t fp = l == kNone ? v0 : f;
      if (in) out[i] = make_uint2(lower ? vp + 1u : l + 1u, fp);  // kNone + 1 = 0
      const bool top = in && (peers >> lane) == 1ull;  // the slot's latest element
      const uint32_t tot = (l == kNone ? 0u : c) + (uint32_t)__popcll(peers);
      if (top) most = max(most, tot);
      if (top && tab) {
        T.last[s] = v;
        T.first[s] = fp;
        T.cnt[s] = tot;
      }
      if (const uint64_t m0 = __ballot(top && !tab)) {
        const int q = __builtin_ctzll(m0);
        z.last = (uint32_t)__builtin_amdgcn_readlane((int)v, q);
        z.first = (uint32_t)__builtin_amdgcn_readlane((int)fp, q);
        z.cnt = (uint32_t)__builtin_amdgcn_readlane((int)tot, q);
      }
    }
    if (end || full) break;
    k = k1;
    v = v1;
    k1 = k2;
    v1 = v2;
  }
  if (full && lane == 0) atomicOr(&st->full, 1u);
  pt_most(most, st);
  if (full || part == kNone || !(piece || to == stop)) return;
  // the part's blocks, by their first elements
  __syncthreads();
  const uint64_t base = (uint64_t)part * kPiece;
  uint32_t m = 0;
  for (uint32_t r = from; r < to; r += 64) {
    const uint32_t i = r + lane;
    const bool is = i < to && out[min(i, to - 1)].x == 0u;
    const uint64_t who = __ballot(is);
    if (!who) continue;
    uint32_t fresh;  // none: every block is there
    const uint32_t s = pt_slot(T, is ? K[i] : 0ull, is, sshift, fresh);
    if (is) {
      const uint64_t q = base + m + (uint32_t)__popcll(who & lt);
      pl.elem[q] = i;
      pl.last[q] = s < kLkSlots ? T.last[s] : z.last;
      pl.cnt[q] = s < kLkSlots ? T.cnt[s] : z.cnt;
    }
    m += (uint32_t)__popcll(who);
  }
  if (lane == 0) pl.count[part] = m;
}

// Joins the parts of cut stretches: one wavefront per stretch goes through
// them in order with the stretch's blocks in a table as above, and gives each
// block's first access in a part its previous access and the block's first
// one, out of the parts before.  (The part's other accesses keep that access
// as their first one: k_names goes on from there.)  Bound by the chain of
// loads and LDS operations per part, so the lists and what they point to are
// loaded ahead.  Every wavefront looks at kJoinCuts multiples of kPiece for
// first cuts of stretches; mostly there are few or none.
__global__ __launch_bounds__(64) void k_pt_join(const uint64_t* __restrict__ K,
                                                const uint32_t* __restrict__ V, uint32_t n,
                                                int bits, uint2* __restrict__ out, PtLists pl,
                                                DevStats* st) {
  __shared__ PtTable T;
  if (st->full) return;
  const uint32_t lane = lane_id();
  const int dshift = 64 - bits, sshift = 64 - bits - kLkBits;
  uint64_t heads;
  {
    const uint32_t q = blockIdx.x * kJoinCuts + lane;
    heads = __ballot(lane < kJoinCuts && pt_cut(K, n, dshift, q * kPiece) &&
                     !pt_cut(K, n, dshift, (q - 1) * kPiece));
  }
  uint32_t most = 0;
  for (; heads; heads &= heads - 1) {
    const uint32_t p0 = blockIdx.x * kJoinCuts + (uint32_t)__builtin_ctzll(heads) - 1;
    const uint64_t dg = K[(uint64_t)(p0 + 1) * kPiece] >> dshift;
    pt_clear(T);
    PtZero z;
    uint32_t occ = 0;
    // a part's list: its number of blocks (0 past the stretch), and the first
    // 64 of them; then their hashes and first positions
    struct List {
      uint32_t m, elem, last, cnt;
    };
    const auto load = [&](uint32_t p) {
      const uint32_t at = p * kPiece, i = min(at + lane, n - 1);  // (no overflow: n is at most 2^29)
      const uint64_t kp = K[min(at, n - 1)];
      List x{pl.count[min(p, (n - 1) / kPiece)], pl.elem[i], pl.last[i], pl.cnt[i]};
      if (p > p0 && (p > (n - 1) / kPiece || (kp >> dshift) != dg)) x.m = 0;
      return x;
    };
    // groups of kU parts: one in hand, the next one's blocks and the one after's lists under way
    constexpr int kU = 4;
    List a[kU], b[kU], c[kU];
    uint64_t ka[kU], kb[kU];
    uint32_t va[kU], vb[kU];
    const auto blocks = [&](const List (&x)[kU], uint64_t (&k)[kU], uint32_t (&v)[kU]) {
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const uint32_t el = lane < x[u].m ? x[u].elem : 0u;
        k[u] = K[el];
        v[u] = V[el];
      }
    };
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      a[u] = load(p0 + u);
      b[u] = load(p0 + kU + u);
    }
    blocks(a, ka, va);
    for (uint32_t p = p0; a[0].m; p += kU) {
#pragma unroll
      for (int u = 0; u < kU; ++u) c[u] = load(p + 2 * kU + u);
      blocks(b, kb, vb);
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        for (uint32_t e = 0; e < a[u].m; e += 64) {
          const bool in = e + lane < a[u].m;
          uint32_t el = a[u].elem, last = a[u].last, cnt = a[u].cnt, v = va[u];
          uint64_t k = ka[u];
          if (e) {
            const uint32_t i = (p + u) * kPiece + min(e + lane, a[u].m - 1);
            el = pl.elem[i];
            last = pl.last[i];
            cnt = pl.cnt[i];
            k = K[el];
            v = V[el];
          }
          if (occ + 64 > kLkSlots) {  // too many distinct blocks: the load is redone by sorting
            if (lane == 0) atomicOr(&st->full, 1u);
            return;
          }
          uint32_t fresh;
          const uint32_t s = pt_slot(T, k, in, sshift, fresh);
          occ += fresh;
          const bool tab = in && s < kLkSlots;
          const uint32_t l = tab ? T.last[s] : z.last;
          const uint32_t f = l == kNone ? v : tab ? T.first[s] : z.first;
          if (in && l != kNone) {
            out[el] = make_uint2(l + 1u, f);
            cnt += tab ? T.cnt[s] : z.cnt;
          }
          if (in) most = max(most, cnt);
          if (tab) {
            T.last[s] = last;
            T.first[s] = f;
            T.cnt[s] = cnt;
          }
          if (const uint64_t m0 = __ballot(in && !tab)) {
            const int q = __builtin_ctzll(m0);
            z.last = (uint32_t)__builtin_amdgcn_readlane((int)last, q);
            z.first = (uint32_t)__builtin_amdgcn_readlane((int)f, q);
            z.cnt = (uint32_t)__builtin_amdgcn_readlane((int)cnt, q);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        a[u] = b[u];
        b[u] = c[u];
        ka[u] = kb[u];
        va[u] = vb[u];
      }
    }
  }
  pt_most(most, st);
}

// One partition pass undone: out[i] = in[dst[i]].
__global__ __launch_bounds__(256) void k_pt_undo(const uint2* __restrict__ in,
                                                 const uint32_t* __restrict__ dst, uint64_t n,
                                                 uint2* __restrict__ out, const DevStats* st) {
  if (st->full) return;
  constexpr int kU = 4;
  for (uint64_t b = (uint64_t)blockIdx.x * (256 * kU) + threadIdx.x; b < n;
       b += (uint64_t)gridDim.x * (256 * kU)) {
    uint32_t d[kU];
    uint2 x[kU];
#pragma unroll
    for (int e = 0; e < kU; ++e) d[e] = dst[min(b + e * 256, n - 1)];
#pragma unroll
    for (int e = 0; e < kU; ++e) x[e] = in[d[e]];
#pragma unroll
    for (int e = 0; e < kU; ++e)
      if (b + e * 256 < n) out[b + e * 256] = x[e];
  }
}

// The first pass undone: links and first positions in trace order; the first
// accesses as bits, and their number, per 64 positions; no next links yet.
__global__ __launch_bounds__(256) void k_place(const uint2* __restrict__ in,
                                               const uint32_t* __restrict__ dst, uint64_t n,
                                               uint32_t* __restrict__ key,
                                               uint32_t* __restrict__ fpos,
                                               uint32_t* __restrict__ nxt,
                                               uint64_t* __restrict__ fbits,
                                               uint32_t* __restrict__ fcnt, const DevStats* st) {
  if (st->full) return;  // not every link was made
  constexpr int kU = 4;
  const uint64_t words = (n + 63) / 64;
  // a wavefront takes kU words of 64 positions
  for (uint64_t w0 = ((uint64_t)blockIdx.x * 4 + threadIdx.x / 64) * kU; w0 < words;
       w0 += (uint64_t)gridDim.x * 4 * kU) {
    uint32_t d[kU];
    uint2 x[kU];
#pragma unroll
    for (int e = 0; e < kU; ++e) d[e] = dst[min((w0 + e) * 64 + lane_id(), n - 1)];
#pragma unroll
    for (int e = 0; e < kU; ++e) x[e] = in[d[e]];
#pragma unroll
    for (int e = 0; e < kU; ++e) {
      const uint64_t i = (w0 + e) * 64 + lane_id();
      const uint64_t m = __ballot(i < n && x[e].x == 0u);
      if (i < n) {
        key[i] = x[e].x;
        fpos[i] = x[e].y;
        nxt[i] = kNone;
      }
      if (lane_id() == 0 && w0 + e < words) {
        fbits[w0 + e] = m;
        fcnt[w0 + e] = (uint32_t)__popcll(m);
      }
    }
  }
}

// Dense ids (the rank of the block's first access among all first accesses, so
// that blocks met close together in the trace sit close together in the
// per-block state arrays), next links, per-block tables and totals; every
// access carries the weight and group of its block's first.
__global__ __launch_bounds__(256) void k_names(const uint32_t* __restrict__ key,
                                               const uint32_t* __restrict__ fpos, uint64_t n,
                                               const uint64_t* __restrict__ fbits,
                                               const uint32_t* __restrict__ fpre,
                                               const uint8_t* __restrict__ w8,
                                               const uint8_t* __restrict__ g8,
                                               uint32_t* __restrict__ nxt,
                                               uint32_t* __restrict__ bid,
                                               uint8_t* __restrict__ blk_w,
                                               uint8_t* __restrict__ blk_g, DevStats* st) {
  __shared__ unsigned long long su[KV_MAX_GROUPS], suw[KV_MAX_GROUPS];
  if (st->full) return;  // the first positions are not all there
  if (threadIdx.x < KV_MAX_GROUPS) {
    su[threadIdx.x] = 0;
    suw[threadIdx.x] = 0;
  }
  __syncthreads();
  constexpr int kU = 4;
  bool bad = false;
  uint32_t cg = 0xFFFFFFFFu;
  unsigned long long cn = 0, cw = 0;
  for (uint64_t b = (uint64_t)blockIdx.x * (256 * kU) + threadIdx.x; b < n;
       b += (uint64_t)gridDim.x * (256 * kU)) {
    uint32_t k[kU], f[kU], w[kU], g[kU];
#pragma unroll
    for (int e = 0; e < kU; ++e) {
      const uint64_t i = min(b + e * 256, n - 1);
      k[e] = key[i];
      f[e] = fpos[i];
      w[e] = w8[i];
      g[e] = g8[i];
    }
    uint64_t m[kU];
    uint32_t p[kU], wf[kU], gf[kU];
#pragma unroll
    for (int e = 0; e < kU; ++e) {
      m[e] = fbits[f[e] >> 6];
      p[e] = fpre[f[e] >> 6];
      wf[e] = w8[f[e]];
      gf[e] = g8[f[e]];
    }
    // the first access of a later part of a cut stretch: on to the block's own
#pragma unroll
    for (int e = 0; e < kU; ++e) {
      if ((m[e] >> (f[e] & 63)) & 1ull) continue;
      f[e] = fpos[f[e]];
      m[e] = fbits[f[e] >> 6];
      p[e] = fpre[f[e] >> 6];
    }
#pragma unroll
    for (int e = 0; e < kU; ++e) {
      const uint64_t i = b + e * 256;
      if (i >= n) continue;
      const uint32_t id = p[e] + (uint32_t)__popcll(m[e] & ((1ull << (f[e] & 63)) - 1));
      bid[i] = id;
      if (k[e]) nxt[k[e] - 1u] = (uint32_t)i;
      bad |= w[e] != wf[e] || g[e] != gf[e];
      if (k[e] == 0u) {
        blk_w[id] = (uint8_t)w[e];
        blk_g[id] = (uint8_t)g[e];
        if (g[e] != cg) {
          if (cn) {
            atomicAdd(&su[cg], cn);
            atomicAdd(&suw[cg], cw);
          }
          cg = g[e];
          cn = 0;
          cw = 0;
        }
        ++cn;
        cw += w[e];
      }
      if (i + 1 == n) {
        const uint64_t wl = i >> 6;
        st->u = fpre[wl] + (uint32_t)__popcll(fbits[wl]);
      }
    }
  }
  if (cn) {
    atomicAdd(&su[cg], cn);
    atomicAdd(&suw[cg], cw);
  }
  if (__ballot(bad) != 0ull && lane_id() == 0) atomicOr(&st->err, (uint32_t)kErrInconsistent);
  __syncthreads();
  if (threadIdx.x < KV_MAX_GROUPS) {
    if (su[threadIdx.x]) atomicAdd(&st->u_g[threadIdx.x], su[threadIdx.x]);
    if (suw[threadIdx.x]) atomicAdd(&st->u_w_g[threadIdx.x], suw[threadIdx.x]);
  }
}

// Digit histogram of one tile: counts[digit * ntiles + tile].
__global__ __launch_bounds__(kRsNT) void k_rs_count(const uint64_t* __restrict__ keys, uint64_t n,
                                                    int shift, uint32_t* __restrict__ counts,
                                                    uint32_t ntiles) {
  __shared__ uint32_t h[kRsDigits];
  if (threadIdx.x < kRsDigits) h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t base = (uint64_t)blockIdx.x * kRsTile;
  const uint32_t lane = lane_id();
#pragma unroll
  for (int e = 0; e < kRsItems; ++e) {
    const uint64_t i = base + (uint64_t)e * kRsNT + threadIdx.x;
    const bool valid = i < n;
    const uint32_t d = valid ? (uint32_t)(keys[i] >> shift) & 255u : 0u;
    // lanes of the wavefront with the same digit (8 ballots): the highest
    // adds their number, so no two lanes of one atomic share an address
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    if (valid && (peers >> lane) == 1ull) atomicAdd(&h[d], (uint32_t)__popcll(peers));
  }
  __syncthreads();
  if (threadIdx.x < kRsDigits) counts[(uint64_t)threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one tile given the exclusive digit offsets.  The tile
// is first put in digit order in LDS, then written out position by position,
// so that neighbouring threads write neighbouring words of one digit's run.
__global__ __launch_bounds__(kRsNT) void k_rs_scatter(const uint64_t* __restrict__ kin,
                                                      const uint32_t* __restrict__ vin,
                                                      uint64_t* __restrict__ kout,
                                                      uint32_t* __restrict__ vout, uint64_t n,
                                                      int shift,
                                                      const uint32_t* __restrict__ offsets,
                                                      uint32_t ntiles) {
  __shared__ uint32_t wcnt[kRsWaves][kRsDigits];
  __shared__ uint32_t gbase[kRsDigits];   // the digit's first output position, less its tile start
  __shared__ uint32_t red[kRsWaves];
  __shared__ uint64_t sk[kRsTile];
  __shared__ uint32_t sv[kRsTile];
  const int w = threadIdx.x / 64;
  const uint32_t lane = lane_id();
  for (int d = threadIdx.x; d < kRsWaves * kRsDigits; d += kRsNT) (&wcnt[0][0])[d] = 0;
  const uint32_t g0 =
      threadIdx.x < kRsDigits ? offsets[(uint64_t)threadIdx.x * ntiles + blockIdx.x] : 0u;
  __syncthreads();
  const uint64_t t0 = (uint64_t)blockIdx.x * kRsTile;
  const uint64_t base = t0 + (uint64_t)w * (kRsItems * 64);
  uint64_t k[kRsItems];
  uint32_t v[kRsItems], d[kRsItems], rk[kRsItems];
  const uint64_t lt = lanemask_lt();
#pragma unroll
  for (int r = 0; r < kRsItems; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    const bool valid = i < n;
    k[r] = valid ? kin[i] : 0ull;
    v[r] = valid ? vin[i] : 0u;
    d[r] = (uint32_t)(k[r] >> shift) & 255u;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d[r] >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t before = (uint32_t)__popcll(peers & lt);
    const uint32_t cnt = (uint32_t)__popcll(peers);
    const uint32_t cur = wcnt[w][d[r]];
    rk[r] = cur + before;
    const bool leader = valid && ((peers >> lane) == 1ull);
    if (leader) wcnt[w][d[r]] = cur + cnt;
  }
  __syncthreads();
  {
    // per digit (one per thread of the first kRsDigits): the tile's count,
    // its start in the tile's digit order (a block scan), and each wave's
    // start inside it
    const int dg = threadIdx.x;
    const bool has = dg < kRsDigits;
    uint32_t tot = 0;
    if (has) {
#pragma unroll
      for (int ww = 0; ww < kRsWaves; ++ww) tot += wcnt[ww][dg];
    }
    uint32_t all;
    const uint32_t ls = block_excl_scan_u32<kRsNT, false>(tot, red, all);
    if (has) {
      uint32_t run = ls;
#pragma unroll
      for (int ww = 0; ww < kRsWaves; ++ww) {
        const uint32_t c = wcnt[ww][dg];
        wcnt[ww][dg] = run;
        run += c;
      }
      gbase[dg] = g0 - ls;
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRsItems; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    if (i < n) {
      const uint32_t lp = wcnt[w][d[r]] + rk[r];
      sk[lp] = k[r];
      sv[lp] = v[r];
    }
  }
  __syncthreads();
  const uint32_t m = (uint32_t)min<uint64_t>(kRsTile, n - t0);
  for (uint32_t p = threadIdx.x; p < m; p += kRsNT) {
    const uint64_t key = sk[p];
    const uint32_t dst = gbase[(uint32_t)(key >> shift) & 255u] + p;
    kout[dst] = key;
    vout[dst] = sv[p];
  }
}

// Run starts in hash order: the first element of every group of equal
// hashes (its first occurrence: ties in the sort go by position).
__global__ __launch_bounds__(256) void k_run_flags(const uint64_t* __restrict__ K, uint64_t n,
                                                   uint32_t* __restrict__ newflag) {
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (uint64_t)gridDim.x * blockDim.x)
    newflag[k] = (k == 0 || K[k - 1] != K[k]) ? 1u : 0u;
}

// Neighbours in hash order are the previous / next occurrences.  Both links
// of a position and its block id go out in one 16-byte scatter (link, next,
// id), split into the three arrays by a pass in position order.  Dense block
// ids follow the order of first occurrence (the rank of the block's first
// position among all first positions), so that blocks met close together in
// the trace sit close together in the per-block state arrays.  At a run
// start the block's weight and group go into the per-block tables.
__global__ __launch_bounds__(256) void k_links(const uint64_t* __restrict__ K,
                                               const uint32_t* __restrict__ V, uint64_t n,
                                               const uint32_t* __restrict__ incl,
                                               const uint32_t* __restrict__ newflag,
                                               const uint32_t* __restrict__ firstpos,
                                               const uint32_t* __restrict__ fincl,
                                               uint4* __restrict__ kn,
                                               uint8_t* __restrict__ blk_w,
                                               uint8_t* __restrict__ blk_g,
                                               uint32_t* __restrict__ runstart,
                                               const uint8_t* __restrict__ w8,
                                               const uint8_t* __restrict__ g8, DevStats* st) {
  __shared__ unsigned long long su[KV_MAX_GROUPS], suw[KV_MAX_GROUPS];
  if (threadIdx.x < KV_MAX_GROUPS) {
    su[threadIdx.x] = 0;
    suw[threadIdx.x] = 0;
  }
  __syncthreads();
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (uint64_t)gridDim.x * blockDim.x) {
    const uint64_t h = K[k];
    const uint32_t pos = V[k];
    const bool sp = newflag[k] == 0u;
    const bool sn = k + 1 < n && K[k + 1] == h;
    const uint32_t key = sp ? V[k - 1] + 1u : 0u;
    const uint32_t nx = sn ? V[k + 1] : kNone;
    const uint32_t run = incl[k] - 1u;
    const uint32_t id = fincl[firstpos[run]] - 1u;
    // a streaming store: each record lands alone in its line
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 rec = {key, nx, id, 0u};
    __builtin_nontemporal_store(rec, reinterpret_cast<u32x4*>(kn) + pos);
    if (!sp) {
      const uint8_t w = w8[pos], g = g8[pos];
      blk_w[id] = w;
      blk_g[id] = g;
      runstart[run] = (uint32_t)k;
      atomicAdd(&su[g], 1ull);
      atomicAdd(&suw[g], (unsigned long long)w);
    }
  }
  __syncthreads();
  if (threadIdx.x < KV_MAX_GROUPS) {
    if (su[threadIdx.x]) atomicAdd(&st->u_g[threadIdx.x], su[threadIdx.x]);
    if (suw[threadIdx.x]) atomicAdd(&st->u_w_g[threadIdx.x], suw[threadIdx.x]);
  }
}

__global__ __launch_bounds__(256) void k_split_links(const uint4* __restrict__ kn, uint64_t n,
                                                     uint32_t* __restrict__ key,
                                                     uint32_t* __restrict__ nxt,
                                                     uint32_t* __restrict__ bid) {
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
       p += (uint64_t)gridDim.x * blockDim.x) {
    const uint4 x = kn[p];
    key[p] = x.x;
    nxt[p] = x.y;
    bid[p] = x.z;
  }
}

// Every access carries its block's weight and group (those of the block's
// first occurrence): read in position order, against the per-block tables.
__global__ __launch_bounds__(256) void k_check_blocks(const uint32_t* __restrict__ bid,
                                                      const uint8_t* __restrict__ blk_w,
                                                      const uint8_t* __restrict__ blk_g,
                                                      const uint8_t* __restrict__ w8,
                                                      const uint8_t* __restrict__ g8, uint64_t n,
                                                      DevStats* st) {
  bool bad = false;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n;
       p += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t id = bid[p];
    bad |= w8[p] != blk_w[id] || g8[p] != blk_g[id];
  }
  if (__ballot(bad) != 0ull && lane_id() == 0) atomicOr(&st->err, (uint32_t)kErrInconsistent);
}

// Position of each hash group's first element (its first occurrence), and
// a flag at that position in trace order.
__global__ __launch_bounds__(256) void k_first_pos(const uint32_t* __restrict__ V,
                                                   const uint32_t* __restrict__ incl,
                                                   const uint32_t* __restrict__ newflag,
                                                   uint64_t n, uint32_t* __restrict__ firstpos,
                                                   uint32_t* __restrict__ firstflag) {
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (uint64_t)gridDim.x * blockDim.x)
    if (newflag[k]) {
      const uint32_t pos = V[k];
      firstpos[incl[k] - 1u] = pos;
      firstflag[pos] = 1u;
    }
}

__global__ __launch_bounds__(256) void k_mult(const uint32_t* __restrict__ incl,
                                              const uint32_t* __restrict__ newflag, uint64_t n,
                                              const uint32_t* __restrict__ runstart,
                                              DevStats* st) {
  unsigned long long best = 0;
  for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
       k += (uint64_t)gridDim.x * blockDim.x) {
    const bool last = (k + 1 == n) || newflag[k + 1];
    if (last) {
      const uint32_t id = incl[k] - 1u;
      best = max(best, (unsigned long long)(k - runstart[id] + 1));
    }
  }
#pragma unroll
  for (int dd = 32; dd >= 1; dd >>= 1) best = max(best, (unsigned long long)__shfl_xor(best, dd, 64));
  // one global atomic per block: atomics of many blocks on one address
  // are taken one at a time
  __shared__ unsigned long long sb[256 / 64];
  if (lane_id() == 0) sb[threadIdx.x / 64] = best;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = 0;
    for (int w = 0; w < 256 / 64; ++w) m = max(m, sb[w]);
    if (m) atomicMax(&st->mult, m);
  }
}

// Partitioned order: inverse permutation and remapped links.
__global__ __launch_bounds__(256) void k_part_inverse(const uint32_t* __restrict__ perm,
                                                      uint64_t n, uint32_t* __restrict__ ppos) {
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (uint64_t)gridDim.x * blockDim.x)
    ppos[perm[q]] = (uint32_t)q;
}

__global__ __launch_bounds__(256) void k_part_build(
    const uint32_t* __restrict__ perm, const uint32_t* __restrict__ ppos, uint64_t n,
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ nxt,
    const uint32_t* __restrict__ bid, const uint8_t* __restrict__ w8,
    const uint8_t* __restrict__ g8, uint32_t* __restrict__ pkey, uint32_t* __restrict__ pnxt,
    uint32_t* __restrict__ pbid, uint8_t* __restrict__ pw, uint8_t* __restrict__ pg) {
  for (uint64_t q = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n;
       q += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t i = perm[q];
    const uint32_t kk = key[i];
    const uint32_t nx = nxt[i];
    pkey[q] = kk ? ppos[kk - 1u] + 1u : 0u;
    pnxt[q] = (nx != kNone) ? ppos[nx] : kNone;
    pbid[q] = bid[i];
    pw[q] = w8[i];
    pg[q] = g8[i];
  }
}

__global__ void k_group_keys(const uint8_t* __restrict__ g8, uint64_t n,
                             uint64_t* __restrict__ keys, uint32_t* __restrict__ vals) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    keys[i] = g8[i];
    vals[i] = (uint32_t)i;
  }
}

uint32_t grid_of(uint64_t m, uint64_t cap = 32768) {
  uint64_t g = (m + 255) / 256;
  if (g > cap) g = cap;
  return (uint32_t)(g ? g : 1);
}

// Grids of the kernels that end with global atomics on one address per
// block (trace statistics): a few blocks per compute unit, so that few
// atomics queue on each address.
constexpr uint64_t kReduceGrid = 1024;

// Unused entries of the block tables from which on they are cut to size.
constexpr uint64_t kTrimBlocks = 1u << 24;

// Test hooks, read at every load: KVCFG_TEST_LOAD_SORT=1 takes the radix sort;
// KVCFG_TEST_LOAD_BITS lowers the most partition bits, so that a short trace
// has long stretches, and has them cut.
bool sort_forced() {
  const char* e = std::getenv("KVCFG_TEST_LOAD_SORT");
  return e && e[0] == '1';
}

int most_bits() {
  const char* e = std::getenv("KVCFG_TEST_LOAD_BITS");
  return e ? std::min(2 * kPtBits, std::max(1, std::atoi(e))) : 2 * kPtBits;
}

// One stable LSD pass over (keys, vals) on digit `shift`.
kv_status radix_pass(const uint64_t* kin, const uint32_t* vin, uint64_t* kout, uint32_t* vout,
                     uint64_t n, int shift, uint32_t* counts, uint32_t* scan_scratch,
                     hipStream_t s) {
  const uint32_t ntiles = div_up(n, kRsTile);
  hipLaunchKernelGGL(k_rs_count, dim3(ntiles), dim3(kRsNT), 0, s, kin, n, shift, counts, ntiles);
  KV_HIP(hipGetLastError());
  kv_status st = scan_u32(counts, counts, (uint64_t)ntiles * 256, false, scan_scratch, s);
  if (st != KV_OK) return st;
  hipLaunchKernelGGL(k_rs_scatter, dim3(ntiles), dim3(kRsNT), 0, s, kin, vin, kout, vout, n,
                     shift, counts, ntiles);
  KV_HIP(hipGetLastError());
  return KV_OK;
}

}  // namespace

// Links, ids and block tables by a stable radix sort of (hash, position)
// pairs; the statistics of k_load_tiles are there already.
static kv_status canon_sorted(Trace& t, const kv_trace_desc& d, DevStats* dstats, DevBuf& counts,
                              DevBuf& scratch, hipStream_t s) {
  const uint64_t n = d.n;
  kv_status st;
  Order& o = t.shared;
  const uint32_t ntiles = div_up(n, kRsTile);
  const uint64_t ncount = (uint64_t)ntiles * 256;
  const uint64_t scratch_elems = std::max(scan_scratch_elems(ncount), scan_scratch_elems(n));
  DevBuf ka, kb, va, vb, kn, fl;
  if ((st = ka.reserve(n * 8)) != KV_OK) return st;
  if ((st = kb.reserve(n * 8)) != KV_OK) return st;
  if ((st = va.reserve(n * 4)) != KV_OK) return st;
  if ((st = vb.reserve(n * 4)) != KV_OK) return st;
  if ((st = kn.reserve(n * 16)) != KV_OK) return st;
  // trace-order first-occurrence flags, their inclusive sums, the groups'
  // first positions (u <= n)
  if ((st = fl.reserve(n * 12)) != KV_OK) return st;
  if ((st = counts.reserve(std::max<uint64_t>(ncount, 1) * 4)) != KV_OK) return st;
  if ((st = scratch.reserve(std::max<uint64_t>(scratch_elems, 1) * 4)) != KV_OK) return st;
  uint64_t *kin = ka.as<uint64_t>(), *kout = kb.as<uint64_t>();
  uint32_t *vin = va.as<uint32_t>(), *vout = vb.as<uint32_t>();
  {
    StageTimer tm(kStLoadSort, s);
    hipLaunchKernelGGL(k_sort_pairs, dim3(grid_of(n)), dim3(256), 0, s, d.hash, n, kin, vin);
    KV_HIP(hipGetLastError());
    for (int shift = 0; shift < 64; shift += 8) {
      st = radix_pass(kin, vin, kout, vout, n, shift, counts.as<uint32_t>(),
                      scratch.as<uint32_t>(), s);
      if (st != KV_OK) return st;
      std::swap(kin, kout);
      std::swap(vin, vout);
    }
  }
  // kin / vin now hold the sorted pairs; the other pair of buffers is free.
  uint32_t* newflag = reinterpret_cast<uint32_t*>(kout);          // n u32
  uint32_t* incl = reinterpret_cast<uint32_t*>(kout) + n;         // n u32
  uint32_t* firstflag = fl.as<uint32_t>();
  uint32_t* fincl = firstflag + n;
  uint32_t* firstpos = fincl + n;
  uint32_t* runstart = vout;  // n >= u entries available
  StageTimer tm(kStLoadLinks, s);
  hipLaunchKernelGGL(k_run_flags, dim3(grid_of(n)), dim3(256), 0, s, kin, n, newflag);
  KV_HIP(hipGetLastError());
  if ((st = scan_u32(newflag, incl, n, true, scratch.as<uint32_t>(), s)) != KV_OK) return st;
  if ((st = fill_u32(firstflag, 0u, n, s)) != KV_OK) return st;
  hipLaunchKernelGGL(k_first_pos, dim3(grid_of(n)), dim3(256), 0, s, vin, incl, newflag, n,
                     firstpos, firstflag);
  KV_HIP(hipGetLastError());
  if ((st = scan_u32(firstflag, fincl, n, true, scratch.as<uint32_t>(), s)) != KV_OK) return st;
  hipLaunchKernelGGL(k_links, dim3(grid_of(n, 4 * kReduceGrid)), dim3(256), 0, s, kin, vin, n,
                     incl, newflag, firstpos, fincl, reinterpret_cast<uint4*>(kn.p),
                     t.blk_w.as<uint8_t>(),
                     t.blk_g.as<uint8_t>(), runstart, o.w.as<uint8_t>(), o.g.as<uint8_t>(),
                     dstats);
  KV_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_split_links, dim3(grid_of(n)), dim3(256), 0, s,
                     reinterpret_cast<const uint4*>(kn.p), n, o.key.as<uint32_t>(),
                     o.nxt.as<uint32_t>(), o.bid.as<uint32_t>());
  KV_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_mult, dim3(grid_of(n, kReduceGrid)), dim3(256), 0, s, incl, newflag, n,
                     runstart, dstats);
  KV_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_check_blocks, dim3(grid_of(n)), dim3(256), 0, s, o.bid.as<uint32_t>(),
                     t.blk_w.as<uint8_t>(), t.blk_g.as<uint8_t>(), o.w.as<uint8_t>(),
                     o.g.as<uint8_t>(), n, dstats);
  KV_HIP(hipGetLastError());
  KV_HIP(hipMemcpyAsync(&dstats->u, incl + (n - 1), 4, hipMemcpyDeviceToDevice, s));
  KV_HIP(hipStreamSynchronize(s));  // the buffers above go back to the cache
  return KV_OK;
}

kv_status canon_build(Trace& t, const kv_trace_desc& d, hipStream_t s) {
  const uint64_t n = d.n;
  kv_status st;
  Order& o = t.shared;
  if ((st = o.key.reserve(n * 4)) != KV_OK) return st;
  if ((st = o.nxt.reserve(n * 4)) != KV_OK) return st;
  if ((st = o.bid.reserve(n * 4)) != KV_OK) return st;
  if ((st = o.w.reserve(n)) != KV_OK) return st;
  if ((st = o.g.reserve(n)) != KV_OK) return st;
  // per block, for up to n of them: their number is known only at the end
  if ((st = t.blk_w.reserve(n)) != KV_OK) return st;
  if ((st = t.blk_g.reserve(n)) != KV_OK) return st;
  // the request of every access and the request times, kept for the
  // inter-arrival times of the TTL curves
  if ((st = t.req.reserve(n * 4)) != KV_OK) return st;
  if ((st = t.req_time.reserve((uint64_t)d.n_req * 8)) != KV_OK) return st;

  // Partition bits: stretches of 256 to 512 accesses on average, whose distinct
  // blocks, with those a stretch may start with, stay below the linking
  // table's 960; two digits from 10 bits on.
  int bits = 1;
  while (bits < most_bits() && (n >> bits) > 512) ++bits;
  const int hi_bits = bits < kPtBits ? bits : (bits + 1) / 2, lo_bits = bits - hi_bits;
  const uint32_t hi = 1u << hi_bits, lo = 1u << lo_bits;
  const bool two = lo_bits > 0;
  const uint32_t ntiles = div_up(n, kRsTile);
  const uint64_t words = (n + 63) / 64;
  const uint64_t ncount = (uint64_t)ntiles * std::max(hi, lo);
  const uint64_t scratch_elems = std::max(scan_scratch_elems(ncount), scan_scratch_elems(words));
  DevBuf ka, kb, va, vb, d1, d2, counts, scratch, dst;
  if ((st = ka.reserve(n * 8)) != KV_OK) return st;
  if ((st = va.reserve(n * 4)) != KV_OK) return st;
  if ((st = d1.reserve(n * 4)) != KV_OK) return st;
  if ((st = kb.reserve(n * 8)) != KV_OK) return st;
  if (two) {
    if ((st = vb.reserve(n * 4)) != KV_OK) return st;
    if ((st = d2.reserve(n * 4)) != KV_OK) return st;
  }
  if ((st = counts.reserve(ncount * 4)) != KV_OK) return st;
  if ((st = scratch.reserve(std::max<uint64_t>(scratch_elems, 1) * 4)) != KV_OK) return st;
  if ((st = dst.reserve(sizeof(DevStats))) != KV_OK) return st;
  DevStats* dstats = dst.as<DevStats>();
  uint32_t* cnt = counts.as<uint32_t>();
  {
    StageTimer tm(kStLoadValidate, s);
    hipLaunchKernelGGL(k_load_init, dim3(1), dim3(64), 0, s, dstats,
                       t.err.as<uint32_t>());
    KV_HIP(hipGetLastError());
    const uint32_t grid = (uint32_t)std::min<uint64_t>(
        std::max<uint64_t>(ntiles, div_up(d.n_req, kRsTile)), kReduceGrid);
    hipLaunchKernelGGL(k_load_tiles, dim3(grid), dim3(kRsNT), 0, s, d.hash, d.req, d.group,
                       d.weight, n, d.req_time, d.n_req, d.n_groups, t.req.as<uint32_t>(),
                       t.req_time.as<double>(), o.g.as<uint8_t>(), o.w.as<uint8_t>(),
                       two ? 64 - bits : 64 - hi_bits, two ? lo : hi, cnt, ntiles, dstats);
    KV_HIP(hipGetLastError());
  }
  const bool sorted = sort_forced();
  if (!sorted) {
    // low digit first, then the high one: in the end equal top bits are consecutive
    uint64_t *K = ka.as<uint64_t>(), *K2 = kb.as<uint64_t>();
    uint32_t *V = va.as<uint32_t>(), *V2 = vb.as<uint32_t>();
    uint2* links;   // (key, first position), partitioned
    {
      StageTimer tm(kStLoadSort, s);
      const uint32_t dg = two ? lo : hi;
      if ((st = scan_u32(cnt, cnt, (uint64_t)ntiles * dg, false, scratch.as<uint32_t>(), s)) !=
          KV_OK)
        return st;
      // digits of 10 bits only past 2^27 accesses: their runs of 8 elements a
      // tile are scattered more slowly
      const auto scatter = [&](auto narrow, auto wide, uint32_t digits, const uint64_t* kin,
                               const uint32_t* vin, uint64_t* kout, uint32_t* vout, uint32_t* to,
                               int shift) {
        hipLaunchKernelGGL(digits < kPtDigits ? narrow : wide, dim3(ntiles), dim3(kRsNT), 0, s, kin,
                           vin, kout, vout, to, n, shift, digits, cnt, ntiles);
      };
      scatter(k_pt_scatter<true, kPtBits - 1>, k_pt_scatter<true, kPtBits>, dg, d.hash, nullptr, K, V,
              d1.as<uint32_t>(), two ? 64 - bits : 64 - hi_bits);
      KV_HIP(hipGetLastError());
      if (two) {
        hipLaunchKernelGGL(k_pt_count, dim3(ntiles), dim3(kRsNT), 0, s, K, n, 64 - hi_bits, hi,
                           cnt, ntiles);
        KV_HIP(hipGetLastError());
        if ((st = scan_u32(cnt, cnt, (uint64_t)ntiles * hi, false, scratch.as<uint32_t>(), s)) !=
            KV_OK)
          return st;
        scatter(k_pt_scatter<false, kPtBits - 1>, k_pt_scatter<false, kPtBits>, hi, K, V, K2, V2,
                d2.as<uint32_t>(), 64 - hi_bits);
        KV_HIP(hipGetLastError());
        std::swap(K, K2);
        std::swap(V, V2);
      }
    }
    StageTimer tm(kStLoadLinks, s);
    links = reinterpret_cast<uint2*>(K2);  // free now
    // wavefronts enough to fill the chip, of whole stretches
    // some 8192 wavefronts, four to each that the chip holds, of 256 to 4096
    // elements (shorter ones only look for a first stretch).  With 256, 512,
    // 1024, 2048, 4096: 26, 35, 44, 69, 100 us for 2.4e5 accesses, 90, 79, 82,
    // 97, 105 us for 4.6e6, 2.29, 2.03, 1.86, 1.76, 1.67 ms for 1.09e8.
    uint32_t chunk = 256;
    while (chunk < 4096 && n >= (uint64_t)chunk * 16384) chunk *= 2;
    // cut stretches' lists, in memory that is written only later
    const PtLists pl{o.key.as<uint32_t>(), o.nxt.as<uint32_t>(), o.bid.as<uint32_t>(), cnt};
    // (one block's 2^14 accesses take one wavefront 0.23 ms, 2^16 0.9 ms; to look
    // for cuts costs each load 5 us)
    const bool cut = n > kCutFrom || most_bits() < 2 * kPtBits;
    const uint32_t chunks = div_up(n, chunk), cuts = cut ? ((uint32_t)n - 1) / kPiece : 0;
    hipLaunchKernelGGL(k_pt_link, dim3(chunks + cuts), dim3(64), 0, s, K, V, (uint32_t)n,
                       cut ? (uint32_t)n : 0u, bits, chunk, chunks, links, pl, dstats);
    KV_HIP(hipGetLastError());
    if (cuts) {
      hipLaunchKernelGGL(k_pt_join, dim3(cuts / kJoinCuts + 1), dim3(64), 0, s, K, V, (uint32_t)n,
                         bits, links, pl, dstats);
      KV_HIP(hipGetLastError());
    }
    uint32_t* fpos = V;                    // free now, as is K
    uint64_t* fbits;
    if (two) {
      uint2* back = reinterpret_cast<uint2*>(K);
      hipLaunchKernelGGL(k_pt_undo, dim3(grid_of(div_up(n, 4))), dim3(256), 0, s, links,
                         d2.as<uint32_t>(), n, back, dstats);
      KV_HIP(hipGetLastError());
      std::swap(links, back);
      fbits = reinterpret_cast<uint64_t*>(back);
    } else {
      fbits = K;
    }
    uint32_t* fpre = reinterpret_cast<uint32_t*>(fbits + words);
    hipLaunchKernelGGL(k_place, dim3(grid_of(div_up(n, 4))), dim3(256), 0, s, links,
                       d1.as<uint32_t>(), n, o.key.as<uint32_t>(), fpos, o.nxt.as<uint32_t>(),
                       fbits, fpre, dstats);
    KV_HIP(hipGetLastError());
    if ((st = scan_u32(fpre, fpre, words, false, scratch.as<uint32_t>(), s)) != KV_OK) return st;
    hipLaunchKernelGGL(k_names, dim3(grid_of(div_up(n, 4), 4 * kReduceGrid)), dim3(256), 0, s,
                       o.key.as<uint32_t>(), fpos, n, fbits, fpre, o.w.as<uint8_t>(),
                       o.g.as<uint8_t>(), o.nxt.as<uint32_t>(), o.bid.as<uint32_t>(),
                       t.blk_w.as<uint8_t>(), t.blk_g.as<uint8_t>(), dstats);
    KV_HIP(hipGetLastError());
  }
  // the statistics come back through the handle's pinned block
  static_assert(sizeof(DevStats) % 16 == 0 && sizeof(DevStats) + 256 <= 4096, "copied in words of 16");
  DevStats& hs = *reinterpret_cast<DevStats*>(t.err_pin->host + 256);
  if ((st = copy_words(dstats, t.err_pin->dev + 256, sizeof(DevStats), s)) != KV_OK) return st;
  KV_HIP(hipStreamSynchronize(s));
  if (sorted || hs.full) {
    // (nothing of the blocks was counted or checked when a table was full)
    for (DevBuf* b : {&ka, &kb, &va, &vb, &d1, &d2}) b->release();
    if ((st = canon_sorted(t, d, dstats, counts, scratch, s)) != KV_OK) return st;
    if ((st = copy_words(dstats, t.err_pin->dev + 256, sizeof(DevStats), s)) != KV_OK) return st;
    KV_HIP(hipStreamSynchronize(s));
  }
  if (hs.err) {
    std::string why;
    if (hs.err & kErrGroup) why += " group id >= n_groups;";
    if (hs.err & kErrWeight) why += " zero weight;";
    if (hs.err & kErrReq) why += " request index out of range or decreasing;";
    if (hs.err & kErrInconsistent) why += " a block hash carries two weights or groups;";
    if (hs.err & kErrTime) why += " request times decreasing or NaN;";
    return fail(KV_ERR_INVALID, "kv_trace_load: invalid trace:" + why);
  }
  const uint64_t u = hs.u;
  // the block tables had room for n blocks; kept for the handle's life, they
  // get what u need where that saves more than the copy's 20 us are worth
  if (n - u >= kTrimBlocks) {
    for (DevBuf* b : {&ka, &kb, &va, &vb, &d1, &d2}) b->release();
    DevBuf own[2];
    DevBuf* const tab[2] = {&t.blk_w, &t.blk_g};
    for (int q = 0; q < 2; ++q) {
      if (own[q].reserve(u) != KV_OK) continue;  // the large table serves as well
      if ((st = copy_words(tab[q]->p, own[q].p, (u + 15) & ~15ull, s)) != KV_OK) return st;
      own[q].swap(*tab[q]);
    }
    KV_HIP(hipStreamSynchronize(s));  // the large tables go back to the cache
  }
  kv_trace_stats& ts = t.st;
  ts = kv_trace_stats{};
  ts.n = n;
  ts.n_distinct = u;
  ts.n_req = d.n_req;
  ts.n_groups = d.n_groups;
  ts.w_min = hs.w_min;
  ts.w_max = hs.w_max;
  ts.max_multiplicity = hs.mult;
  ts.span = hs.t1 - hs.t0;
  for (uint32_t g = 0; g < KV_MAX_GROUPS; ++g) {
    ts.n_g[g] = hs.n_g[g];
    ts.n_w_g[g] = hs.n_w_g[g];
    ts.u_g[g] = hs.u_g[g];
    ts.u_w_g[g] = hs.u_w_g[g];
    ts.n_w += hs.n_w_g[g];
    ts.distinct_w += hs.u_w_g[g];
  }
  o.seg[0] = 0;
  o.seg[1] = n;
  for (uint32_t g = 2; g <= KV_MAX_GROUPS; ++g) o.seg[g] = n;
  o.built = true;
  t.n = n;
  t.u = u;
  t.n_groups = d.n_groups;
  return KV_OK;
}

kv_status canon_partition(Trace& t, hipStream_t s) {
  if (t.part.built) return KV_OK;
  const uint64_t n = t.n;
  kv_status st;
  Order& p = t.part;
  Order& o = t.shared;
  if ((st = p.key.reserve(n * 4)) != KV_OK) return st;
  if ((st = p.nxt.reserve(n * 4)) != KV_OK) return st;
  if ((st = p.bid.reserve(n * 4)) != KV_OK) return st;
  if ((st = p.w.reserve(n)) != KV_OK) return st;
  if ((st = p.g.reserve(n)) != KV_OK) return st;
  const uint32_t ntiles = div_up(n, kRsTile);
  const uint64_t ncount = (uint64_t)ntiles * 256;
  DevBuf ka, kb, va, vb, counts, scratch;
  if ((st = ka.reserve(n * 8)) != KV_OK) return st;
  if ((st = kb.reserve(n * 8)) != KV_OK) return st;
  if ((st = va.reserve(n * 4)) != KV_OK) return st;
  if ((st = vb.reserve(n * 4)) != KV_OK) return st;
  if ((st = counts.reserve(ncount * 4)) != KV_OK) return st;
  if ((st = scratch.reserve(std::max<uint64_t>(scan_scratch_elems(ncount), 1) * 4)) != KV_OK)
    return st;
  StageTimer tm(kStPartition, s);
  hipLaunchKernelGGL(k_group_keys, dim3(grid_of(n)), dim3(256), 0, s, o.g.as<uint8_t>(), n,
                     ka.as<uint64_t>(), va.as<uint32_t>());
  KV_HIP(hipGetLastError());
  st = radix_pass(ka.as<uint64_t>(), va.as<uint32_t>(), kb.as<uint64_t>(), vb.as<uint32_t>(), n,
                  0, counts.as<uint32_t>(), scratch.as<uint32_t>(), s);
  if (st != KV_OK) return st;
  const uint32_t* perm = vb.as<uint32_t>();
  uint32_t* ppos = va.as<uint32_t>();
  hipLaunchKernelGGL(k_part_inverse, dim3(grid_of(n)), dim3(256), 0, s, perm, n, ppos);
  KV_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_part_build, dim3(grid_of(n)), dim3(256), 0, s, perm, ppos, n,
                     o.key.as<uint32_t>(), o.nxt.as<uint32_t>(), o.bid.as<uint32_t>(),
                     o.w.as<uint8_t>(), o.g.as<uint8_t>(), p.key.as<uint32_t>(),
                     p.nxt.as<uint32_t>(), p.bid.as<uint32_t>(), p.w.as<uint8_t>(),
                     p.g.as<uint8_t>());
  KV_HIP(hipGetLastError());
  KV_HIP(hipStreamSynchronize(s));
  p.seg[0] = 0;
  for (uint32_t g = 0; g < KV_MAX_GROUPS; ++g)
    p.seg[g + 1] = p.seg[g] + (g < t.n_groups ? t.st.n_g[g] : 0);
  p.built = true;
  return KV_OK;
}

}  // namespace kv
