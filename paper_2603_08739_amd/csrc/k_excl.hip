// k_excl.hip - exclusive (write-back demotion) hierarchies that are no split
// stack: FIFO and LFU tiers, and LRU tiers over blocks of mixed weights.
//
// In the tier hierarchy of a KV cache (Section 4.1's DRAM and disk below
// HBM) a block can live in one tier at a time: a hit in a lower tier
// promotes the block to the top tier, and a tier that overflows demotes its
// victim to the next tier, dropping it past the last one.  A block entering a
// tier (a miss, a promotion, a demotion) is that tier's newest member - LRU:
// most recently used; FIFO: newest insertion; LFU: count 1, touched now - and
// the tier passes its own victims down before it admits the block.
//
// Two facts take the place of an access-by-access replay of lists:
//  * The top tier never depends on the tiers below it (a hit there enters it
//    as a miss does), so it is an ordinary cache of its policy.
//  * In a lower tier no block is ever touched (a hit takes it out), so under
//    every policy its victim is its oldest entry: each lower tier is a queue,
//    and as a tier's victims leave in the order they entered, all lower tiers
//    are consecutive ranges of one queue - the top tier's demotions in order.
// So a hierarchy is one queue of entries and a head per tier: tier t holds
// the entries from its head to the head above that are still alive (not
// taken out again).  Which entry an access takes out, and when an entry is
// taken out, does not depend on the heads: both are known before the walk.
//
// The queue of each policy:
//  LRU:  entries are the accesses themselves; an access takes out the entry
//        of its block's previous access, and the top tier is the newest
//        range of the same queue.  Nothing has to be prepared: links and
//        weights are the trace's.
//  FIFO: entries are the insertions (the misses of the top tier), again with
//        the top tier as the newest range; a hit of the top tier changes
//        nothing.  The misses come from the chunked FIFO replay.
//  LFU:  entries are the top tier's evictions in order, from the chunked LFU
//        replay; the heads are those of the lower tiers only.
// One such stream serves every configuration with the same top tier; each
// configuration then walks it with its own heads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <tuple>
#include <vector>

#include "kv_device.h"
#include "kv_internal.h"

namespace kv {
namespace {

constexpr int kXNT = 64;           // one wavefront per configuration
constexpr uint32_t kXIt = 4;       // events, and queue entries, per lane and step
constexpr uint32_t kXStep = kXNT * kXIt;
constexpr uint32_t kXStage = 2048; // events staged in LDS at a time
constexpr uint32_t kXWin = 1024;   // queue entries staged in LDS per tier
constexpr uint32_t kXBatch = 16;   // loads of one array in flight per lane
constexpr uint32_t kXShort = 4;    // a step of fewer events is not worth its chain
constexpr uint32_t kXBurst = 64;   // most events taken one by one in a row
static_assert(kXStage % (64 * kXBatch) == 0, "slices are staged in whole batches");
constexpr int kXPrep = 1024;       // threads of the per-stream scans

// A queue and the events that change it.  Event k takes out entry e[k] - 1
// (0: none), whose weight is w[k], and then appends entries until pt[k]
// granules have been appended in all (pt null: one entry per event, of the
// event's weight).  Entry q is taken out at event out[q] (kNone: never).
struct XStream {
  // LRU: the order's links, which are absolute: `base` is the first position
  const uint32_t *e, *pt, *out;
  const uint8_t *w, *g, *qw, *qg;
  const uint32_t* meta;   // {events, entries}; null: `n` of both
  uint32_t n, base;
  // FIFO / LFU preparation
  uint32_t policy;
  uint64_t cap, begin, end;
  const uint32_t *key, *nxt;       // the order's links
  const uint8_t *w8, *g8;          // and its weights and groups
  const uint64_t* bits;            // top tier's hits, words from begin / 64
  const uint32_t* emit;            // the replay's emission, from begin
  const unsigned long long* jcnt;  // the replay's counters [n_groups][4]
  uint32_t *wpre, *ev_e, *ev_pt, *pwi, *en_out, *pq, *cnt;
  uint8_t *ev_w, *ev_g, *en_w, *en_g;
};

// One hierarchy of a configuration.
struct XWalk {
  uint32_t cfg, group;    // group: KV_MAX_GROUPS for a shared hierarchy
  uint32_t stream;        // kNone: no victims at all (the top tier holds every block)
  uint32_t nt;            // heads
  uint32_t cap[KV_TIERS]; // capacity of each head's tier
  uint32_t nlive;         // live tiers
  uint8_t live[KV_TIERS + 1];  // live tiers, fastest first
};

// ---------------------------------------------------------------------------
// preparation of FIFO and LFU streams
// ---------------------------------------------------------------------------

// Misses of word `wi` of a job's hits: the accesses of [begin, end) not hit.
__device__ __forceinline__ uint64_t miss_word(const XStream& x, uint64_t wi) {
  const uint64_t p0 = ((x.begin >> 6) + wi) << 6;
  uint64_t m = ~x.bits[wi];
  if (p0 < x.begin) m &= ~0ull << (x.begin - p0);
  if (p0 + 64 > x.end) m &= ~0ull >> (p0 + 64 - x.end);
  return m;
}

// The number of misses before position p.
__device__ __forceinline__ uint32_t miss_rank(const XStream& x, uint64_t p) {
  const uint64_t wi = (p >> 6) - (x.begin >> 6);
  return x.wpre[wi] + (uint32_t)__popcll(miss_word(x, wi) & ((1ull << (p & 63)) - 1));
}

// Misses before each word of hits; the numbers of events and entries.  One
// workgroup per stream: a few thousand words for a trace of some hundred
// thousand accesses.
__global__ __launch_bounds__(kXPrep) void k_x_rank(const XStream* __restrict__ xs,
                                                   uint32_t n_groups) {
  __shared__ uint32_t sh[2 * (kXPrep / 64)];
  const XStream x = xs[blockIdx.x];
  const uint64_t nw = ((x.end + 63) >> 6) - (x.begin >> 6);
  uint32_t run = 0;
  for (uint64_t w0 = 0; w0 < nw; w0 += kXPrep) {
    const uint64_t wi = w0 + threadIdx.x;
    const uint32_t c = wi < nw ? (uint32_t)__popcll(miss_word(x, wi)) : 0u;
    uint32_t tot;
    const uint32_t pre = block_excl_scan_u32<kXPrep>(c, sh, tot);
    if (wi < nw) x.wpre[wi] = run + pre;
    run += tot;
  }
  if (threadIdx.x == 0) {
    unsigned long long ev = run;
    if (x.policy == KV_POLICY_LFU) {
      ev = 0;
      for (uint32_t g = 0; g < n_groups; ++g) ev += x.jcnt[g * 4 + 2];
    }
    x.cnt[0] = run;
    x.cnt[1] = (uint32_t)ev;
  }
}

// Events and entries of every access: weights, groups, and for LFU which
// entry an event takes out and when an entry is taken out.  (A stay of the
// top tier that ended with an eviction is followed by a miss of its block.)
__global__ __launch_bounds__(256) void k_x_gather(const XStream* __restrict__ xs) {
  const XStream x = xs[blockIdx.y];
  const bool lfu = x.policy == KV_POLICY_LFU;
  for (uint64_t i = x.begin + (uint64_t)blockIdx.x * 256 + threadIdx.x; i < x.end;
       i += (uint64_t)gridDim.x * 256) {
    const uint64_t wi = (i >> 6) - (x.begin >> 6);
    const uint32_t w = x.w8[i], g = x.g8[i];
    const uint32_t em = x.emit[i - x.begin];
    if ((miss_word(x, wi) >> (i & 63)) & 1ull) {
      const uint32_t k = miss_rank(x, i);
      x.ev_w[k] = (uint8_t)w;
      x.ev_g[k] = (uint8_t)g;
      if (lfu) {
        const uint32_t p = x.key[i];
        x.ev_e[k] = p ? x.emit[p - 1 - x.begin] + 1u : 0u;  // evicted, as this is a miss
      } else {
        x.ev_e[k] = em;  // weight before the superseded insertion (k_x_link)
        x.en_out[k] = kNone;
      }
    }
    if (lfu && em != kNone) {
      const uint32_t nx = x.nxt[i];
      x.en_w[em] = (uint8_t)w;
      x.en_g[em] = (uint8_t)g;
      x.en_out[em] = nx == kNone ? kNone : miss_rank(x, nx);
    }
  }
}

// Weight of the events (y = 0) or LFU entries (y = 1) before each, and in all.
__global__ __launch_bounds__(kXPrep) void k_x_weights(const XStream* __restrict__ xs) {
  constexpr uint32_t kIt = 4;
  __shared__ uint32_t sh[2 * (kXPrep / 64)];
  const XStream x = xs[blockIdx.x];
  const bool entries = blockIdx.y != 0;
  if (entries && x.policy != KV_POLICY_LFU) return;
  const uint32_t m = x.cnt[entries ? 1 : 0];
  const uint8_t* w = entries ? x.en_w : x.ev_w;
  uint32_t* out = entries ? x.pq : x.pwi;
  uint32_t run = 0;
  for (uint32_t b = 0; b < m; b += kXPrep * kIt) {
    const uint32_t i0 = b + threadIdx.x * kIt;
    uint32_t v[kIt], s = 0;
#pragma unroll
    for (uint32_t q = 0; q < kIt; ++q) {
      v[q] = i0 + q < m ? w[i0 + q] : 0u;
      s += v[q];
    }
    uint32_t tot;
    uint32_t pre = run + block_excl_scan_u32<kXPrep>(s, sh, tot);
#pragma unroll
    for (uint32_t q = 0; q < kIt; ++q) {
      if (i0 + q < m) out[i0 + q] = pre;
      pre += v[q];
    }
    run += tot;
  }
  if (threadIdx.x == 0) out[m] = run;
}

// FIFO: the entry an event takes out, from the weight inserted before it.
// LFU: the weight evicted by each event - the fewest evictions, in order,
// after which the cached weight with the event's block fits.
__global__ __launch_bounds__(256) void k_x_link(const XStream* __restrict__ xs) {
  const XStream x = xs[blockIdx.y];
  const uint32_t m = x.cnt[0], ne = x.cnt[1];
  for (uint32_t k = blockIdx.x * 256 + threadIdx.x; k < m; k += gridDim.x * 256) {
    if (x.policy == KV_POLICY_LFU) {
      const uint32_t in = x.pwi[k + 1];
      x.ev_pt[k] = in > x.cap ? x.pq[lower_bound(x.pq, 0u, ne, (uint32_t)(in - x.cap))] : 0u;
    } else {
      const uint32_t s = x.ev_e[k];
      uint32_t e = 0;
      if (s != kNone) {
        const uint32_t q = lower_bound(x.pwi, 0u, k, s);  // weights are positive: one such q
        e = q + 1;
        x.en_out[q] = k;
      }
      x.ev_e[k] = e;
    }
  }
}

// ---------------------------------------------------------------------------
// the walk
// ---------------------------------------------------------------------------
struct WalkLds {
  uint32_t e[kXStage], pt[kXStage];
  uint8_t w[kXStage], g[kXStage];
  uint32_t out[KV_TIERS][kXWin];
  uint8_t qw[KV_TIERS][kXWin];
  uint32_t pref[kXStep];
  unsigned long long hit[KV_MAX_GROUPS][KV_TIERS][2], ev[KV_MAX_GROUPS][KV_TIERS][2];
};

__device__ __forceinline__ uint32_t lane_u32(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

// Inclusive prefix sums of the lanes' kXIt consecutive values (lane by lane),
// and the total of all.
__device__ __forceinline__ uint32_t step_scan(const uint32_t (&v)[kXIt], uint32_t (&incl)[kXIt]) {
  uint32_t s = 0;
#pragma unroll
  for (uint32_t r = 0; r < kXIt; ++r) {
    s += v[r];
    incl[r] = s;
  }
  const uint32_t through = wave_incl_scan_u32(s);
#pragma unroll
  for (uint32_t r = 0; r < kXIt; ++r) incl[r] += through - s;
  return lane_u32(through, 63);
}

// Walks one hierarchy's events, up to 256 at a time, four consecutive ones per
// lane.  With the entries alive at the step's first event, tier t must have
// let go, by event k, of  max over j <= k of (arrived by j - taken out by j -
// room): both sums are prefix sums over the step, and the entries that go are
// the shortest stretch from the head that weighs as much.  What leaves a tier
// arrives in the next.  This holds as long as no event of the step takes out
// an entry that a head passes in the same step; the events before the first
// such event are taken alone, and that event by itself.  Heads stand far
// behind the entries in use unless a tier is small, so steps are nearly always
// whole (638 steps for 160,001 accesses at the smallest capacities of a
// weighted mix).
//
// Where blocks come back within the few entries of small tiers, that event
// comes after a few others time and again.  Then events are taken one by one,
// the lanes searching a tier's next 64 entries: one at first, and up to
// kXBurst in a row while steps stay under kXShort events.  An event by itself
// takes a microsecond; a step takes two, whatever its length, and a short one
// up to three tries (500 accesses to 125 blocks, tiers of 4 to 40 granules: 1.4
// to 1.6 ms with a step for every such event, 0.65 to 0.95 with lists replayed
// access by access, now 0.55 to 1.05; kXShort = 12 doubled the time of some
// hierarchies that steps of 5 to 10 events serve well).
//
// Bound by the wavefront's dependent chain per step (a few scans and LDS
// round trips per tier), so a lane takes four events; the events and queue
// entries are streamed through LDS in slices, 16 loads in flight per lane
// (one load at a time: 3.8 ms instead of 2.0 ms for the walks below; one
// event per lane: 6.6 ms).  Measured: 64 FIFO and LFU hierarchies over
// 238,313 accesses of unit weight walk in 2.0 ms, 48 of every policy over
// 160,001 accesses of weights 1 and 4 in 4.2 ms; whole evaluations 355 ->
// 3.6 ms and 460 -> 6.7 ms (lists replayed access by access, before; the
// second 6.2 to 9.6 ms by the trace).
// wu: the weight of every block, or 0 when weights differ.
template <bool kOne>
__device__ void walk(const XStream& x, const XWalk& j, uint32_t wu, WalkLds& S, uint32_t g0,
                     bool& bad) {
  const uint32_t lane = lane_id();
  const uint32_t n_ev = x.meta ? x.meta[0] : x.n, n_en = x.meta ? x.meta[1] : x.n;
  const uint32_t nt = j.nt;
  uint32_t H[KV_TIERS] = {0, 0, 0}, room[KV_TIERS], wb[KV_TIERS];
  // hits and departures: each lane's number, all lanes' weight (no sum of
  // weights reaches 2^32)
  uint32_t hc[KV_TIERS] = {0, 0, 0}, hw[KV_TIERS] = {0, 0, 0};
  uint32_t ec[KV_TIERS] = {0, 0, 0}, ew[KV_TIERS] = {0, 0, 0};
#pragma unroll
  for (uint32_t t = 0; t < KV_TIERS; ++t) {
    room[t] = j.cap[t];
    wb[t] = kNone;  // no window staged
  }
  uint32_t send = 0, sbase = 0, ptb = 0, step = kXStep, burst = 0, k0 = 0;
  // stages tier t's window of the queue, from entry `base` on
  const auto window = [&](uint32_t t, uint32_t base) {
    __syncthreads();
    uint32_t so[kXWin / 64], sq[kXWin / 64];
#pragma unroll
    for (uint32_t r = 0; r < kXWin / 64; ++r) {
      const uint32_t q = min(base + lane + 64 * r, n_en - 1);
      so[r] = x.out[x.base + q];
      sq[r] = x.qw[x.base + q];
    }
#pragma unroll
    for (uint32_t r = 0; r < kXWin / 64; ++r) {
      const bool is = base + lane + 64 * r < n_en;  // past the queue: no weight
      S.out[t][lane + 64 * r] = so[r] == kNone ? kNone : so[r] - x.base;
      S.qw[t][lane + 64 * r] = is ? (uint8_t)sq[r] : (uint8_t)0;
    }
    __syncthreads();
  };
  // takes staged events one by one up to `end`; false if the queue ends before
  // what a tier must let go
  const auto one_by_one = [&](uint32_t end) -> bool {
    for (; k0 < end; ++k0) {
      const uint32_t at = k0 - sbase;
      const uint32_t e = lane_u32(S.e[at], 0), w = lane_u32(S.w[at], 0);
      uint32_t arr = w;
      if (x.pt) {
        const uint32_t p = lane_u32(S.pt[at], 0);
        arr = p - ptb;
        ptb = p;
      }
      uint32_t d = nt;  // the tier that holds the event's entry
#pragma unroll
      for (int t = KV_TIERS - 1; t >= 0; --t)
        if ((uint32_t)t < nt && e > H[t]) d = (uint32_t)t;
      if (!kOne && d < nt && lane == 0) {
        const uint32_t g = S.g[at];
        atomicAdd(&S.hit[g][d][0], 1ull);
        atomicAdd(&S.hit[g][d][1], (unsigned long long)w);
      }
#pragma unroll
      for (uint32_t t = 0; t < KV_TIERS; ++t) {
        if (t >= nt) continue;
        if (d == t) {
          room[t] += w;
          if (kOne) {
            hc[t] += lane == 0 ? 1u : 0u;
            hw[t] += w;
          }
        }
        uint32_t gone = 0;
        const int32_t over = (int32_t)arr - (int32_t)min(room[t], 1u << 30);
        while (over > 0 && gone < (uint32_t)over) {
          const uint32_t base = H[t];
          if (base >= n_en) return false;
          if (base < wb[t] || base + 64 > wb[t] + kXWin) {
            wb[t] = base;
            window(t, base);
          }
          const uint32_t i = base - wb[t] + lane;
          // alive unless taken out by now, this event's own entry among them
          const uint32_t v = S.out[t][i] > k0 ? (uint32_t)S.qw[t][i] : 0u;
          const uint32_t pre = gone + wave_incl_scan_u32(v);
          const uint64_t enough = __ballot(pre >= (uint32_t)over);
          const uint32_t l = enough ? (uint32_t)__builtin_ctzll(enough) : 63u;
          const bool goes = v != 0u && lane <= l;
          const uint32_t upto = lane_u32(pre, l);
          if (kOne) {
            ec[t] += goes ? 1u : 0u;
            ew[t] += upto - gone;
          } else if (goes) {
            const uint32_t g = x.qg[x.base + base + lane];
            atomicAdd(&S.ev[g][t][0], 1ull);
            atomicAdd(&S.ev[g][t][1], (unsigned long long)v);
          }
          gone = upto;
          H[t] = base + l + 1;
        }
        room[t] += gone - arr;
        arr = gone;
      }
    }
    return true;
  };
  while (k0 < n_ev) {
    if (k0 + kXStep > send && send < n_ev) {
      // stage the next events (the previous ones are read already)
      sbase = k0;
      send = min(n_ev, k0 + kXStage);
      __syncthreads();
      // 16 loads of each array in flight per lane, clamped to the last event
      for (uint32_t b = lane; b < send - sbase; b += 64 * kXBatch) {
        uint32_t se[kXBatch], sw[kXBatch], sp[kXBatch], sg[kXBatch];
#pragma unroll
        for (uint32_t r = 0; r < kXBatch; ++r) {
          const uint32_t k = min(sbase + b + 64 * r, n_ev - 1);
          se[r] = x.e[x.base + k];
          sw[r] = x.w[x.base + k];
          sp[r] = x.pt ? x.pt[k] : 0u;
          sg[r] = kOne ? 0u : x.g[x.base + k];
        }
#pragma unroll
        for (uint32_t r = 0; r < kXBatch; ++r) {
          const uint32_t i = b + 64 * r;  // below kXStage, a multiple of the batch
          S.e[i] = se[r] ? se[r] - x.base : 0u;
          S.w[i] = (uint8_t)sw[r];
          S.pt[i] = sp[r];
          if (!kOne) S.g[i] = (uint8_t)sg[r];
        }
      }
      __syncthreads();
    }
    if (step < kXShort) {  // (burst is set: only a short clash makes steps short)
      if (!one_by_one(min(min(n_ev, send), k0 + burst))) {
        bad = true;
        return;
      }
      step = min(kXStep, burst * 16);
      continue;
    }
    const uint32_t m = min(step, n_ev - k0);
    const uint32_t i0 = lane * kXIt, at = k0 - sbase + i0;
    bool in[kXIt];
    uint32_t e[kXIt], w[kXIt], d[kXIt], arr[kXIt];
#pragma unroll
    for (uint32_t r = 0; r < kXIt; ++r) {
      in[r] = i0 + r < m;
      const uint32_t q = in[r] ? at + r : 0u;
      e[r] = in[r] ? S.e[q] : 0u;
      w[r] = in[r] ? (uint32_t)S.w[q] : 0u;
      arr[r] = x.pt ? S.pt[q] - ptb : 0u;  // past the step: not used
      d[r] = nt;  // the tier that holds the event's entry
#pragma unroll
      for (int t = KV_TIERS - 1; t >= 0; --t)
        if ((uint32_t)t < nt && e[r] > H[t]) d[r] = (uint32_t)t;
    }
    // weight that arrives by each event, and in all
    uint32_t total;
    if (x.pt) total = S.pt[k0 - sbase + m - 1] - ptb;
    else total = step_scan(w, arr);
    // an entry is alive for the step unless taken out before its first event
    const uint32_t alive = k0;
    uint32_t clash = kXIt;  // the lane's first event that takes out a passed entry
    uint32_t newH[KV_TIERS], nc[KV_TIERS], nR[KV_TIERS], nA[KV_TIERS], nP[KV_TIERS];
#pragma unroll
    for (uint32_t t = 0; t < KV_TIERS; ++t) {
      newH[t] = H[t];
      nc[t] = nR[t] = nA[t] = nP[t] = 0;
      if (t >= nt) continue;
      nA[t] = total;
      uint32_t out[kXIt], R[kXIt], need[kXIt];
#pragma unroll
      for (uint32_t r = 0; r < kXIt; ++r) out[r] = d[r] == t ? w[r] : 0u;
      nR[t] = step_scan(out, R);
      const int32_t have = (int32_t)min(room[t], 1u << 30);
      uint32_t top = 0;
#pragma unroll
      for (uint32_t r = 0; r < kXIt; ++r) {
        const int32_t over = (int32_t)(arr[r] - R[r]) - have;
        top = max(top, in[r] && over > 0 ? (uint32_t)over : 0u);
        need[r] = top;
      }
      const uint32_t through = wave_incl_max_u32(top);
      const uint32_t most = lane_u32(through, 63);
      // the lanes below (wave_shr:1; lane 0 gets 0)
      const uint32_t below =
          (uint32_t)__builtin_amdgcn_update_dpp(0, (int)through, 0x138, 0xf, 0xf, false);
      uint32_t gone[kXIt];  // weight that left the tier by this event
#pragma unroll
      for (uint32_t r = 0; r < kXIt; ++r) {
        need[r] = max(need[r], below);
        gone[r] = 0;
      }
      // with one weight the entries that go weigh the need rounded up; the
      // last tier's departures arrive nowhere
      const bool search = t + 1 < nt && wu == 0;
      if (t + 1 < nt && wu > 1) {
#pragma unroll
        for (uint32_t r = 0; r < kXIt; ++r) gone[r] = (need[r] + wu - 1) / wu * wu;
      } else if (t + 1 < nt && wu == 1) {
#pragma unroll
        for (uint32_t r = 0; r < kXIt; ++r) gone[r] = need[r];
      }
      if (most) {
        uint32_t acc = 0, base = H[t];
        for (;;) {
          if (base >= n_en) {  // the queue holds what the tier must let go: never reached
            bad = true;
            return;
          }
          if (base < wb[t] || base + kXStep > wb[t] + kXWin) {
            wb[t] = base;
            window(t, base);
          }
          uint32_t qw[kXIt], pre[kXIt];
#pragma unroll
          for (uint32_t r = 0; r < kXIt; ++r) {
            const uint32_t i = base - wb[t] + i0 + r;
            qw[r] = S.out[t][i] >= alive ? (uint32_t)S.qw[t][i] : 0u;
          }
          const uint32_t tot = acc + step_scan(qw, pre);
#pragma unroll
          for (uint32_t r = 0; r < kXIt; ++r) pre[r] += acc;
          if (search) {
            *reinterpret_cast<uint4*>(&S.pref[i0]) = make_uint4(pre[0], pre[1], pre[2], pre[3]);
            __syncthreads();
            // the first prefix >= need, four ways at a time (256 = 4^4)
            uint32_t lo[kXIt] = {0, 0, 0, 0};
#pragma unroll
            for (uint32_t h = kXStep / 4; h; h /= 4) {
              uint32_t c[kXIt][3];
#pragma unroll
              for (uint32_t r = 0; r < kXIt; ++r)
#pragma unroll
                for (uint32_t z = 0; z < 3; ++z) c[r][z] = S.pref[lo[r] + (z + 1) * h - 1];
#pragma unroll
              for (uint32_t r = 0; r < kXIt; ++r)
#pragma unroll
                for (uint32_t z = 0; z < 3; ++z) lo[r] += c[r][z] < need[r] ? h : 0u;
            }
#pragma unroll
            for (uint32_t r = 0; r < kXIt; ++r)
              if (need[r] > acc && need[r] <= tot) gone[r] = S.pref[lo[r]];
            __syncthreads();
          }
          uint32_t n_go = 0;  // entries before the lane's first one past the stretch
#pragma unroll
          for (uint32_t r = 0; r < kXIt; ++r) {
            nc[t] += qw[r] != 0u && pre[r] - qw[r] < most ? 1u : 0u;
            n_go += pre[r] < most ? 1u : 0u;
          }
          if (most <= tot) {
            const uint32_t l =
                (uint32_t)__ffsll((long long)__ballot(pre[kXIt - 1] >= most)) - 1u;
            const uint32_t r = lane_u32(n_go, l);
            newH[t] = base + l * kXIt + r + 1;
            const uint32_t v = r == 0 ? pre[0] : r == 1 ? pre[1] : r == 2 ? pre[2] : pre[3];
            nP[t] = lane_u32(v, l);
            break;
          }
          acc = tot;
          base += kXStep;
        }
#pragma unroll
        for (int r = kXIt - 1; r >= 0; --r)
          if (e[r] > H[t] && e[r] <= newH[t]) clash = min(clash, (uint32_t)r);
      }
      total = nP[t];
#pragma unroll
      for (uint32_t r = 0; r < kXIt; ++r) arr[r] = gone[r];
    }
    if (const uint64_t c = __ballot(clash < kXIt)) {
      const uint32_t l = (uint32_t)__ffsll((long long)c) - 1u;
      step = l * kXIt + lane_u32(clash, l);
      if (step < kXShort) burst = burst ? min(kXBurst, burst * 4) : 1u;
      continue;
    }
    // the step stands
#pragma unroll
    for (uint32_t t = 0; t < KV_TIERS; ++t) {
      if (t >= nt) continue;
      if (kOne) {
#pragma unroll
        for (uint32_t r = 0; r < kXIt; ++r) hc[t] += d[r] == t ? 1u : 0u;
        hw[t] += nR[t];
        ec[t] += nc[t];
        ew[t] += nP[t];
      } else if (nP[t]) {
        for (uint32_t q = H[t] + lane; q < newH[t]; q += 64) {
          uint32_t o = x.out[x.base + q];
          if (o != kNone) o -= x.base;
          if (o < alive) continue;
          const uint32_t g = x.qg[x.base + q];
          atomicAdd(&S.ev[g][t][0], 1ull);
          atomicAdd(&S.ev[g][t][1], (unsigned long long)x.qw[x.base + q]);
        }
      }
      room[t] = room[t] + nR[t] + nP[t] - nA[t];
      H[t] = newH[t];
    }
    if (!kOne) {
#pragma unroll
      for (uint32_t r = 0; r < kXIt; ++r) {
        if (!in[r] || d[r] >= nt) continue;
        const uint32_t g = S.g[at + r];
        atomicAdd(&S.hit[g][d[r]][0], 1ull);
        atomicAdd(&S.hit[g][d[r]][1], (unsigned long long)w[r]);
      }
    }
    if (x.pt) ptb += nA[0];
    k0 += m;
    step = min(kXStep, m * 16);
    if (m >= kXShort) burst = 0;
  }
  if (kOne) {
#pragma unroll
    for (uint32_t t = 0; t < KV_TIERS; ++t) {
      const uint32_t h = wave_sum(hc[t]), v = wave_sum(ec[t]);
      if (lane != 0) continue;
      S.hit[g0][t][0] = h;
      S.hit[g0][t][1] = hw[t];
      S.ev[g0][t][0] = v;
      S.ev[g0][t][1] = ew[t];
    }
  }
}

__global__ __launch_bounds__(kXNT) void k_excl_walk(const XStream* __restrict__ xs,
                                                    const XWalk* __restrict__ walks,
                                                    const GroupStats* __restrict__ gs,
                                                    uint32_t n_groups, uint32_t wu,
                                                    uint64_t* __restrict__ counts,
                                                    uint32_t* __restrict__ err) {
  __shared__ WalkLds S;
  const XWalk j = walks[blockIdx.x];
  const uint32_t lane = lane_id();
  for (uint32_t i = lane; i < (uint32_t)(KV_MAX_GROUPS * KV_TIERS * 2); i += kXNT) {
    (&S.hit[0][0][0])[i] = 0;
    (&S.ev[0][0][0])[i] = 0;
  }
  __syncthreads();
  const bool shared = j.group == KV_MAX_GROUPS;
  const uint32_t g0 = shared ? 0u : j.group;
  bool bad = false;
  const unsigned long long* jcnt = nullptr;
  uint32_t first = 0;  // the live tier of head 0
  if (j.stream != kNone) {
    const XStream x = xs[j.stream];
    jcnt = x.jcnt;
    first = x.policy == KV_POLICY_LFU ? 1u : 0u;
    if (n_groups == 1 || !shared) walk<true>(x, j, wu, S, g0, bad);
    else walk<false>(x, j, wu, S, g0, bad);
  }
  __syncthreads();
  // The records this walk owns, one lane per group.  An access the top tier
  // does not serve misses there and enters it; what a tier does not serve
  // the next one sees, and what a tier evicts enters the next one.
  if (lane < n_groups && (shared || lane == j.group)) {
    const uint32_t g = lane;
    const GroupStats q = gs[g];
    uint64_t* c = counts + ((uint64_t)j.cfg * n_groups + g) * KV_TIERS * 8;
    for (uint32_t i = 0; i < (uint32_t)(KV_TIERS * 8); ++i) c[i] = 0;
    for (uint32_t f = 0; f < 2; ++f) {  // counts, weights
      const unsigned long long all = f ? q.n_w_g : q.n_g, u = f ? q.u_w_g : q.u_g;
      unsigned long long miss = all, ins = 0;
      for (uint32_t d = 0; d < j.nlive; ++d) {
        unsigned long long hit = 0, ev = 0;
        if (j.stream == kNone) {
          if (d == 0) hit = all - u;
        } else if (d < first || (d == 0 && jcnt)) {
          hit = all - jcnt[g * 4 + f];
          ev = jcnt[g * 4 + 2 + f];
        } else {
          hit = S.hit[g][d - first][f];
          ev = S.ev[g][d - first][f];
        }
        miss -= hit;
        if (d == 0) ins = miss;
        const uint32_t at = j.live[d] * 8 + 4 * f;
        c[at + KV_F_HIT] = hit;
        c[at + KV_F_MISS] = miss;
        c[at + KV_F_INS] = ins;
        c[at + KV_F_EVICT] = ev;
        ins = ev;
      }
    }
  }
  if (lane == 0 && bad && atomicCAS(&err[0], 0u, 2u) == 0u) atomicExch(&err[1], j.cfg);
}

uint64_t excl_test_budget() {
  const char* e = std::getenv("KVCFG_TEST_REPLAY_BUDGET");
  return e ? std::strtoull(e, nullptr, 10) : 0;
}

// Where a stream's arrays lie in the buffer it shares with its wave.  Arrays
// take the place of others that nothing reads any more: when an entry is taken
// out that of the replay's state, weights before events that of the emission,
// weights evicted by events (LFU, written where they are computed from) that
// of the weights before events.  20.2 bytes per access for LFU, 14.2 for FIFO
// (37 and 18, and 4 per block, with a place for each: calls whose memory the
// lists replayed per configuration, 33 and 9 bytes per block, had fitted
// failed).
struct Slab {
  uint64_t state, classes, bits, emit, wpre, ev_e, ev_w, ev_g, pwi, en_out, ev_pt, en_w, en_g, pq;
  uint64_t bytes;
  Slab(const Trace& t, uint32_t policy, uint64_t begin, uint64_t end) {
    const uint64_t n = end - begin, words = ((end + 63) >> 6) - (begin >> 6);
    const bool lfu = policy == KV_POLICY_LFU;
    const EmitLayout l = emit_layout(t, policy, n);
    uint64_t at = 0;
    auto put = [&](uint64_t b) {
      const uint64_t r = at;
      at += (b + 255) & ~255ull;
      return r;
    };
    state = en_out = put(std::max(l.state, n * 4));
    classes = put(l.classes);
    bits = put(words * 8);
    emit = pwi = put((n + 1) * 4);
    ev_pt = pwi + 4;
    wpre = put(words * 4);
    ev_e = put(n * 4);
    ev_w = put(n);
    ev_g = put(n);
    en_w = put(lfu ? n : 0);
    en_g = put(lfu ? n : 0);
    pq = put(lfu ? (n + 1) * 4 : 0);
    bytes = at;
  }
};

}  // namespace

bool excl_replayed(const kv_config& C, uint32_t g, bool mixed) {
  if (C.mode != KV_MODE_EXCLUSIVE_DEMOTE) return false;
  const uint32_t pol = C.partitioned ? C.policy[g] : C.policy[0];
  return pol != KV_POLICY_LRU || mixed;
}

kv_status excl_run(Trace& t, const kv_config* cfg_host, uint32_t n_cfg, const GroupStats* gs_dev,
                   uint64_t* counts, hipStream_t s) {
  const uint32_t G = t.n_groups;
  const bool mixed = t.st.w_min != t.st.w_max;
  // the walks, and the distinct streams under them
  std::vector<XWalk> walks;
  std::vector<ReplayJob> tops;  // stream i's top tier (LRU: capacity 0)
  std::map<std::tuple<uint32_t, uint32_t, uint32_t, uint64_t>, uint32_t> stream_of;
  for (uint32_t c = 0; c < n_cfg; ++c) {
    const kv_config& C = cfg_host[c];
    if (C.mode != KV_MODE_EXCLUSIVE_DEMOTE) continue;
    for (uint32_t h = 0; h < (C.partitioned ? G : 1u); ++h) {
      if (!excl_replayed(C, h, mixed)) continue;
      const uint32_t pol = C.partitioned ? C.policy[h] : C.policy[0];
      const bool part = C.partitioned && G > 1;
      XWalk w{};
      w.cfg = c;
      w.group = C.partitioned ? h : (uint32_t)KV_MAX_GROUPS;
      w.stream = kNone;
      uint64_t caps[KV_TIERS] = {};
      for (uint32_t k = 0; k < (uint32_t)KV_TIERS; ++k) {
        const uint64_t x = C.partitioned ? C.cap_group[k][h] : C.cap[k];
        if (!x) continue;
        caps[w.nlive] = x;
        w.live[w.nlive++] = (uint8_t)k;
      }
      const uint64_t distinct = C.partitioned ? t.st.u_w_g[h] : t.st.distinct_w;
      if (w.nlive && caps[0] < distinct) {
        const bool lru = pol == KV_POLICY_LRU;
        const uint32_t first = pol == KV_POLICY_LFU ? 1u : 0u;  // the LFU queue starts below the top
        w.nt = w.nlive - first;
        for (uint32_t d = 0; d < w.nt; ++d)
          w.cap[d] = (uint32_t)std::min<uint64_t>(caps[d + first], 0xFFFFFFFFull);
        const uint32_t grp = part ? h : (uint32_t)KV_MAX_GROUPS;
        const auto key = std::make_tuple(part ? 1u : 0u, grp, pol, lru ? 0ull : caps[0]);
        auto it = stream_of.find(key);
        if (it == stream_of.end()) {
          ReplayJob r{};
          r.order = part ? 1u : 0u;
          r.group = grp;
          r.policy = pol;
          r.cap = caps[0];
          r.begin = part ? t.part.seg[h] : 0;
          r.end = part ? t.part.seg[h + 1] : t.n;
          it = stream_of.emplace(key, (uint32_t)tops.size()).first;
          tops.push_back(r);
        }
        w.stream = it->second;
      }
      walks.push_back(w);
    }
  }
  if (walks.empty()) return KV_OK;
  StageTimer tm(kStReplayExcl, s);
  // LRU streams (and walks without one) need no replay; the others run in
  // waves whose arrays fit one buffer (all at once when they fit)
  const uint32_t ns = (uint32_t)tops.size();
  std::vector<uint32_t> order, rank(ns);
  for (uint32_t pass = 0; pass < 2; ++pass)
    for (uint32_t i = 0; i < ns; ++i)
      if ((tops[i].policy == KV_POLICY_LRU) == (pass == 0)) order.push_back(i);
  uint32_t n_lru = 0;
  for (uint32_t i = 0; i < ns; ++i) {
    rank[order[i]] = i;
    n_lru += tops[i].policy == KV_POLICY_LRU;
  }
  for (XWalk& w : walks)
    if (w.stream != kNone) w.stream = rank[w.stream];
  std::stable_sort(walks.begin(), walks.end(), [](const XWalk& a, const XWalk& b) {
    return a.stream + 1 < b.stream + 1;  // walks without a stream first
  });
  std::vector<Slab> slabs;
  std::vector<uint64_t> off(ns, 0);
  uint64_t total = 0, largest = 0;
  for (uint32_t i = n_lru; i < ns; ++i) {
    const ReplayJob& r = tops[order[i]];
    slabs.emplace_back(t, r.policy, r.begin, r.end);
    total += slabs.back().bytes;
    largest = std::max(largest, slabs.back().bytes);
  }
  DevBuf& bslab = t.ws[20];
  uint64_t budget = std::max<uint64_t>(total, 1);
  if (total > excl_budget(total, 0, bslab.bytes)) {
    size_t fr = 0, all = 0;
    KV_HIP(hipMemGetInfo(&fr, &all));
    budget = excl_budget(total, fr, bslab.bytes);
  }
  if (const uint64_t tb = excl_test_budget()) budget = std::max<uint64_t>(tb, 1);
  DevBuf& btab = t.ws[21];
  kv_status st;
  std::vector<uint32_t> lo;  // first stream of each wave
  for (;;) {
    lo.assign(1, n_lru);
    uint64_t cur = 0, most = 0;
    for (uint32_t i = n_lru; i < ns; ++i) {
      const uint64_t b = slabs[i - n_lru].bytes;
      if (cur && cur + b > std::max(budget, largest)) {
        lo.push_back(i);
        cur = 0;
      }
      off[i] = cur;
      cur += b;
      most = std::max(most, cur);
    }
    if ((st = bslab.reserve(std::max<uint64_t>(most, 1))) == KV_OK) break;
    if (st != KV_ERR_NOMEM || budget <= largest) return st;
    budget /= 2;
  }
  lo.push_back(ns);
  // device tables: streams, walks, {events, entries}, replay counters, jobs
  auto align = [](uint64_t b) { return (b + 255) & ~255ull; };
  const uint64_t t_walk = align(ns * sizeof(XStream));
  const uint64_t t_meta = t_walk + align(walks.size() * sizeof(XWalk));
  const uint64_t t_jcnt = t_meta + align(8ull * ns);
  const uint64_t t_jobs = t_jcnt + align(32ull * ns * G);
  if ((st = btab.reserve(t_jobs + emit_table_bytes() * ns)) != KV_OK) return st;
  uint8_t* tab = btab.as<uint8_t>();
  uint8_t* slab = bslab.as<uint8_t>();
  std::vector<XStream> xs(ns);
  for (uint32_t i = 0; i < ns; ++i) {
    const ReplayJob& r = tops[order[i]];
    const Order& o = r.order ? t.part : t.shared;
    XStream& x = xs[i];
    x.policy = r.policy;
    x.cap = r.cap;
    x.begin = r.begin;
    x.end = r.end;
    x.key = o.key.as<uint32_t>();
    x.nxt = o.nxt.as<uint32_t>();
    x.w8 = o.w.as<uint8_t>();
    x.g8 = o.g.as<uint8_t>();
    if (r.policy == KV_POLICY_LRU) {
      x.e = x.key;
      x.out = x.nxt;
      x.w = x.qw = x.w8;
      x.g = x.qg = x.g8;
      x.n = (uint32_t)(r.end - r.begin);
      x.base = (uint32_t)r.begin;
      continue;
    }
    const Slab& b = slabs[i - n_lru];
    uint8_t* p = slab + off[i];
    auto u32 = [&](uint64_t a) { return reinterpret_cast<uint32_t*>(p + a); };
    x.bits = reinterpret_cast<uint64_t*>(p + b.bits);
    x.emit = u32(b.emit);
    x.jcnt = reinterpret_cast<unsigned long long*>(tab + t_jcnt) + 4ull * G * i;
    x.cnt = reinterpret_cast<uint32_t*>(tab + t_meta) + 2 * i;
    x.wpre = u32(b.wpre);
    x.ev_e = u32(b.ev_e);
    x.ev_w = p + b.ev_w;
    x.ev_g = p + b.ev_g;
    x.pwi = u32(b.pwi);
    x.en_out = u32(b.en_out);
    const bool lfu = r.policy == KV_POLICY_LFU;
    x.ev_pt = lfu ? u32(b.ev_pt) : nullptr;
    x.pq = lfu ? u32(b.pq) : nullptr;
    x.en_w = lfu ? p + b.en_w : x.ev_w;
    x.en_g = lfu ? p + b.en_g : x.ev_g;
    x.e = x.ev_e;
    x.pt = lfu ? x.ev_pt : x.pwi + 1;
    x.out = x.en_out;
    x.w = x.ev_w;
    x.g = x.ev_g;
    x.qw = x.en_w;
    x.qg = x.en_g;
    x.meta = x.cnt;
  }
  // the tables are staged in the trace so they outlive the async copies
  t.excl_stage.assign(t_meta, 0);
  std::memcpy(t.excl_stage.data(), xs.data(), ns * sizeof(XStream));
  std::memcpy(t.excl_stage.data() + t_walk, walks.data(), walks.size() * sizeof(XWalk));
  KV_HIP(hipMemcpyAsync(tab, t.excl_stage.data(), t_meta, hipMemcpyHostToDevice, s));
  const XStream* xs_dev = reinterpret_cast<const XStream*>(tab);
  const XWalk* walks_dev = reinterpret_cast<const XWalk*>(tab + t_walk);
  // the walks of streams [a, b) (kNone + 1 = 0: those without a stream)
  auto walk_range = [&](uint32_t a, uint32_t b) -> kv_status {
    const auto by = [](const XWalk& w, uint32_t v) { return w.stream + 1 < v; };
    const size_t w0 = std::lower_bound(walks.begin(), walks.end(), a, by) - walks.begin();
    const size_t w1 = std::lower_bound(walks.begin(), walks.end(), b, by) - walks.begin();
    if (w0 == w1) return KV_OK;
    hipLaunchKernelGGL(k_excl_walk, dim3((uint32_t)(w1 - w0)), dim3(kXNT), 0, s, xs_dev,
                       walks_dev + w0, gs_dev, G, mixed ? 0u : t.st.w_max, counts,
                       t.err.as<uint32_t>());
    KV_HIP(hipGetLastError());
    return KV_OK;
  };
  const uint32_t err_base = t.err_first + (uint32_t)t.err_jobs.size();
  const uint32_t job0 = (uint32_t)t.err_jobs.size() - t.err_call;  // after the inclusive replays
  for (uint32_t i = n_lru; i < ns; ++i) {
    const ReplayJob& r = tops[order[i]];
    t.err_add(r.policy, r.group, r.cap);
  }
  uint32_t w0 = 0;  // the first wave walks the LRU streams too
  t.emit_stage.clear();
  t.emit_stage.reserve(emit_table_bytes() * ns);  // staged copies stay where they are
  for (size_t v = 0; v + 1 < lo.size(); ++v) {
    std::vector<EmitJob> ej;
    uint64_t longest = 0;
    for (uint32_t i = lo[v]; i < lo[v + 1]; ++i) {
      const ReplayJob& r = tops[order[i]];
      const Slab& b = slabs[i - n_lru];
      ej.push_back(EmitJob{r, off[i] + b.state, off[i] + b.classes, off[i] + b.bits,
                           off[i] + b.emit});
      longest = std::max(longest, r.end - r.begin);
    }
    if (ej.empty()) break;
    if ((st = replay_emit(t, ej, slab, tab + t_jobs + emit_table_bytes() * (lo[v] - n_lru),
                          t.emit_stage,
                          reinterpret_cast<unsigned long long*>(tab + t_jcnt) + 4ull * G * lo[v],
                          err_base + lo[v] - n_lru, job0 + lo[v] - n_lru, s)) != KV_OK)
      return st;
    const uint32_t nj = lo[v + 1] - lo[v];
    const XStream* x = xs_dev + lo[v];
    const dim3 grid(std::min<uint32_t>(div_up(longest, 256), 2048), nj);
    hipLaunchKernelGGL(k_x_rank, dim3(nj), dim3(kXPrep), 0, s, x, G);
    KV_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_x_gather, grid, dim3(256), 0, s, x);
    KV_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_x_weights, dim3(nj, 2), dim3(kXPrep), 0, s, x);
    KV_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_x_link, grid, dim3(256), 0, s, x);
    KV_HIP(hipGetLastError());
    if ((st = walk_range(w0, lo[v + 1] + 1)) != KV_OK) return st;
    w0 = lo[v + 1] + 1;
  }
  if (w0 == 0 && (st = walk_range(0, n_lru + 1)) != KV_OK) return st;
  // a failed state check is reported by the next call on this trace
  KV_HIP(hipMemcpyAsync(t.err_host, t.err.p, 2 * sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  KV_HIP(hipEventRecord(t.err_pin->ev, s));
  t.err_pending = true;
  return KV_OK;
}

}  // namespace kv
