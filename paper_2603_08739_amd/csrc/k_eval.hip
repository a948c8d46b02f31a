// k_eval.hip - per-configuration counts, objectives and the Pareto filter.
#include "kv_device.h"
#include "kv_internal.h"

namespace kv {
namespace {

// One group's cumulative histogram at a capacity: accesses with a stack
// distance of at most it, their weight, blocks that end no deeper, theirs.
struct Cum {
  uint64_t hit, hit_w, fin, fin_w;
};

// Threshold index of a capacity in group g.
__device__ __forceinline__ uint32_t thr_index(const OrderView& ov, uint32_t g, uint64_t cap) {
  const uint32_t c = cap > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)cap;
  return lower_bound(ov.thr, ov.off[g], ov.off[g + 1], c);
}

// All zero for an absent tier.
__device__ __forceinline__ Cum cum_at(const OrderView& ov, uint32_t g, uint64_t cap, uint32_t idx) {
  Cum r{0, 0, 0, 0};
  if (cap == 0) return r;
  const ulonglong2* h = reinterpret_cast<const ulonglong2*>(ov.hist + (uint64_t)(idx + g) * 4);
  const ulonglong2 a = h[0], b = h[1];
  r.hit = a.x;
  r.hit_w = a.y;
  r.fin = b.x;
  r.fin_w = b.y;
  return r;
}

// LRU records from the stack-distance histograms.
//  inclusive: hit_k = hits(C_k) - hits(M) if C_k > M (M = largest faster
//             capacity), miss_k = N - hits(max(M, C_k)), ins_k = N - hits(C_k),
//             evict_k = ins_k - final residents at C_k.
//  exclusive (uniform weight w0): the tiers are one LRU stack cut at the
//             cumulative block capacities S_k; hit_k = hits(S_k) - hits(S_{k-1}),
//             miss_k = N - hits(S_k), evict_k = N - hits(S_k) - finals(S_k)
//             (a block crosses depth S_k once per reuse interval whose distance
//             exceeds S_k and once more if it ends deeper); ins of the top tier
//             = N - hit_top, of a lower tier = evictions of the tier above.
// Cumulative joint value of field f over accesses (or final blocks, `fin`)
// with stack distance <= cap (cap = ~0: any, cold accesses included) and gap
// <= the TTL value at index k of group g.
__device__ __forceinline__ uint64_t joint_at(const OrderView& ov, const JointView& jv,
                                             uint32_t g, uint64_t cap, uint32_t k, int f,
                                             bool fin) {
  if (cap == 0) return 0;
  const uint32_t lo = ov.off[g], hi = ov.off[g + 1];
  const uint32_t d = cap == ~0ull ? hi - lo
                                  : lower_bound(ov.thr, lo, hi,
                                                cap > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)cap) - lo;
  const uint32_t nt = jv.toff[g + 1] - jv.toff[g] + 1;
  const uint64_t b = jv.jbase[g] + (uint64_t)d * nt + k;
  return (fin ? jv.fh : jv.jh)[2 * b + f];
}

// Tier 2 as a disk TTL tier (trace order): present at an access iff its
// stack distance fits cap2 (unbounded: cap2 = ~0) and its gap fits the TTL;
// the faster tiers' largest capacity M decides which accesses reach it.
__device__ __forceinline__ void ttl_tier_record(const OrderView& ov, const JointView& jv,
                                                const kv_config& C, uint32_t g, uint64_t M,
                                                const GroupStats& s, uint64_t* r,
                                                double* store) {
  const double t = C.ttl[g];
  const uint32_t tlo = jv.toff[g], thi = jv.toff[g + 1];
  const uint32_t k = lower_bound(jv.tthr, tlo, thi, t) - tlo;
  const uint64_t c2 = C.cap[2] ? C.cap[2] : ~0ull;
  const uint64_t N = s.n_g, NW = s.n_w_g;
  const uint64_t pc = joint_at(ov, jv, g, c2, k, 0, false), pw = joint_at(ov, jv, g, c2, k, 1, false);
  const uint64_t lo_cap = (M == 0) ? 0 : (M < c2 ? M : c2);
  const uint64_t mc = joint_at(ov, jv, g, lo_cap, k, 0, false);
  const uint64_t mw = joint_at(ov, jv, g, lo_cap, k, 1, false);
  const uint64_t hc = pc - mc, hw = pw - mw;
  const Cum m = cum_at(ov, g, M, M ? thr_index(ov, g, M) : 0u);
  const uint64_t rc = N - m.hit, rw = NW - m.hit_w;  // reach the disk
  r[KV_F_HIT] = hc;
  r[KV_F_HIT_W] = hw;
  r[KV_F_MISS] = rc - hc;
  r[KV_F_MISS_W] = rw - hw;
  r[KV_F_INS] = N - pc;
  r[KV_F_INS_W] = NW - pw;
  r[KV_F_EVICT] = (N - pc) - joint_at(ov, jv, g, c2, k, 0, true);
  r[KV_F_EVICT_W] = (NW - pw) - joint_at(ov, jv, g, c2, k, 1, true);
  if (C.cap[2] == 0) {
    // W_g t + sum over gaps <= t of w gap + t (weight of the longer gaps)
    const double sd = jv.wd[tlo + g + k];
    const uint64_t gapw = NW - s.u_w_g;               // re-accesses
    const uint64_t inw = joint_at(ov, jv, g, ~0ull, k, 1, false);  // re-accesses within t
    *store = ((double)s.u_w_g * t + sd) + t * (double)(gapw - inw);
  }
}

// One thread per (configuration, group, tier): a record needs the histogram
// at its own capacity and at the largest faster one (the sum of the faster
// ones in the exclusive mode).  Bound by the chain of a threshold search, so
// a tier has a thread of its own (one thread for all three, each field
// searched for by itself: 13 us for 25 configurations, 22 us for 527; now 9
// and 11 us).
__global__ __launch_bounds__(256) void k_lru_counts(const kv_config* __restrict__ cfg,
                                                    uint32_t n_cfg, uint32_t G, OrderView sh,
                                                    OrderView pt, OrderView px, OrderView lf,
                                                    JointView jv,
                                                    const GroupStats* __restrict__ gs,
                                                    uint32_t mixed,
                                                    uint64_t* __restrict__ counts,
                                                    double* __restrict__ store_cg) {
  const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= (uint64_t)n_cfg * G * KV_TIERS) return;
  const uint32_t k = (uint32_t)(tid % KV_TIERS), cg = (uint32_t)(tid / KV_TIERS);
  const uint32_t c = cg / G, g = cg % G;
  const kv_config& C = cfg[c];
  const bool part = C.partitioned != 0;
  const uint32_t pol = part ? C.policy[g] : C.policy[0];
  if (pol != KV_POLICY_LRU && pol != KV_POLICY_LEAF) return;
  // an exclusive hierarchy over mixed weights is no split stack: walked
  if (C.mode == KV_MODE_EXCLUSIVE_DEMOTE && mixed) return;
  // radix-tree eviction: distances of the re-touched order (shared tiers only)
  const OrderView& ov = pol == KV_POLICY_LEAF ? lf : (part && G > 1) ? pt : sh;
  uint64_t cap[3];
  for (int q = 0; q < 3; ++q) cap[q] = part ? C.cap_group[q][g] : C.cap[q];
  const GroupStats s = gs[g];
  const uint64_t N = s.n_g, NW = s.n_w_g;
  uint64_t* r = counts + ((uint64_t)cg * KV_TIERS + k) * KV_FIELDS;
  if (k == 2 && store_cg) store_cg[cg] = 0.0;
  if (k == 2 && C.disk_ttl) {
    double st = 0.0;
    ttl_tier_record(ov, jv, C, g, cap[0] > cap[1] ? cap[0] : cap[1], s, r, &st);
    if (store_cg) store_cg[cg] = st;
    return;
  }
  const uint64_t ck = k == 0 ? cap[0] : k == 1 ? cap[1] : cap[2];
  if (ck == 0) {
    for (int f = 0; f < KV_FIELDS; ++f) r[f] = 0;
    return;
  }
  if (C.mode == KV_MODE_EXCLUSIVE_DEMOTE) {
    uint64_t sp = 0;  // blocks of the faster tiers
    for (uint32_t q = 0; q < k; ++q) sp += (q == 0 ? cap[0] : cap[1]) / s.w0;
    const uint64_t sk = (sp + ck / s.w0) * s.w0;
    const bool top = sp == 0;
    sp *= s.w0;
    const Cum a = cum_at(ov, g, sk, thr_index(ov, g, sk));
    const Cum p = cum_at(ov, g, sp, top ? 0u : thr_index(ov, g, sp));
    const uint64_t hit = a.hit - p.hit;
    const uint64_t miss = N - a.hit;
    const uint64_t ev = N - a.hit - a.fin;
    const uint64_t ins = top ? N - hit : N - p.hit - p.fin;  // what the tier above evicts
    r[KV_F_HIT] = hit;
    r[KV_F_MISS] = miss;
    r[KV_F_INS] = ins;
    r[KV_F_EVICT] = ev;
    r[KV_F_HIT_W] = hit * s.w0;
    r[KV_F_MISS_W] = miss * s.w0;
    r[KV_F_INS_W] = ins * s.w0;
    r[KV_F_EVICT_W] = ev * s.w0;
    return;
  }
  // which accesses a tier serves: by stack distance, or with prefix reuse
  // by the running maximum over the request; what it holds: by distance
  const uint64_t M = k == 0 ? 0 : k == 1 ? cap[0] : (cap[0] > cap[1] ? cap[0] : cap[1]);
  const uint32_t ik = thr_index(ov, g, ck), im = M ? thr_index(ov, g, M) : 0u;
  const Cum a = cum_at(ov, g, ck, ik);
  const OrderView& sv = C.mode == KV_MODE_INCLUSIVE_PREFIX ? px : ov;
  const Cum sa = cum_at(sv, g, ck, ik), sm = cum_at(sv, g, M, im);
  const bool more = ck > M;
  r[KV_F_HIT] = more ? sa.hit - sm.hit : 0;
  r[KV_F_HIT_W] = more ? sa.hit_w - sm.hit_w : 0;
  r[KV_F_MISS] = N - (more ? sa.hit : sm.hit);
  r[KV_F_MISS_W] = NW - (more ? sa.hit_w : sm.hit_w);
  r[KV_F_INS] = N - a.hit;
  r[KV_F_INS_W] = NW - a.hit_w;
  r[KV_F_EVICT] = (N - a.hit) - a.fin;
  r[KV_F_EVICT_W] = (NW - a.hit_w) - a.fin_w;
}

struct CostArgs {
  double pg, p0, p1, p2, bw_dram, ssd_base, ssd_per_gib, ssd_max, tpf;
  double gb, tpg, span, n_req;
  uint64_t n_w;
  uint32_t n_media;
  kv_disk_medium media[KV_MAX_MEDIA];
};

// (cost, throughput, latency) in IEEE double, left to right, no contraction.
__global__ __launch_bounds__(256) void k_objectives(const kv_config* __restrict__ cfg,
                                                    uint32_t n_cfg, uint32_t G,
                                                    const uint64_t* __restrict__ counts,
                                                    const double* __restrict__ store_cg,
                                                    CostArgs a, double* __restrict__ obj) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n_cfg) return;
  uint64_t hw0 = 0, hw1 = 0, hw2 = 0, iw2 = 0;
  for (uint32_t g = 0; g < G; ++g) {
    const uint64_t* r = counts + ((uint64_t)c * G + g) * 24;
    hw0 += r[0 * 8 + KV_F_HIT_W];
    hw1 += r[1 * 8 + KV_F_HIT_W];
    hw2 += r[2 * 8 + KV_F_HIT_W];
    iw2 += r[2 * 8 + KV_F_INS_W];
  }
  const uint64_t rw = a.n_w - (hw0 + hw1 + hw2);
  const double kGiB = 1073741824.0;
  const double c0 = ((double)cfg[c].cap[0] * a.gb) / kGiB;
  const double c1 = ((double)cfg[c].cap[1] * a.gb) / kGiB;
  double c2 = ((double)cfg[c].cap[2] * a.gb) / kGiB;
  if (cfg[c].disk_ttl && cfg[c].cap[2] == 0) {
    // an unbounded TTL tier: its mean occupancy over the span
    double st = 0.0;
    for (uint32_t g = 0; g < G; ++g) st += store_cg[(uint64_t)c * G + g];
    c2 = a.span > 0 ? ((st * a.gb) / kGiB) / a.span : 0.0;
  }
  double p2 = a.p2, base = a.ssd_base, per_gib = a.ssd_per_gib, bmax = a.ssd_max;
  if (a.n_media) {
    const kv_disk_medium& md = a.media[cfg[c].medium];
    p2 = md.price_per_gib_hour;
    base = md.bw_base;
    per_gib = md.bw_per_gib;
    bmax = md.bw_max;
  }
  const double bw_lin = base + per_gib * c2;
  const double bw_ssd = (bmax < bw_lin) ? bmax : bw_lin;
  const double t_dram = ((double)hw1 * a.gb) / a.bw_dram;
  const double t_ssd = ((double)(hw2 + iw2) * a.gb) / bw_ssd;
  const double t_rec = ((double)rw * a.tpg) * a.tpf;
  const double t_busy = (t_rec + t_dram) + t_ssd;
  const double t_wall = (a.span < t_busy) ? t_busy : a.span;
  const double thr = ((double)a.n_w * a.tpg) / t_wall;
  const double lat = t_busy / a.n_req;
  const double cost = (((a.pg + c0 * a.p0) + c1 * a.p1) + c2 * p2) * (t_wall / 3600.0);
  obj[3 * (uint64_t)c + 0] = cost;
  obj[3 * (uint64_t)c + 1] = thr;
  obj[3 * (uint64_t)c + 2] = lat;
}

struct Bounds {
  double b0, b1, b2;
};

__device__ __forceinline__ bool feasible(double o0, double o1, double o2, const Bounds& b) {
  if (o0 != o0 || o1 != o1 || o2 != o2) return false;
  if (b.b0 == b.b0 && !(o0 <= b.b0)) return false;
  if (b.b1 == b.b1 && !(o1 >= b.b1)) return false;
  if (b.b2 == b.b2 && !(o2 <= b.b2)) return false;
  return true;
}

// a dominates b, both of one segment.
__device__ __forceinline__ bool dominates(double a0, double a1, double a2, double b0, double b1,
                                          double b2) {
  // (no short cuts: the loads behind every operand go out together)
  return bool(int(a0 <= b0) & int(a1 >= b1) & int(a2 <= b2) &
              (int(a0 < b0) | int(a1 > b1) | int(a2 < b2)));
}

__device__ __forceinline__ double lane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

constexpr int kPaNT = 256;  // points of a tile, one thread each

// A tile's points that may still be on the front, packed.
struct PaTile {
  double o[3][kPaNT];
  uint32_t seg[kPaNT];
  uint32_t idx[kPaNT];  // row
  uint32_t dom[kPaNT];  // found dominated
  uint32_t wsum[kPaNT / 64];
  uint32_t n;
};

// Packs the rows of the threads with `keep` into t (any earlier reader of t
// is past a barrier).  Two barriers.
__device__ __forceinline__ void pa_pack(PaTile& t, bool keep, uint32_t row, uint32_t seg, double o0,
                                        double o1, double o2) {
  const uint64_t m = __ballot(keep);
  const int w = wave_id();
  if (lane_id() == 0) t.wsum[w] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t at = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kPaNT / 64; ++i) {
    if (i < w) at += t.wsum[i];
    all += t.wsum[i];
  }
  at += (uint32_t)__popcll(m & lanemask_lt());
  if (keep) {
    t.o[0][at] = o0;
    t.o[1][at] = o1;
    t.o[2][at] = o2;
    t.seg[at] = seg;
    t.idx[at] = row;
    t.dom[at] = 0;
  }
  if (threadIdx.x == 0) t.n = all;
  __syncthreads();
}

// Marks the points of `p` that a candidate of `c` dominates.  With few
// points, k threads share one point's candidates, so the block stays busy.
// Bound by the LDS reads' latency, so kPaU candidates are read side by side
// (one at a time, each operand as the comparison came to it: 43 us for 256
// points of which none is dominated, now 26).
constexpr uint32_t kPaU = 4;
__device__ __forceinline__ void pa_compare(PaTile& p, const PaTile& c) {
  const uint32_t np = p.n, nc = c.n;
  uint32_t k = 1;
  while (2 * k * np <= (uint32_t)kPaNT && k < 64) k *= 2;
  const uint32_t i = threadIdx.x / k;
  if (i >= np || p.dom[i]) return;
  const double b0 = p.o[0][i], b1 = p.o[1][i], b2 = p.o[2][i];
  const uint32_t sb = p.seg[i];
  bool dom = false;
  uint32_t j = threadIdx.x % k;
  for (; j + (kPaU - 1) * k < nc && !dom; j += kPaU * k) {
    uint32_t s[kPaU];
    double a0[kPaU], a1[kPaU], a2[kPaU];
#pragma unroll
    for (uint32_t q = 0; q < kPaU; ++q) {
      const uint32_t r = j + q * k;
      s[q] = c.seg[r];
      a0[q] = c.o[0][r];
      a1[q] = c.o[1][r];
      a2[q] = c.o[2][r];
    }
#pragma unroll
    for (uint32_t q = 0; q < kPaU; ++q)
      dom |= s[q] == sb && dominates(a0[q], a1[q], a2[q], b0, b1, b2);
  }
  for (; j < nc && !dom; j += k)
    dom = c.seg[j] == sb && dominates(c.o[0][j], c.o[1][j], c.o[2][j], b0, b1, b2);
  if (dom) p.dom[i] = 1;
}

// Flag of every point: 1 if it meets the bounds (and has no NaN) and no
// other such point of its tile of 256 and its segment dominates it.  First
// each wavefront's 64 points against each other, the candidate broadcast
// from a lane, then the tile's remaining points against each other.  With
// one tile (n <= 256) that is the front, and `result` (or null) receives
// {flagged rows, NaN seen}; with more, a NaN sets *nan_seen (or null).
// Comparisons bound this filter, and a point dominated inside its tile need
// not be compared with the other tiles' points at all.  A call over 11,000
// sweep objectives takes 47 us (163 us with all pairs in one pass, whose
// kernel ran 141 us); for 512 points, whose two tiles left the chip idle
// for 66 us, the whole load-and-evaluate step shortens by 92 us.
__global__ __launch_bounds__(kPaNT) void k_pareto_tile(const double* __restrict__ obj,
                                                       const uint32_t* __restrict__ seg, uint32_t n,
                                                       Bounds bd, uint8_t* __restrict__ flag,
                                                       uint32_t* __restrict__ nan_seen,
                                                       uint32_t* __restrict__ result) {
  __shared__ PaTile t;
  __shared__ uint32_t left[kPaNT / 64], bad[kPaNT / 64];
  const uint32_t b = blockIdx.x * kPaNT + threadIdx.x;
  double o0 = 0, o1 = 0, o2 = 0;
  uint32_t sb = 0;
  bool live = false, nan = false;
  if (b < n) {
    o0 = obj[3 * (uint64_t)b];
    o1 = obj[3 * (uint64_t)b + 1];
    o2 = obj[3 * (uint64_t)b + 2];
    sb = seg ? seg[b] : 0u;
    live = feasible(o0, o1, o2, bd);
    nan = o0 != o0 || o1 != o1 || o2 != o2;
  }
  const uint64_t any_nan = __ballot(nan);
  const uint64_t cand = __ballot(live);
  bool dom = false;
  for (uint64_t left_c = cand; left_c; left_c &= left_c - 1) {
    const int j = (int)__builtin_ctzll(left_c);
    const double a0 = lane_f64(o0, j), a1 = lane_f64(o1, j), a2 = lane_f64(o2, j);
    const uint32_t sa = (uint32_t)__builtin_amdgcn_readlane((int)sb, j);
    dom |= sa == sb && dominates(a0, a1, a2, o0, o1, o2);
  }
  live = live && !dom;
  if (b < n && !live) flag[b] = 0;
  pa_pack(t, live, b, sb, o0, o1, o2);
  pa_compare(t, t);
  __syncthreads();
  const bool on = threadIdx.x < t.n && !t.dom[threadIdx.x];
  if (threadIdx.x < t.n) flag[t.idx[threadIdx.x]] = on ? 1 : 0;
  if (nan_seen && any_nan && lane_id() == 0) atomicOr(nan_seen, 1u);
  if (result) {
    const uint64_t m = __ballot(on);
    if (lane_id() == 0) {
      left[wave_id()] = (uint32_t)__popcll(m);
      bad[wave_id()] = any_nan != 0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      result[0] = left[0] + left[1] + left[2] + left[3];
      result[1] = bad[0] | bad[1] | bad[2] | bad[3];
    }
  }
}

// Dominance between tiles over a grid of (point tile, candidate slice):
// block (x, y) tests the points of tile x still flagged against the points
// still flagged in tiles [y * per, (y + 1) * per) and clears the flag of
// every point a candidate dominates.  Every writer stores 0, so the blocks
// need no ordering; whichever flags a block still sees set, the result is the
// same: dominance is transitive, so a point dominated by a cleared candidate
// is dominated by the one that cleared it or one that never is.
__global__ __launch_bounds__(kPaNT) void k_pareto_cross(const double* __restrict__ obj,
                                                        const uint32_t* __restrict__ seg,
                                                        uint32_t n, uint32_t per, uint8_t* flag) {
  __shared__ PaTile p, c;
  auto pack = [&](PaTile& t, uint32_t tile) {
    const uint32_t b = tile * kPaNT + threadIdx.x;
    const bool keep = b < n && flag[b];
    double o0 = 0, o1 = 0, o2 = 0;
    uint32_t sb = 0;
    if (keep) {
      o0 = obj[3 * (uint64_t)b];
      o1 = obj[3 * (uint64_t)b + 1];
      o2 = obj[3 * (uint64_t)b + 2];
      sb = seg ? seg[b] : 0u;
    }
    pa_pack(t, keep, b, sb, o0, o1, o2);
  };
  pack(p, blockIdx.x);
  if (p.n == 0) return;
  const uint32_t tiles = (n + kPaNT - 1) / kPaNT;
  const uint32_t t1 = min(tiles, (blockIdx.y + 1) * per);
  for (uint32_t t = blockIdx.y * per; t < t1; ++t) {
    if (t == blockIdx.x) continue;  // its own pairs are settled
    pack(c, t);
    pa_compare(p, c);
    __syncthreads();
  }
  if (threadIdx.x < p.n && p.dom[threadIdx.x]) flag[p.idx[threadIdx.x]] = 0;
}

// {points left on the front, NaN seen} into `result`, by one block; *nan_seen
// is cleared for the next call.
__global__ __launch_bounds__(1024) void k_pareto_count(const uint8_t* __restrict__ flag, uint32_t n,
                                                       uint32_t* __restrict__ nan_seen,
                                                       uint32_t* __restrict__ result) {
  __shared__ uint32_t sh[16];
  uint32_t v = 0;
  for (uint32_t i = threadIdx.x; i < n; i += 1024) v += flag[i];
  v = block_sum<1024>(v, sh);
  if (threadIdx.x == 0) {
    result[0] = v;
    result[1] = *nan_seen;
    *nan_seen = 0;
  }
}

}  // namespace

kv_status lru_counts(const kv_config* cfg_dev, uint32_t n_cfg, uint32_t n_groups,
                     OrderView shared, OrderView part, OrderView prefix, OrderView leaf,
                     JointView joint,
                     const GroupStats* gs_dev, bool mixed, uint64_t* counts, double* store_cg,
                     hipStream_t s) {
  const uint64_t m = (uint64_t)n_cfg * n_groups * KV_TIERS;
  if (m == 0) return KV_OK;
  StageTimer tm(kStLruCounts, s);
  hipLaunchKernelGGL(k_lru_counts, dim3(div_up(m, 256)), dim3(256), 0, s, cfg_dev, n_cfg,
                     n_groups, shared, part, prefix, leaf, joint, gs_dev, mixed ? 1u : 0u, counts,
                     store_cg);
  KV_HIP(hipGetLastError());
  return KV_OK;
}

kv_status objectives(const kv_config* cfg_dev, uint32_t n_cfg, uint32_t n_groups,
                     const uint64_t* counts, const double* store_cg, const kv_cost_model& m,
                     double gb, double tpg, double span, double n_req, uint64_t n_w,
                     double* obj, hipStream_t s) {
  if (n_cfg == 0) return KV_OK;
  CostArgs a{m.price_gpu_per_hour, m.price_per_gib_hour[0], m.price_per_gib_hour[1],
             m.price_per_gib_hour[2], m.bw_dram, m.ssd_bw_base, m.ssd_bw_per_gib,
             m.ssd_bw_max, m.t_prefill_per_token, gb, tpg, span, n_req, n_w, m.n_media, {}};
  for (uint32_t i = 0; i < KV_MAX_MEDIA; ++i) a.media[i] = m.media[i];
  StageTimer tm(kStObjectives, s);
  hipLaunchKernelGGL(k_objectives, dim3(div_up(n_cfg, 256)), dim3(256), 0, s, cfg_dev, n_cfg,
                     n_groups, counts, store_cg, a, obj);
  KV_HIP(hipGetLastError());
  return KV_OK;
}

kv_status pareto(const double* obj, const uint32_t* segment, uint32_t n, const double* bounds,
                 uint8_t* flag, uint32_t* nan_seen, uint32_t* result, hipStream_t s) {
  const double nan = __builtin_nan("");
  Bounds bd{bounds ? bounds[0] : nan, bounds ? bounds[1] : nan, bounds ? bounds[2] : nan};
  StageTimer tm(kStPareto, s);
  if (n == 0) return KV_OK;
  const uint32_t nt = div_up(n, kPaNT);
  hipLaunchKernelGGL(k_pareto_tile, dim3(nt), dim3(kPaNT), 0, s, obj, segment, n, bd, flag,
                     nt > 1 && result ? nan_seen : (uint32_t*)nullptr,
                     nt == 1 ? result : (uint32_t*)nullptr);
  KV_HIP(hipGetLastError());
  if (nt == 1) return KV_OK;
  // point tiles x candidate slices: about 2,048 blocks, eight to a compute unit
  const uint32_t ny = std::max<uint32_t>(1, std::min<uint32_t>(nt, div_up(2048, nt)));
  const uint32_t per = div_up(nt, ny);
  hipLaunchKernelGGL(k_pareto_cross, dim3(nt, div_up(nt, per)), dim3(kPaNT), 0, s, obj, segment, n,
                     per, flag);
  KV_HIP(hipGetLastError());
  if (result) {
    hipLaunchKernelGGL(k_pareto_count, dim3(1), dim3(1024), 0, s, flag, n, nan_seen, result);
    KV_HIP(hipGetLastError());
  }
  return KV_OK;
}

}  // namespace kv
