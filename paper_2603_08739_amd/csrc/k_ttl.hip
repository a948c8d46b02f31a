// k_ttl.hip - TTL retention curves of the disk tier (Section 4.3).
//
// Under a time-to-live t a block stays on disk for t seconds after each of
// its accesses, so an access hits iff the gap delta to its block's previous
// access is at most t, and a block with accesses a_1 < ... < a_m occupies
// storage for sum_j min(t, a_{j+1} - a_j) + t seconds.  Per group, the hits
// H_g(t) and the storage integral C_g(t) for every t of a sorted list follow
// from one histogram of the gaps over the list's bins:
//   bin(delta) = #{k : ttl[k] < delta}, so delta <= ttl[k] <=> bin <= k;
//   H_g(ttl[k])  = sum of the counts of bins 0..k
//   C_g(ttl[k])  = W_g*ttl[k] + sum_{delta <= ttl[k]} w*delta
//                  + ttl[k] * (weight of the gaps above ttl[k]).
// The pass is a stream over the trace with one dependent gather per access
// (the request of the previous access); the histogram lives in LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "kv_device.h"
#include "kv_internal.h"

namespace kv {
namespace {

constexpr int kTtlNT = 1024;       // threads per workgroup
constexpr int kTtlU = 8;           // accesses per thread per step (gathers in flight)
static_assert(kTtlU % 4 == 0, "accesses are read four at a time");
constexpr uint32_t kTtlMax = 1024; // TTL values per call
constexpr uint32_t kTtlBins = 4096;  // groups * (TTL values + 1)

// Gap histogram: per (group, bin) the number of gaps, their summed weight
// and the summed weight * gap, added into the zeroed global arrays.  In LDS
// the count and the weight share one 64-bit word (count << 32 | weight: with
// n <= 2^29 over up to 1024 workgroups a workgroup sees at most 2^19
// accesses of at most 255 granules each, so the weight never carries).
//
// A request's blocks were mostly last read by one earlier request, so
// neighbouring accesses share a gap.  A thread first joins its consecutive
// accesses of one (request, previous request, group) into runs, and a
// wavefront then joins the lanes' runs of one such triple, so that a search
// and two LDS atomics serve all of them (per access they were most of the
// time, the atomics on few addresses taken one lane at a time); what four
// triples do not cover goes lane by lane.  1e8 accesses, 64 TTLs: 809 -> 286 us
// (3.5 TB/s of the 10 bytes per access that have to be read).  A wavefront
// with a thread of kTtlMany runs or more joins no lanes and takes its runs side
// by side, so that their loads and searches overlap: neighbours are strangers
// there, and run after run they cost more than they save (1e7 random accesses,
// 8 TTLs: 160 us, 149 without any joining, now 150; 500 accesses 8.6, 4.3 and
// 4.0 us; 1e6 accesses whose group changes at every block 16, 10.5 and 10.6).
constexpr int kTtlMany = 4;
__global__ __launch_bounds__(kTtlNT) void k_ttl_hist(
    const uint32_t* __restrict__ key, const uint32_t* __restrict__ req,
    const double* __restrict__ rt, const uint8_t* __restrict__ w8,
    const uint8_t* __restrict__ g8, uint64_t n, const double* __restrict__ ttl, uint32_t n_ttl,
    uint32_t bins, unsigned long long* __restrict__ cnt, unsigned long long* __restrict__ wsum,
    double* __restrict__ wd) {
  __shared__ unsigned long long hcw[kTtlBins];
  __shared__ double hd[kTtlBins];
  __shared__ double tt[kTtlMax];
  const uint32_t tid = threadIdx.x;
  const uint32_t nb = n_ttl + 1;
  for (uint32_t i = tid; i < bins; i += kTtlNT) {
    hcw[i] = 0;
    hd[i] = 0.0;
  }
  for (uint32_t i = tid; i < n_ttl; i += kTtlNT) tt[i] = ttl[i];
  __syncthreads();
  const uint64_t step = (uint64_t)gridDim.x * kTtlNT * kTtlU;
  for (uint64_t p0 = (uint64_t)blockIdx.x * kTtlNT * kTtlU; p0 < n; p0 += step) {
    // each thread takes kTtlU consecutive accesses, read as vectors (the
    // arrays hold 16 readable bytes past n; accesses past n are dropped)
    uint32_t k[kTtlU], r[kTtlU], rp[kTtlU], w[kTtlU], g[kTtlU];
    const uint64_t pt = p0 + (uint64_t)tid * kTtlU;
#pragma unroll
    for (int q = 0; q < kTtlU / 4; ++q) {
      const uint64_t pq = min<uint64_t>(pt + 4 * q, n & ~3ull);
      const uint4 kv = *reinterpret_cast<const uint4*>(key + pq);
      const uint4 rv = *reinterpret_cast<const uint4*>(req + pq);
      const uint32_t wv = *reinterpret_cast<const uint32_t*>(w8 + pq);
      const uint32_t gv = *reinterpret_cast<const uint32_t*>(g8 + pq);
      const uint32_t ka[4] = {kv.x, kv.y, kv.z, kv.w}, ra[4] = {rv.x, rv.y, rv.z, rv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool in = pq == pt + 4 * q && pt + 4 * q + e < n;
        k[4 * q + e] = in ? ka[e] : 0u;
        r[4 * q + e] = ra[e];
        w[4 * q + e] = (wv >> (8 * e)) & 0xFFu;
        g[4 * q + e] = (gv >> (8 * e)) & 0xFFu;
      }
    }
#pragma unroll
    for (int u = 0; u < kTtlU; ++u) rp[u] = k[u] ? req[k[u] - 1] : 0u;
    // cum[u]: count << 16 | weight of the accesses with a gap up to u; ends:
    // the last accesses of runs
    uint32_t cum[kTtlU], ends = 0, run = 0;
#pragma unroll
    for (int u = 0; u < kTtlU; ++u) {
      if (k[u]) run += (1u << 16) | w[u];  // no earlier access: no gap
      cum[u] = run;
      const int v = u + 1 < kTtlU ? u + 1 : u;
      const bool same = u + 1 < kTtlU && k[v] && r[v] == r[u] && rp[v] == rp[u] && g[v] == g[u];
      ends |= (k[u] && !same ? 1u : 0u) << u;
    }
    if (__ballot(__popc(ends) >= kTtlMany)) {
      uint32_t before = 0;
#pragma unroll
      for (int u = 0; u < kTtlU; ++u) {
        if (!((ends >> u) & 1u)) continue;
        const uint32_t c = cum[u] - before, wt = c & 0xFFFFu;
        before = cum[u];
        const double delta = rt[r[u]] - rt[rp[u]];
        const uint32_t b = lower_bound(tt, 0u, n_ttl, delta);
        const uint32_t idx = g[u] * nb + b;
        atomicAdd(&hcw[idx], (unsigned long long)(c >> 16) << 32 | wt);
        atomicAdd(&hd[idx], (double)wt * delta);
      }
      continue;
    }
    uint32_t done = 0;
    while (__ballot(ends != 0u)) {
      const int at = ends ? __builtin_ctz(ends) : 0;
      uint32_t rr = r[0], pp = rp[0], gg = g[0], cc = cum[0];
#pragma unroll
      for (int u = 1; u < kTtlU; ++u) {
        rr = at == u ? r[u] : rr;
        pp = at == u ? rp[u] : pp;
        gg = at == u ? g[u] : gg;
        cc = at == u ? cum[u] : cc;
      }
      bool has = ends != 0u;
      const uint32_t c0 = has ? cc - done : 0u;
      done = has ? cc : done;
      ends &= ends - 1u;
      // count << 20 | weight: a wavefront's at most 512 accesses and 130,560 granules
      uint32_t sum = (c0 >> 16) << 20 | (c0 & 0xFFFFu);
      uint64_t left = __ballot(has);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        if (!left) break;
        const int l = (int)__builtin_ctzll(left);
        const uint32_t lr = (uint32_t)__builtin_amdgcn_readlane((int)rr, l);
        const uint32_t lp = (uint32_t)__builtin_amdgcn_readlane((int)pp, l);
        const uint32_t lg = (uint32_t)__builtin_amdgcn_readlane((int)gg, l);
        const bool mine = has && rr == lr && pp == lp && gg == lg;
        const uint64_t peers = __ballot(mine);
        const uint32_t all = wave_add_dpp(mine ? sum : 0u);
        left &= ~peers;
        if (mine) {
          if ((int)lane_id() == l) sum = all;
          else has = false;
        }
      }
      if (has) {
        const double delta = rt[rr] - rt[pp];
        const uint32_t b = lower_bound(tt, 0u, n_ttl, delta);
        const uint32_t idx = gg * nb + b, wt = sum & 0xFFFFFu;
        atomicAdd(&hcw[idx], (unsigned long long)(sum >> 20) << 32 | wt);
        atomicAdd(&hd[idx], (double)wt * delta);
      }
    }
  }
  __syncthreads();
  for (uint32_t i = tid; i < bins; i += kTtlNT) {
    const unsigned long long x = hcw[i];
    if (!x) continue;
    atomicAdd(&cnt[i], x >> 32);
    atomicAdd(&wsum[i], x & 0xFFFFFFFFull);
    atomicAdd(&wd[i], hd[i]);
  }
}

struct GroupWeights {
  unsigned long long w[KV_MAX_GROUPS];  // distinct weight per group
};

// Cumulative curves, one workgroup per group.  Its bins are read at once;
// the sums run in bin order (the double one as it always did), one thread
// for each.
__global__ __launch_bounds__(256) void k_ttl_fin(const unsigned long long* __restrict__ cnt,
                          const unsigned long long* __restrict__ wsum,
                          const double* __restrict__ wd, const double* __restrict__ ttl,
                          uint32_t n_ttl, GroupWeights W,
                          uint64_t* __restrict__ hits, uint64_t* __restrict__ hitw,
                          double* __restrict__ store) {
  __shared__ unsigned long long c[kTtlMax + 1], ws[kTtlMax + 1];
  __shared__ double d[kTtlMax + 1];
  const uint32_t g = blockIdx.x, nb = n_ttl + 1;
  for (uint32_t b = threadIdx.x; b < nb; b += 256) {
    c[b] = cnt[(uint64_t)g * nb + b];
    ws[b] = wsum[(uint64_t)g * nb + b];
    d[b] = wd[(uint64_t)g * nb + b];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long run = 0;
    for (uint32_t b = 0; b < nb; ++b) c[b] = run += c[b];
  } else if (threadIdx.x == 64) {
    unsigned long long run = 0;
    for (uint32_t b = 0; b < nb; ++b) ws[b] = run += ws[b];
  } else if (threadIdx.x == 128) {
    double run = 0.0;
    for (uint32_t b = 0; b < nb; ++b) d[b] = run += d[b];
  }
  __syncthreads();
  const double Wg = (double)W.w[g];
  const unsigned long long P = ws[n_ttl];  // weight of every gap of the group
  for (uint32_t k = threadIdx.x; k < n_ttl; k += 256) {
    const double t = ttl[k];
    hits[(uint64_t)g * n_ttl + k] = c[k];
    hitw[(uint64_t)g * n_ttl + k] = ws[k];
    store[(uint64_t)g * n_ttl + k] = Wg * t + d[k] + t * (double)(P - ws[k]);
  }
}

}  // namespace

// The no-allocation variant's device memory: the TTL values, then the three
// gap histograms (count, weight, weight * gap) of at most kTtlBins bins.
// Each device holds its own copy for the life of the process; host code
// reaches it only through the address hipGetSymbolAddress returns.
constexpr size_t kScratchTtlBytes = (size_t)kTtlMax * sizeof(double);
constexpr size_t kScratchBytes = kScratchTtlBytes + (size_t)kTtlBins * 3 * sizeof(uint64_t);
static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {
kv_status scratch_ptr(uint8_t** out) {
  static std::mutex mu;
  static void* per_dev[64] = {};
  int d = 0;
  KV_HIP(hipGetDevice(&d));
  if (d < 0 || d >= 64) return fail(KV_ERR_DEVICE, "device index out of range");
  std::lock_guard<std::mutex> lk(mu);
  if (!per_dev[d]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      (void)hipGetLastError();
      return fail(KV_ERR_DEVICE, std::string("kv_ttl_curves_noalloc: no address for the "
                                             "scratch array: ") + hipGetErrorString(e));
    }
    per_dev[d] = p;
  }
  *out = static_cast<uint8_t*>(per_dev[d]);
  return KV_OK;
}
}  // namespace

kv_status ttl_curves_noalloc(Trace& t, const double* ttl_host, uint32_t n_ttl, uint64_t* hits,
                             uint64_t* hitw, double* store, hipStream_t s) {
  if (n_ttl > kTtlMax || (uint64_t)t.n_groups * (n_ttl + 1) > kTtlBins)
    return fail(KV_ERR_UNSUPPORTED,
                "kv_ttl_curves_noalloc: n_groups * (n_ttl + 1) must be <= 4096");
  uint8_t* base = nullptr;
  kv_status st;
  if ((st = scratch_ptr(&base)) != KV_OK) return st;
  double* ttl_dev = reinterpret_cast<double*>(base);
  KV_HIP(hipMemcpyAsync(ttl_dev, ttl_host, (size_t)n_ttl * sizeof(double),
                        hipMemcpyHostToDevice, s));
  return ttl_curves_into(t, ttl_dev, n_ttl,
                         reinterpret_cast<unsigned long long*>(base + kScratchTtlBytes), hits,
                         hitw, store, s);
}

kv_status ttl_curves(Trace& t, const double* ttl_dev, uint32_t n_ttl, uint64_t* hits,
                     uint64_t* hitw, double* store, hipStream_t s) {
  const uint32_t G = t.n_groups;
  const uint32_t bins = G * (n_ttl + 1);
  if (n_ttl > kTtlMax || bins > kTtlBins)
    return fail(KV_ERR_UNSUPPORTED, "kv_ttl_curves: n_groups * (n_ttl + 1) must be <= 4096");
  DevBuf& bh = t.ws[22];
  kv_status st;
  if ((st = bh.reserve((uint64_t)bins * 24)) != KV_OK) return st;
  return ttl_curves_into(t, ttl_dev, n_ttl, bh.as<unsigned long long>(), hits, hitw, store, s);
}

kv_status ttl_curves_into(Trace& t, const double* ttl_dev, uint32_t n_ttl,
                          unsigned long long* cnt, uint64_t* hits, uint64_t* hitw,
                          double* store, hipStream_t s) {
  const uint32_t G = t.n_groups;
  const uint32_t bins = G * (n_ttl + 1);
  kv_status st;
  unsigned long long* wsum = cnt + bins;
  double* wd = reinterpret_cast<double*>(wsum + bins);
  StageTimer tm(kStTtl, s);
  if ((st = fill_u64(reinterpret_cast<uint64_t*>(cnt), 0, (uint64_t)bins * 3, s)) != KV_OK)
    return st;
  const uint64_t per_block = (uint64_t)kTtlNT * kTtlU;
  const uint32_t nblk = (uint32_t)std::min<uint64_t>((t.n + per_block - 1) / per_block, 1024);
  hipLaunchKernelGGL(k_ttl_hist, dim3(nblk), dim3(kTtlNT), 0, s, t.shared.key.as<uint32_t>(),
                     t.req.as<uint32_t>(), t.req_time.as<double>(), t.shared.w.as<uint8_t>(),
                     t.shared.g.as<uint8_t>(), t.n, ttl_dev, n_ttl, bins, cnt, wsum, wd);
  KV_HIP(hipGetLastError());
  GroupWeights W{};
  for (uint32_t g = 0; g < KV_MAX_GROUPS; ++g) W.w[g] = t.st.u_w_g[g];
  hipLaunchKernelGGL(k_ttl_fin, dim3(G), dim3(256), 0, s, cnt, wsum, wd, ttl_dev, n_ttl, W, hits,
                     hitw, store);
  KV_HIP(hipGetLastError());
  return KV_OK;
}

}  // namespace kv
