// Standalone batched scorer (Section III-A cost equation + per-pool argmin)
// and the per-replica goodput reduction (Section IV-B SLO targets, Table II
// goodput), for gfx950.
//
// Shared snapshot (inst_stride 0), many requests: the instance terms that do
// not depend on the request, w_b * backlog and w_q * queue, are formed once
// per block into LDS (the same float32 operations the equation performs
// first), then each thread scores kReq requests against every instance,
// reading each LDS entry once for all of its requests.  VALU-bound.
//
// Per-request snapshot (inst_stride >= n_inst), or a shared one for few
// requests: L lanes per request, U instances per lane and pass with every
// load of the pass issued before its first cost.  Rows of at most 64
// instances laid out for 16-byte loads have a kernel of their own (16 lanes
// per request, four consecutive instances per lane).  HBM-bound.
#include <algorithm>

#include "lane_ops.h"
#include "rt_internal.h"

namespace rt {
namespace {

constexpr int kReq = 2;       // requests per thread (shared snapshot)
constexpr int kBlock = 256;

struct SnapEntry {
  float lb;    // w_b * backlog
  float qq;    // w_q * (float)queue
  int32_t kv;  // occupancy
  float kvf;   // ... in float32
};

__device__ __forceinline__ bool req_ok(int32_t pool, int32_t p, int32_t oh, uint32_t c) {
  if (p < 1 || c >= (uint32_t)kMaxClasses) return false;
  if (pool == 1 && (oh < 1 || (int64_t)p + oh > INT32_MAX)) return false;
  return true;
}

// One thread's kReq requests against every snapshot entry, any values.  kNonNeg:
// no occupancy is negative, so occupancy + need < 2^32 and the sum converts
// exactly through the unsigned 32-bit path (same value and rounding as int64;
// 300,000 requests x 300 instances with occupancies above 2^24: 46 us, 80 us
// through int64).
template <bool kNonNeg>
__device__ __forceinline__ void score_loop(const SnapEntry* snap, int n, const ScoreArgs& a, const float* sg,
                                           const float* work, const int64_t* need, uint32_t* bkey,
                                           int32_t* bi) {
  for (int j = 0; j < n; ++j) {
    const SnapEntry e = snap[j];
#pragma unroll
    for (int r = 0; r < kReq; ++r) {
      float press;
      if constexpr (kNonNeg)
        press = (float)((uint32_t)e.kv + (uint32_t)need[r]) * a.inv_cap;
      else
        press = (float)((int64_t)e.kv + need[r]) * a.inv_cap;
      const float load = e.lb * sg[r];
      const float size = work[r] * (1.0f + a.rho * press) * sg[r];
      const float cost = load + size + e.qq;
      const uint32_t k = cost_key(cost);
      if (k < bkey[r]) {
        bkey[r] = k;
        bi[r] = j;
      }
    }
  }
}

// The same where no cost can be NaN, -0 or negative and every occupancy +
// need is below 2^24 (see the kernel): the sum is then exact in float32 and
// float minima order as the keys do.  Costs are taken four at a time: their
// minimum (two instructions), one compare and two selects per four instead of
// per one; the index within the winning four is found afterwards by taking
// its costs again.  10.4 VALU instructions a pair (9.4 with rho 1, whose product
// changes nothing: four products, four sums, a quarter of five for the minimum and
// the loop's own) against 17 above; 2^20 requests x 64 instances: 25.9 us with the
// loop above, 16.8 us so.
template <bool kRho1>
__device__ __forceinline__ float plain_cost(const SnapEntry& e, const ScoreArgs& a, float sg, float work, float need) {
  const float press = (e.kvf + need) * a.inv_cap;
  const float load = e.lb * sg;
  const float size = work * (1.0f + (kRho1 ? press : a.rho * press)) * sg;
  return load + size + e.qq;
}

template <bool kRho1>
__device__ __forceinline__ void plain_loop(const SnapEntry* snap, int n, const ScoreArgs& a, const float* sg,
                                           const float* work, const int64_t* need, uint32_t* bkey, int32_t* bi) {
  float best[kReq], needf[kReq];
  int32_t bg[kReq];
#pragma unroll
  for (int r = 0; r < kReq; ++r) {
    best[r] = __builtin_huge_valf();
    bg[r] = 0;
    needf[r] = (float)need[r];
  }
#pragma unroll 2
  for (int j = 0; j < n; j += 4) {
    SnapEntry e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = snap[j + u];
#pragma unroll
    for (int r = 0; r < kReq; ++r) {
      float c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) c[u] = plain_cost<kRho1>(e[u], a, sg[r], work[r], needf[r]);
      const float m = __builtin_fminf(__builtin_fminf(__builtin_fminf(c[0], c[1]), c[2]), c[3]);
      const bool b = m < best[r];
      best[r] = b ? m : best[r];
      bg[r] = b ? j : bg[r];
    }
  }
#pragma unroll
  for (int r = 0; r < kReq; ++r) {
    int32_t at = 3;
#pragma unroll
    for (int u = 2; u >= 0; --u)
      at = plain_cost<kRho1>(snap[bg[r] + u], a, sg[r], work[r], needf[r]) == best[r] ? u : at;
    bi[r] = bg[r] + at;
    bkey[r] = __float_as_uint(best[r]);
  }
}

__global__ void __launch_bounds__(kBlock) score_shared_kernel(ScoreArgs a) {
  extern __shared__ SnapEntry snap[];
  __shared__ uint32_t kv_max;  // (of the bits: from 2^31 on where an occupancy is negative)
  const int n = a.n_inst;
  if (threadIdx.x == 0) kv_max = 0;
  __syncthreads();
  int plain = 1;
  uint32_t kvm = 0;
  for (int j = threadIdx.x; j < n; j += kBlock) {
    SnapEntry e;
    e.lb = a.w_b * a.backlog[j];
    e.qq = a.w_q * (float)a.queue[j];
    e.kv = a.kv[j];
    e.kvf = (float)e.kv;
    plain &= e.lb >= 0.0f && e.lb < __builtin_huge_valf() && e.qq >= 0.0f;
    kvm = max(kvm, (uint32_t)e.kv);
    snap[j] = e;
  }
  // entries past the last, up to a multiple of four: never the first minimum
  for (int j = n + threadIdx.x; j < ((n + 3) & ~3); j += kBlock)
    snap[j] = SnapEntry{__builtin_huge_valf(), 0.0f, 0, 0.0f};
  if (kvm > 0) atomicMax(&kv_max, kvm);
  plain = __syncthreads_and(plain);
  kvm = kv_max;

  const int64_t first = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * kReq;
  float sg[kReq], work[kReq];
  int64_t need[kReq];
  int32_t bi[kReq];
  uint32_t bkey[kReq];
  bool ok[kReq];
#pragma unroll
  for (int r = 0; r < kReq; ++r) {
    const int64_t i = first + r;
    ok[r] = false;
    sg[r] = 0.0f;
    work[r] = 0.0f;
    need[r] = 0;
    bi[r] = -1;
    bkey[r] = 0xffffffffu;
    if (i < a.n_req) {
      const int32_t p = a.plen[i];
      const int32_t oh = a.pool == 1 ? a.ohat[i] : 0;
      const uint32_t c = a.cls[i];
      ok[r] = req_ok(a.pool, p, oh, c);
      if (ok[r]) {
        sg[r] = a.sigma[c];
        work[r] = a.pool == 1 ? a.w_s * (float)oh * a.tau : a.w_s * (float)p * a.tau;
        need[r] = a.pool == 1 ? (int64_t)p + oh : (int64_t)p;
      }
    }
    // The plain loop's conditions (from ten instances on: taking the winning four
    // again costs what the loop saves on fewer; 4,000,000 requests x 5 23.8 us and
    // 21.0 with the other loop, x 10 26.0 and 25.9, x 12 26.0 and 28.3).  The
    // snapshot's terms are finite and not negative; occupancy + need stays below
    // 2^24 for the largest occupancy (a negative one counts as one of 2^31 or
    // more); and work * (1 + rho * press) is finite for it, so for every one (each
    // operation is monotone).  Then every product and sum of a cost is +0,
    // positive or +inf (weights are +0 or positive), and +inf meets neither
    // 0 * inf nor inf - inf: sigma and the reciprocal capacity are finite.
    const float top = work[r] * (1.0f + a.rho * ((float)((int64_t)kvm + need[r]) * a.inv_cap));
    plain &= (int64_t)kvm + need[r] < (1 << 24) && top < __builtin_huge_valf();
  }
  if (n >= 10 && __all(plain)) {
    if (a.rho == 1.0f)
      plain_loop<true>(snap, n, a, sg, work, need, bkey, bi);
    else
      plain_loop<false>(snap, n, a, sg, work, need, bkey, bi);
  } else if ((int32_t)kvm >= 0) {
    score_loop<true>(snap, n, a, sg, work, need, bkey, bi);
  } else {
    score_loop<false>(snap, n, a, sg, work, need, bkey, bi);
  }
#pragma unroll
  for (int r = 0; r < kReq; ++r) {
    const int64_t i = first + r;
    if (i < a.n_req) {
      a.out_idx[i] = ok[r] ? bi[r] : -1;
      a.out_score[i] = __uint_as_float(ok[r] ? bkey[r] : 0x7fc00000u);
    }
  }
}

// L lanes per request, 64 / L requests per wave and G such groups at once; a
// lane takes instances (lane mod L) + L * u of its request's row, U of them
// per pass, every load of a pass issued before its first cost.  Within a lane
// the first of equal keys stays; then the lanes of a request reduce the key,
// and the lowest index that holds it.  Stride 0 (one snapshot for every
// request) is a row like any other.  Against one 64-lane segment, one load
// per array in flight and a 64-bit shuffle reduction per request: 300,007 rows
// of 37 instances 87.7 -> 30.6 us; 48 requests x 1,000 shared instances
// 90 us with a thread per request, 10 us (the launch itself) so.
template <int L, int U, int G>
__global__ void __launch_bounds__(kBlock) score_rows_kernel(ScoreArgs a) {
  constexpr int kSegs = 64 / L;
  const int lane = threadIdx.x & 63;
  const int sl = lane & (L - 1);
  const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int64_t first = wave * (kSegs * G) + lane / L;
  const int n = a.n_inst;
  int32_t p[G], oh[G];
  uint32_t c[G];
  bool live[G];
  const float* bl[G];
  const int32_t *qu[G], *kv[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int64_t i = first + g * kSegs;
    live[g] = i < a.n_req;
    const int64_t ii = live[g] ? i : 0;
    p[g] = a.plen[ii];
    oh[g] = a.pool == 1 ? a.ohat[ii] : 0;
    c[g] = a.cls[ii];
    bl[g] = a.backlog + ii * a.stride;
    qu[g] = a.queue + ii * a.stride;
    kv[g] = a.kv + ii * a.stride;
  }
  uint32_t bkey[G];
  int32_t bj[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    bkey[g] = 0xffffffffu;
    bj[g] = sl;
  }
  for (int j0 = 0; j0 < n; j0 += L * U) {
    float b4[G][U];
    int32_t q4[G][U], k4[G][U];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = min(j0 + u * L + sl, n - 1);
        b4[g][u] = bl[g][j];
        q4[g][u] = qu[g][j];
        k4[g][u] = kv[g][j];
      }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float sg = a.sigma[c[g] & (kMaxClasses - 1)];
      const float work = a.pool == 1 ? a.w_s * (float)oh[g] * a.tau : a.w_s * (float)p[g] * a.tau;
      const uint32_t need = a.pool == 1 ? (uint32_t)p[g] + (uint32_t)oh[g] : (uint32_t)p[g];  // < 2^31 when ok
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * L + sl;
        // occupancy + need, exact in 32 bits: unsigned when the occupancy is
        // >= 0 (the sum is < 2^32), signed otherwise (the sum is < 2^31)
        const uint32_t sum = (uint32_t)k4[g][u] + need;
        const float kvn = k4[g][u] >= 0 ? (float)sum : (float)(int32_t)sum;
        const float press = kvn * a.inv_cap;
        const float load = a.w_b * b4[g][u] * sg;
        const float size = work * (1.0f + a.rho * press) * sg;
        const float cost = load + size + a.w_q * (float)q4[g][u];
        uint32_t k = cost_key(cost);
        k = j < n ? k : 0xffffffffu;
        const bool b = k < bkey[g];
        bkey[g] = b ? k : bkey[g];
        bj[g] = b ? j : bj[g];
      }
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint32_t m = seg_min<L>(bkey[g]);
    const uint32_t idx = seg_min<L>(bkey[g] == m ? (uint32_t)bj[g] : 0xffffffffu);
    const int64_t i = first + g * kSegs;
    const bool ok = req_ok(a.pool, p[g], oh[g], c[g]);
    if (live[g] && sl == 0) {
      a.out_idx[i] = ok ? (int32_t)idx : -1;
      a.out_score[i] = __uint_as_float(ok ? m : 0x7fc00000u);
    }
  }
}

// Per-request rows of at most 64 instances, n_inst and the stride multiples
// of 4 and the snapshot arrays 16-byte aligned: 16 lanes per request, four
// consecutive instances per lane (one 16-byte load per array), four
// requests per wave and kRowGroups groups of four per wave, every load of a
// wave issued before its first cost.  Within a lane the four costs are taken
// in index order (the first of equal keys stays); the 16 lanes of a request
// reduce the key, then the lowest index holding it, with DPP within their
// row.
constexpr int kRowGroups = 4;

__global__ void __launch_bounds__(kBlock) score_rows16_kernel(ScoreArgs a) {
  constexpr int G = kRowGroups;
  const int lane = threadIdx.x & 63;
  const int rq = lane >> 4, ql = lane & 15;
  const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const int64_t first = wave * 4 * G;
  const int j0 = 4 * ql;  // this lane's first instance
  const bool lane_in = j0 < a.n_inst;
  float4 b4[G];
  int4 q4[G], k4[G];
  int32_t p[G], oh[G];
  uint32_t c[G];
  bool live[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int64_t i = first + 4 * g + rq;
    live[g] = i < a.n_req;
    const int64_t ii = live[g] ? i : 0;
    p[g] = a.plen[ii];
    oh[g] = a.pool == 1 ? a.ohat[ii] : 0;
    c[g] = a.cls[ii];
    const int64_t e = ii * a.stride + (lane_in ? j0 : 0);
    b4[g] = *reinterpret_cast<const float4*>(a.backlog + e);
    q4[g] = *reinterpret_cast<const int4*>(a.queue + e);
    k4[g] = *reinterpret_cast<const int4*>(a.kv + e);
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const bool ok = live[g] && req_ok(a.pool, p[g], oh[g], c[g]);
    const float sg = a.sigma[c[g] & (kMaxClasses - 1)];
    const float work = a.pool == 1 ? a.w_s * (float)oh[g] * a.tau : a.w_s * (float)p[g] * a.tau;
    const uint32_t need = a.pool == 1 ? (uint32_t)p[g] + (uint32_t)oh[g] : (uint32_t)p[g];  // < 2^31 when ok
    const float bb[4] = {b4[g].x, b4[g].y, b4[g].z, b4[g].w};
    const int32_t qq[4] = {q4[g].x, q4[g].y, q4[g].z, q4[g].w};
    const int32_t kk[4] = {k4[g].x, k4[g].y, k4[g].z, k4[g].w};
    uint32_t bkey = 0xffffffffu;
    int32_t bj = j0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      // occupancy + need, exact in 32 bits: unsigned when the occupancy is
      // >= 0 (the sum is < 2^32), signed otherwise (the sum is < 2^31)
      const uint32_t sum = (uint32_t)kk[u] + need;
      const float kvn = kk[u] >= 0 ? (float)sum : (float)(int32_t)sum;
      const float press = kvn * a.inv_cap;
      const float load = a.w_b * bb[u] * sg;
      const float size = work * (1.0f + a.rho * press) * sg;
      const float cost = load + size + a.w_q * (float)qq[u];
      uint32_t k = cost_key(cost);
      k = lane_in ? k : 0xffffffffu;
      const bool b = k < bkey;
      bkey = b ? k : bkey;
      bj = b ? j0 + u : bj;
    }
    const uint32_t m = seg_min<16>(bkey);
    const uint32_t idx = seg_min<16>(bkey == m ? (uint32_t)bj : 0xffffffffu);
    const int64_t i = first + 4 * g + rq;
    if (live[g] && ql == 0) {
      a.out_idx[i] = ok ? (int32_t)idx : -1;
      a.out_score[i] = __uint_as_float(ok ? m : 0x7fc00000u);
    }
  }
}

__global__ void __launch_bounds__(kBlock) goodput_kernel(GoodputArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t rep = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (rep >= a.n_replicas) return;  // whole wave leaves together
  const int64_t lo = a.offsets[rep], hi = a.offsets[rep + 1];
  const int pid = a.param_point ? a.param_point[rep] : 0;
  if (lo < 0 || hi < lo || hi > a.n_requests || pid < 0 || pid >= a.n_points) {
    // a replica this trace does not describe consistently: no read outside it
    if (lane == 0) {
      a.goodput[rep] = 0.0;
      if (a.met) a.met[rep] = -1;
      atomicOr(a.flag, kFlagBadTrace);
    }
    return;
  }
  // the point's targets, lane k < 8 holding class k's (read per request
  // with a cross-lane shuffle instead of a dependent load)
  const DevPoint& pp = a.points[pid];
  const int k8 = lane & (kMaxClasses - 1);
  const int64_t my_ttft = pp.slo_ttft[k8], my_tpot = pp.slo_tpot[k8];
  int64_t met = 0;
  // four 64-request chunks per iteration, their loads issued together
  constexpr int kU = 4;
  for (int64_t i0 = lo; i0 < hi; i0 += 64 * kU) {
    int64_t tt[kU], sp[kU];
    int32_t o[kU];
    uint32_t c[kU];
    bool in[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int64_t i = i0 + u * 64 + lane;
      in[u] = i < hi;
      const int64_t j = in[u] ? i : lo;
      tt[u] = a.ttft[j];
      sp[u] = a.span[j];
      o[u] = a.olen[j];
      c[u] = a.cls[j];
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool valid = in[u] && tt[u] >= 0 && c[u] < (uint32_t)kMaxClasses;
      const int cc = valid ? (int)c[u] : 0;
      const int64_t lim_ttft = __shfl(my_ttft, cc, 64), lim_tpot = __shfl(my_tpot, cc, 64);
      const bool ok_ttft = tt[u] <= lim_ttft;
      const bool ok_tpot = o[u] <= 1 || sp[u] <= lim_tpot * (int64_t)(o[u] - 1);
      met += (valid && ok_ttft && ok_tpot) ? 1 : 0;
    }
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) {
    const uint32_t l = (uint32_t)__shfl_xor((int)(uint32_t)met, m, 64);
    const uint32_t h = (uint32_t)__shfl_xor((int)(uint32_t)((uint64_t)met >> 32), m, 64);
    met += (int64_t)(((uint64_t)h << 32) | l);
  }
  if (lane == 0) {
    const int64_t n = hi - lo;
    a.goodput[rep] = n > 0 ? (double)met / (double)n : 0.0;
    if (a.met) a.met[rep] = met;
  }
}

}  // namespace

template <int L, int U>
static hipError_t launch_rows(const ScoreArgs& a, hipStream_t stream) {
  constexpr int G = L <= 2 ? 1 : (U <= 2 ? 4 : 2);  // groups of requests at once
  const int64_t per_block = (kBlock / 64) * (64 / L) * G;
  hipLaunchKernelGGL((score_rows_kernel<L, U, G>), dim3((unsigned)((a.n_req + per_block - 1) / per_block)), dim3(kBlock),
                     0, stream, a);
  return hipGetLastError();
}

template <int L>
static hipError_t launch_rows(const ScoreArgs& a, hipStream_t stream) {
  switch ((a.n_inst + L - 1) / L) {
    case 1: return launch_rows<L, 1>(a, stream);
    case 2: return launch_rows<L, 2>(a, stream);
    case 3: return launch_rows<L, 3>(a, stream);
    default: return launch_rows<L, 4>(a, stream);
  }
}

// Lanes per request of the rows kernel: few instances per lane, and few idle
// lanes (4,000,000 rows of one instance: 49 us with four lanes and four requests
// at once, 17.8 with one of each).
static int rows_lanes(int n) { return n <= 2 ? n : (n <= 16 ? 4 : (n <= 64 ? 16 : 64)); }

// A shared snapshot takes a thread per kReq requests from a number of requests
// on.  That thread walks the whole snapshot alone (30 to 40 ns an instance,
// however few the requests are), while lanes per request cost about 0.7 ps per
// place they have for an instance, idle ones and the last pass's included.
// Lanes and thread: 65,000 requests x 66 instances 14.6 and 11.6 us, x 100 14.7
// and 11.5, x 1,000 45.3 and 45.8; 48,000 x 300 20.7 and 16.6; 30,000 x 300 14.5
// and 16.5.
static bool thread_per_request(const ScoreArgs& a) {
  const int64_t L = rows_lanes(a.n_inst), pass = L * std::min<int64_t>(4, (a.n_inst + L - 1) / L);
  const int64_t places = (a.n_inst + pass - 1) / pass * pass;
  return a.stride == 0 && (double)a.n_req * (double)places >= 55000.0 * (double)a.n_inst;
}

hipError_t launch_score(const ScoreArgs& a, hipStream_t stream) {
  if (a.n_req <= 0) return hipSuccess;
  if (thread_per_request(a)) {
    const int64_t per_block = (int64_t)kBlock * kReq;
    const int64_t blocks = (a.n_req + per_block - 1) / per_block;
    const size_t lds = sizeof(SnapEntry) * (((size_t)a.n_inst + 3) & ~(size_t)3);
    hipLaunchKernelGGL(score_shared_kernel, dim3((unsigned)blocks), dim3(kBlock), lds, stream, a);
    return hipGetLastError();
  }
  const bool aligned = ((uintptr_t)a.backlog | (uintptr_t)a.queue | (uintptr_t)a.kv) % 16 == 0;
  if (a.n_inst <= 64 && a.n_inst % 4 == 0 && a.stride % 4 == 0 && aligned) {
    const int64_t per_block = (kBlock / 64) * 4 * kRowGroups;
    const unsigned blocks = (unsigned)((a.n_req + per_block - 1) / per_block);
    hipLaunchKernelGGL(score_rows16_kernel, dim3(blocks), dim3(kBlock), 0, stream, a);
    return hipGetLastError();
  }
  switch (rows_lanes(a.n_inst)) {
    case 1: return launch_rows<1, 1>(a, stream);
    case 2: return launch_rows<2, 1>(a, stream);
    case 4: return launch_rows<4>(a, stream);
    case 16: return launch_rows<16>(a, stream);
    default: return launch_rows<64>(a, stream);
  }
}

hipError_t launch_goodput(const GoodputArgs& a, hipStream_t stream) {
  if (a.n_replicas <= 0) return hipSuccess;
  const unsigned blocks = (unsigned)((a.n_replicas + 3) / 4);
  hipLaunchKernelGGL(goodput_kernel, dim3(blocks), dim3(kBlock), 0, stream, a);
  return hipGetLastError();
}

}  // namespace rt
