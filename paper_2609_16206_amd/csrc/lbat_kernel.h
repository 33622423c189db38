// Replica-batched simulation of the learned prefill/decode router under
// continuous batching, for pools of at most 128 instances, on gfx950: one
// replica per aligned segment of S <= 64 lanes of one wave, M instances per
// lane (prefill instance j on lane j / M, slot j % M; decode instance d on lane
// ceil(P / M) + d / M, slot d % M), every instance's state in registers and its
// queues in LDS.  (The model and the arithmetic are those of bat_kernel.hip.)
//
// Order of work.  The prefill pool needs nothing from the decode pool, so it
// runs one request ahead: iteration u takes the prefill instances' events up to
// arrival u and places request u there, and the decode instances' events up to
// arrival u - 1 and places request u - 1.  Both pools then run through the same
// instructions, lanes of both at once: the rounds, the score, the argmins and
// the admission.  A prefill that ends in iteration u (up to arrival u, so a
// request before u, placed on its decode instance by the end of the iteration)
// leaves a record in its segment's list in LDS; at the end of the iteration
// the decode lanes take the transfers meant for them from the list, none of
// which lands before arrival u - 1.  A prefill lane that finds the list full
// waits, and the iteration is repeated for its pool after the list was taken; in
// the wave's other segments the request just placed does not join meanwhile (one
// without prefill work would end in the iteration that placed it, before its
// decode placement).
//
// Events.  An instance has members (the batch, sorted by finish virtual time)
// and joins to come: KV transfers sorted by landing time, or, on a prefill
// instance, the request it was given last, which joins at its arrival with the
// next iteration's events.  A round takes, on every lane and slot, a join that
// comes before the next completion, then a completion that comes no later than
// the next join; rounds go on while some lane had an event.  A prefill instance's
// join comes before any completion: those up to its arrival were taken before it
// was placed.  (The completion taken again from the clock at that arrival can
// round to the arrival itself; the batch has the new member by then.)
//
// Queues.  The front entry is in registers, with all that the event needs; the
// next ones are a sorted ring in LDS (32 bytes each; as many as the waves that
// are to share a compute unit leave room for), and those beyond it a sorted
// ring in HBM, which holds key and request alone (the rest is read back from
// the trace, a decode member's prefill end from its span slot, where it is
// parked).  While something lies in HBM the LDS ring is full, so a queue is
// always in order front, LDS, HBM.  Nothing waits for HBM on the common path:
// the trace comes a block of S requests ahead, by way of records in LDS, and
// outcomes are stored and forgotten.
//
// What bounds it: the instructions of a step's chain (clock, score, argmin,
// admission, and as many rounds as the busiest lane of the wave has events: about
// 2.4 for four replicas of 2 + 6), some 720 a step at about 1.8 issue slots
// each.  Batches are short (2 + 6 at its own rate: one member in the median, 90 %
// at most four; transfers in flight: one), so an insertion into an empty queue, a
// departure that leaves one empty and a clock step of batches of one (no
// division) each have a short way, taken where all active lanes can.
// Measured, before (a kernel with the rings in HBM and the prefill pool's rounds
// before the decode pool's: 4.0 us a step, its vector unit 29 % busy between
// waits for loads behind stores) and now: 4,096 replicas of 2 + 6 x 3,000
// 12.1 and 7.0 ms; 8,192 of 8 + 64 x 500 6.9 and 5.6 ms.  Two waves per SIMD with
// half the replicas each took the same 7.0 ms; three instances per lane (two
// replicas of 8 + 64 a wave) spill and took 5.9 ms.
#pragma once

#include <algorithm>

#include "lane_ops.h"
#include "rt_internal.h"

namespace rt {
namespace bat {

constexpr int kLbatWaves = 4;  // waves of a workgroup, at most

// A member of a batch, or a join to come.
struct alignas(16) Member {
  double t;      // finish virtual time; landing time (prefill: arrival)
  int32_t r;     // request
  int32_t f;     // cache tokens it holds: p (prefill), p + o (decode)
  double x0;     // what its outcome is measured from: arrival; prefill end
  int32_t o, oh;
};
static_assert(sizeof(Member) == 32, "two 16-byte words");

// Later than every event.
constexpr double kFar = 1.7976931348623157e308;

// A request as a step reads it.
struct alignas(16) BReq {
  double now;  // arrival if accepted, -1 if rejected, kFar beyond the replica
  int32_t p;   // 0: nothing to place
  int32_t o, oh;
  float sg;
  int32_t pad[2];
};
static_assert(sizeof(BReq) == 32, "two 16-byte words");

typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
typedef __attribute__((address_space(3))) int32_t lds_i32;
typedef __attribute__((address_space(3))) uint16_t lds_u16;

__device__ __forceinline__ void lds_min(uint32_t at, int32_t v) {
  __hip_atomic_fetch_min((lds_i32*)(uintptr_t)at, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

template <typename T>
__device__ __forceinline__ T lds_get32(uint32_t at) {
  const u32x4 v[2] = {*(const lds_u32x4*)(uintptr_t)at, *(const lds_u32x4*)(uintptr_t)(at + 16)};
  T x;
  __builtin_memcpy(&x, v, sizeof v);
  return x;
}
template <typename T>
__device__ __forceinline__ void lds_put32(uint32_t at, const T& x) {
  u32x4 v[2];
  __builtin_memcpy(v, &x, sizeof v);
  *(lds_u32x4*)(uintptr_t)at = v[0];
  *(lds_u32x4*)(uintptr_t)(at + 16) = v[1];
}

// A sorted queue of one instance.
struct Queue {
  Member fr;     // the front; t = +inf where the queue is empty
  int32_t cnt;   // entries in all
  int32_t n;     // in the LDS ring
  int32_t x;     // beyond it
  int32_t hx;    // head of those
  uint32_t hd;   // head of the LDS ring (bytes, taken modulo the ring)
  double tt;     // the last entry in the LDS ring
  int32_t tr;
};

struct LInst {
  double v, tl, left, kv, pend, owed;
  double tc;   // the batch's next completion (+inf where it has no member)
  double nd;   // members
  double sd;   // slowdown at that many
  int32_t q;
  int32_t d0;  // prefill: the decode instance of the batch's front, -1 where not at hand
  Queue b, j;  // the batch, the joins to come
};

// Layout of a launch: every instance slot of a wave has (bmask + tmask) / 32 +
// 2 entries and a gap of one (so that the slots' rings do not start on one
// LDS bank); the waves' records follow at rec_at.
struct LBat {
  uint32_t bmask, tmask;  // ring bytes - 32 of the batch and of the joins
  uint32_t stride;        // bytes of an instance slot
  uint32_t max_inst;      // instance slots of a segment
  uint32_t rec_at;
  uint32_t wave_bytes;    // records, list, table and candidates of a wave
};

template <int S>
struct LbatDims {
  static constexpr int kSegs = 64 / S;
  static constexpr int kRecs = 2 * S;                     // records of a segment: two blocks
  static constexpr int kRecBytes = kRecs * 32 + 32;       // and a gap, as above
  static constexpr int kList = S / 2 < 4 ? 4 : S / 2;     // departures listed at once
  static constexpr int kTable = kRecs < 32 ? 32 : kRecs;  // latest requests whose decode instance is at hand
  static constexpr int kStop = kSegs < 2 ? 16 : kSegs * 8;  // where each replica first rejected a request and stopped
  static constexpr int kList0 = kSegs * kRecBytes, kDst0 = kList0 + kSegs * kList * 32,
                       kTable0 = kDst0 + kSegs * kList * 4, kStop0 = kTable0 + kSegs * kTable * 2,
                       kCand0 = kStop0 + kStop;
  static constexpr int kCandBytes = kSegs * kRecs * 16;
  static_assert(kCand0 % 16 == 0, "16-byte words");
};

template <int S, int M, int kOcc>
__global__ void __launch_bounds__(64 * kLbatWaves, kOcc) lbat_kernel(SimArgs a, BatScratch b, LBat g) {
  using Dm = LbatDims<S>;
  const int lane = (int)(threadIdx.x & 63);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t wave_id = blockIdx.x * (blockDim.x >> 6) + wave;
  const int sl = lane & (S - 1);
  const int sg0 = lane & ~(S - 1);  // the segment's first lane
  const int seg = lane / S;
  const int64_t item = (int64_t)wave_id * (64 / S) + seg;
  const bool has = item < a.n_work;
  const int32_t rep = has ? a.work[item] : 0;
  const int64_t lo = has ? a.offsets[rep] : 0;
  const int32_t R = has ? (int32_t)(a.offsets[rep + 1] - lo) : 0;
  const DevPoint& pt = a.points[(has && a.param_point) ? a.param_point[rep] : 0];
  const int32_t P = pt.P, D = pt.D;
  const int32_t LP = (P + M - 1) / M, LD = (D + M - 1) / M;  // lanes holding each pool
  const bool isP = has && sl < LP;
  const bool isD = has && sl >= LP && sl < LP + LD;
  const int32_t npool = isP ? P : D;
  const int32_t j0 = (isP ? sl : sl - LP) * M;  // the lane's first instance in its pool
  bool ok[M];                                    // the slot holds an instance
#pragma unroll
  for (int m = 0; m < M; ++m) ok[m] = (isP || isD) && j0 + m < npool;
  const double beta = isP ? pt.beta_pre : pt.beta_dec;
  const double xfer = (double)pt.xfer_tok_ns;
  const int32_t ncls = pt.n_classes, pol = pt.policy, len_thr = pt.len_thr, bmode = pt.mode;
  const float w_b = pt.w_b, w_s = pt.w_s, w_q = pt.w_q, rho = pt.rho;
  const float tau = isP ? pt.tau_pre : pt.tau_dec;
  const float basec = isP ? pt.pre_base : 0.0f;
  const float inv = isP ? pt.inv_cap_pre : pt.inv_cap_dec;
  // stand-alone work: base + tokens (prefill: p, decode: o - 1) x price
  const double wbase = isP ? (double)pt.pre_base_ns : 0.0;
  const double wtok = isP ? (double)pt.pre_tok_ns : (double)pt.dec_tok_ns;
  const float sig_l = pt.sigma[sl & (kMaxClasses - 1)];  // lane k: sigma of class k mod 8 (S = 4: the first four)
  const float sig_h = pt.sigma[(sl & 3) + 4];
  // wave-uniform: which scoring terms some replica of the wave needs
  const bool lrn = pol == kPolicyLearned || pol == kPolicyLearnedSampled;
  const bool any_true = __any(has && lrn && bmode == 0), any_proxy = __any(has && lrn && bmode != 0);
  const bool any_samp = __any(has && pol == kPolicyLearnedSampled), any_base = __any(has && !lrn);
  const int32_t C = b.C;

  // LDS (a kernel without static shared memory: addresses from 0)
  const uint32_t w0 = g.rec_at + wave * g.wave_bytes;
  const uint32_t rec0 = w0 + (uint32_t)(seg * Dm::kRecBytes);
  const uint32_t list0 = w0 + Dm::kList0 + (uint32_t)(seg * Dm::kList * 32);
  const uint32_t dst0 = w0 + Dm::kDst0 + (uint32_t)(seg * Dm::kList * 4);
  const uint32_t tab0 = w0 + Dm::kTable0 + (uint32_t)(seg * Dm::kTable * 2);
  // the segment's first request rejected, and the first that found a queue full:
  // the replica stops there, and rejections after it do not count (in LDS:
  // rarely written)
  const uint32_t rej_at = w0 + Dm::kStop0 + (uint32_t)(seg * 8), full_at = rej_at + 4;
  *(lds_i32*)(uintptr_t)rej_at = *(lds_i32*)(uintptr_t)full_at = INT32_MAX;
  const uint32_t cand0 = w0 + Dm::kCand0 + (uint32_t)(seg * Dm::kRecs * 16);
  // ring entries: never more than the queue's capacity leaves behind its front
  const int32_t limb = min((int32_t)(g.bmask >> 5) + 1, C - 1), limt = min((int32_t)(g.tmask >> 5) + 1, C - 1);
  uint32_t bring[M], jring[M];
  Entry* hb[M];
  Entry* hj[M];
  const int64_t gl = (int64_t)wave_id * 64 + lane;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const uint32_t slot = (wave * (uint32_t)Dm::kSegs + (uint32_t)seg) * g.max_inst +
                          (ok[m] ? (uint32_t)((isP ? 0 : P) + j0 + m) : 0u);
    bring[m] = slot * g.stride;
    jring[m] = bring[m] + g.bmask + 32;
    hb[m] = reinterpret_cast<Entry*>(b.ring) + (gl * M + m) * (int64_t)C;
    hj[m] = reinterpret_cast<Entry*>(b.wring) + (gl * M + m) * (int64_t)C;
  }
  uint64_t segm = ~0ull, below = (1ull << lane) - 1ull;  // lanes of the segment; those before this one
  if constexpr (S < 64) segm = ((1ull << (S & 63)) - 1ull) << sg0;
  below &= segm;

  LInst in[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    LInst& x = in[m];
    x.v = x.tl = x.left = x.kv = x.pend = x.owed = x.nd = 0.0;
    x.sd = 1.0;
    x.tc = kInf;
    x.q = 0;
    x.d0 = -1;
    x.b = Queue{Member{kInf, 0, 0, 0.0, 0, 0}, 0, 0, 0, 0, 0u, 0.0, 0};
    x.j = x.b;
  }
  bool full = false, dead = false;

  auto any_lane = [](bool c) __attribute__((always_inline)) { return __builtin_amdgcn_ballot_w64(c) != 0; };
  auto before = [](double t, int32_t r, double t2, int32_t r2) __attribute__((always_inline)) {
    return t < t2 || (t == t2 && r < r2);
  };
  // An entry goes to HBM: a decode request's prefill end is parked in its span
  // slot (its outcome replaces it there).
  auto park = [&](int32_t r, double x0) __attribute__((always_inline)) {
    if (isD) a.span[lo + r] = __double_as_longlong(x0);
  };

  // e into a queue (on the active lanes), on the way to the placement of request
  // `step`.
  auto insert = [&](Queue& Q, uint32_t ring, uint32_t mask, int32_t lim, Entry* hbm, const Member& e, int32_t step)
                    __attribute__((always_inline)) {
    if (__builtin_expect(!any_lane(Q.cnt > 0), 1)) {  // alone in it
      Q.fr = e;
      Q.cnt = 1;
      return;
    }
    auto at = [&](int32_t i) __attribute__((always_inline)) { return ring + ((Q.hd + (uint32_t)i * 32u) & mask); };
    bool put = true;
    if (__builtin_expect(any_lane(Q.n >= lim), 0)) {
      if (Q.n >= lim) {
        if (Q.cnt >= C) {
          full = true;
          lds_min(full_at, step);
          put = false;
        } else if (!before(e.t, e.r, Q.tt, Q.tr)) {  // behind the LDS ring
          int32_t i = Q.hx + Q.x;
          while (i > Q.hx) {
            const Entry z = hbm[(i - 1) & (C - 1)];
            if (!before(e.t, e.r, z.t, z.r)) break;
            hbm[i & (C - 1)] = z;
            --i;
          }
          hbm[i & (C - 1)] = Entry{e.t, e.r, 0};
          park(e.r, e.x0);
          Q.x += 1;
          Q.cnt += 1;
          put = false;
        } else {  // the ring's last entry makes room
          const Member z = lds_get32<Member>(at(Q.n - 1));
          Q.hx -= 1;
          hbm[Q.hx & (C - 1)] = Entry{z.t, z.r, 0};
          park(z.r, z.x0);
          Q.x += 1;
          Q.n -= 1;
          const Member y = lds_get32<Member>(at(Q.n - 1));  // (not used where none is left)
          Q.tt = y.t;
          Q.tr = y.r;
        }
      }
    }
    if (put) {
      const bool had = Q.cnt > 0;
      const bool lt = !had || before(e.t, e.r, Q.fr.t, Q.fr.r);
      int32_t i = Q.n;  // the ring position taken, from the head
      const bool shift = !lt && Q.n > 0 && before(e.t, e.r, Q.tt, Q.tr);
      if (any_lane(shift)) {
        if (shift) {
          while (i > 0) {
            const Member z = lds_get32<Member>(at(i - 1));
            if (!before(e.t, e.r, z.t, z.r)) break;
            lds_put32(at(i), z);
            --i;
          }
        }
      }
      // a new front sends the old one to the ring (an empty queue's: nothing
      // reads it there)
      Member s;
      s.t = lt ? Q.fr.t : e.t;
      s.r = lt ? Q.fr.r : e.r;
      s.f = lt ? Q.fr.f : e.f;
      s.x0 = lt ? Q.fr.x0 : e.x0;
      s.o = lt ? Q.fr.o : e.o;
      s.oh = lt ? Q.fr.oh : e.oh;
      const bool last = lt ? Q.n == 0 : i == Q.n;
      lds_put32(at(lt ? -1 : i), s);
      Q.fr.t = lt ? e.t : Q.fr.t;
      Q.fr.r = lt ? e.r : Q.fr.r;
      Q.fr.f = lt ? e.f : Q.fr.f;
      Q.fr.x0 = lt ? e.x0 : Q.fr.x0;
      Q.fr.o = lt ? e.o : Q.fr.o;
      Q.fr.oh = lt ? e.oh : Q.fr.oh;
      Q.hd -= lt ? 32u : 0u;
      Q.tt = last ? s.t : Q.tt;
      Q.tr = last ? s.r : Q.tr;
      Q.n += had ? 1 : 0;
      Q.cnt += 1;
    }
  };
  // The front leaves a queue (on the active lanes; the queue is not empty).
  auto pop = [&](Queue& Q, uint32_t ring, uint32_t mask, const Entry* hbm) __attribute__((always_inline)) {
    Q.fr.t = kInf;
    if (__builtin_expect(!any_lane(Q.n > 0), 1)) {
      Q.cnt = 0;
      return;
    }
    const bool more = Q.n > 0;
    const Member f = lds_get32<Member>(ring + (Q.hd & mask));
    Q.fr = f;
    Q.fr.t = more ? f.t : kInf;
    Q.hd += more ? 32u : 0u;
    Q.n -= more ? 1 : 0;
    Q.cnt -= 1;
    if (__builtin_expect(any_lane(Q.x > 0), 0)) {
      if (Q.x > 0) {  // the ring's place is taken by the first entry beyond it
        const Entry z = hbm[Q.hx & (C - 1)];
        const int64_t gi = lo + z.r;
        const int32_t p = a.plen[gi], o = a.olen[gi], oh = a.ohat[gi];
        const int64_t w = isP ? a.arrival[gi] : a.span[gi];
        const double x0 = isP ? i64_to_f64(w) : __longlong_as_double(w);
        lds_put32(ring + ((Q.hd + (uint32_t)Q.n * 32u) & mask), Member{z.t, z.r, isP ? p : p + o, x0, o, oh});
        Q.tt = z.t;
        Q.tr = z.r;
        Q.n += 1;
        Q.x -= 1;
        Q.hx += 1;
      }
    }
  };
  // The next completion, after the batch or its clock changed.
  auto next_done = [&](LInst& x) __attribute__((always_inline)) {
    x.tc = x.tl + max_f64(x.b.fr.t - x.v, 0.0) * x.sd;
  };
  auto resize = [&](LInst& x, double by) __attribute__((always_inline)) {
    x.nd = x.nd + by;
    x.sd = 1.0 + beta * max_f64(x.nd - 1.0, 0.0);
    next_done(x);
  };
  // The clock to time t (the caller brings x.tc up to date).  A batch of one
  // runs at full speed: x / 1 = x.
  auto clock_to = [&](LInst& x, double t) __attribute__((always_inline)) {
    double dv = t - x.tl;
    if (any_lane(x.nd > 1.0)) {
      asm volatile("" : "+v"(dv));  // (keeps the division under the branch)
      dv = dv / x.sd;
    }
    dv = x.nd > 0.0 ? dv : 0.0;  // (an idle batch's clock stands still, its work is 0)
    x.v = x.v + dv;
    x.left = x.left - x.nd * dv;
    x.tl = t;
  };

  const int32_t Rmax = __builtin_amdgcn_readfirstlane(wave_max_nonneg(R));

  // Raw trace of a block, lane k of the segment holding request (block start +
  // k) (clamped into the replica; request 0 of the trace for a segment without
  // one).
  const int64_t rd_base = R > 0 ? lo : 0;
  const uint32_t rd_last = R > 0 ? (uint32_t)(R - 1) : 0u;
  struct Raw {
    int64_t arr;
    int32_t p, o, oh;
    uint32_t c;
    uint4 w;
  };
  auto load_raw = [&](Raw& f, uint32_t blk) __attribute__((always_inline)) {
    const int64_t i = rd_base + min(blk + (uint32_t)sl, rd_last);
    f.arr = a.arrival[i];
    f.p = a.plen[i];
    f.o = a.olen[i];
    f.oh = a.ohat[i];
    f.c = a.cls[i];
    if (any_samp) f.w = *reinterpret_cast<const uint4*>(a.samp + 4 * i);
  };
  // The records of a block.  A request is accepted if it is valid and its
  // arrival equals the running maximum of the valid arrivals so far.
  double carry = 0.0;  // largest valid arrival before the block
  auto derive = [&](const Raw& f, uint32_t blk) __attribute__((always_inline)) {
    const int32_t p = f.p, o = f.o, oh = f.oh;
    const int32_t po = (int32_t)((uint32_t)p + (uint32_t)o), poh = (int32_t)((uint32_t)p + (uint32_t)oh);
    const uint32_t i = blk + (uint32_t)sl;
    const bool inside = i < (uint32_t)R;
    const int32_t vm = min(min(min(p, o), min(oh, po)), min(poh, ncls - (int32_t)f.c));
    const bool valid = inside && opaque(vm) >= 1;
    const double x = valid ? i64_to_f64(f.arr) : -1.0;
    double incl = x;
#pragma unroll
    for (int d = 1; d < S; d *= 2) {
      const double y = __shfl_up(incl, d, S);
      incl = sl >= d ? __builtin_fmax(incl, y) : incl;
    }
    incl = __builtin_fmax(incl, carry);
    carry = __shfl(incl, S - 1, S);
    const bool acc = valid && x == incl;
    BReq r;
    r.now = !inside ? kFar : (acc ? x : -1.0);
    r.p = acc ? p : 0;
    r.o = o;
    r.oh = oh;
    const int32_t cl = (int32_t)(f.c & (kMaxClasses - 1));
    r.sg = __shfl(sig_l, cl, S);
    if constexpr (S < kMaxClasses) {
      const float hi = __shfl(sig_h, cl & (S - 1), S);
      r.sg = cl >= S ? hi : r.sg;
    }
    r.pad[0] = r.pad[1] = 0;
    lds_put32(rec0 + (i & (Dm::kRecs - 1)) * 32u, r);
    if (any_samp) {
      uint32_t c1, c2, d1, d2;
      c1 = __umulhi(f.w.x, (uint32_t)P);
      c2 = __umulhi(f.w.y, (uint32_t)(P - 1));
      c2 = P > 1 ? c2 + (c2 >= c1 ? 1u : 0u) : c1;
      d1 = __umulhi(f.w.z, (uint32_t)D);
      d2 = __umulhi(f.w.w, (uint32_t)(D - 1));
      d2 = D > 1 ? d2 + (d2 >= d1 ? 1u : 0u) : d1;
      *(lds_u32x4*)(uintptr_t)(cand0 + (i & (Dm::kRecs - 1)) * 16u) = u32x4{c1, c2, d1, d2};
    }
    if (inside && !acc) {
      lds_min(rej_at, (int32_t)i);
      a.ttft[lo + i] = a.span[lo + i] = -1;
    }
  };
  struct Cur {
    BReq r;
    u32x4 c;
  };
  auto read_rec = [&](Cur& q, uint32_t i) __attribute__((always_inline)) {
    q.r = lds_get32<BReq>(rec0 + (i & (Dm::kRecs - 1)) * 32u);
    if (any_samp) q.c = *(const lds_u32x4*)(uintptr_t)(cand0 + (i & (Dm::kRecs - 1)) * 16u);
  };

  int64_t* const o_t = (isP ? a.ttft : a.span) + lo;
  const uint32_t lag = isP ? 0u : 1u;  // the lane's request of iteration u is u - lag
  int32_t ndep = 0;    // departures in the segment's list
  uint64_t stall = 0;  // lanes waiting for room in it
  int32_t idc = -1;    // the decode instance of the latest decode placement

  // Every event up to `now` (prefill lanes: as far as the list has room).
  auto rounds = [&](double now, uint32_t u) __attribute__((always_inline)) {
    for (;;) {
      bool act = false;
      stall = 0;
      static_for<M>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        LInst& x = in[m];
        const double tj = x.j.fr.t;
        const bool join = tj <= now && tj < x.tc;
        if (join) {
          Member e = x.j.fr;
          pop(x.j, jring[m], g.tmask, hj[m]);
          clock_to(x, tj);
          const double w = wbase + (double)(isP ? e.f : e.o - 1) * wtok;
          x.owed = x.owed - w;
          x.left = x.left + w;
          e.t = x.v + w;
          // (a prefill instance took the request when it was placed)
          insert(x.b, bring[m], g.bmask, limb, hb[m], e, isP ? e.r : (int32_t)(u - 1u));
          x.d0 = x.b.fr.r == e.r ? -1 : x.d0;
          resize(x, 1.0);
        }
        bool fire = x.tc <= now && x.tc <= x.j.fr.t;
        int32_t pos = 0;
        const uint64_t wm = __builtin_amdgcn_ballot_w64(fire && isP);
        if (wm != 0) {
          pos = ndep + __popcll(wm & below);
          stall |= __builtin_amdgcn_ballot_w64(fire && isP && pos >= Dm::kList);
          fire = fire && (isD || pos < Dm::kList);
          ndep = min(ndep + (int32_t)__popcll(wm & segm), Dm::kList);
        }
        if (fire) {
          const Member e = x.b.fr;
          const double tc = x.tc;
          x.left = x.left - x.nd * (e.t - x.v);
          x.v = e.t;
          x.tl = tc;
          x.q -= 1;
          x.kv = x.kv - (double)e.f;
          x.pend = x.pend - (double)(isP ? e.f : e.oh);
          o_t[e.r] = round_ns(tc - e.x0);
          if (isP) {
            lds_put32(list0 + (uint32_t)pos * 32u,
                      Member{tc + (double)e.f * xfer, e.r, e.f + e.o, tc, e.o, e.oh});
            // (request u - 1 is yet to be placed; one that was not at the
            // front when it was placed is in the table, or was written out
            // since)
            int32_t d = x.d0;
            const bool look = d < 0 && (uint32_t)e.r != u - 1u;
            if (__builtin_expect(any_lane(look), 0)) {
              if (look) {
                if (u - (uint32_t)e.r < (uint32_t)Dm::kTable)
                  d = *(const lds_u16*)(uintptr_t)(tab0 + ((uint32_t)e.r & (Dm::kTable - 1)) * 2u);
                else
                  d = a.i_dec[lo + e.r];
              }
              d = opaque(d);  // (waits for the load here, not on the common path)
            }
            *(lds_i32*)(uintptr_t)(dst0 + (uint32_t)pos * 4u) = d;
          }
          pop(x.b, bring[m], g.bmask, hb[m]);
          x.d0 = -1;
          x.left = x.b.cnt == 0 ? 0.0 : x.left;
          resize(x, -1.0);
        }
        act = act || join || fire;
      });
      if (!any_lane(act)) return;
    }
  };

  // outcomes of the block's iterations, lane k keeping the k-th
  int32_t b_ip = -1, b_id = -1;

  Raw raw;
  load_raw(raw, 0);
  derive(raw, 0);
  if (sl == S - 1) lds_put32(rec0 + (Dm::kRecs - 1) * 32u, BReq{-1.0, 0, 1, 1, 0.0f, {0, 0}});  // "request -1"
  load_raw(raw, (uint32_t)S);
  Cur cur;
  read_rec(cur, 0u - lag);
  const uint32_t end = (uint32_t)Rmax + 2u;  // (one iteration drains the prefill pool, one more the decode pool)
  for (uint32_t blk = 0; blk < end; blk += S) {
    derive(raw, blk + S);
    load_raw(raw, blk + 2 * S);
    const uint32_t ue = min(blk + (uint32_t)S, end);
#pragma unroll 1
    for (uint32_t u = blk; u < ue; ++u) {
      if (dead) {
        cur.r.now = -1.0;
        cur.r.p = 0;
      }
      const double now = cur.r.now;
      bool again = false;
      for (;;) {
        rounds(now, u);
        const bool held = isP && (stall & segm) != 0;
        const bool go = cur.r.p > 0 && !held;
        const int32_t p = cur.r.p, o = cur.r.o, oh = cur.r.oh;
        const float sg = cur.r.sg;
        const float work = w_s * (float)(isP ? p : oh) * tau;
        const double need = (double)(isP ? p : p + oh);
        uint32_t bkey = 0xffffffffu;
        int32_t bm = 0;
        static_for<M>([&](auto mc) __attribute__((always_inline)) {
          constexpr int m = decltype(mc)::value;
          LInst& x = in[m];
          if (go) {
            clock_to(x, now);
            next_done(x);
          }
          float bl = 0.0f;
          if (any_true) {
            double w = x.left < 0.0 ? 0.0 : x.left;
            w = w + x.owed;
            bl = (float)w * 1e-9f;
          }
          if (any_proxy) {
            const float bp = tau * (float)x.pend + basec * (float)x.q;
            bl = bmode == 0 ? bl : bp;
          }
          const float press = (float)(x.kv + need) * inv;
          const float load = w_b * bl * sg;
          const float size = work * (1.0f + rho * press) * sg;
          uint32_t key = cost_key(load + size + w_q * (float)x.q);
          const int32_t jj = j0 + m;
          if (any_samp) {
            const uint32_t c1 = isP ? cur.c[0] : cur.c[2], c2 = isP ? cur.c[1] : cur.c[3];
            key = pol != kPolicyLearnedSampled || (uint32_t)jj == c1 || (uint32_t)jj == c2 ? key : 0xffffffffu;
          }
          if (any_base) {
            // round robin; least loaded; or least loaded within the decode
            // part the request's predicted length picks (length threshold)
            const bool part = isP || npool == 1 || ((jj >= (npool + 1) / 2) == (oh >= len_thr));
            const uint32_t rr = (uint32_t)jj == (u - lag) % (uint32_t)npool ? 0u : 1u;
            const uint32_t kb = pol == kPolicyRoundRobin ? rr
                                : pol == kPolicyLengthThreshold && !part ? 0xffffffffu : (uint32_t)x.q;
            key = lrn ? key : kb;
          }
          key = ok[m] && go ? key : 0xffffffffu;
          const bool lower = m == 0 || key < bkey;
          bkey = lower ? key : bkey;
          bm = lower ? m : bm;
        });
        uint32_t kp = isP ? bkey : 0xffffffffu, kd = isD ? bkey : 0xffffffffu;
        seg_min2<S>(kp, kd);
        const int32_t wp = seg_first<S>(isP && bkey == kp, lane);  // winning lanes
        const int32_t wd = seg_first<S>(isD && bkey == kd, lane);
        int32_t ip = wp * M, id = (wd - LP) * M;
        if constexpr (M > 1) {
          ip += (int32_t)seg_or<S>(sl == wp ? (uint32_t)bm : 0u);
          id += (int32_t)seg_or<S>(sl == wd ? (uint32_t)bm : 0u);
        }
        // (no key: nothing was placed)
        const bool keep = (u & (S - 1)) == (uint32_t)sl;
        b_ip = keep && kp != 0xffffffffu ? ip : b_ip;
        b_id = keep && kd != 0xffffffffu ? id : b_id;
        idc = kd != 0xffffffffu ? id : idc;
        static_for<M>([&](auto mc) __attribute__((always_inline)) {
          LInst& x = in[decltype(mc)::value];
          x.d0 = kd != 0xffffffffu && x.b.fr.r == (int32_t)(u - 1u) ? idc : x.d0;
        });

        // admission: the instance holds the request's tokens and owes its
        // work from now on; a prefill instance takes it into its batch with
        // the next events, a decode instance once its KV lands
        if (go && sl == (isP ? wp : wd)) {
          const double w = wbase + (double)(isP ? p : o - 1) * wtok;
          const double f = (double)(isP ? p : p + o), k = (double)(isP ? p : oh);
          static_for<M>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            LInst& x = in[m];
            if (M > 1 && bm != m) return;
            x.owed = x.owed + w;
            x.q += 1;
            x.kv = x.kv + f;
            x.pend = x.pend + k;
            if (isP) {
              x.j.fr = Member{now, (int32_t)u, p, now, o, oh};
              x.j.cnt = 1;
              x.tc = kInf;  // (no completion before it joins)
            }
          });
          if (isD) *(lds_u16*)(uintptr_t)(tab0 + ((u - 1u) & (Dm::kTable - 1)) * 2u) = (uint16_t)(j0 + bm);
        }
        // the listed transfers go to their decode instances
        for (int32_t i = 0; any_lane(i < ndep); ++i) {
          const Member e = lds_get32<Member>(list0 + (uint32_t)i * 32u);
          int32_t d = *(const lds_i32*)(uintptr_t)(dst0 + (uint32_t)i * 4u);
          d = (uint32_t)e.r == u - 1u ? idc : d;
          const bool mine = isD && i < ndep;
          static_for<M>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value;
            if (mine && d == j0 + m) insert(in[m].j, jring[m], g.tmask, limt, hj[m], e, (int32_t)u);
          });
        }
        ndep = 0;
        if (__builtin_expect(stall == 0, 1)) break;
        again = true;
        if (!held) {
          cur.r.p = 0;  // placed already; it joins with the next iteration
          static_for<M>([&](auto mc) __attribute__((always_inline)) {
            LInst& x = in[decltype(mc)::value];
            if (isP && x.j.fr.t < kInf) x.tc = __builtin_nan("");
          });
        }
      }
      if (__builtin_expect(again, 0)) {
        static_for<M>([&](auto mc) __attribute__((always_inline)) {
          LInst& x = in[decltype(mc)::value];
          x.tc = x.tc != x.tc ? kInf : x.tc;
        });
      }
      if (__builtin_expect(any_lane(full), 0)) dead = seg_or<S>(full ? 1u : 0u) != 0;  // (the replica stops)
      read_rec(cur, u + 1u - lag);
    }
    if (blk + (uint32_t)sl < (uint32_t)R) a.i_pre[lo + blk + sl] = b_ip;
    if (blk + (uint32_t)sl - 1u < (uint32_t)R) a.i_dec[lo + blk + sl - 1] = b_id;
    b_ip = b_id = -1;
  }
  // (an instance's clock never goes back: its last value is the latest time it reached)
  // (what is left after the drain had no finite time to end at)
  bool late = false;
#pragma unroll
  for (int m = 0; m < M; ++m)
    late = late || (ok[m] && (in[m].tl >= kTimeLimit || (!dead && in[m].b.cnt + in[m].j.cnt > 0)));
  const bool rej = *(const lds_i32*)(uintptr_t)rej_at < *(const lds_i32*)(uintptr_t)full_at;
  const uint32_t flag = (late ? kFlagTimeRange : 0u) | (rej ? kFlagRejected : 0u) | (full ? kFlagBatchCap : 0u);
  if (flag) atomicOr(a.flag, flag);
}

template <int S, int M, int kOcc>
hipError_t launch_lbat_occ(const SimArgs& a, const BatScratch& b, hipStream_t stream) {
  using Dm = LbatDims<S>;
  const int64_t waves = (a.n_work + Dm::kSegs - 1) / Dm::kSegs;
  const LdsShare share = lds_share(a.call_waves, 4 * kOcc);
  const uint32_t wpb = share.wpb;
  LBat g{};
  g.max_inst = (uint32_t)a.max_inst;
  g.wave_bytes = (uint32_t)(Dm::kCand0 + (a.samp ? Dm::kCandBytes : 0));
  const uint32_t slots = (uint32_t)Dm::kSegs * g.max_inst;  // of a wave
  const uint32_t room = share.bytes - g.wave_bytes;
  // entries of the two rings: what the compute unit's waves leave each slot
  uint32_t kb = 16, kt = 8;
  while (kb > 1 && slots * 32u * (kb + kt + 1) > room) {
    kb /= 2;
    kt = std::max(1u, kt / 2);
  }
  g.bmask = (kb - 1) * 32;
  g.tmask = (kt - 1) * 32;
  g.stride = 32 * (kb + kt + 1);
  g.rec_at = wpb * slots * g.stride;
  const uint32_t lds = g.rec_at + wpb * g.wave_bytes;
  if (lds > 64 * 1024) {
    // (per device, so at every launch; the whole of a compute unit's, so that
    // a smaller launch of another thread takes nothing from this one)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lbat_kernel<S, M, kOcc>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((lbat_kernel<S, M, kOcc>), dim3((unsigned)((waves + wpb - 1) / wpb)), dim3(64 * wpb), lds, stream, a,
                     b, g);
  return hipGetLastError();
}

// Three waves per SIMD where a call has more than two, two otherwise.  Segments
// of 32 and 64 lanes gain from the third (with rings of at least two and one
// entries, one and one where all waves then fit in one pass): 16,384 replicas of
// 3 + 14 x 500 4.62 and 3.84 ms, 5,120 x 400 1.54 and 1.16, 2,560 of 10 + 29 x 300
// 0.98 and 0.75, 2,300 of 2 + 62 x 150 0.49 and 0.37.  Narrower ones have more
// replicas, so more slots a wave, and their rings would be too short for the
// batches of small pools: 65,536 of 1 + 2 x 1,000 8.4 ms with two waves and 17.7
// with three, of 2 + 6 13.1 and 20.9.  With three, segments of 32 lanes spill 36
// registers a lane and those of 64 four (the figures have that in them); two
// instances per lane fill the registers of two waves.
template <int S, int M>
hipError_t launch_lbat(const SimArgs& a, const BatScratch& b, hipStream_t stream) {
  if constexpr (M == 1 && S >= 32) {
    using Dm = LbatDims<S>;
    const int64_t per_cu = waves_per_cu(a.call_waves);
    const uint32_t slots = (uint32_t)Dm::kSegs * (uint32_t)a.max_inst, places = per_cu <= 12 ? 1 + 1 + 1 : 2 + 1 + 1;
    const uint32_t bytes = slots * 32 * places + Dm::kCand0 + (a.samp ? Dm::kCandBytes : 0);
    if (per_cu > 8 && bytes <= lds_share(a.call_waves, 12).bytes)
      return launch_lbat_occ<S, M, 3>(a, b, stream);
  }
  return launch_lbat_occ<S, M, 2>(a, b, stream);
}

}  // namespace bat
}  // namespace rt
