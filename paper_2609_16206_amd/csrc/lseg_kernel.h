// Replica-batched simulation of the learned prefill/decode router for pools
// of at most 32 instances a side, FIFOs in LDS, on gfx950.
//
// Method: Algorithm 1 per admission (score every instance of both pools with
// the Section III-A cost equation, take each pool's argmin, prefill, transfer
// the KV cache, decode, record), on the serial-service simulator of Section
// III-D / Section VI.
//
// Mapping.  A replica is a chain of admissions; replicas are independent.
// One replica occupies an aligned segment of S lanes of one wave (64 / S
// replicas per wave); its prefill instances are on the lower half of the
// segment's lanes and its decode instances on the upper half, one per lane.
// Each half then takes its own pool's argmin with one reduction, and hands
// the other half what it needs in one exchange.  Per-instance state lives in
// registers, the FIFOs of requests in flight in LDS.
//
// What bounds it: a replica's steps follow one another, so a launch of few
// waves is as long as one wave's step times the requests, and the slowest
// wave's at that.  A wave issues an instruction every four cycles, so the
// step is written for few instructions (about 130, 820 cycles where no queue
// is deep; the kernel of seg_kernel.h, which keeps the FIFO's front in
// registers and the rest in HBM, takes about 270 and 1,270), and for few
// waits on its one chain (releases, score, argmin, winner's busy-until,
// serve, append).  Measured, before (seg_kernel.h) and now: one replica of
// 3 + 3 instances x 2,000 requests 1.18 and 0.75 ms; 4,096 of 2 + 6 x 4,000
// 2.83 and 2.16 ms; the 1,225-point sweep (32,768 x 2,000) 14.5 and 11.5 ms.
// Of the 2 + 6 launch's 1,200 cycles a step, about 400 are what its slowest
// waves spend on queues beyond their rings.
//
// Requests.  The terms a step needs (arrival, service times, priced work and
// cache need of each pool, sigma, the sampled candidates or the range of
// instances a baseline policy offers) are derived once per block of S
// requests, lane k working on request (block start + k), and left in LDS, a
// record per pool; a lane reads its pool's record of the next request a step
// ahead (three 16-byte reads).  A request is accepted if it is valid and its
// arrival equals the running maximum of the valid arrivals so far (a prefix
// maximum over the segment).
//
// FIFOs.  Service is in admission order, so an instance releases its
// requests in admission order.  A ring per instance in LDS (16-byte entries:
// release time, cache tokens, ledger tokens; a power of two of them, as many
// as the waves that share a compute unit leave room for, 64 for 4,096 replicas
// of 2 + 6) holds the front of its FIFO.  The first three entries are also in
// registers, re-read after the releases of every step and used at the append,
// so that up to three releases between two arrivals take one pass and no wait
// (two: four replicas of 2 + 6 release more on 35 % of the steps; three: on
// 11 %; a fourth would cost as much as it saves).  Requests beyond the ring
// are a list in HBM in which a request's record holds its two successors;
// such a ring is refilled by up to two requests every four steps, loaded four
// steps before they are put (a wait for a load is one for every store before
// it), and at once where fewer than three entries are left.  That, and
// releases beyond three, lie under one wave-uniform branch.
//
// Outcomes.  Each half keeps its pool's placement and time (prefill: TTFT,
// decode: span), lane k of the half the outcome of step (block start + k),
// and writes them every S / 2 steps with one coalesced store per array.
//
// Arithmetic of the cost: evaluated exactly as the equation is written, left
// to right in float32, one rounding per operation (built with
// -ffp-contract=off).  Times and token totals are integers held in doubles
// (exact below 2^53; simulated times are kept below 2^52).
#pragma once

#include <algorithm>

#include "seg_kernel.h"

namespace rt {
namespace seg {

// A request as one pool's lanes read it.
struct alignas(16) LReq {
  double now;      // arrival (ns) if the request is accepted, else -1
  double svc;      // service time on the pool
  double need;     // cache tokens it needs there
  float work, sg;  // priced work, sigma of its class
  double xfer;     // KV transfer delay (read by the decode half)
  int32_t fp, tk;  // cache and ledger tokens it holds until release
};
static_assert(sizeof(LReq) == 48, "three 16-byte words");

// A FIFO entry in LDS.
struct alignas(16) LEntry {
  double t;
  int32_t f, k;
};
constexpr int kEntryBytes = (int)sizeof(LEntry);

struct LSlot {
  double busy;     // end of everything admitted so far
  double kv;       // cache tokens in flight
  double pend;     // ledger tokens in flight
  int32_t q;       // requests in flight
  int32_t x;       // those beyond the ring
  int32_t qa;      // q after the last append
  uint32_t hd;     // ring position of the head (bytes, taken modulo the ring)
  int32_t tail;    // last admitted request
  int32_t tail2, tail3;  // the two admitted before it
  int32_t last;    // last request in the ring (where some lie beyond it)
  double ht, nt, ot;               // positions 0, 1, 2: release times ...
  int32_t hf, hk, nf, nk, of, ok;  // ... cache and ledger tokens
  int32_t lp;      // requests of the refill in flight (0 .. 2)
  u32x4 l1, l2;    // ... themselves, as loaded (nothing reads a part of them
  uint2 lk;        // before they are put: a copy would wait for the load)
};

// The records of a wave: one per pool and request of each segment's block.
// The 96 bytes after each segment's records spread the segments' reads of
// one word over the LDS banks.
template <int S>
constexpr int lreq_bytes() { return (64 / S) * (S * 2 * (int)sizeof(LReq) + 96); }
constexpr bool mode_range(int m) { return mode_sampled(m) || m == kModeBase; }  // two more words per record and pool
// (one pair more than the wave's records: each block's last step reads the
// words of record S, its next, which are behind the last segment's)
constexpr int kCandBytes = (64 + 1) * 2 * (int)sizeof(uint2);
template <int S, int kMode>
constexpr int lseg_fixed_lds() { return lreq_bytes<S>() + (mode_range(kMode) ? kCandBytes : 0); }

// The rings of a launch: every instance slot of a workgroup's waves has one
// of mask / 16 + 1 entries, a power of two, at LDS address (slot * bytes);
// the waves' records follow at rec_at.
struct LRings {
  uint32_t mask;       // ring bytes - 16
  uint32_t log_bytes;  // log2 of the ring bytes
  uint32_t max_inst;   // instance slots of a segment
  uint32_t rec_at;
};

template <int S>
__device__ __forceinline__ double seg_prefix_max(double x, int sl) {
  // within rows of 16 lanes: shifts that stay inside the segment
  auto shr = [&](auto cc, int k) __attribute__((always_inline)) {
    constexpr int C = decltype(cc)::value;
    const double y = __hiloint2double((int)dpp<C>((uint32_t)__double2hiint(x)), (int)dpp<C>((uint32_t)__double2loint(x)));
    x = sl >= k ? __builtin_fmax(x, y) : x;
  };
  shr(std::integral_constant<int, 0x111>{}, 1);
  shr(std::integral_constant<int, 0x112>{}, 2);
  shr(std::integral_constant<int, 0x114>{}, 4);
  if constexpr (S >= 16) shr(std::integral_constant<int, 0x118>{}, 8);
  // the last lane of each row into the rows after it
  if constexpr (S >= 32) {
    const int lane15 = ((threadIdx.x & 63) & ~31) + 15;
    const double y = __shfl(x, lane15);
    x = sl >= 16 && (sl & 31) >= 16 ? __builtin_fmax(x, y) : x;
  }
  if constexpr (S >= 64) {
    const double y = __shfl(x, 31);
    x = sl >= 32 ? __builtin_fmax(x, y) : x;
  }
  return x;
}

// The lower half's value of each segment, read by its upper half (every lane
// of a half holds the same value).
template <int S>
__device__ __forceinline__ uint32_t from_lower_half(uint32_t v) {
  if constexpr (S == 8) return dpp<0x141>(v);   // row_half_mirror
  else if constexpr (S == 16) return dpp<0x140>(v);  // row_mirror
  else if constexpr (S == 32) return __builtin_amdgcn_permlane16_swap(v, v, false, false)[0];
  else return __builtin_amdgcn_permlane32_swap(v, v, false, false)[0];
}

// c ? a : b of values.  (The operator on two lvalues selects between their
// addresses, which moves register-resident slots to scratch memory.)
template <typename T>
__device__ __forceinline__ T pick(bool c, T a, T b) { return c ? a : b; }

// 16 bytes of LDS at a byte address.
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
__device__ __forceinline__ u32x4 lds_get4(uint32_t at) { return *(const lds_u32x4*)(uintptr_t)at; }
__device__ __forceinline__ void lds_put4(uint32_t at, u32x4 v) { *(lds_u32x4*)(uintptr_t)at = v; }
typedef __attribute__((address_space(3))) uint64_t lds_u64;

// Does `c` hold on some lane (wave-uniform)?
__device__ __forceinline__ bool any_lane(bool c) { return __builtin_amdgcn_ballot_w64(c) != 0; }

template <int S, int kMode>
__global__ void __launch_bounds__(64 * kSegWaves) lseg_kernel(SimArgs a, LRings g) {
  constexpr bool kTok = mode_ledger(kMode);    // the ledger is priced
  constexpr bool kKv = kMode != kModeBase;     // occupancy is priced
  constexpr bool kSamp = mode_sampled(kMode);  // two candidates per pool
  constexpr bool kRange = mode_range(kMode);
  constexpr int Sh = S / 2;
  const int lane = threadIdx.x & 63;
  const int sl = lane & (S - 1), hl = lane & (Sh - 1);
  const int seg = lane / S;
  // a workgroup has 1 .. kSegWaves waves (chosen at launch), each with LDS of its own
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t wave_id = blockIdx.x * (blockDim.x >> 6) + wave;
  const int64_t item = (int64_t)wave_id * (64 / S) + seg;
  const bool live = item < a.n_work;
  const int rep = live ? a.work[item] : 0;
  const int64_t base = live ? a.offsets[rep] : 0;
  const int32_t R = live ? (int32_t)(a.offsets[rep + 1] - base) : 0;
  const int pid = (live && a.param_point) ? a.param_point[rep] : 0;
  const DevPoint& pt = a.points[pid];
  const int32_t P = pt.P, D = pt.D, ncls = pt.n_classes, policy = pt.policy, len_thr = pt.len_thr;
  const bool isp = sl < Sh;
  const int32_t npool = isp ? P : D;
  const float w_b = pt.w_b, w_s = pt.w_s, w_q = pt.w_q, rho = pt.rho;
  const float tau = isp ? pt.tau_pre : pt.tau_dec;
  const float tau_pre = pt.tau_pre, tau_dec = pt.tau_dec;
  const float basec = isp ? pt.pre_base : 0.0f;  // proxy ledger: base per in-flight prefill
  // (a lane without an instance prices NaN, which orders after every cost, on a
  // lane after every instance of its pool)
  const bool mine = live && hl < npool;
  const float inv = !mine ? __builtin_nanf("") : (isp ? pt.inv_cap_pre : pt.inv_cap_dec);
  const double pre_base_ns = (double)pt.pre_base_ns, pre_tok_ns = (double)pt.pre_tok_ns;
  const double dec_tok_ns = (double)pt.dec_tok_ns, xfer_tok_ns = (double)pt.xfer_tok_ns;
  char* const recr = (isp ? a.rec[0] : a.rec[1]) + rec_off<kTok>(base);
  const int64_t dmy = -1 - (int64_t)(wave_id & (kDummyRecords - 1)) - base;  // the wave's dummy record
  const float sig_l = pt.sigma[sl & (kMaxClasses - 1)];  // lane k: sigma of class k mod 8

  // LDS (a kernel without static shared memory: addresses from 0): the
  // rings, then every wave's records and candidates
  constexpr uint32_t kSegRec = (uint32_t)(S * 2 * (int)sizeof(LReq) + 96);
  const uint32_t wave_at = g.rec_at + wave * (uint32_t)lseg_fixed_lds<S, kMode>();
  const uint32_t rec0 = wave_at + (uint32_t)seg * kSegRec;
  const uint32_t my_rec = rec0 + (isp ? 0u : (uint32_t)sizeof(LReq));
  const uint32_t pad_at = rec0 + kSegRec - 96;  // written by nobody else
  const uint32_t cand0 = wave_at + (uint32_t)lreq_bytes<S>() + (uint32_t)(seg * S * 2 * (int)sizeof(uint2));
  const uint32_t my_cand = cand0 + (isp ? 0u : (uint32_t)sizeof(uint2));
  const int32_t K = (int32_t)(g.mask >> 4) + 1;
  // the lane's ring and the mask of its positions (bytes); a lane without an
  // instance has the pad
  const uint32_t slot = (wave * (64 / S) + (uint32_t)seg) * g.max_inst + (uint32_t)((isp ? 0 : P) + hl);
  const uint32_t ring_base = mine ? slot << g.log_bytes : pad_at, ring_mask = mine ? g.mask : 0u;
  auto ring_at = [&](uint32_t pos) __attribute__((always_inline)) -> uint32_t { return (pos & ring_mask) | ring_base; };
  auto ring_put = [&](uint32_t at, double t, int32_t f, int32_t k) __attribute__((always_inline)) {
    lds_put4(at, u32x4{(uint32_t)__double2loint(t), (uint32_t)__double2hiint(t), (uint32_t)f, (uint32_t)k});
  };

  LSlot x;
  x.busy = x.kv = x.pend = 0.0;
  x.q = x.x = x.qa = x.lp = 0;
  x.hd = 0;
  x.tail = x.tail2 = x.tail3 = x.last = -1;
  x.l1 = x.l2 = u32x4{0, 0, 0, 0};
  x.lk = make_uint2(0u, 0u);
  x.ht = x.nt = x.ot = kInf;
  x.hf = x.hk = x.nf = x.nk = x.of = x.ok = 0;

  const int32_t Rmax = __builtin_amdgcn_readfirstlane(wave_max_nonneg(R));

  // Raw trace of a block, lane k of the segment holding request (block start
  // + k) (clamped into the replica; request 0 of the trace for a segment
  // without one).
  const int64_t rd_base = R > 0 ? base : 0;
  const int32_t rd_last = R > 0 ? R - 1 : 0;
  struct Raw {
    int64_t arr;
    int32_t p, o, oh;
    uint32_t c;
    uint4 w;
  };
  auto load_raw = [&](Raw& f, int32_t blk) __attribute__((always_inline)) {
    const int64_t i = rd_base + min((uint32_t)blk + (uint32_t)sl, (uint32_t)rd_last);
    f.arr = a.arrival[i];
    f.p = a.plen[i];
    f.o = a.olen[i];
    f.oh = a.ohat[i];
    f.c = a.cls[i];
    if constexpr (kSamp) f.w = *reinterpret_cast<const uint4*>(a.samp + 4 * i);
  };
  auto put_rec = [&](uint32_t at, const LReq& r) __attribute__((always_inline)) {
    u32x4 v[3];
    __builtin_memcpy(v, &r, sizeof v);
    lds_put4(at, v[0]);
    lds_put4(at + 16, v[1]);
    lds_put4(at + 32, v[2]);
  };
  double carry = 0.0;  // largest valid arrival before the block
  bool rej = false;    // a request of this lane was rejected
  auto derive = [&](const Raw& f, int32_t blk) __attribute__((always_inline)) {
    const int32_t p = f.p, o = f.o, oh = f.oh;
    const int32_t po = (int32_t)((uint32_t)p + (uint32_t)o), poh = (int32_t)((uint32_t)p + (uint32_t)oh);
    const int32_t vm = min(min(min(p, o), min(oh, po)), min(min(poh, ncls - (int32_t)f.c), (int32_t)((uint32_t)R - ((uint32_t)blk + (uint32_t)sl))));
    const bool valid = opaque(vm) >= 1;
    const double x = valid ? i64_to_f64(f.arr) : -1.0;
    const double incl = __builtin_fmax(seg_prefix_max<S>(x, sl), carry);
    carry = __shfl(incl, (lane & ~(S - 1)) + S - 1);
    const bool acc = valid && x == incl;
    rej = rej || (!acc && blk + sl < R);
    const float sg = __builtin_bit_cast(
        float, __builtin_amdgcn_ds_bpermute((int)(((lane & ~7) + (f.c & (kMaxClasses - 1))) << 2),
                                            __builtin_bit_cast(int, sig_l)));
    LReq r;
    r.now = acc ? x : -1.0;
    r.svc = __builtin_fma((double)p, pre_tok_ns, pre_base_ns);
    r.need = (double)p;
    r.work = w_s * (float)p * tau_pre;
    r.sg = sg;
    r.xfer = 0.0;
    r.fp = p;
    r.tk = p;
    const uint32_t d = rec0 + (uint32_t)sl * 2 * (uint32_t)sizeof(LReq);
    put_rec(d, r);
    r.svc = (double)(o - 1) * dec_tok_ns;
    r.need = (double)poh;
    r.work = w_s * (float)oh * tau_dec;
    r.xfer = (double)p * xfer_tok_ns;
    r.fp = po;
    r.tk = oh;
    put_rec(d + (uint32_t)sizeof(LReq), r);
    if constexpr (kRange) {
      uint2 cp, cd;  // sampled: the two candidates; baselines: first instance offered and how many
      if constexpr (kSamp) {
        sample_pair(f.w.x, f.w.y, (uint32_t)P, cp.x, cp.y);
        sample_pair(f.w.z, f.w.w, (uint32_t)D, cd.x, cd.y);
      } else {
        cp = make_uint2(0u, (uint32_t)P);
        cd = make_uint2(0u, (uint32_t)D);
        if (policy == kPolicyRoundRobin) {
          cp = make_uint2((uint32_t)(blk + sl) % (uint32_t)P, 1u);
          cd = make_uint2((uint32_t)(blk + sl) % (uint32_t)D, 1u);
        } else if (policy == kPolicyLengthThreshold && D > 1) {
          const uint32_t half = (uint32_t)(D + 1) / 2;
          cd = oh >= len_thr ? make_uint2(half, (uint32_t)D - half) : make_uint2(0u, half);
        }
      }
      lds_put4(cand0 + (uint32_t)sl * 2 * (uint32_t)sizeof(uint2), u32x4{cp.x, cp.y, cd.x, cd.y});
    }
  };
  struct Cur {
    LReq r;
    uint2 c;
  };
  // (record S of a block, and its candidates, lie in a pad or are the next
  // segment's: read, not used)
  static_assert((64 / S - 1) * (int)kSegRec + (S + 1) * 2 * (int)sizeof(LReq) <= lreq_bytes<S>(), "record S is in the wave's LDS");
  static_assert((64 / S - 1) * S * 16 + (S + 1) * 16 <= kCandBytes, "and so are its candidates");
  auto read_rec = [&](Cur& q, uint32_t i) __attribute__((always_inline)) {
    const uint32_t at = my_rec + i * 2 * (uint32_t)sizeof(LReq);
    const u32x4 v[3] = {lds_get4(at), lds_get4(at + 16), lds_get4(at + 32)};
    __builtin_memcpy(&q.r, v, sizeof v);
    if constexpr (kRange) {
      const uint64_t w = *(const lds_u64*)(uintptr_t)(my_cand + i * 2 * (uint32_t)sizeof(uint2));
      q.c = make_uint2((uint32_t)w, (uint32_t)(w >> 32));
    }
  };

  // Queues beyond the ring.  Everything here runs without divergent branches
  // (lanes with nothing to do use the wave's dummy record, or the pad).
  // The next one or two requests behind a slot's ring, loaded where the ring
  // has room for two.
  auto load_next = [&](bool c) __attribute__((always_inline)) {
    const char* const rp = rec_at<kTok>(recr, sel_index(c, x.last, dmy));
    x.l1 = *reinterpret_cast<const u32x4*>(rp);
    x.l2 = *reinterpret_cast<const u32x4*>(rp + 16);
    if constexpr (kTok) x.lk = *reinterpret_cast<const uint2*>(rp + kRecTok);
    x.lp = c ? min(x.x, 2) : 0;
  };
  // ... and put there.
  auto put_next = [&]() __attribute__((always_inline)) {
    const bool c1 = x.lp >= 1, c2 = x.lp >= 2;
    const uint32_t pos = x.hd + (uint32_t)(x.q - x.x) * kEntryBytes;
    // (an entry {time, index, cache tokens} of the record becomes {time, cache
    // tokens, ledger tokens} in the ring)
    lds_put4(pick(c1, ring_at(pos), pad_at), u32x4{x.l1[0], x.l1[1], x.l1[3], x.lk.x});
    lds_put4(pick(c2, ring_at(pos + kEntryBytes), pad_at), u32x4{x.l2[0], x.l2[1], x.l2[3], x.lk.y});
    x.x -= x.lp;
    x.last = pick(c2, (int32_t)x.l2[2], pick(c1, (int32_t)x.l1[2], x.last));
    x.lp = 0;
  };
  // Positions 0, 1, 2 into the registers (whatever lies there; the count says
  // what is valid).
  auto read_front = [&]() __attribute__((always_inline)) {
    const u32x4 h = lds_get4(ring_at(x.hd)), n = lds_get4(ring_at(x.hd + kEntryBytes)),
                o = lds_get4(ring_at(x.hd + 2 * kEntryBytes));
    x.ht = __hiloint2double((int)h[1], (int)h[0]);
    x.hf = (int32_t)h[2];
    x.nt = __hiloint2double((int)n[1], (int)n[0]);
    x.nf = (int32_t)n[2];
    x.ot = __hiloint2double((int)o[1], (int)o[0]);
    x.of = (int32_t)o[2];
    if constexpr (kTok) {
      x.hk = (int32_t)h[3];
      x.nk = (int32_t)n[3];
      x.ok = (int32_t)o[3];
    }
  };

  // outcomes of the current block of Sh steps: this half's placement and time
  int32_t b_i = -1;
  double b_v = 0.0;
  int32_t* const o_i = isp ? a.i_pre : a.i_dec;
  int64_t* const o_t = isp ? a.ttft : a.span;
  auto flush = [&](uint32_t t0) __attribute__((always_inline)) {
    const uint32_t tl = t0 + (uint32_t)hl;
    if (tl < (uint32_t)R) {
      o_i[base + tl] = b_i;
      o_t[base + tl] = b_i < 0 ? -1 : f64_to_i64(b_v);
    }
  };

  const int grp = lane & ~(Sh - 1);  // the half's first lane
  uint64_t beyond = 0;               // lanes with a queue beyond its ring (not empty: some lane has one)
  // The last append, as the lane's queue beyond its ring sees it.
  bool ap = false;  // the lane admitted the last request
  double ap_end = 0.0;
  int32_t ap_f = 0, ap_k = 0;

  // Step t of record `rq`; the next record is read into `rn` from LDS address
  // `next`.
  auto step = [&](const int32_t t, const int32_t k, const Cur& rq, Cur& rn, uint32_t next) __attribute__((always_inline)) {
    const LReq& r = rq.r;
    const bool go = r.now >= 0.0;

    // 1. releases: up to three from the registers
    const int32_t phase = t & 3;
    bool more = false;
    auto pop = [&]() __attribute__((always_inline)) {
      const bool p1 = x.ht <= r.now, p2 = x.nt <= r.now, p3 = x.ot <= r.now;  // p3 implies p2 implies p1
      const int32_t np = (p1 ? 1 : 0) + (p2 ? 1 : 0) + (p3 ? 1 : 0);
      // (the sum of three may pass 2^32, that of two does not)
      if constexpr (kKv)
        x.kv = x.kv - ((double)((p1 ? (uint32_t)x.hf : 0u) + (p2 ? (uint32_t)x.nf : 0u)) + (double)(p3 ? x.of : 0));
      if constexpr (kTok)
        x.pend = x.pend - ((double)((p1 ? (uint32_t)x.hk : 0u) + (p2 ? (uint32_t)x.nk : 0u)) + (double)(p3 ? x.ok : 0));
      x.q -= np;
      x.hd += (uint32_t)np * kEntryBytes;
      more = p3;
    };
    beyond |= __builtin_amdgcn_ballot_w64(x.q > K);
    pop();
    uint64_t again = __builtin_amdgcn_ballot_w64(more);
    if (__builtin_expect((again | beyond) != 0, 0)) {
      uint64_t low = 0;  // lanes with fewer than three entries in the ring of a queue that lies beyond it
      auto check_low = [&]() __attribute__((always_inline)) {
        low = __builtin_amdgcn_ballot_w64((x.x > 0) & (x.q - x.x < 3));
      };
      if (beyond) {
        // the last request, where it was admitted beyond the ring (the append
        // left x unchanged): the first successor of the one before it in its
        // FIFO and the second of the one before that
        const bool out = ap & ((x.x > 0) | (x.qa > K));
        x.last = pick(out & (x.x == 0), x.tail2, x.last);
        x.x += out ? 1 : 0;
        // the refill loaded four steps ago (ahead of the stores: its wait
        // is one for every access before it)
        if (phase == 0) put_next();
        char* const r1 = rec_at<kTok>(recr, sel_index(out, x.tail2, dmy));
        char* const r2 = rec_at<kTok>(recr, sel_index(out, x.tail3, dmy));
        *reinterpret_cast<Entry*>(r1) = Entry{ap_end, x.tail, ap_f};
        *reinterpret_cast<Entry*>(r2 + 16) = Entry{ap_end, x.tail, ap_f};
        if constexpr (kTok) {
          *reinterpret_cast<int32_t*>(r1 + kRecTok) = ap_k;
          *reinterpret_cast<int32_t*>(r2 + kRecTok + 4) = ap_k;
        }
        check_low();
      }
      while ((again | low) != 0) {
        while (low != 0) {
          put_next();
          load_next((x.x > 0) & (x.q - x.x < 3));
          put_next();
          check_low();
        }
        if (again == 0) break;
        read_front();
        x.ht = pick(x.q >= 1, x.ht, kInf);
        x.nt = pick(x.q >= 2, x.nt, kInf);
        x.ot = pick(x.q >= 3, x.ot, kInf);
        pop();
        again = __builtin_amdgcn_ballot_w64(more);
        if (beyond) check_low();
      }
      if (beyond && phase == 0) {
        load_next((x.x > 0) & (x.q - x.x + 2 <= K));
        beyond = __builtin_amdgcn_ballot_w64(x.x > 0);
      }
    }
    // the front again (used at the append), then the next record
    read_front();
    read_rec(rn, next);

    // 2. score this lane's instance
    uint32_t key;
    if constexpr (kMode == kModeBase) {
      key = mine && (uint32_t)hl - rq.c.x < rq.c.y ? (uint32_t)x.q : 0xffffffffu;
    } else {
      float bl;
      if constexpr (!kTok)
        bl = (float)__builtin_fmax(x.busy - r.now, 0.0) * 1e-9f;
      else
        bl = tau * (float)x.pend + basec * (float)x.q;
      const float press = (float)(x.kv + r.need) * inv;
      const float load = w_b * bl * r.sg;
      const float size = r.work * (1.0f + rho * press) * r.sg;
      const float cost = load + size + w_q * (float)x.q;
      key = cost != cost ? 0x7fc00000u : __float_as_uint(cost);
    }
    if constexpr (kSamp) key = (uint32_t)hl == rq.c.x || (uint32_t)hl == rq.c.y ? key : 0xffffffffu;

    // 3. each half's argmin, lowest index on equal keys, and the winner's
    // busy-until on every lane of the half
    const uint32_t kmin = seg_min<Sh>(key);
    // (some lane of the half holds the minimum: the lowest bit from the half's first lane up)
    const int32_t wl = __builtin_ctz((uint32_t)(__builtin_amdgcn_ballot_w64(key == kmin) >> grp));
    const bool won = wl == hl;
    double busyw;
    if constexpr (Sh <= 16) {
      busyw = __hiloint2double((int)seg_or<Sh>(won ? (uint32_t)__double2hiint(x.busy) : 0u),
                               (int)seg_or<Sh>(won ? (uint32_t)__double2loint(x.busy) : 0u));
    } else {
      const int wa = (grp + wl) << 2;
      busyw = __hiloint2double(__builtin_amdgcn_ds_bpermute(wa, __double2hiint(x.busy)),
                               __builtin_amdgcn_ds_bpermute(wa, __double2loint(x.busy)));
    }

    // 4. serve: the lower half forms the prefill end, the upper half takes
    // it from there and forms the decode end (exact integers in doubles)
    const double pf = max_f64(r.now, busyw) + r.svc;
    const double pfd = __hiloint2double((int)from_lower_half<S>((uint32_t)__double2hiint(pf)),
                                        (int)from_lower_half<S>((uint32_t)__double2loint(pf)));
    const double de = max_f64(pfd + r.xfer, busyw) + r.svc;
    const double end = pick(isp, pf, de);
    const double ref = pick(isp, r.now, pfd);
    const int32_t wg = go ? wl : -1;
    const bool own = opaque(wg) == hl;

    // 5. append to the winner's FIFO
    ap_end = end;
    ap_f = r.fp;
    ap_k = r.tk;
    // (a lane that admits nothing writes a position behind its last entry;
    // where the ring is full, the pad)
    ring_put(pick(x.q < K, ring_at(x.hd + (uint32_t)x.q * kEntryBytes), pad_at), end, r.fp, r.tk);
    // positions 0, 1, 2 as they are now: re-read after the releases (when
    // there were x.q entries), then this request at position x.q; +inf (or
    // NaN) where there is none
    const bool w0 = x.q == 0, w1 = x.q == 1, w2 = x.q == 2, lt2 = x.q < 2;
    const double e0 = __hiloint2double(own ? __double2hiint(end) : 0x7ff00000, __double2loint(end));
    x.ht = pick(w0, e0, x.ht);
    x.hf = pick(w0, r.fp, x.hf);
    x.nt = pick(w1, e0, x.nt);
    x.nf = pick(w1, r.fp, x.nf);
    x.nt = __hiloint2double(w0 ? 0x7ff80000 : __double2hiint(x.nt), __double2loint(x.nt));
    x.ot = pick(w2, e0, x.ot);
    x.of = pick(w2, r.fp, x.of);
    x.ot = __hiloint2double(lt2 ? 0x7ff80000 : __double2hiint(x.ot), __double2loint(x.ot));
    if constexpr (kTok) {
      x.hk = pick(w0, r.tk, x.hk);
      x.nk = pick(w1, r.tk, x.nk);
      x.ok = pick(w2, r.tk, x.ok);
      x.pend = x.pend + (own ? (double)r.tk : 0.0);
    }
    if constexpr (kKv) x.kv = x.kv + (own ? (double)r.fp : 0.0);
    x.q += own ? 1 : 0;
    ap = own;
    x.qa = x.q;
    x.tail3 = pick(own, x.tail2, x.tail3);
    x.tail2 = pick(own, x.tail, x.tail2);
    x.tail = pick(own, t, x.tail);
    x.busy = pick(own, end, x.busy);

    // 6. the outcome
    const bool keep = k == hl;
    b_i = pick(keep, wg, b_i);
    b_v = pick(keep, end - ref, b_v);
  };

  Raw raw;
  load_raw(raw, 0);
  // per block of S steps: its records, then two halves of Sh steps, the
  // outcomes written after each (a last block's steps past the longest
  // replica change nothing)
  for (uint32_t t0 = 0; t0 < (uint32_t)Rmax; t0 += S) {
    derive(raw, (int32_t)t0);
    load_raw(raw, (int32_t)(t0 + S));
    uint32_t at = 0;
    Cur ra, rb;
    read_rec(ra, 0);
#pragma unroll 1
    for (uint32_t h = 0; h < 2; ++h) {
      const uint32_t tb = t0 + h * Sh;
#pragma unroll 1
      for (uint32_t k = 0; k < (uint32_t)Sh; k += 2) {
        step((int32_t)(tb + k), (int32_t)k, ra, rb, at + 1);
        step((int32_t)(tb + k + 1), (int32_t)(k + 1), rb, ra, at + 2);
        at += 2;
      }
      flush(tb);
    }
  }
  // (busy-until never decreases, so the last one is the latest time reached)
  const uint32_t flag = (x.busy >= kTimeLimit ? kFlagTimeRange : 0u) | (rej ? kFlagRejected : 0u);
  if (flag) atomicOr(a.flag, flag);
}

// Rings of a wave with `bytes` of LDS, `fixed` of them for its records, over
// `slots` instances: log2 of a ring's bytes, a power of two (4 to 256 entries).
inline uint32_t ring_log_bytes(uint32_t bytes, uint32_t fixed, uint32_t slots) {
  uint32_t lg = 6;
  while (lg < 12 && (slots << (lg + 1)) <= bytes - fixed) ++lg;
  return lg;
}

// A compute unit holds two waves per SIMD of a launch that has so many, and a
// third, in segments of 16 lanes and more, where that costs the rings no more
// than half their entries and leaves eight, and where it does not only move the
// last pass over the GPU (13 to 16 waves a compute unit: two passes of eight).
// 9,000 replicas of 2 + 6 x 1,000: 1.10 ms with two, 0.95 with three; 14,336:
// 1.30 and 1.34; 24,576: 1.94 and 1.80; 32,768 of 4 + 8 x 300 (eight entries)
// 0.71 and 0.66, least loaded (four) 0.48 and 0.72.  Segments of 8 lanes: 65,536
// of 1 + 3 x 300 0.99 and 1.12.
template <int S>
int64_t lseg_most_waves(int64_t call_waves, uint32_t fixed, uint32_t slots) {
  if (S < 16) return 8;
  const int64_t per_cu = waves_per_cu(call_waves);
  if (per_cu <= 8 || (per_cu > 12 && per_cu <= 16)) return 8;
  const uint32_t two = ring_log_bytes(lds_share(call_waves, 8).bytes, fixed, slots);
  const uint32_t three = ring_log_bytes(lds_share(call_waves, 12).bytes, fixed, slots);
  return three >= 7 && three + 1 >= two ? 12 : 8;
}

template <int S, int kMode>
hipError_t launch_lseg(const SimArgs& a, hipStream_t stream) {
  constexpr int64_t kSegs = 64 / S;
  constexpr uint32_t kFixed = (uint32_t)lseg_fixed_lds<S, kMode>();
  const int64_t waves = (a.n_work + kSegs - 1) / kSegs;
  const uint32_t slots = (uint32_t)(kSegs * a.max_inst);  // of a wave
  const LdsShare share = lds_share(a.call_waves, lseg_most_waves<S>(a.call_waves, kFixed, slots));
  const uint32_t wpb = share.wpb;
  LRings g{};
  g.max_inst = (uint32_t)a.max_inst;
  g.log_bytes = ring_log_bytes(share.bytes, kFixed, slots);
  g.mask = (1u << g.log_bytes) - kEntryBytes;
  g.rec_at = wpb * slots << g.log_bytes;
  const uint32_t lds = g.rec_at + wpb * kFixed;
  if (lds > 64 * 1024) {
    // (per device, so at every launch; the whole of a compute unit's, so that
    // a smaller launch of another thread takes nothing from this one)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&lseg_kernel<S, kMode>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((lseg_kernel<S, kMode>), dim3((unsigned)((waves + wpb - 1) / wpb)), dim3(64 * wpb), lds,
                     stream, a, g);
  return hipGetLastError();
}

// The segment widths compiled for every mode, one instance per lane.  (Narrower
// ones were slower for every pool, also with many replicas: a wave of 32 or 16
// replicas has a lane with more than three releases, or a queue beyond its
// ring, on almost every step.  Two to four instances per lane were slower than
// the kernel of seg_kernel.h, which skips the slots that no lane needs.)
#define RT_LSEG_FOR_EACH(X) X(8) X(16) X(32) X(64)

template <int kMode>
hipError_t launch_lseg_mode(int S, const SimArgs& a, hipStream_t stream);

}  // namespace seg
}  // namespace rt
