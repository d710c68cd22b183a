// Batched negacyclic NTT / inverse NTT for gfx950 on FP64 lanes.
//
// One workgroup transforms one N-word polynomial (N = 4096 / 8192 / 16384), exchanging
// values through LDS (N doubles + 1/16 padding, 136 KiB at N = 16384 against 160 KiB per
// CU).  Each of the N/PT work-items keeps PT = 16 (or 32) values in registers and runs up to
// four (five) radix-2 stages on them per pass; the first pass reads global memory and the last
// writes it, so a transform costs (passes - 1) LDS round trips.  The forward transform is the
// Cooley-Tukey ordering with twiddles psi^brv(m+i) (natural in, bit-reversed out, value j is
// the evaluation at psi^(2 brv(j) + 1)); the inverse is the Gentleman-Sande ordering with
// psi^-brv(m+i) followed by N^-1.  Polys are addressed through a descriptor table so a
// launch can gather from arbitrary buffers and moduli.
#include "blb_internal.h"
#include "blb_kernels.h"
#include <algorithm>
#include <type_traits>

namespace {

// Values per work-item (the radix of a pass: log2 of it is the number of radix-2 stages a pass
// runs in registers).  16 (passes of 4 stages, N/16 work-items) or 32 (passes of 5 stages, N/32
// work-items, one LDS round trip fewer); chosen per context by the autotuner, never changing a
// result.
constexpr int kPT16 = 16, kPT32 = 32;

// Where a launch finds its polynomials: a descriptor table, or (descs == null) a regular
// batch of `count` limb-polys stored back to back at `base`, transformed in place, poly p
// taken modulo prime p mod nl (the [item][limb][N] layout of ciphertexts and plaintexts), or
// (coef set) a plan batch: poly p reads the integer coefficients of plaintext p / nl and goes to
// base + p x out_bytes.
struct NttSrc {
  const PolyDesc* descs;
  uint64_t* base;
  int nl;
  int log_n;
  int group = 1;  // runs of this many of the first `split` descriptors read the same words,
  int split = 0;
  int tail = 1;   // of this many of the rest
  int count = 0;
  const uint64_t* coef = nullptr;
  size_t out_bytes = 0;
  // Workgroup w of the launch takes descriptor at(w): workgroups go round-robin over the 8 XCDs, so the
  // `group` descriptors of a run are given to workgroups 8 apart and meet in one XCD's L2.
  __device__ __forceinline__ int at(int w) const {
    const int lo = w < split ? 0 : split, end = w < split ? split : count, run = w < split ? group : tail;
    const int span = 8 * run;
    if (run <= 1 || end - lo < span) return w;
    const int base = lo + (w - lo) / span * span;
    if (base + span > end) return w;
    return base + (w - base) % 8 * run + (w - base) / 8;
  }
  __device__ __forceinline__ PolyDesc get(int w) const { return desc(at(w)); }
  __device__ __forceinline__ PolyDesc desc(int p) const {
    if (descs) {
      // scalar loads (the table is read-only while the kernel runs): they do not join the
      // in-order vector-memory counter, so fetching a descriptor never waits for the stores
      // of the previous polynomial
      typedef __attribute__((address_space(4))) const uint64_t ku64;
      static_assert(sizeof(PolyDesc) == 64, "descriptor layout");
      const ku64* w = (const ku64*)(descs + p);
      union {
        uint64_t u[8];
        PolyDesc d;
      } r;
#pragma unroll
      for (int i = 0; i < 8; ++i) r.u[i] = w[i];
      return r.d;
    }
    PolyDesc d;
    d.src = coef ? coef + ((size_t)(p / nl) << log_n) : base + ((size_t)p << log_n);
    d.dst = coef ? (uint64_t*)((uint8_t*)base + (size_t)p * out_bytes) : base + ((size_t)p << log_n);
    d.src2 = nullptr;
    d.src3 = nullptr;
    d.aux = 0.0;
    d.aux2 = 0.0;
    d.mod = (int16_t)(p % nl);
    d.n_src = 1;
    d.gal = 0;
    d.log_n = log_n;
    d.flags = 0;
    return d;
  }
};

__host__ __device__ constexpr int pad_idx(int j) { return j + (j >> 4); }

// Bounds (in units of q) of the GS = 2^R_LOG slots of a Gentleman-Sande pass whose operands are below
// `in`: pre[u][k] marks the operands of stage u to reduce first (a sum would pass 8 otherwise),
// post[k] the slots that leave the pass above `out`.
template <int R_LOG>
struct GsBounds {
  static constexpr int GS = 1 << R_LOG;
  bool pre[R_LOG][GS] = {};
  bool post[GS] = {};
  constexpr GsBounds(double in, double out) {
    double b[GS] = {};
    for (int k = 0; k < GS; ++k) b[k] = in;
    for (int u = R_LOG - 1; u >= 0; --u) {
      const int t = GS >> (u + 1);
      for (int k = 0; k < GS; ++k) {
        if (k & t) continue;
        double &x = b[k], &y = b[k + t];
        if (x + y > 8.0) {  // the larger one first
          const bool first = x >= y;
          (first ? x : y) = 0.5;
          pre[u][first ? k : k + t] = true;
        }
        if (x + y > 8.0) {
          x = y = 0.5;
          pre[u][k] = pre[u][k + t] = true;
        }
        const double sum = x + y;
        x = sum;
        y = 0.5 + 0.1875 * sum;
      }
    }
    for (int k = 0; k < GS; ++k) post[k] = b[k] > out;
  }
};

// One pass of R_LOG radix-2 stages starting at global stage S0.  Work-item `tid` holds
// PT values in registers: GPT groups of GS = 2^R_LOG values each, group h being the
// butterfly group g = tid + h T (T = N / PT) whose members sit TL = N >> (S0 + R_LOG)
// words apart.
template <int LOGN, int PT, int S0, int R_LOG>
struct Pass {
  static constexpr int N = 1 << LOGN;
  static constexpr int T = N / PT;
  static constexpr int GS = 1 << R_LOG;
  static constexpr int GPT = PT / GS;
  static constexpr int TL = N >> (S0 + R_LOG);
  static_assert(S0 + R_LOG <= LOGN && GS <= PT, "pass shape");
  // twiddles differ across the lanes of a wave (vector loads) unless the pass spans whole
  // columns (TL >= T) or a butterfly tree covers at least 64 work-items (TL >= 64)
  static constexpr bool LANE_TW = !(TL >= T || TL >= 64);

  // coefficient index of register slot i (= h GS + k)
  __host__ __device__ static constexpr int idx(int tid, int i) {
    const int h = i / GS, k = i % GS;
    const int g = tid + h * T;
    return (g / TL) * (TL << R_LOG) + (g % TL) + k * TL;
  }

  // Padded LDS word of slot i relative to slot 0.  In every pass shape used here it does not
  // depend on the work-item (asserted for all work-items at compile time below), so an exchange
  // needs one address per work-item and the slots become immediate offsets.
  static constexpr int lds_off(int i) { return pad_idx(idx(0, i)) - pad_idx(idx(0, 0)); }

  // Twiddle k of group h in stage S0 + u.  SUB: this is a transform of half the ring's polynomial, whose
  // first stage is done; `half` picks the half's twiddles (stage s has 2^(s+1) of them in the whole
  // transform, the second half's after the first's).
  template <bool SUB>
  struct TwMem {
    const double* __restrict__ tw;
    int tid, half;
    __device__ double operator()(int h, int u, int k) const {
      // group index; compile-time when a pass spans whole columns (first pass), and uniform
      // over the 64-lane wave when TL >= 64, so the twiddles come through scalar loads
      int hi = (tid + h * T) / TL;
      if constexpr (TL >= T) hi = (h * T) / TL;
      else if constexpr (TL >= 64) hi = __builtin_amdgcn_readfirstlane(hi);
      return tw[(1 << (S0 + u)) + (SUB ? (1 + half) << (S0 + u) : 0) + (hi << u) + k];
    }
  };
  // the pass's twiddles in registers, loaded ahead of the pass
  struct TwRegs {
    double w[GPT][GS - 1];
    template <bool FWD, class Mem>
    __device__ void load(const Mem& mem) {  // in the order of use: loads complete in the order of issue
#pragma unroll
      for (int uu = 0; uu < R_LOG; ++uu)
#pragma unroll
        for (int h = 0; h < GPT; ++h)
#pragma unroll
          for (int k = 0; k < 1 << (FWD ? uu : R_LOG - 1 - uu); ++k) {
            const int u = FWD ? uu : R_LOG - 1 - uu;
            w[h][(1 << u) - 1 + k] = mem(h, u, k);
          }
      __builtin_amdgcn_sched_barrier(0);
    }
    __device__ double operator()(int h, int u, int k) const { return w[h][(1 << u) - 1 + k]; }
  };

  // FWD: Cooley-Tukey stages in increasing order; else Gentleman-Sande in decreasing order.
  // mid() runs after the first executed stage, when every operand has been read; sink(i) after
  // register slot i has its last value, so that what follows (the exchange's LDS writes) is issued
  // between the last stage's arithmetic instead of after it.  FIRST / LAST: the executed first /
  // last pass of the transform.
  template <bool FWD, bool FIRST, bool LAST, class Tw, class Mid, class Sink>
  __device__ static __forceinline__ void run(double (&x)[PT], const Tw& tw, double q, double qi, const Mid& mid, const Sink& sink) {
    // Lazy reduction.  Twiddles are centred (|w| <= q/2), so for |b| <= B q a product is below q/2 +
    // 0.1875 B q (the quotient estimate is off by < B 2^-53 q, the dropped low part of b w is below
    // that too), and every FP64 sum and product step is exact up to 8 q < 2^53.
    // Forward: B' = 1.1875 B + 1/2.  From 1 (canonical words) six stages stay below 7.62, from 1/2
    // (reduced) six below 6.22 and two below 1.8: values are reduced after stage (log2 N - 2) / 2 and
    // after stage log2 N - 2, and come out below 1.8 q (canon2 makes them canonical).
    // Inverse: a + b adds the bounds; GsBounds tracks each slot's through the pass and reduces only
    // the operands whose sum could pass 8 (the all-sum slots) and, at the end of a pass, slots above 2.
    // Against a reduction of every value each fourth (second, inverse) stage this is 10 % fewer
    // instructions a transform.
    constexpr GsBounds<R_LOG> gs(FIRST ? 1.0 : 2.0, LAST ? 8.0 : 2.0);
#pragma unroll
    for (int uu = 0; uu < R_LOG; ++uu) {
      const int u = FWD ? uu : (R_LOG - 1 - uu);
      const int t_loc = GS >> (u + 1);
#pragma unroll
      for (int h = 0; h < GPT; ++h) {
#pragma unroll
        for (int k = 0; k < GS; ++k) {
          if (k & t_loc) continue;
          const double w = tw(h, u, k >> (R_LOG - u));
          double& a = x[h * GS + k];
          double& b = x[h * GS + k + t_loc];
          if (FWD) {
            const bool red = S0 + u + 1 == (LOGN - 2) / 2 || S0 + u + 1 == LOGN - 2;
            const double v = mulmod_s(b, w, q, qi);
            const double sum = a + v, dif = a - v;
            a = red ? reduce_s(sum, q, qi) : sum;
            b = red ? reduce_s(dif, q, qi) : dif;
          } else {
            if (gs.pre[u][k]) a = reduce_s(a, q, qi);
            if (gs.pre[u][k + t_loc]) b = reduce_s(b, q, qi);
            const double sum = a + b, dif = a - b;
            a = sum;
            b = mulmod_s(dif, w, q, qi);
            if (uu == R_LOG - 1) {
              if (gs.post[k]) a = reduce_s(a, q, qi);
              if (gs.post[k + t_loc]) b = reduce_s(b, q, qi);
            }
          }
          if (uu == R_LOG - 1) {
            sink(h * GS + k);
            sink(h * GS + k + t_loc);
          }
        }
      }
      if (uu == 0) mid();
    }
  }
};

// Workgroup barrier that orders LDS accesses only: global loads in flight (the persistent
// kernel's prefetch of the next polynomial) are not waited for, unlike __syncthreads().
// Global memory is never exchanged between work-items of a workgroup here: each work-item
// consumes its own loads before its first barrier, and stores come after the last one.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Slot i's LDS word for the writer (pass PA's layout) and all slots read in PB's layout.  The exchange
// needs a barrier before the writes (behind every read of the previous exchange, also of the
// previous polynomial in the persistent kernel): it stands inside pass PA, after its first stage.
template <class P, int PT>
struct LdsSink {
  double* base;
  const double (&x)[PT];
  __device__ void operator()(int i) const { base[P::lds_off(i)] = x[i]; }
};
template <class PB, bool FWD, int PT>
__device__ __forceinline__ void read_layout(const double* lds, double (&x)[PT], int tid) {
  const double* lb = lds + pad_idx(PB::idx(tid, 0));
  lds_barrier();
  // in the order the next pass's first stage takes them: (k, k + GS/2) forward, (k, k + 1) inverse
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int h = i / PB::GS, r = i % PB::GS;
    const int slot = FWD ? h * PB::GS + (r >> 1) + (r & 1) * (PB::GS / 2) : i;
    x[slot] = lb[PB::lds_off(slot)];
  }
}

// lds_off(i) is the same for every work-item of pass P
template <class P>
constexpr bool lds_affine() {
  for (int i = 1; i < P::GS * P::GPT; ++i) {
    const int off = P::lds_off(i);
    for (int tid = 1; tid < P::T; ++tid)
      if (pad_idx(P::idx(tid, i)) - pad_idx(P::idx(tid, 0)) != off) return false;
  }
  return true;
}

// Pass schedule (forward order).  PT = 16: three passes of four stages, then the remaining
// LOGN - 12 stages; PT = 32: two passes of five stages, then the remaining LOGN - 10.  The first
// pass reads its operands straight from global memory and the last pass writes straight to
// global memory, so a transform makes (passes - 1) LDS round trips.
template <int LOGN, int PT>
struct Sched {
  static constexpr int R = PT == 32 ? 5 : 4;
  static constexpr int REM = LOGN - 3 * R;  // stages of a fourth pass (PT = 16 only)
  static_assert(PT == 16 || PT == 32, "values per work-item");
  static_assert(PT == 16 || LOGN - 2 * R >= 1, "third pass");
  using P0 = Pass<LOGN, PT, 0, R>;
  using P1 = Pass<LOGN, PT, R, R>;
  using P2 = Pass<LOGN, PT, 2 * R, (PT == 32 ? LOGN - 2 * R : R)>;
  using P3 = Pass<LOGN, PT, 3 * R, (PT == 16 && REM > 0 ? REM : 1)>;
  static constexpr bool HAS3 = PT == 16 && REM > 0;
  using Tail = std::conditional_t<HAS3, P3, P2>;  // forward-last / inverse-first pass
  static_assert(lds_affine<P0>(), "LDS offsets of the first pass depend on the work-item");
  static_assert(lds_affine<P1>(), "LDS offsets of the second pass depend on the work-item");
  static_assert(lds_affine<P2>(), "LDS offsets of the third pass depend on the work-item");
  static_assert(lds_affine<Tail>(), "LDS offsets of the last pass depend on the work-item");
  static constexpr int NP = HAS3 ? 4 : 3;  // passes
  // passes (in execution order) that run before the persistent kernel's prefetch is issued:
  // the leading run of passes with per-lane twiddles
  template <bool FWD>
  static constexpr int issue_after() {
    const bool lane[4] = {P0::LANE_TW, P1::LANE_TW, P2::LANE_TW, HAS3 ? Tail::LANE_TW : false};
    int k = 0;
    while (k < NP && lane[FWD ? k : NP - 1 - k]) ++k;
    return k;
  }
};
template <int LOGN, int PT, bool FWD>
using FirstPass = std::conditional_t<FWD, typename Sched<LOGN, PT>::P0, typename Sched<LOGN, PT>::Tail>;
template <int LOGN, int PT, bool FWD>
using LastPass = std::conditional_t<FWD, typename Sched<LOGN, PT>::Tail, typename Sched<LOGN, PT>::P0>;

struct NoIssue {
  __device__ void operator()() const {}
};

struct LdsMid {
  __device__ void operator()() const { lds_barrier(); }
};
struct NoMid {
  __device__ void operator()() const {}
};
struct NoSink {
  __device__ void operator()(int) const {}
};
// x holds the first pass's operands on entry and the last pass's results on exit.  issue()
// enqueues the persistent kernel's prefetch of the next polynomial.  Vector loads complete in
// issue order, so a per-lane twiddle load issued after the prefetch is waited for only once
// the whole prefetch has arrived: issue() runs after the leading passes that load per-lane
// twiddles (before the first pass when it has none).  REUSED: the LDS may still be read by the
// previous polynomial's last exchange (persistent kernel), so the first exchange needs its barrier too.
template <int LOGN, int PT, bool FWD, bool REUSED, bool SUB = false, class Issue = NoIssue>
__device__ __forceinline__ void ntt_core(double* lds, double (&x)[PT], const double* tw, double q, double qi, int tid,
                                         const Issue& issue = Issue(), int half = 0) {
  using S = Sched<LOGN, PT>;
  using P0 = typename S::P0;
  using P1 = typename S::P1;
  using P2 = typename S::P2;
  using P3 = typename S::P3;
  using FirstMid = std::conditional_t<REUSED, LdsMid, NoMid>;
  constexpr int at = S::template issue_after<FWD>();  // passes run before issue()
  auto sink = [&](auto pass) { return LdsSink<decltype(pass), PT>{lds + pad_idx(decltype(pass)::idx(tid, 0)), x}; };
  auto mem = [&](auto pass) { return typename decltype(pass)::template TwMem<SUB>{tw, tid, half}; };
  // One polynomial (or half) per workgroup: each pass's per-lane twiddles are loaded during the pass
  // before it, so that no stage waits for its own (8192 limb-polys of N = 8192: 248 / 262 -> 234 / 238 us
  // forward / inverse; of N = 4096, inverse: 99 -> 88-95 us; few limb-polys: equal).  Not forward at
  // N = 4096, whose four workgroups per CU hide them (1024: 20.9 -> 21.7 us), nor in the persistent kernel,
  // whose registers hold the next polynomial instead.
  constexpr bool AHEAD = !REUSED && (LOGN == 13 || !FWD);
  auto ahead = [&](auto pass, auto& regs) {
    if constexpr (AHEAD && decltype(pass)::LANE_TW) regs.template load<FWD>(mem(pass));
  };
  auto use = [&](auto pass, const auto& regs) {
    if constexpr (AHEAD && decltype(pass)::LANE_TW) return regs;
    else return mem(pass);
  };
  typename P0::TwRegs t0;
  typename P1::TwRegs t1;
  typename P2::TwRegs t2;
  typename S::Tail::TwRegs t3;
  if constexpr (FWD) {
    if constexpr (at == 0) issue();
    P0::template run<true, true, false>(x, mem(P0()), q, qi, [&] { FirstMid()(); ahead(P1(), t1); }, sink(P0()));
    if constexpr (at == 1) issue();
    read_layout<P1, true>(lds, x, tid);
    P1::template run<true, false, false>(x, use(P1(), t1), q, qi, [&] { LdsMid()(); ahead(P2(), t2); }, sink(P1()));
    if constexpr (at == 2) issue();
    read_layout<P2, true>(lds, x, tid);
    if constexpr (S::HAS3) {
      P2::template run<true, false, false>(x, use(P2(), t2), q, qi, [&] { LdsMid()(); ahead(P3(), t3); }, sink(P2()));
      if constexpr (at == 3) issue();
      read_layout<P3, true>(lds, x, tid);
      P3::template run<true, false, true>(x, use(P3(), t3), q, qi, NoMid(), NoSink());
      if constexpr (at == 4) issue();
    } else {
      P2::template run<true, false, true>(x, use(P2(), t2), q, qi, NoMid(), NoSink());
      if constexpr (at == 3) issue();
    }
  } else {
    // pass k of the inverse runs Pass index NP - 1 - k
    if constexpr (at == 0) issue();
    if constexpr (S::HAS3) {
      ahead(P3(), t3);
      P3::template run<false, true, false>(x, use(P3(), t3), q, qi, [&] { FirstMid()(); ahead(P2(), t2); }, sink(P3()));
      if constexpr (at == 1) issue();
      read_layout<P2, false>(lds, x, tid);
      P2::template run<false, false, false>(x, use(P2(), t2), q, qi, [&] { LdsMid()(); ahead(P1(), t1); }, sink(P2()));
    } else {
      ahead(P2(), t2);
      P2::template run<false, true, false>(x, use(P2(), t2), q, qi, [&] { FirstMid()(); ahead(P1(), t1); }, sink(P2()));
    }
    if constexpr (at == S::NP - 2) issue();
    read_layout<P1, false>(lds, x, tid);
    P1::template run<false, false, false>(x, use(P1(), t1), q, qi, [&] { LdsMid()(); ahead(P0(), t0); }, sink(P1()));
    if constexpr (at == S::NP - 1) issue();
    read_layout<P0, false>(lds, x, tid);
    P0::template run<false, false, true>(x, use(P0(), t0), q, qi, NoMid(), NoSink());
    if constexpr (at == S::NP) issue();
  }
}

template <int LOGN, int PT, bool FWD, class LoadOp>
__device__ __forceinline__ void ntt_load(double (&x)[PT], const PolyDesc& d, const LoadOp& ld, double q, double qi, int tid) {
  if constexpr (LoadOp::kAll) {
    ld.template load_all<LOGN, PT, FWD>(x, d, q, qi, tid);
  } else {
#pragma unroll
    for (int i = 0; i < PT; ++i) x[i] = ld(d, FirstPass<LOGN, PT, FWD>::idx(tid, i), q, qi);
  }
}

// results of the last pass to global memory, canonical unless the epilogue multiplies them anyway
// (kLazy: it takes |v| < 1.8 q).  The inverse applies its scale (N^-1) here: |x| <= 8 q comes out of the
// product below 2 q.
template <int LOGN, int PT, bool FWD, class StoreOp>
__device__ __forceinline__ void ntt_store(double (&x)[PT], const PolyDesc& d, const StoreOp& st, double q, double qi, double ninv, int tid,
                                          double* lds) {
  if constexpr (StoreOp::kAll) {  // the epilogue takes all of a work-item's results at once
    int j[PT];
    double v[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      j[i] = LastPass<LOGN, PT, FWD>::idx(tid, i);
      const double y = FWD ? x[i] : mulmod_s(x[i], ninv, q, qi);
      v[i] = FWD && StoreOp::kLazy ? y : canon2(y, q, qi);
    }
    st.template put_all<LOGN, PT, LastPass<LOGN, PT, FWD>::GS>(d, j, v, q, qi, lds, tid);
  } else {
    // Every operand load of the epilogue is issued before the first store: vector-memory
    // completion is tracked in issue order, so a load issued after a store could only be
    // consumed once that store had completed.
    typename StoreOp::Operand e[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) e[i] = st.fetch(d, LastPass<LOGN, PT, FWD>::idx(tid, i));
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const int j = LastPass<LOGN, PT, FWD>::idx(tid, i);
      const double y = FWD ? x[i] : mulmod_s(x[i], ninv, q, qi);
      const double v = FWD && StoreOp::kLazy ? y : canon2(y, q, qi);
      st.put(d, j, v, e[i], q, qi);
    }
  }
}

// waves per SIMD the launch bounds promise: 4 (PT 16: 16 waves per workgroup at N = 16384, up
// to 128 VGPRs each) or 2 (PT 32: up to 256 VGPRs, room for 32 values and their prefetch)
template <int PT>
constexpr int waves_per_eu() { return PT == 32 ? 2 : 4; }

// One workgroup per polynomial.
template <int LOGN, int PT, bool FWD, class LoadOp, class StoreOp>
__global__ __launch_bounds__((1 << LOGN) / PT) __attribute__((amdgpu_waves_per_eu(waves_per_eu<PT>()))) void k_ntt(
    NttSrc descs, const double* __restrict__ tw_all, ModTable mt, LoadOp ld, StoreOp st) {
  constexpr int N = 1 << LOGN;
  __shared__ double lds[N + N / 16];
  const PolyDesc d = descs.get(blockIdx.x);
  const double q = mt.m[d.mod].q, qi = mt.m[d.mod].qinv;
  const int tid = threadIdx.x;
  double x[PT];
  ntt_load<LOGN, PT, FWD>(x, d, ld, q, qi, tid);
  ntt_core<LOGN, PT, FWD, false>(lds, x, tw_all + (size_t)d.mod * N, q, qi, tid);
  ntt_store<LOGN, PT, FWD>(x, d, st, q, qi, !FWD && !LoadOp::kAll && d.aux2 != 0.0 ? d.aux2 : mt.m[d.mod].ninv, tid, lds);
}

// Half a polynomial per workgroup (forward, N = 2^(LOGN + 1)): the first stage, x_j +- w x_{j + N/2}, is
// done while the words are read, and each half is a transform of its own.  At N = 16384 a whole
// polynomial's exchange buffer leaves one workgroup per CU with nothing to run while it loads, stages or
// stores; two halves fit a CU, and few polynomials spread over twice the CUs.  Both halves read all
// words (the same XCD's L2 serves the second) and form the first stage's products.  Bound by FP64 issue
// and LDS in turn; ModDown conversions of the attention output 2400 -> 2165 us in 10 launches, rescales
// 629 -> 533 us in 7.
template <int LOGN, int PT, class LoadOp, class StoreOp>
__global__ __launch_bounds__((1 << LOGN) / PT) __attribute__((amdgpu_waves_per_eu(waves_per_eu<PT>()))) void k_ntt_half(
    NttSrc descs, const double* __restrict__ tw_all, ModTable mt, LoadOp ld, StoreOp st) {
  constexpr int H = 1 << LOGN;
  __shared__ double lds[H + H / 16];
  const int w = descs.at(blockIdx.x), half = w & 1;
  PolyDesc d = descs.desc(w >> 1);
  const double q = mt.m[d.mod].q, qi = mt.m[d.mod].qinv;
  const int tid = threadIdx.x;
  const double* tw = tw_all + (size_t)d.mod * 2 * H;
  const double w1 = half ? -tw[1] : tw[1];
  double x[PT];
  const auto cst = ld.half_constants(d, w1, q, qi);
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int j = FirstPass<LOGN, PT, true>::idx(tid, i);
    x[i] = ld.half(d, j, H, cst, q, qi);
  }
  ntt_core<LOGN, PT, true, false, true>(lds, x, tw, q, qi, tid, NoIssue(), half);
  d.dst += half * H;
  d.src2 += half * H;
  if (d.src3) d.src3 += half * H;
  d.flags |= half ? kUpperHalf : 0;
  ntt_store<LOGN, PT, true>(x, d, st, q, qi, 0.0, tid, lds);
}

// Persistent, software-pipelined variant: a grid of resident workgroups walks the descriptor
// list with a grid stride; the next polynomial's operands are loaded into registers while the
// current one is transformed, hiding the global-memory latency that a one-shot workgroup (one
// per CU at N = 16384) exposes.
template <int LOGN, int PT, bool FWD, class LoadOp, class StoreOp>
__global__ __launch_bounds__((1 << LOGN) / PT) __attribute__((amdgpu_waves_per_eu(waves_per_eu<PT>()))) void k_ntt_pipe(
    NttSrc descs, const double* __restrict__ tw_all, ModTable mt, LoadOp ld, StoreOp st, int count) {
  constexpr int N = 1 << LOGN;
  constexpr int PF = PT;
  using First = FirstPass<LOGN, PT, FWD>;
  __shared__ double lds[N + N / 16];
  const int tid0 = threadIdx.x;
  int p = blockIdx.x;
  if (p >= count) return;
  // The next polynomial's words are prefetched raw (converted only when its iteration starts, so
  // nothing waits for them earlier).  Vector-memory completion is tracked in issue order,
  // stores included: the only wait in an iteration is for its own prefetch, issued before the
  // previous iteration's stores.
  uint64_t nx[PF];
  {
    const PolyDesc d = descs.get(p);
#pragma unroll
    for (int i = 0; i < PF; ++i) nx[i] = ld.raw(d, First::idx(tid0, i));
    // the first polynomial's loads complete before the loop: registers still pending on entry
    // would make the loop head wait for the previous iteration's stores as well
#pragma unroll
    for (int i = 0; i < PF; ++i) asm volatile("" : "+v"(nx[i]));
  }
  for (;;) {
    // an opaque copy of the work-item index: keeps the compiler from hoisting every
    // index computation of the loop body out of the loop (which would spill registers)
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const PolyDesc d = descs.get(p);
    const double q = mt.m[d.mod].q, qi = mt.m[d.mod].qinv;
    double x[PT];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
      uint64_t u = nx[i];
      asm volatile("" : "+v"(u));  // the conversion stays in this iteration
      x[i] = ld.cvt(d, u, q, qi);
    }
#pragma unroll
    for (int i = PF; i < PT; ++i) x[i] = ld(d, First::idx(tid, i), q, qi);
    const int pn = p + gridDim.x;
    auto prefetch = [&] {
      // unconditional (the last iteration re-reads its own polynomial), so the loads land in nx
      // directly and are only waited for when the next iteration starts
      const PolyDesc dn = descs.get(pn < count ? pn : p);
#pragma unroll
      for (int i = 0; i < PF; ++i) nx[i] = ld.raw(dn, First::idx(tid, i));
    };
    ntt_core<LOGN, PT, FWD, true>(lds, x, tw_all + (size_t)d.mod * N, q, qi, tid, prefetch);
    ntt_store<LOGN, PT, FWD>(x, d, st, q, qi, !FWD && !LoadOp::kAll && d.aux2 != 0.0 ? d.aux2 : mt.m[d.mod].ninv, tid, lds);
    p = pn;
    if (p >= count) break;
  }
}

template <int PT, bool FWD, class LoadOp, class StoreOp>
void launch_ntt_pt(blb_ctx* c, NttSrc d_descs, int count, LoadOp ld, StoreOp st) {
  const double* tw = FWD ? c->d_tw_fwd : c->d_tw_inv;
  const int threads = c->n / PT;
  // At N = 16384 the transforms that read scratch (base conversions, rescale) run as two halves: 12-head
  // Q K^T 3558 -> 3321 us, attention output 7358 -> 6977 us, a rotate-and-sum over 1 / 24 / 64
  // ciphertexts (4 primes + 2 special) 1154 / 1538 / 2889 -> 1033 / 1503 / 2793 us (with one special prime
  // 953 / 1587 / 3291 -> 824 / 1468 / 2998 us).  Not plan transforms: their coefficients' reductions, which
  // both halves would do, make them slower (145 us against the persistent grid's 130).
  constexpr bool kHalf = FWD && LoadOp::kHalf;
  if constexpr (kHalf) {
    if (c->log_n == 14) {
      NttSrc src = d_descs;
      src.group = 2 * src.group;
      src.split = 2 * src.split;
      src.tail = 2 * src.tail;
      src.count = 2 * count;
      emit(c, [=, stream = c->stream] { k_ntt_half<13, PT><<<2 * count, threads / 2, 0, stream>>>(src, tw, c->mt, ld, st); });
      return;
    }
  }
  // The persistent grid pays at N = 16384, where one polynomial fills a CU's LDS and nothing else hides
  // its loads, from the third round of polynomials on (2048 of them: 125-135 us against 137-144 one per
  // workgroup; 512: equal; 256: 23 against 21).  At N = 4096 / 8192 four / two workgroups per CU overlap
  // by themselves: one polynomial each is faster at every count (1024 at N = 8192: 34 us against 38-40).
  if constexpr (StoreOp::kPersistent && LoadOp::kPersistent) {
    if (c->ntt_variant == 1 && c->log_n == 14 && count > 2 * c->n_cu) {
      emit(c, [=, stream = c->stream] { k_ntt_pipe<14, PT, FWD><<<c->n_cu, threads, 0, stream>>>(d_descs, tw, c->mt, ld, st, count); });
      return;
    }
  }
  switch (c->log_n) {
    case 12: emit(c, [=, stream = c->stream] { k_ntt<12, PT, FWD><<<count, threads, 0, stream>>>(d_descs, tw, c->mt, ld, st); }); break;
    case 13: emit(c, [=, stream = c->stream] { k_ntt<13, PT, FWD><<<count, threads, 0, stream>>>(d_descs, tw, c->mt, ld, st); }); break;
    case 14:
      if constexpr (!kHalf)
        emit(c, [=, stream = c->stream] { k_ntt<14, PT, FWD><<<count, threads, 0, stream>>>(d_descs, tw, c->mt, ld, st); });
      break;
    default: break;
  }
}
template <bool FWD, class LoadOp, class StoreOp>
void launch_ntt_generic(blb_ctx* c, NttSrc d_descs, int count, LoadOp ld, StoreOp st) {
  if (count <= 0) return;
  if (c->ntt_radix == 32) launch_ntt_pt<kPT32, FWD>(c, d_descs, count, ld, st);
  else launch_ntt_pt<kPT16, FWD>(c, d_descs, count, ld, st);
}

}  // namespace

// ---------------------------------------------------------------------------------------
// Load / store variants.  Descriptor pointers are global memory; accessing them through the
// global address space (not generic) keeps the loads off the LDS counter, so the LDS-only
// barriers do not wait for them, and lets a uniform base pointer stay in scalar registers.
// ---------------------------------------------------------------------------------------
typedef __attribute__((address_space(1))) uint64_t gu64;
__device__ __forceinline__ uint64_t gld(const uint64_t* p, int j) { return ((const gu64*)p)[j]; }
__device__ __forceinline__ void gst(uint64_t* p, int j, uint64_t v) { ((gu64*)p)[j] = v; }
// words j, j + 1 (ciphertexts need 8-byte alignment only)
typedef uint64_t u64pair __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ u64pair gld2(const uint64_t* p, int j) { return *(const __attribute__((address_space(1))) u64pair*)((const gu64*)p + j); }
__device__ __forceinline__ void gst2(uint64_t* p, int j, double a, double b) {
  *(__attribute__((address_space(1))) u64pair*)((gu64*)p + j) = u64pair{d2u(a), d2u(b)};
}

// Loads: raw(d, j) fetches word j, cvt() turns it into this pass's double operand.
// kHalf: k_ntt_half may run it; half_constants() and half() then give the first forward stage's result
// x_j + w x_{j + H} (w the twiddle, negated for the upper half), reduced.  Only for loads whose source
// is scratch that nothing writes meanwhile: both halves read all of it.
// kPersistent: whether the persistent kernel, which prefetches one raw word per value, may run it.
struct LdPlain {
  static constexpr bool kAll = false;
  static constexpr bool kHalf = false;
  static constexpr bool kPersistent = true;
  __device__ uint64_t raw(const PolyDesc& d, int j) const { return gld(d.src, j); }
  __device__ double cvt(const PolyDesc&, uint64_t u, double, double) const { return u2d(u); }
  __device__ double operator()(const PolyDesc& d, int j, double q, double qi) const { return cvt(d, raw(d, j), q, qi); }
};
// Stores: fetch(d, j) loads the epilogue's global operand for word j, put() writes word j; or (kAll)
// put_all() loads and writes all of a work-item's words.
// In k_ntt_half the words at dst, src2 and src3 are the half's; kUpperHalf in the flags tells which.
// kPersistent: whether the persistent kernel may run this epilogue (the ModDown epilogue's operands do
// not fit 128 VGPRs next to a prefetch of the following polynomial).
struct StPlain {
  static constexpr bool kLazy = false;
  static constexpr bool kPersistent = true;
  static constexpr bool kAll = false;
  struct Operand {};
  __device__ Operand fetch(const PolyDesc&, int) const { return {}; }
  __device__ void put(const PolyDesc& d, int j, double v, Operand, double, double) const { gst(d.dst, j, d2u(v)); }
};
// load an integer coefficient (int64) and reduce it into this modulus: plan transforms
struct LdCoef {
  static constexpr bool kAll = false;
  static constexpr bool kHalf = false;
  static constexpr bool kPersistent = true;
  __device__ uint64_t raw(const PolyDesc& d, int j) const { return gld(d.src, j); }
  __device__ double cvt(const PolyDesc&, uint64_t u, double q, double qi) const { return i64_mod(u, q, qi); }
  __device__ double operator()(const PolyDesc& d, int j, double q, double qi) const { return cvt(d, raw(d, j), q, qi); }
};
// load a residue of another modulus and lift it centred into this modulus: used by rescale (last limb ->
// limb i).  That modulus is the descriptor's aux, or (GIVEN: the descriptors hold masks) q_last.
template <bool GIVEN>
struct LdLift {
  double q_last;
  static constexpr bool kAll = false;
  static constexpr bool kHalf = true;
  static constexpr bool kPersistent = false;
  __device__ uint64_t raw(const PolyDesc& d, int j) const { return gld(d.src, j); }
  __device__ double cvt(const PolyDesc& d, uint64_t u, double q, double qi) const {
    const double v = u2d(u);
    const double ql = GIVEN ? q_last : d.aux;
    const double t = v > 0.5 * ql ? v - ql : v;  // centred, |t| < q_l / 2
    return reduce_s(t, q, qi);
  }
  __device__ double operator()(const PolyDesc& d, int j, double q, double qi) const { return cvt(d, raw(d, j), q, qi); }
  __device__ double half_constants(const PolyDesc&, double w, double, double) const { return w; }
  __device__ double half(const PolyDesc& d, int j, int H, double w, double q, double qi) const {
    const uint64_t a = raw(d, j), b = raw(d, j + H);
    return reduce_s(cvt(d, a, q, qi) + mulmod_s(cvt(d, b, q, qi), w, q, qi), q, qi);
  }
};
// Masked rescale (a mask product or a sum of two, then the rescale) without the masked ciphertext in
// memory: the inverse transform of the last limb forms src2 mx + src3 my (src3 may be null) while it reads,
// and the other limbs' epilogue forms theirs.  The descriptor's aux2 and aux hold the addresses of mx, my.
__device__ __forceinline__ const uint64_t* mask_of(double bits) { return (const uint64_t*)__double_as_longlong(bits); }
struct LdMasked {
  static constexpr bool kAll = true;
  static constexpr bool kHalf = false;
  static constexpr bool kPersistent = false;
  template <int LOGN, int PT, bool FWD>
  __device__ void load_all(double (&x)[PT], const PolyDesc& d, double q, double qi, int tid) const {
    auto idx = [&](int i) { return FirstPass<LOGN, PT, FWD>::idx(tid, i); };
#pragma unroll
    for (int i = 0; i < PT; ++i) x[i] = mulmod_s(u2d(gld(d.src2, idx(i))), u2d(gld(mask_of(d.aux2), idx(i))), q, qi);
    if (d.src3)  // uniform over the workgroup (one descriptor)
#pragma unroll
      for (int i = 0; i < PT; ++i) x[i] = reduce_s(x[i] + mulmod_s(u2d(gld(d.src3, idx(i))), u2d(gld(mask_of(d.aux), idx(i))), q, qi), q, qi);
  }
};
// Base conversion (no centring) of n_src limbs into this modulus, sum_i y_i cst_i with y_i < q_i of
// limb i: the ModUp of a digit and the ModDown of the special limbs, done while the transform reads
// its operands instead of in a pass of its own that wrote every converted limb and had it read
// back (the conversions' write and read were a third of a key switch's ModDown traffic).  A single
// limb's constant is 1 and its words, below 2^50, are operands as they are.
// Wider digits read their limbs once for each limb they give (the runs of descriptors keep that in the L2), and
// at N = 16384 more than two are converted by whole polynomials; against the pass of its own and the in-place
// transforms a rotate-and-sum step over 16 / 64 ciphertexts took, two steps, us: 6 primes in digits of 3,
// 2 special, N = 16384 436 / 1280 -> 230 / 655; 8 in 4, 4 special 502 / 1672 -> 288 / 1012; 8 in 8, 1 special
// 445 / 1263 -> 270 / 553; 12 in 4, 3 special, N = 8192 482 / 1333 -> 268 / 775.
// MOST: bound on n_src (1: one limb always); STRIDE: distance of the constants.
template <int MOST, int STRIDE>
struct LdConv {
  static constexpr bool kAll = false;
  static constexpr bool kPersistent = false;
  static constexpr bool kHalf = MOST <= 2;  // more: the stage's constants would not fit the registers
  __device__ double operator()(const PolyDesc& d, int j, double q, double qi) const {
    if constexpr (MOST == 1) return u2d(gld(d.src, j));
    typedef __attribute__((address_space(4))) const double kdouble;
    uint64_t u[MOST];
#pragma unroll
    for (int i = 0; i < MOST; ++i)
      if (i < d.n_src) u[i] = gld(d.src + ((size_t)i << d.log_n), j);
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < MOST; ++i)  // |acc| < 8 x 0.875 q
      if (i < d.n_src) acc += mulmod_s(u2d(u[i]), ((const kdouble*)d.cst)[i * STRIDE], q, qi);
    return reduce_s(acc, q, qi);
  }
  // sum_i y_i[j] cst_i + y_i[j + H] (w cst_i): the stage's product costs no more than the conversion's
  struct HalfConst {
    double c[MOST], wc[MOST];
  };
  __device__ HalfConst half_constants(const PolyDesc& d, double w, double q, double qi) const {
    typedef __attribute__((address_space(4))) const double kdouble;
    HalfConst h;
#pragma unroll
    for (int i = 0; i < MOST; ++i) {
      h.c[i] = MOST == 1 ? 1.0 : i < d.n_src ? ((const kdouble*)d.cst)[i * STRIDE] : 0.0;
      h.wc[i] = MOST == 1 ? w : reduce_s(mulmod_s(h.c[i], w, q, qi), q, qi);
    }
    return h;
  }
  __device__ double half(const PolyDesc& d, int j, int H, const HalfConst& h, double q, double qi) const {
    if constexpr (MOST == 1) {
      const uint64_t a = gld(d.src, j), b = gld(d.src, j + H);
      return reduce_s(u2d(a) + mulmod_s(u2d(b), h.wc[0], q, qi), q, qi);
    } else {
      uint64_t a[MOST], b[MOST];
#pragma unroll
      for (int i = 0; i < MOST; ++i)
        if (i < d.n_src) {
          a[i] = gld(d.src + ((size_t)i << d.log_n), j);
          b[i] = gld(d.src + ((size_t)i << d.log_n), j + H);
        }
      double acc = 0.0;
#pragma unroll
      for (int i = 0; i < MOST; ++i)
        if (i < d.n_src) {
          if (i > 0 && (i & 3) == 0) acc = reduce_s(acc, q, qi);  // four limbs: |acc| < q/2 + 8 x 0.875 q
          acc += mulmod_s(u2d(a[i]), h.c[i], q, qi) + mulmod_s(u2d(b[i]), h.wc[i], q, qi);
        }
      return reduce_s(acc, q, qi);
    }
  }
};
// rescale epilogue: dst[j] <- (c_i[j] - v) * q_l^-1 mod q_i, c_i = d.src2, aux2 = q_l^-1 mod q_i
struct StRescale {
  static constexpr bool kLazy = true;
  static constexpr bool kPersistent = true;
  static constexpr bool kAll = false;
  using Operand = uint64_t;
  __device__ Operand fetch(const PolyDesc& d, int j) const { return gld(d.src2, j); }
  __device__ void put(const PolyDesc& d, int j, double v, Operand ci, double q, double qi) const {
    const double r = mulmod_s(u2d(ci) - v, d.aux2, q, qi);  // |c_i - v| < 2.8 q: |r| < 1.6 q
    gst(d.dst, j, d2u(canon2(r, q, qi)));
  }
};
// ModDown epilogue: dst[j] <- (u_i[j] - v) * P^-1 (+ add[j] if src3), u_i = src2 (u64).
// For a rotation add = sigma_g(c0), a permuted read of src3 (kAddBoth: sigma_g(c0) + c0).  g is odd, so
// sigma_g keeps aligned runs of 2^k words together (their exponents differ in the top k bits only): a
// wave's permuted read covers whole lines, and a pair of words is one load, swapped or not.  Against
// staging src3 in LDS (two barriers, and two waits for memory in turn): ModDowns of the attention output
// 2090-2185 -> 1984 us in 10 launches (N = 16384), of 24 rotate-and-sums 154 -> 146 us in 11 (N = 8192), of a
// single rotation 7.8 -> 7.4 us (N = 4096).
struct StModDown {
  static constexpr bool kLazy = true;
  static constexpr bool kPersistent = false;
  static constexpr bool kAll = true;
  template <int LOGN, int PT, int GS>
  __device__ void put_all(const PolyDesc& d, const int (&j)[PT], const double (&v)[PT], double q, double qi, double*, int) const {
    static_assert(GS % 2 == 0, "runs of pairs");
    constexpr int P = PT / 2;
    u64pair u[P], a[P];
    uint32_t swap = 0;
    // (a rotation's element is 1 mod 4, so it keeps the exponents' bit that tells the halves apart)
    const int up = d.flags & kUpperHalf ? 1 << (d.log_n - 1) : 0;
    auto load_add = [&](int m) {
      const int jp = d.gal ? (int)gal_perm((uint32_t)(j[2 * m] + up), d.gal, d.log_n) - up : j[2 * m];
      a[m] = gld2(d.src3, jp & ~1);
      swap |= (uint32_t)(jp & 1) << m;
    };
    auto add = [&](double& x, uint64_t y) {
      x += u2d(y);
      x = x >= q ? x - q : x;
    };
#pragma unroll
    for (int m = 0; m < P; ++m) u[m] = gld2(d.src2, j[2 * m]);
    if (d.src3) {  // uniform over the workgroup (one descriptor)
#pragma unroll
      for (int m = 0; m < P / 2; ++m) load_add(m);
    }
    double r[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i)
      r[i] = canon2(mulmod_s(u2d(u[i / 2][i % 2]) - v[i], d.aux2, q, qi), q, qi);  // |u_i - v| < 2.8 q: |product| < 1.6 q
    if (d.src3) {
#pragma unroll
      for (int m = P / 2; m < P; ++m) load_add(m);  // (all P at once do not fit 128 VGPRs)
#pragma unroll
      for (int m = 0; m < P; ++m) {
        const bool s = swap >> m & 1;
        add(r[2 * m], s ? a[m][1] : a[m][0]);
        add(r[2 * m + 1], s ? a[m][0] : a[m][1]);
      }
      if (d.flags & kAddBoth) {
#pragma unroll
        for (int m = 0; m < P; ++m) a[m] = gld2(d.src3, j[2 * m]);
#pragma unroll
        for (int i = 0; i < PT; ++i) add(r[i], a[i / 2][i % 2]);
      }
      // dst may be src3 itself: every work-item's permuted reads have arrived before any store
      if (d.gal) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        lds_barrier();
      }
    }
#pragma unroll
    for (int m = 0; m < P; ++m) gst2(d.dst, j[2 * m], r[2 * m], r[2 * m + 1]);
  }
};

// masked rescale epilogue: dst[j] <- (src2[j] mx[j] + src3[j] my[j] - v) * q_l^-1 mod q_i (src3 may be null)
struct StMaskRescale {
  double inv[BLB_MAXQ];  // q_l^-1 modulo each prime
  static constexpr bool kLazy = true;
  static constexpr bool kPersistent = false;
  static constexpr bool kAll = true;
  template <int LOGN, int PT, int GS>
  __device__ void put_all(const PolyDesc& d, const int (&j)[PT], const double (&v)[PT], double q, double qi, double*, int) const {
    static_assert(GS % 2 == 0, "runs of pairs");
    const int up = d.flags & kUpperHalf ? 1 << (d.log_n - 1) : 0;
    double r[PT];
    auto add = [&](const uint64_t* x, const uint64_t* m, const double (&to)[PT], double sign) {
#pragma unroll
      for (int i = 0; i < PT; i += 2) {
        const u64pair a = gld2(x, j[i]), b = gld2(m + up, j[i]);
        r[i] = mulmod_s(u2d(a[0]), u2d(b[0]), q, qi) + sign * to[i];
        r[i + 1] = mulmod_s(u2d(a[1]), u2d(b[1]), q, qi) + sign * to[i + 1];
      }
    };
    add(d.src2, mask_of(d.aux2), v, -1.0);
    if (d.src3) add(d.src3, mask_of(d.aux), r, 1.0);  // uniform over the workgroup (one descriptor)
    const double w = inv[d.mod];
#pragma unroll
    for (int i = 0; i < PT; i += 2)  // |r| < 0.875 q + 0.875 q + 1.8 q: |product| < 1.84 q
      gst2(d.dst, j[i], canon2(mulmod_s(r[i], w, q, qi), q, qi), canon2(mulmod_s(r[i + 1], w, q, qi), q, qi));
  }
};

// Plan epilogue: canonical results in the 50-bit plan format (low 32 bits, next 16, top 2 in u32
// words of 16; see pt50_bytes) at dst.  A work-item holds runs of GS consecutive words (the last
// pass's groups), so its top-bit codes fill whole words (GS = 16), whole bytes (GS = 4) or half a byte
// (GS = 2: the neighbour lane's half joins it); passes of other sizes gather the codes in LDS (free
// after the last pass).
struct StPack50 {
  static constexpr bool kLazy = false;
  static constexpr bool kPersistent = true;
  static constexpr bool kAll = true;
  template <int LOGN, int PT, int GS>
  __device__ void put_all(const PolyDesc& d, const int (&j)[PT], const double (&v)[PT], double, double, double* lds, int tid) const {
    constexpr int N = 1 << LOGN, T = N / PT;
    typedef __attribute__((address_space(1))) uint32_t g32;
    typedef __attribute__((address_space(1))) uint16_t g16;
    typedef __attribute__((address_space(1))) uint8_t g8;
    g32* lo = (g32*)(uint8_t*)d.dst;
    g16* mid = (g16*)((uint8_t*)d.dst + (size_t)4 * N);
    uint8_t* top = (uint8_t*)d.dst + (size_t)6 * N;
    uint32_t code[PT];
#pragma unroll
    for (int i = 0; i < PT; ++i) {
      const uint64_t w = d2u(v[i]);
      lo[j[i]] = (uint32_t)w;
      mid[j[i]] = (uint16_t)(w >> 32);
      code[i] = (uint32_t)(w >> 48);
    }
    if constexpr (GS == 16 || GS == 4 || GS == 2) {
#pragma unroll
      for (int h = 0; h < PT / GS; ++h) {
        uint32_t bits = 0;
#pragma unroll
        for (int k = 0; k < GS; ++k) bits |= code[h * GS + k] << (2 * k);
        if constexpr (GS == 16) ((g32*)top)[j[h * GS] >> 4] = bits;
        else if constexpr (GS == 4) ((g8*)top)[j[h * GS] >> 2] = (uint8_t)bits;
        else {  // lanes t, t + 1 hold words 4m, 4m + 1 and 4m + 2, 4m + 3
          const uint32_t other = __shfl_xor(bits, 1);
          if ((tid & 1) == 0) ((g8*)top)[j[h * GS] >> 2] = (uint8_t)(bits | (other << 4));
        }
      }
      return;
    }
    uint8_t* codes = (uint8_t*)lds;
    lds_barrier();  // every work-item is past its reads of the last exchange
#pragma unroll
    for (int i = 0; i < PT; ++i) codes[j[i]] = (uint8_t)code[i];
    lds_barrier();
    for (int t = tid; t < N / 16; t += T) {
      const uint32_t* c4 = (const uint32_t*)(codes + 16 * t);
      uint32_t word = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint32_t x = c4[b];  // codes of words 4b .. 4b + 3, one per byte
        const uint32_t c = (x & 3u) | ((x >> 6) & 0xCu) | ((x >> 12) & 0x30u) | ((x >> 18) & 0xC0u);
        word |= c << (8 * b);
      }
      ((g32*)top)[t] = word;
    }
  }
};

// add-into epilogue: dst[j] <- src2[j] + v mod q  (mask added to c0 in evaluation form)
struct StAddTo {
  static constexpr bool kLazy = false;
  static constexpr bool kPersistent = true;
  static constexpr bool kAll = false;
  using Operand = uint64_t;
  __device__ Operand fetch(const PolyDesc& d, int j) const { return gld(d.src2, j); }
  __device__ void put(const PolyDesc& d, int j, double v, Operand a, double q, double) const {
    double r = u2d(a) + v;
    r = r >= q ? r - q : r;
    gst(d.dst, j, d2u(r));
  }
};

static NttSrc table(blb_ctx* c, const PolyDesc* d_descs) { return NttSrc{d_descs, nullptr, 1, c->log_n}; }
void launch_ntt_addto(blb_ctx* c, const PolyDesc* d_descs, int count) {
  launch_ntt_generic<true>(c, table(c, d_descs), count, LdPlain{}, StAddTo{});
}
void launch_ntt(blb_ctx* c, const PolyDesc* d_descs, int count, bool fwd) {
  if (fwd) launch_ntt_generic<true>(c, table(c, d_descs), count, LdPlain{}, StPlain{});
  else launch_ntt_generic<false>(c, table(c, d_descs), count, LdPlain{}, StPlain{});
}
void launch_ntt_rescale(blb_ctx* c, const PolyDesc* d_descs, int count) {
  launch_ntt_generic<true>(c, table(c, d_descs), count, LdLift<false>{}, StRescale{});
}
void launch_intt_masked(blb_ctx* c, const PolyDesc* d_descs, int count) {
  launch_ntt_generic<false>(c, table(c, d_descs), count, LdMasked{}, StPlain{});
}
void launch_ntt_rescale_masked(blb_ctx* c, const PolyDesc* d_descs, int count, int level, const double* inv) {
  StMaskRescale st{};
  for (int i = 0; i < level; ++i) st.inv[i] = inv[i];
  launch_ntt_generic<true>(c, table(c, d_descs), count, LdLift<true>{(double)c->mod[level]}, st);
}
static NttSrc grouped(blb_ctx* c, const PolyDesc* d_descs, int count, NttRuns r) {
  return NttSrc{d_descs, nullptr, 1, c->log_n, r.group, r.split, r.tail, count};
}
void launch_ntt_modup(blb_ctx* c, const PolyDesc* d_descs, int count, int most, NttRuns runs) {
  const NttSrc src = grouped(c, d_descs, count, runs);
  if (most <= 1) launch_ntt_generic<true>(c, src, count, LdConv<1, BLB_MAXM>{}, StPlain{});
  else if (most <= 2) launch_ntt_generic<true>(c, src, count, LdConv<2, BLB_MAXM>{}, StPlain{});
  else launch_ntt_generic<true>(c, src, count, LdConv<BLB_MAXALPHA, BLB_MAXM>{}, StPlain{});
}
void launch_ntt_moddown(blb_ctx* c, const PolyDesc* d_descs, int count, int most, NttRuns runs) {
  const NttSrc src = grouped(c, d_descs, count, runs);
  if (most <= 1) launch_ntt_generic<true>(c, src, count, LdConv<1, BLB_MAXQ>{}, StModDown{});
  else if (most <= 2) launch_ntt_generic<true>(c, src, count, LdConv<2, BLB_MAXQ>{}, StModDown{});
  else launch_ntt_generic<true>(c, src, count, LdConv<BLB_MAXSP, BLB_MAXQ>{}, StModDown{});
}
void launch_ntt_regular(blb_ctx* c, uint64_t* base, int count, int nl, bool fwd) {
  const NttSrc src{nullptr, base, nl, c->log_n};
  if (fwd) launch_ntt_generic<true>(c, src, count, LdPlain{}, StPlain{});
  else launch_ntt_generic<false>(c, src, count, LdPlain{}, StPlain{});
}
void launch_ntt_plan(blb_ctx* c, const uint64_t* coef, uint8_t* out, int count, int nl, int p50) {
  NttSrc src{nullptr, (uint64_t*)out, nl, c->log_n, nl, count * nl, 1, count * nl};  // a plaintext's limbs read the same words
  src.coef = coef;
  src.out_bytes = pt_poly_bytes(c->n, p50);
  if (p50) launch_ntt_generic<true>(c, src, count * nl, LdCoef{}, StPack50{});
  else launch_ntt_generic<true>(c, src, count * nl, LdCoef{}, StPlain{});
}
