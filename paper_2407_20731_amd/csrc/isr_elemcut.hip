// Per-element cut: a variant of the lossy step's selection in which every
// element is cut alone by the plain value rule, at its own share of the
// budget (Sec. IV-B: the lossy step's sorting kernels; the global cut's
// threshold rule applied inside one element).  FP64 path.
//
// One wavefront per element.  Its norm terms and energies are formed from
// the field and the FP64 coefficients, and the element's threshold is found by
// a binary search over the energies' keys (their bit patterns, monotone for
// non-negative doubles), between bounds that need no sum: energies of at most
// the budget over twice their number all fit, one above the budget never does.
// It stops once no energy lies strictly inside the interval.  Bound by VALU
// issue: at N = 7 a probe costs ~190 instructions of a wavefront, the exact
// sums and the transform ~1500 (8,192 elements, 3 components: 362 -> 136 us).
// Each probe decides RN(exact sum of
// energies below the key) <= B_e: an FP64 wave sum with a rigorous error
// bound settles almost every probe, and the rest are summed exactly.  Exact
// sums: every lane splits its terms by error-free extraction against 2^m >=
// the wave's largest term into three FP64 sums (exact), their wave totals
// form one 192-bit integer in a wave big integer (X units of 2^-1075), and
// the rare terms far below 2^m go through 32-bit digits in LDS;
// the result is rounded once.  The workgroup adds every element's exact norm
// and dropped energy into per-component digit totals, and the finishing
// kernel rounds the component totals.  The kept counts are known per element
// by then, so the offset scan and pass B of the streaming path follow, on the
// per-element thresholds.
#include "isr.h"
#include "isr_engine.cuh"

namespace isr {

namespace {

constexpr int ED = 68;       // digits of one element's sum (top term bit < 2^2099, 12 bits of count)
constexpr int GD = 128;      // digits of a component total (the 64 words of a wave big integer)
constexpr int EC_WAVES = 4;  // wavefronts per workgroup
constexpr u64 INF_KEY = 0x7ff0000000000000ull;

DEV double jw1(const double* jac, long long e, double t) { return jac ? jac[e] * t : t; }

struct ElemLds {
  u64 d[EC_WAVES][ED];             // per wavefront: the sum being formed
  u64 tot[ISR_MAX_COMP][2][GD];    // per component: norm (0) and dropped energy (1)
  u64 kept[ISR_MAX_COMP];
};

// LDS operations of one wavefront complete in issue order; the fence keeps
// the compiler from moving the accesses around each other.
DEV void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

DEV void ed_clear(u64* D) {
  const int l = lane_id();
  D[l] = 0ull;
  if (l < ED - 64) D[64 + l] = 0ull;
  wave_order();
}

// Adds a finite x >= 0: its significand at X-unit shift max(E, 1) spans
// three 32-bit digits.
DEV void ed_add(u64* D, double x) {
  const u64 bits = dbits(x);
  if (bits == 0ull) return;
  const int E = (int)(bits >> 52);
  const u64 sig = (bits & M52) | (E ? (1ull << 52) : 0ull);
  const int sh = E ? E : 1;
  const int d = sh >> 5, r = sh & 31;
  const u64 lo = sig << r;
  const u64 hi = r ? (sig >> (64 - r)) : 0ull;
  atomicAdd((unsigned long long*)&D[d], (unsigned long long)(lo & 0xffffffffull));
  atomicAdd((unsigned long long*)&D[d + 1], (unsigned long long)(lo >> 32));
  if (hi) atomicAdd((unsigned long long*)&D[d + 2], (unsigned long long)hi);
}

// Digits (each below 2^64, digit i of weight 2^(32 i)) as a wave big
// integer: lane l holds bits [64 l, 64 l + 64).
DEV u64 digits_to_words(u64 a, u64 b) {
  const u64 lo = a + (b << 32);
  const u64 hi = (b >> 32) + (lo < a ? 1ull : 0ull);
  u64 w = lo;
  u64 up = shfl_up64(hi, 1);
  if (lane_id() == 0) up = 0ull;
  wb_add(w, up);
  return w;
}

DEV u64 ed_words(const u64* D) {
  wave_order();
  const int l = lane_id();
  const u64 a = 2 * l < ED ? D[2 * l] : 0ull;
  const u64 b = 2 * l + 1 < ED ? D[2 * l + 1] : 0ull;
  return digits_to_words(a, b);
}

// A wave big integer (each word split in two 32-bit digits) into totals.
DEV void tot_add(u64* T, u64 w) {
  if (w == 0ull) return;
  const int l = lane_id();
  atomicAdd((unsigned long long*)&T[2 * l], (unsigned long long)(w & 0xffffffffull));
  atomicAdd((unsigned long long*)&T[2 * l + 1], (unsigned long long)(w >> 32));
}

// X-unit wave big integer of the exact sum of the terms x[k] with take[k]
// (finite, >= 0) over the wave's lanes.
template <int CNT>
DEV u64 exact_words(const double (&x)[CNT], const bool (&take)[CNT], u64* D) {
  u64 mk = 0ull;
#pragma unroll
  for (int k = 0; k < CNT; ++k) {
    const u64 b = take[k] ? dbits(x[k]) : 0ull;
    mk = b > mk ? b : mk;
  }
  mk = wave_max_dpp(mk);
  if (mk == 0ull) return 0ull;
  // every term is below 2^m (exponent of the largest term plus one)
  int m = (int)(mk >> 52) - 1022;
  m = m < XM_MIN ? XM_MIN : (m > XM_MAX ? XM_MAX : m);
  constexpr int h = 7;  // a lane adds at most 64 = 2^(h-1) terms
  const XParm P = xparm(m, h);
  const XRange R = xrange(P);
  XRun A = xrun(P);
  bool rem = false;
#pragma unroll
  for (int k = 0; k < CNT; ++k) {
    const double y = take[k] ? x[k] : 0.0;
    rem = (xrun_left(A, R, y) && y != 0.0) || rem;
  }
  long long K[3];
  xints(xrun_sums(A, P), P, K);
  I192 z = {{0ull, 0ull, 0ull}};
  const int sft[3] = {107 - 2 * h, 53 - h, 0};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    // (a lane's sum is below 2^53 in magnitude, the wave's below 2^59)
    i192_add_shl(z, (__int128)(long long)wave_sum_dpp((u64)K[i]), sft[i]);
  }
  // z counts units u3 = 2^(m + 3h - 159), i.e. X units shifted by sh (>= 61)
  const int sh = m + 3 * h - 159 + 1075;
  u64 w = part_at(z.w[0], z.w[1], sh);
  wb_add(w, part_at(z.w[2], 0ull, sh + 128));
  if (ballot(rem)) {
    ed_clear(D);
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
      const double y = take[k] ? x[k] : 0.0;
      if (!xin(R, y) && y != 0.0) ed_add(D, y);
    }
    wb_add(w, ed_words(D));
  }
  return w;
}

// RN(exact sum of the energies whose key is below K) <= B, the same answer
// in every lane.  Padding slots carry key ~0 and never count.  The FP64 sum
// of C non-negative terms, in any order, is within (C - 1) 2^-53 of the
// exact sum (first order); twice that settles the probe when B (or the
// successor of B) lies outside the band.
template <int CNT>
DEV bool ec_feasible(const double (&x)[CNT], const u64 (&key)[CNT], u64 K, double B, double succB, u64* D) {
  double s = 0.0;
  int c = 0;
#pragma unroll
  for (int k = 0; k < CNT; ++k) {
    const bool in = key[k] < K;
    s = s + (in ? x[k] : 0.0);
    c += __popcll(ballot(in));
  }
  const double S = wave_sum_dpp(s);
  const double C = (double)c;
  const double bound = ((2.0 * C) * 0x1p-53) * S;
  if (S + bound <= B) return true;
  if (S - bound > succB) return false;
  bool in[CNT];
#pragma unroll
  for (int k = 0; k < CNT; ++k) in[k] = key[k] < K;
  return wb_round(exact_words<CNT>(x, in, D)) <= B;
}

}  // namespace

struct ElemScale {
  double s[ISR_MAX_COMP];  // budget scale per component (1 until a repair)
};

template <int N>
struct ElemXform {};  // transform buffers, one a wavefront
template <>
struct ElemXform<7> {
  double buf[EC_WAVES][Eng<7, P_FP64>::LDSW];
};

template <int N>
__global__ __launch_bounds__(256) void k_elemsel(Job j, const double* coef, double* tau_out, u64* G, ElemScale sc) {
  constexpr int n = N + 1, n3 = n * n * n, CNT = (n3 + 63) / 64;
  __shared__ ElemLds L;
  __shared__ ElemXform<N> X;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < ISR_MAX_COMP * 2 * GD; i += 256) (&L.tot[0][0][0])[i] = 0ull;
  if (tid < ISR_MAX_COMP) L.kept[tid] = 0ull;
  __syncthreads();
  u64* D = L.d[wv];
  const long long E = j.n_elem, pairs = E * j.ncomp;
  const double tt = j.tol * j.tol;
  for (long long p = (long long)blockIdx.x * EC_WAVES + wv; p < pairs; p += (long long)gridDim.x * EC_WAVES) {
    const int comp = (int)(p / E);
    const long long e = p - (long long)comp * E;
    const double* ue = j.u + (size_t)comp * j.comp_stride + (size_t)e * n3;
    double t[CNT], x[CNT];
    u64 key[CNT];
    bool badu = false, bad = false;
    // norm term of field value f and energy of coefficient f (any lane and
    // slot each: both sums are exact), slot k of this lane holding dense
    // position 64 k + lane of the coefficients
    auto take = [&](int k, double uv, int fu, double cv, int fc) {
      t[k] = jw1(j.jac, e, j.tab.w3[fu]) * (uv * uv);
      x[k] = jw1(j.jac, e, j.tab.g3[fc]) * (cv * cv);
      key[k] = dbits(x[k]);
      badu = badu || !__builtin_isfinite(uv);
      bad = bad || !(t[k] >= 0.0 && t[k] <= 0x1.fffffffffffffp+1023) ||
            !(x[k] >= 0.0 && x[k] <= 0x1.fffffffffffffp+1023);
    };
    if constexpr (n == 8) {
      // the wave-tile engine's transform on the spot (its coefficient slots
      // are the dense positions): no coefficient array, no kernel before this
      typedef Eng<N, P_FP64> G;
      static_assert(G::EPW == 1 && G::NS == CNT, "one element, eight slots");
      double u[CNT], c[CNT];
      G::load(ue, 1, (((uintptr_t)ue) & 15) == 0, u, lane);
      G::forward(u, c, X.buf[wv], typename G::Mats(), j.tab, lane);
#pragma unroll
      for (int k = 0; k < CNT; ++k) take(k, u[k], G::w3i(k, lane), c[k], G::g3i(k, lane));
    } else {
      const double* ce = coef + (size_t)p * n3;
#pragma unroll
      for (int k = 0; k < CNT; ++k) {
        const int f = lane + 64 * k;
        if (f < n3) {
          take(k, ue[f], f, ce[f], f);
        } else {
          t[k] = 0.0;
          x[k] = 0.0;
          key[k] = ~0ull;
        }
      }
    }
    const u64 ub = ballot(badu), xb = ballot(bad);
    if (ub | xb) {  // non-finite field value, or an energy or norm term out of range
      if (lane == 0) {
        atomicOr(&j.st[comp].flags, ub ? (int)ST_NONFINITE : (int)ST_OVERFLOW);
        tau_out[p] = __builtin_inf();
        j.cnt[p] = 0u;
      }
      continue;
    }
    // the element's norm, exactly, and its budget
    bool valid[CNT];
#pragma unroll
    for (int k = 0; k < CNT; ++k) valid[k] = lane + 64 * k < n3;
    u64 w = exact_words<CNT>(t, valid, D);
    const double U2e = wb_round(w);
    tot_add(L.tot[comp][0], w);
    const double B = (tt * U2e) * sc.s[comp];
    const double succB = __longlong_as_double((long long)(dbits(B) + 1ull));
    // the element's threshold
    u64 kt;
    if (ec_feasible<CNT>(x, key, INF_KEY, B, succB, D)) {
      kt = INF_KEY;  // everything fits the budget: +inf, nothing kept
    } else {
      // Largest key <= `most` and smallest key >= `least` over the wave (0 /
      // ~0 when there is none; padding slots, key ~0, never count as one).
      auto last_upto = [&](u64 most) {
        u64 m = 0ull;
#pragma unroll
        for (int k = 0; k < CNT; ++k) m = key[k] <= most && key[k] > m ? key[k] : m;
        return wave_max_dpp(m);
      };
      auto first_from = [&](u64 least) {
        u64 m = ~0ull;
#pragma unroll
        for (int k = 0; k < CNT; ++k) m = key[k] >= least && key[k] < m ? key[k] : m;
        return ~wave_max_dpp(~m);
      };
      // S(lo) <= B < S(hi) from the start: energies of at most B over twice
      // their number all fit, and one above B never does
      constexpr double SHARE = CNT <= 1 ? 0x1p-7 : CNT <= 2 ? 0x1p-8 : CNT <= 4 ? 0x1p-9 : CNT <= 8 ? 0x1p-10
                               : CNT <= 16 ? 0x1p-11 : CNT <= 32 ? 0x1p-12 : 0x1p-13;
      static_assert(CNT <= 64, "energies of an element");
      const u64 small = last_upto(dbits(B * SHARE));
      u64 lo = small ? small : first_from(0ull);
      const u64 over = first_from(dbits(B) + 1ull);
      u64 hi = (over != ~0ull ? over : last_upto(INF_KEY)) + 1ull;
      // bisection over the keys themselves: the probe is the first key from
      // the middle on (log2 of the energies inside, some seven probes; over
      // the bits alone the last key is only met after about fifty)
      // (lo < mid <= hi, and mid == hi only when nothing fits between: every
      // step raises lo, lowers hi or ends)
      for (;;) {
        const u64 mid = lo + 1ull + ((hi - lo - 1ull) >> 1);
        const u64 up = first_from(mid);
        if (up < hi) {
          if (ec_feasible<CNT>(x, key, up, B, succB, D))
            lo = up;
          else
            hi = mid;  // (no key in [mid, up))
        } else {
          // nothing from the middle on: down to the last key below it (lo is
          // one: done)
          const u64 dn = last_upto(mid - 1ull);
          if (dn <= lo) break;
          hi = dn + 1ull;
        }
      }
      kt = lo;  // no energy strictly inside, S(lo) <= B < S(hi): lo is an energy's key
    }
    // dropped energy, exactly, and the kept count
    bool drop[CNT];
    u64 kc = 0;
#pragma unroll
    for (int k = 0; k < CNT; ++k) {
      drop[k] = valid[k] && key[k] < kt;
      kc += (valid[k] && !drop[k]) ? 1ull : 0ull;
    }
    w = exact_words<CNT>(x, drop, D);
    tot_add(L.tot[comp][1], w);
    kc = wave_sum_dpp(kc);
    if (lane == 0) {
      atomicAdd((unsigned long long*)&L.kept[comp], (unsigned long long)kc);
      tau_out[p] = __longlong_as_double((long long)kt);
      j.cnt[p] = (u32)kc;
    }
  }
  __syncthreads();
  for (int i = tid; i < j.ncomp * 2 * GD; i += 256) {
    const u64 v = (&L.tot[0][0][0])[i];
    if (v) atomicAdd((unsigned long long*)&G[i], (unsigned long long)v);
  }
  if (tid < j.ncomp && L.kept[tid]) atomicAdd((unsigned long long*)&j.st[tid].kept, (unsigned long long)L.kept[tid]);
}

// Component totals: U2 and the dropped energy rounded from their digits;
// the threshold is per element (NaN here), and the selection is final.
__global__ __launch_bounds__(64) void k_elemfin(Job j, const u64* G) {
  const int comp = blockIdx.x, l = lane_id();
  double v[2];
  for (int k = 0; k < 2; ++k) {
    const u64* T = G + ((size_t)comp * 2 + k) * GD;
    v[k] = wb_round(digits_to_words(T[2 * l], T[2 * l + 1]));
  }
  if (l == 0) {
    CompState* st = j.st + comp;
    st->U2 = v[0];
    st->B = (j.tol * j.tol) * v[0];
    st->tau = __builtin_nan("");
    st->dropped = v[1];
    st->resolved = 1;
    st->bstar = -1;
    // bound on the error terms of pass B, as for the global cut
    int m = st->B > 0.0 ? ilogb(st->B) + 6 : (v[0] > 0.0 ? ilogb(v[0]) - 80 : XM_MIN);
    st->xm_err = m < XM_MIN ? XM_MIN : (m > XM_MAX ? XM_MAX : m);
  }
}

size_t elemcut_digit_bytes(int ncomp) { return (size_t)ncomp * 2 * GD * sizeof(u64); }

hipError_t launch_elemcut(const Job& j, const double* coef, double* tau, u64* G, const double* scale, int grid,
                          hipStream_t s) {
  ElemScale sc;
  for (int k = 0; k < ISR_MAX_COMP; ++k) sc.s[k] = k < j.ncomp ? scale[k] : 1.0;
  switch (j.order) {
#define EC_CASE(NN)                                                                              \
  case NN:                                                                                       \
    hipLaunchKernelGGL((k_elemsel<NN>), dim3(grid), dim3(256), 0, s, j, coef, tau, G, sc);      \
    break;
    EC_CASE(1) EC_CASE(2) EC_CASE(3) EC_CASE(4) EC_CASE(5) EC_CASE(6) EC_CASE(7) EC_CASE(8)
    EC_CASE(9) EC_CASE(10) EC_CASE(11) EC_CASE(12) EC_CASE(13) EC_CASE(14) EC_CASE(15)
#undef EC_CASE
    default:
      return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_elemfin, dim3(j.ncomp), dim3(64), 0, s, j, (const u64*)G);
  return hipGetLastError();
}

}  // namespace isr
