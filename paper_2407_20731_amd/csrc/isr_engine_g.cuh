// Streaming path of the FP64 orders 8..15 ((N+1)^2 > 64): the passes of
// isr_engine.cuh with a workgroup for a wavefront.  A tile is EPI elements
// (Shape<N>: as many as give 256 threads a pencil each), transformed in place
// in LDS with one pencil per thread and the fixed evaluation order of the
// oracle (forward64, inverse64).
//
// What it replaces, the general passes of isr_passes.cuh, put every norm,
// energy and error term into LDS exponent bins (two LDS atomics a value) and
// found the kept values' places by a ticket and a look-back per tile (one
// contended atomic each).  Here the terms go into the running exact sums, the
// per-element counts are known before pass B, and the next tile's field values
// are in flight while a tile is transformed.  What bounds it: FP64 VALU issue
// (6 n multiplies and additions a value and transform) and the LDS round trips
// between its barriers.
// N = 9, 4,097 elements, 3 components: pass A 185 + 59 (second pass) -> 90 us,
// pass B 577 -> 121 us, the request with its decompression 1,006 -> 377 us.
//
// Rows (n values along i) are n | 1 doubles apart in LDS: for even n the
// pencils along i would otherwise meet in few banks (n = 16: two).  Field
// values are read and the error formed in dense order, f = threadIdx + 256 k,
// so that loads are coalesced and a thread's quadrature weights stay the same
// from tile to tile (in registers, as the energy weights of its pencil).
#pragma once

#include "isr_engine.cuh"

namespace isr {

template <int N>
struct EngG {
  typedef Shape<N> S;
  static constexpr int n = S::n, n2 = S::n2, n3 = S::n3, EPI = S::EPI, W = S::W;
  static constexpr int P = n | 1;            // row pitch
  static constexpr int PL = n * P, PE = n2 * P;  // plane, element
  static constexpr int LDSW = EPI * PE;
  static constexpr int PER = (EPI * n3 + 255) / 256;  // dense values per thread
  static_assert(EPI * n2 <= 256 && EPI * W <= 64 && EPI <= 4, "one pencil per thread, one word per lane");

  static DEV int at(int idx) { return (idx / n) * P + idx % n; }  // LDS place of dense value idx

  // dense values of a tile (zero past its end)
  static DEV void load(const double* __restrict__ src, int count, double (&r)[PER], int tid) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = tid + 256 * k;
      r[k] = idx < count ? __builtin_nontemporal_load(&src[idx]) : 0.0;
    }
  }
  static DEV void store(double* w, const double (&r)[PER], int tid) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = tid + 256 * k;
      if (idx < EPI * n3) w[at(idx)] = r[k];
    }
  }

  // forward of the stored tile; thread (el, q = a, p = b) gets c[r].  Ends with
  // every thread past its LDS reads only after the caller's next barrier.
  static DEV void forward(double* w, const DevTables& t, int el, int a, int b, bool act, double (&c)[n]) {
    double x[n];
    __syncthreads();
    if (act) {
      double* row = w + el * PE + (a * n + b) * P;
      double y[n];
#pragma unroll
      for (int i = 0; i < n; ++i) x[i] = row[i];
      forward64<n>(t.A, x, y);
#pragma unroll
      for (int i = 0; i < n; ++i) row[i] = y[i];
    }
    __syncthreads();
    if (act) {
      double* col = w + el * PE + a * PL + b;
      double y[n];
#pragma unroll
      for (int k = 0; k < n; ++k) x[k] = col[k * P];
      forward64<n>(t.A, x, y);
#pragma unroll
      for (int k = 0; k < n; ++k) col[k * P] = y[k];
    }
    __syncthreads();
    if (act) {
      const double* col = w + el * PE + a * P + b;
#pragma unroll
      for (int k = 0; k < n; ++k) x[k] = col[k * PL];
      forward64<n>(t.A, x, c);
    }
  }
  // inverse of the coefficients cm of thread (el, a, b); the field is left in
  // LDS (after the caller's next barrier).  Begins with a barrier.
  static DEV void inverse(double* w, const DevTables& t, int el, int a, int b, bool act, const double (&cm)[n]) {
    double x[n];
    __syncthreads();
    if (act) {
      double y[n];
      inverse64<n>(t.V, cm, y);
      double* col = w + el * PE + a * P + b;
#pragma unroll
      for (int k = 0; k < n; ++k) col[k * PL] = y[k];
    }
    __syncthreads();
    if (act) {
      double* col = w + el * PE + a * PL + b;
      double y[n];
#pragma unroll
      for (int k = 0; k < n; ++k) x[k] = col[k * P];
      inverse64<n>(t.V, x, y);
#pragma unroll
      for (int k = 0; k < n; ++k) col[k * P] = y[k];
    }
    __syncthreads();
    if (act) {
      double* row = w + el * PE + (a * n + b) * P;
      double y[n];
#pragma unroll
      for (int i = 0; i < n; ++i) x[i] = row[i];
      inverse64<n>(t.V, x, y);
#pragma unroll
      for (int i = 0; i < n; ++i) row[i] = y[i];
    }
  }
};

// Workgroups per CU the passes are compiled for: three up to order 12 (168
// VGPRs; at N = 10 and 12 pass B spills about 30 of them and still takes 116 and
// 160 us, against 117..121 and 163..168 us with two), two above (75 spills and
// more with three).
template <int N>
constexpr int wide_minb() {
  return N <= 12 ? 3 : 2;
}

// this thread's weights: w3 of its dense values, g3 of its pencil's coefficients
template <class G>
DEV void g_weights(const DevTables& t, double (&w3)[G::PER], double (&g3)[G::n], int tid, int a, int b) {
#pragma unroll
  for (int k = 0; k < G::PER; ++k) {
    const int idx = tid + 256 * k;
    w3[k] = idx < G::EPI * G::n3 ? t.w3[idx % G::n3] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < G::n; ++r) g3[r] = t.g3[(r * G::n + a) * G::n + b];
}

// ---- sample pass --------------------------------------------------------------
template <int N>
struct SampleLdsG {
  double w[EngG<N>::LDSW];
  float hs[SBINS];  // sums of energy / 2^(bin exponent), each term in [1, 2)
  double u2[4];
  int maxe;
};

template <int N>
__global__ __launch_bounds__(256, 2) void k_sampleG(Job j) {
  typedef EngG<N> G;
  constexpr int n = G::n, n2 = G::n2, n3 = G::n3, EPI = G::EPI, PER = G::PER;
  __shared__ SampleLdsG<N> L;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, comp = blockIdx.y;
  const int el = tid / n2, a = (tid % n2) / n, b = tid % n;
  CompState* st = j.st + comp;
  for (int k = tid; k < SBINS; k += 256) L.hs[k] = 0.0f;
  if (tid == 0) L.maxe = 0;
  const long long E = j.n_elem, tiles = (E + EPI - 1) / EPI;
  const long long ss = j.sample_stride > 0 ? j.sample_stride : 1, stiles = (tiles + ss - 1) / ss;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  double w3[PER], g3[n];
  g_weights<G>(j.tab, w3, g3, tid, a, b);
  double u2 = 0.0;
  int maxe = 0;
  for (long long k0 = blockIdx.x; k0 < stiles; k0 += gridDim.x) {
    const long long e0 = k0 * ss * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    const bool act = tid < EPI * n2 && el < ne;
    double u[PER], c[n];
    G::load(ub + e0 * n3, ne * n3, u, tid);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = tid + 256 * k;
      if (idx >= ne * n3) continue;
      const double x = jw(j.jac, e0 + idx / n3, w3[k]) * (u[k] * u[k]);
      u2 += x;
      const int ex = bits_exp(dbits(x));
      maxe = ex > maxe ? ex : maxe;
    }
    __syncthreads();
    G::store(L.w, u, tid);
    G::forward(L.w, j.tab, el, a, b, act, c);
    const double je = j.jac && act ? j.jac[e0 + el] : 1.0;
    // energies first, then their atomics: none of these waits for the next
    // (rounded sums only place the window)
    int eb[n];
    float em[n];
#pragma unroll
    for (int r = 0; r < n; ++r) {
      const double en = act ? (je * g3[r]) * (c[r] * c[r]) : 0.0;
      eb[r] = bits_exp(dbits(en));
      em[r] = eb[r] < HBINS - 1 ? (float)ldexp(en, 1023 - eb[r]) : 0.0f;
    }
#pragma unroll
    for (int r = 0; r < n; ++r)
      if (em[r] != 0.0f) atomicAdd(&L.hs[eb[r]], em[r]);
  }
  u2 = wave_sum_f64(u2);
  for (int m = 32; m > 0; m >>= 1) {
    const int o = __shfl_xor(maxe, m);
    maxe = o > maxe ? o : maxe;
  }
  __syncthreads();
  if (lane == 0) {
    L.u2[wv] = u2;
    atomicMax(&L.maxe, maxe);
  }
  __syncthreads();
  HistBin* H = j.histEs + (size_t)comp * HBINS;
  for (int k = tid; k < SBINS; k += 256)
    if (L.hs[k] != 0.0f) atomicAdd((double*)&H[k].lo, ldexp((double)L.hs[k], k - 1023));
  if (tid == 0) {
    atomicAdd(&st->samp_u2, L.u2[0] + L.u2[1] + L.u2[2] + L.u2[3]);
    atomicMax(&st->samp_maxe, L.maxe);
  }
}

// slots of terms out of the running sums' range that are staged at a time
constexpr int XF_CH = 8;

// ---- pass A -------------------------------------------------------------------
template <int N>
struct PassALdsG {
  double w[EngG<N>::LDSW];
  u64 key[4][CAPB];
  u32 idx[4][CAPB];
  u32 ecnt[4];
  XFar far[2];  // norm terms, energies
  double stage[4][64 * XF_CH];
  long long red[4][8];
};

// Whether the sample has left a component without a window (all sampled energies
// zero, or all within the budget): the request then goes to the general pipeline
// as a whole, and no component's pass is worth its time (N = 8, 5,753 elements, one of
// 3 components all zero: 1054 -> 925 us; 89 elements: 302 -> 253).
DEV bool no_window(const Job& j) {
  if (j.tol < 0.0) return false;
  for (int c = 0; c < j.ncomp; ++c)
    if (j.st[c].win_lo >= j.st[c].win_hi) return true;
  return false;
}

template <int N>
__global__ __launch_bounds__(256, wide_minb<N>()) void k_passAG(Job j) {
  typedef EngG<N> G;
  constexpr int n = G::n, n2 = G::n2, n3 = G::n3, EPI = G::EPI, PER = G::PER;
  __shared__ PassALdsG<N> L;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, comp = blockIdx.y;
  const int el = tid / n2, a = (tid % n2) / n, b = tid % n;
  CompState* st = j.st + comp;
  if (no_window(j)) {
    if (blockIdx.x == 0 && tid == 0) {
      atomicOr(&st->flags, ST_MISS);
      st->resolved = 1;
    }
    return;
  }
  const int wlo = st->win_lo, whi = st->win_hi;
  const XParm PN = xparm(st->xm_norm, j.xh);
  const XParm PE = xparm(wlo - 1023, j.xh);
  const u32 hwlo = (u32)wlo << 20, hwhi = (u32)whi << 20;
  const XRange RN = xrange(PN);
  XRange RE = xrange(PE);
  RE.lo = RE.lo < hwlo ? RE.lo : hwlo;  // (without a window, wlo = 0, nothing is below it)
  HistBin* gN = j.histN + (size_t)comp * HBINS;
  HistBin* gE = j.histE + (size_t)comp * HBINS;
  u64* list = list_ptr(j, comp, 0);
  u32* lidx = j.lidx + (size_t)comp * j.list_cap;
  const long long E = j.n_elem, tiles = (E + EPI - 1) / EPI;
  u32* cnt = j.cnt + (size_t)comp * E;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  double w3[PER], g3[n];
  g_weights<G>(j.tab, w3, g3, tid, a, b);
  XRun rn = xrun(PN), re = xrun(PE);
  u64 hi_tot = 0ull;
  u32 ncap = 0u;
  double u[PER];
  if (tid < 4) L.ecnt[tid] = 0u;
  xfar_clear(L.far[0], tid);
  xfar_clear(L.far[1], tid);
  __syncthreads();
  long long t = blockIdx.x;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPI;
    G::load(ub + e0 * n3, (int)((E - e0) < EPI ? (E - e0) : EPI) * n3, u, tid);
  };
  if (t < tiles) fetch(t);
  for (; t < tiles; t += gridDim.x) {
    const long long e0 = t * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    const bool act = tid < EPI * n2 && el < ne;
    int dt = tid;  // (per-tile copy: the indexes made from it are not kept across tiles)
    asm volatile("" : "+v"(dt));
    // norm terms of the dense values
    u64 odd = 0ull;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = dt + 256 * k;
      const bool v = idx < ne * n3;
      const double x = v ? jw(j.jac, e0 + idx / n3, w3[k]) * (u[k] * u[k]) : 0.0;
      odd |= __builtin_amdgcn_ballot_w64(xrun_left(rn, RN, x) && v);
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(rn);
    if (odd) {
      double xn[PER];
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int idx = dt + 256 * k;
        xn[k] = idx < ne * n3 ? jw(j.jac, e0 + idx / n3, w3[k]) * (u[k] * u[k]) : 0.0;
      }
      xfar_tile<64, XF_CH, true>(L.far[0], xfar_m(PN.m, j.xh), gN, L.stage, xn, [&](double x) { return !xin(RN, x); });
    }
    odd = 0ull;
    G::store(L.w, u, dt);
    if (t + gridDim.x < tiles) fetch(t + gridDim.x);
    double c[n];
    G::forward(L.w, j.tab, el, a, b, act, c);
    u32 hmine = 0u, hmax = 0u;
    const double je = j.jac && act ? j.jac[e0 + el] : 1.0;  // (1.0 * g3 is g3)
#pragma unroll
    for (int r = 0; r < n; ++r) {
      const double en = act ? (je * g3[r]) * (c[r] * c[r]) : 0.0;
      const u32 hw = hi_word(en);
      const bool hi = act && hw >= hwhi;
      const bool cp = act && hw < hwhi && hw >= hwlo;
      hmax = hw > hmax ? hw : hmax;
      hmine += hi ? 1u : 0u;
      const u64 bc = ballot(cp);
      if (bc) {
        if (cp) {
          const u32 pos = ncap + lane_rank(bc);
          L.key[wv][pos] = dbits(en);
          L.idx[wv][pos] = (u32)(e0 + el);
        }
        ncap += (u32)__popcll(bc);
        if (ncap > (u32)(CAPB - 64)) {
          asm volatile("" ::: "memory");
          cap_flush(L.key[wv], L.idx[wv], ncap, st, list, lidx, j.list_cap, lane);
        }
      }
      const bool tiny = hw < RE.lo;
      xrun_add(re, hw < hwlo && !tiny ? en : 0.0);
      odd |= __builtin_amdgcn_ballot_w64(tiny && act);
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(re);
    if (odd) {
      double xe[n];
#pragma unroll
      for (int r = 0; r < n; ++r) xe[r] = act ? (je * g3[r]) * (c[r] * c[r]) : 0.0;
      xfar_tile<64, XF_CH, true>(L.far[1], xfar_m(PE.m, j.xh), gE, L.stage, xe, [&](double x) { return hi_word(x) < RE.lo; });
    }
    if (hmax >= 0x7ff00000u) slow_bin(gE, __builtin_inf());  // Inf/NaN: counted in the flag bin
    hi_tot += hmine;
    if (hmine) atomicAdd(&L.ecnt[el], hmine);
    __syncthreads();  // counts are whole, and the tile is no longer read
    if (tid < ne) {
      cnt[e0 + tid] = L.ecnt[tid];
      L.ecnt[tid] = 0u;
    }
  }
  asm volatile("" ::: "memory");
  cap_flush(L.key[wv], L.idx[wv], ncap, st, list, lidx, j.list_cap, lane);
  const XParm QN = xparm(again(PN.m), j.xh);
  const XParm QE = xparm(again(PE.m), j.xh);
  long long v[7], kn[3], ke[3];
  xints(xrun_sums(rn, QN), QN, kn);
  xints(xrun_sums(re, QE), QE, ke);
  v[0] = kn[0];
  v[1] = kn[1];
  v[2] = kn[2];
  v[3] = ke[0];
  v[4] = ke[1];
  v[5] = ke[2];
  v[6] = (long long)hi_tot;
  block_sum_i64<7>(v, L.red, tid);
  if (tid < 7) j.slotsA[((size_t)comp * j.gA + blockIdx.x) * 8 + tid] = L.red[0][tid];
  xfar_out(L.far[0], gN, tid);
  if (wlo < whi) xfar_out(L.far[1], gE, tid - 64);
}

// ---- pass B -------------------------------------------------------------------
template <int N>
struct PassBLdsG {
  double w[EngG<N>::LDSW];
  u64 bm[64];  // the tile's bitmap words
  u32 wp[64];  // kept values before each word
  XFar far;  // error terms
  double stage[4][64 * XF_CH];
  long long red[4][8];
};

template <int N>
__global__ __launch_bounds__(256, wide_minb<N>()) void k_passBG(Job j) {
  typedef EngG<N> G;
  constexpr int n = G::n, n2 = G::n2, n3 = G::n3, EPI = G::EPI, PER = G::PER, W = G::W;
  __shared__ PassBLdsG<N> L;
  const int tid = threadIdx.x, lane = tid & 63, comp = blockIdx.y;
  const int el = tid / n2, a = (tid % n2) / n, b = tid % n;
  CompState* st = j.st + comp;
  if (st->flags & ST_MISS) return;
  const XParm PR = xparm(st->xm_err, j.xh);
  const XRange RR = xrange(PR);
  HistBin* gR = j.histR + (size_t)comp * HBINS;
  const double tau_c = st->tau;
  const double* te = j.tau_elem ? j.tau_elem + (size_t)comp * j.n_elem : nullptr;
  u64 voff = 0ull;
  for (int cc = 0; cc < comp; ++cc) voff += j.st[cc].kept;
  const u64 vcap = (u64)j.ncomp * (u64)j.n_elem * (u64)n3;
  const long long E = j.n_elem, tiles = (E + EPI - 1) / EPI;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  u64* gbm = j.bitmap + (size_t)comp * E * W;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  double w3[PER], g3[n];
  g_weights<G>(j.tab, w3, g3, tid, a, b);
  XRun rr = xrun(PR);
  bool bad = false;
  if (tid < 64) L.bm[tid] = 0ull;
  xfar_clear(L.far, tid);  // (before the first tile's first barrier)
  double un[PER];
  long long t = blockIdx.x;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPI;
    G::load(ub + e0 * n3, (int)((E - e0) < EPI ? (E - e0) : EPI) * n3, un, tid);
  };
  if (t < tiles) fetch(t);
  for (; t < tiles; t += gridDim.x) {
    const long long e0 = t * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    const bool act = tid < EPI * n2 && el < ne;
    // (per-tile copies: the compiler would keep every index and mask made from
    // these in registers across tiles)
    int ab = a * n + b, dt = tid;
    asm volatile("" : "+v"(ab), "+v"(dt));
    double c[n];
    __syncthreads();  // (the tile before is no longer read)
    G::store(L.w, un, tid);
    G::forward(L.w, j.tab, el, a, b, act, c);
    if (t + gridDim.x < tiles) fetch(t + gridDim.x);
    const double je = j.jac && act ? j.jac[e0 + el] : 1.0;
    const double tau = te && act ? te[e0 + el] : tau_c;
    const u64 vbase = voff + eptr[e0];
    u32 keep = 0u;
#pragma unroll
    for (int r = 0; r < n; ++r) {
      const double en = (je * g3[r]) * (c[r] * c[r]);
      if (act && !(en < tau)) {  // (a NaN is kept: pass A counts it among the energies above)
        keep |= 1u << r;
        const int f = r * n2 + ab;
        atomicOr((unsigned long long*)&L.bm[el * W + (f >> 6)], 1ull << (f & 63));
      }
    }
    __syncthreads();
    // words out, and the kept values before each of the tile's words (they
    // follow each other in the blob across its elements)
    if (tid < 64) {
      const u64 wd = L.bm[lane];
      const u32 pc = (u32)__popcll(wd);
      u32 incl = pc;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const u32 o = (u32)__shfl_up((int)incl, d);
        incl += lane >= d ? o : 0u;
      }
      L.wp[lane] = incl - pc;
      if (lane < ne * W) gbm[e0 * W + lane] = wd;
      // each element's count against its offsets, and the tile's against the
      // room for values: never written past
      if (lane < ne * W && lane % W == W - 1 && voff + eptr[e0 + lane / W + 1] - vbase != (u64)incl) bad = true;
    }
    __syncthreads();
    const u32 tot = L.wp[EPI * W - 1] + (u32)__popcll(L.bm[EPI * W - 1]);
    const bool fits = vbase <= vcap && (u64)tot <= vcap - vbase;
    if (!fits) bad = true;
    if (keep && fits) {
      double* dst = (double*)j.values + vbase;
#pragma unroll
      for (int r = 0; r < n; ++r) {
        if (!((keep >> r) & 1u)) continue;
        const int f = r * n2 + ab, wi = el * W + (f >> 6);
        dst[L.wp[wi] + (u32)__popcll(L.bm[wi] & ((1ull << (f & 63)) - 1ull))] = c[r];
      }
    }
#pragma unroll
    for (int r = 0; r < n; ++r) c[r] = (keep >> r) & 1u ? c[r] : 0.0;
    G::inverse(L.w, j.tab, el, a, b, act, c);
    if (tid < 64) L.bm[tid] = 0ull;  // (read before the inverse's first barrier, set again after the next tile's)
    double u[PER];
    G::load(ub + e0 * n3, ne * n3, u, tid);
    __syncthreads();
    // error terms of the dense values
    u64 odd = 0ull;
    double xs[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = dt + 256 * k;
      const bool v = idx < ne * n3;
      const double d = v ? u[k] - L.w[G::at(idx)] : 0.0;
      const double x = v ? jw(j.jac, e0 + idx / n3, w3[k]) * (d * d) : 0.0;
      xs[k] = x;
      odd |= __builtin_amdgcn_ballot_w64(xrun_left(rr, RR, x) && v);
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(rr);
    if (odd)
      xfar_tile<64, XF_CH, true>(L.far, xfar_m(PR.m, j.xh), gR, L.stage, xs, [&](double x) { return !xin(RR, x); });
  }
  if (ballot(bad)) {
    if (lane == 0) atomicOr(&st->flags, ST_LIST);
  }
  const XParm QR = xparm(again(PR.m), j.xh);
  long long v[3];
  xints(xrun_sums(rr, QR), QR, v);
  block_sum_i64<3>(v, L.red, tid);
  if (tid < 3) j.slotsB[((size_t)comp * j.gB + blockIdx.x) * 4 + tid] = L.red[0][tid];
  xfar_out(L.far, gR, tid);
}

// ---- reading kept values back ----------------------------------------------------
// Kept coefficients of thread (el, a, b) of a tile whose bitmap words are in
// L.bm, with L.wp kept values before each (wave 0 puts them there): calls
// fn(place, r, index) for each kept one, zero for the others.  base: the place
// of its element's first value.
template <class G, class LDS>
DEV void g_words(LDS& L, u64 wcur, int tid) {
  if (tid >= 64) return;
  const u32 pc = (u32)__popcll(wcur);
  u32 incl = pc;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const u32 o = (u32)__shfl_up((int)incl, d);
    incl += tid >= d ? o : 0u;
  }
  L.bm[tid] = wcur;
  L.wp[tid] = incl - pc;
}
template <class G, class LDS, class FN>
DEV void g_kept(double (&cm)[G::n], const LDS& L, u64 base, int el, int a, int b, bool act, FN fn) {
  constexpr int n = G::n, W = G::W;
  const u32 p0 = act ? L.wp[el * W] : 0u;
#pragma unroll
  for (int r = 0; r < n; ++r) {
    cm[r] = 0.0;
    const int f = (r * n + a) * n + b, wi = el * W + (f >> 6);
    const u64 wd = act ? L.bm[wi] : 0ull;
    if ((wd >> (f & 63)) & 1ull)
      cm[r] = fn(base + (L.wp[wi] - p0 + (u32)__popcll(wd & ((1ull << (f & 63)) - 1ull))), r, f);
  }
}

// ---- decompress ------------------------------------------------------------------
// Blobs of FP64 values and quantisation codes.  A tile's words and offsets are
// in flight while the one before is inverted; the field leaves from LDS in
// dense order in non-temporal stores (what it replaces stored a row of n a
// lane).  Bound by the inverse as pass B is, less its forward.  N = 9, 4,097
// elements, 3 components, FP64: 71 -> 53 us.
template <int N>
struct WordLdsG {
  double w[EngG<N>::LDSW];
  u64 bm[64];  // the tile's bitmap words
  u32 wp[64];  // kept values before each word
};

template <int N, bool OUT64>
__global__ __launch_bounds__(256, 2) void k_decompG(Job j, void* out) {
  typedef EngG<N> G;
  constexpr int n = G::n, n2 = G::n2, n3 = G::n3, EPI = G::EPI, PER = G::PER, W = G::W;
  typedef typename Pick<OUT64, double, float>::type ot;
  __shared__ WordLdsG<N> L;
  const int tid = threadIdx.x, comp = blockIdx.y;
  const int el = tid / n2, a = (tid % n2) / n, b = tid % n;
  const long long E = j.n_elem, tiles = (E + EPI - 1) / EPI;
  const u64* gbm = j.bitmap + (size_t)comp * E * W;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  const u64 voff = j.voff[comp];
  const double qs = j.qstep ? j.qstep[comp] : 0.0;
  ot* ocomp = (ot*)out + (size_t)comp * E * n3;
  u64 wnext = 0ull, bnext = 0ull;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    wnext = tid < 64 && tid < ne * W ? gbm[e0 * W + tid] : 0ull;
    bnext = el < ne ? eptr[e0 + el] : 0ull;
  };
  long long t = blockIdx.x;
  if (t < tiles) fetch(t);
  for (; t < tiles; t += gridDim.x) {
    const long long e0 = t * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    const bool act = tid < EPI * n2 && el < ne;
    g_words<G>(L, wnext, tid);
    const u64 base = voff + bnext;
    if (t + gridDim.x < tiles) fetch(t + gridDim.x);
    __syncthreads();
    double cm[n];
    g_kept<G>(cm, L, base, el, a, b, act, [&](u64 pos, int, int f) -> double {
      if (j.vbytes == 8) return ((const double*)j.values)[pos];
      // quantisation codes: the value is (code * step) / sqrt(g3)
      return ((double)((const float*)j.values)[pos] * qs) / __builtin_sqrt(j.tab.g3[f]);
    });
    G::inverse(L.w, j.tab, el, a, b, act, cm);
    __syncthreads();
    ot* o = ocomp + e0 * n3;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = tid + 256 * k;
      if (idx < ne * n3) __builtin_nontemporal_store((ot)L.w[G::at(idx)], &o[idx]);
    }
  }
}

// ---- quantised variant ------------------------------------------------------------
// The codes of the kept values and the error they leave, as k_quantW
// (isr_engine.cuh) does for the smaller orders.  N = 9, 3,333 elements, 3
// components: 266 -> 71 us.
template <int N>
struct QuantLdsG : WordLdsG<N> {
  XFar far;  // error terms
  double stage[4][64 * XF_CH];
  long long red[4][8];
};

template <int N>
__global__ __launch_bounds__(256, 2) void k_quantG(Job j) {
  typedef EngG<N> G;
  constexpr int n = G::n, n2 = G::n2, n3 = G::n3, EPI = G::EPI, PER = G::PER, W = G::W;
  __shared__ QuantLdsG<N> L;
  const int tid = threadIdx.x, comp = blockIdx.y;
  const int el = tid / n2, a = (tid % n2) / n, b = tid % n;
  const long long E = j.n_elem, tiles = (E + EPI - 1) / EPI;
  const u64* gbm = j.bitmap + (size_t)comp * E * W;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  const u64 voff = j.voff[comp];
  const double step = j.qstep[comp];
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  const XParm PR = xparm(j.qxm[comp], j.xh);
  const XRange RR = xrange(PR);
  XRun rr = xrun(PR);
  HistBin* gR = j.histR + (size_t)comp * HBINS;
  double w3[PER], sq[n];
  g_weights<G>(j.tab, w3, sq, tid, a, b);
#pragma unroll
  for (int r = 0; r < n; ++r) sq[r] = __builtin_sqrt(sq[r]);
  xfar_clear(L.far, tid);  // (before the first tile's first barrier)
  bool big = false;
  u64 wnext = 0ull, bnext = 0ull;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    wnext = tid < 64 && tid < ne * W ? gbm[e0 * W + tid] : 0ull;
    bnext = el < ne ? eptr[e0 + el] : 0ull;
  };
  long long t = blockIdx.x;
  if (t < tiles) fetch(t);
  for (; t < tiles; t += gridDim.x) {
    const long long e0 = t * EPI;
    const int ne = (int)((E - e0) < EPI ? (E - e0) : EPI);
    const bool act = tid < EPI * n2 && el < ne;
    double u[PER];
    G::load(ub + e0 * n3, ne * n3, u, tid);
    g_words<G>(L, wnext, tid);
    const u64 base = voff + bnext;
    if (t + gridDim.x < tiles) fetch(t + gridDim.x);
    __syncthreads();
    double cm[n];
    g_kept<G>(cm, L, base, el, a, b, act, [&](u64 pos, int r, int) -> double {
      const double c = ((const double*)j.values)[pos];
      const double q = __builtin_rint((c * sq[r]) / step);
      if (!(__builtin_fabs(q) < 16777216.0)) big = true;
      j.qvals[pos] = (float)q;
      return (q * step) / sq[r];
    });
    G::inverse(L.w, j.tab, el, a, b, act, cm);
    __syncthreads();
    u64 odd = 0ull;
    double xs[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = tid + 256 * k;
      const bool v = idx < ne * n3;
      const double d = v ? u[k] - L.w[G::at(idx)] : 0.0;
      xs[k] = w3[k] * (d * d);
      odd |= __builtin_amdgcn_ballot_w64(xrun_left(rr, RR, xs[k]) && v);
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(rr);
    if (odd)
      xfar_tile<64, XF_CH, true>(L.far, xfar_m(PR.m, j.xh), gR, L.stage, xs, [&](double x) { return !xin(RR, x); });
  }
  if (big) atomicOr(&j.ticket[1], 1u);
  const XParm QR = xparm(again(PR.m), j.xh);
  long long v[3];
  xints(xrun_sums(rr, QR), QR, v);
  block_sum_i64<3>(v, L.red, tid);
  if (tid < 3) j.slotsB[((size_t)comp * j.gB + blockIdx.x) * 4 + tid] = L.red[0][tid];
  xfar_out(L.far, gR, tid);
}

// ---- launchers ------------------------------------------------------------------
#define ISR_FAST_ORDERS_G(X) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)

inline hipError_t launch_fast_g(int kind, const Job& j, int gx, hipStream_t s) {
  const dim3 grid(gx, j.ncomp), blk(256);
  switch (j.order) {
#define CASE(NN)                                                 \
  case NN:                                                       \
    if (kind == F_SAMPLE)                                        \
      hipLaunchKernelGGL((k_sampleG<NN>), grid, blk, 0, s, j);   \
    else if (kind == F_PASSA)                                    \
      hipLaunchKernelGGL((k_passAG<NN>), grid, blk, 0, s, j);    \
    else if (kind == F_PASSB)                                    \
      hipLaunchKernelGGL((k_passBG<NN>), grid, blk, 0, s, j);    \
    else                                                         \
      return hipErrorInvalidValue;                               \
    break;
    ISR_FAST_ORDERS_G(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

inline hipError_t launch_decomp_g(const Job& j, int gx, int cus, hipStream_t s, void* out, int out_fp64) {
  switch (j.order) {
#define CASE(NN)                                                                                      \
  case NN: {                                                                                          \
    static const int nb = resident_wgs((const void*)k_decompG<NN, true>),                             \
                     nb32 = resident_wgs((const void*)k_decompG<NN, false>);                          \
    if (out_fp64)                                                                                     \
      hipLaunchKernelGGL((k_decompG<NN, true>), decomp_grid(j, gx, nb, cus), dim3(256), 0, s, j, out); \
    else                                                                                              \
      hipLaunchKernelGGL((k_decompG<NN, false>), decomp_grid(j, gx, nb32, cus), dim3(256), 0, s, j, out); \
    break;                                                                                            \
  }
    ISR_FAST_ORDERS_G(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

inline hipError_t launch_quant_g(const Job& j, hipStream_t s) {
  switch (j.order) {
#define CASE(NN)                                                                  \
  case NN:                                                                        \
    hipLaunchKernelGGL((k_quantG<NN>), dim3(j.gB, j.ncomp), dim3(256), 0, s, j);  \
    break;
    ISR_FAST_ORDERS_G(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

inline int resident_fast_g(int kind, int order) {
  switch (order) {
#define CASE(NN)                                                                                        \
  case NN:                                                                                              \
    return resident_wgs(kind == F_SAMPLE  ? (const void*)k_sampleG<NN>                                  \
                        : kind == F_PASSA ? (const void*)k_passAG<NN>                                   \
                        : kind == F_QUANT ? (const void*)k_quantG<NN>                                   \
                                          : (const void*)k_passBG<NN>);
    ISR_FAST_ORDERS_G(CASE)
#undef CASE
    default:
      return 1;
  }
}

}  // namespace isr
