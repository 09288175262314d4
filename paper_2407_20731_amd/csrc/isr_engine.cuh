// Streaming path for orders 1..7 ((N+1)^2 <= 64): one wavefront owns a tile
// of EPW = 64 / (N+1)^2 elements and runs its whole transform chain on its
// own, with no workgroup barriers.
//
//   k_sample  every sample_stride-th tile: rounded exponent histogram of the
//             energies and rounded U2, which place a window of three energy
//             exponent bins around the expected threshold
//   k_passA   exact norm sum, sum of the energies below the window, window
//             energies (with their element) to list 0, per-element count of
//             energies above the window
//   k_passB   keep e >= tau, bitmaps, kept values at per-element offsets
//             (known up front: no look-back), inverse of the kept set, error
//             sum; the last workgroup of a component finalizes it
//
// Exact sums without atomics (isr_xsum.cuh): a non-negative term x <= M is split
// into three parts on fixed grids by error-free extraction (Rump, Ogita and
// Oishi, "Accurate floating-point summation part I", SIAM J. Sci. Comput. 31(1),
// 2008, Alg. 3.2), added to three FP64 sums that stay exact.  On the FP64 path
// every norm, energy and error term is split, against running sums biased to the
// middle of a binade; a tile's terms far below M are summed in the same manner
// against bounds of their own into digits in LDS, and only a term above M goes to
// the global exponent bins.  The MFMA paths, whose energies already carry the
// transform error, add terms in a fixed order per lane (one FP64 add a term) and
// split each lane's total against fixed powers of two, so that their results stay
// deterministic.  Workgroups publish their three integer sums; the consumer turns
// the totals into exact bins.
//
// Transforms on MFMA use a block-diagonal trick for n <= 8: a 16x16 tile
// holds two 8x8 copies of the 1D matrix, the K dimension pairs the contracted
// index of two sets of 16 pencils, so the 64 lanes of every output register
// hold 64 valid (pencil, index) pairs.  Lane l = 16 g + P of block b holds
// pencil 32 b + 16 (g >> 1) + P and indices 4 (g & 1) + m, m = 0..3, in
// four registers, for the input and for the output of every stage alike.
// Between stages the tile is transposed through a per-wave LDS buffer.
// The FP64 path keeps one pencil per lane and the fixed evaluation order of
// the oracle (forward64, inverse64).
#pragma once

#include "isr_passes.cuh"
#include "isr_fastsel.cuh"
#include "isr_selbody.cuh"
#include "isr_xsum.cuh"

// Minimum resident workgroups per CU the streaming passes are compiled for
// (bounds their registers: 4 -> 128 VGPRs, 3 -> 168, 2 -> 256).  FP64 four: the
// table entries sit in scalar registers, so the passes fit 128 (with three or two
// both take 1 to 3 % longer at N = 7, and as long at the other orders; pass B of N = 5
// with two, 9,710 elements, 69 us for 61).  But pass B of N = 6 three: with four it
// spills 37 registers (6,115 elements, 3 components: the request 291 us for 276).
// MFMA paths three.
#ifndef ISR_FAST_MINB_F64
#define ISR_FAST_MINB_F64 4
#endif
#ifndef ISR_FAST_MINB_MIX
#define ISR_FAST_MINB_MIX 3
#endif
#define ISR_FAST_MINB (PREC == P_FP64 ? ISR_FAST_MINB_F64 : ISR_FAST_MINB_MIX)

namespace isr {

template <int N, int PREC>
constexpr int fast_minb_b() {
  return PREC == P_FP64 && N != 6 ? ISR_FAST_MINB_F64 : 3;
}

template <bool C, class A, class B>
struct Pick {
  typedef A type;
};
template <class A, class B>
struct Pick<false, A, B> {
  typedef B type;
};

// ---- the wave-tile engine --------------------------------------------------------
template <int N, int PREC>
struct Eng {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  static_assert(n >= 2 && n <= 8, "streaming engine covers orders 1..7");
  static constexpr bool MF = PREC != P_FP64;
  static constexpr int EPW = 64 / n2;      // elements per tile
  static constexpr int PT = EPW * n2;      // pencils per tile (<= 64)
  static constexpr int NB = MF ? 2 : 1;    // pencil blocks (32 pencils each on MFMA)
  static constexpr int SPB = MF ? 4 : n;   // registers per block
  static constexpr int NS = NB * SPB;      // slots per lane
  static_assert(NS <= 8, "slot tables hold 8 slots");
  static constexpr int P0 = n + 1;         // LDS row pitch
  static constexpr int LDSW = EPW * n * n * P0;
  static constexpr int W = (n3 + 63) / 64;  // bitmap words per element
  typedef typename Pick<MF, float, double>::type wt;

  struct Mats {
    float fa[4], fv[4];  // FP32 A-operand fragments (forward A, inverse V)
    s4 ha, la, hv, lv;   // BF16 hi / lo fragments
  };

  DEV static int pencil(int s, int lane) { return MF ? 32 * (s >> 2) + 16 * (lane >> 5) + (lane & 15) : lane; }
  DEV static int axis(int s, int lane) { return MF ? 4 * ((lane >> 4) & 1) + (s & 3) : s; }
  DEV static bool pvalid(int s, int lane) { return pencil(s, lane) < PT && axis(s, lane) < n; }
  DEV static bool valid(int s, int lane, int ne) { return pencil(s, lane) < ne * n2 && axis(s, lane) < n; }
  DEV static int elem(int s, int lane) { return pencil(s, lane) / n2; }

  static DEV void frag(float (&f)[4], s4& h, s4& l, const float* M, int lane) {
    const int row = lane & 15, g = lane >> 4;
    const bool same = (row >> 3) == (g >> 1);
    const int b = row & 7;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 4 * (g & 1) + v;
      const float m = (same && b < n && a < n) ? M[b * n + a] : 0.0f;
      f[v] = m;
      const short hi = to_bf16(m);
      h[v] = hi;
      l[v] = to_bf16(m - from_bf16(hi));
    }
  }
  static DEV void init(Mats& mt, const DevTables& t, int lane) {
    if constexpr (MF) {
      frag(mt.fa, mt.ha, mt.la, t.A32, lane);
      frag(mt.fv, mt.hv, mt.lv, t.V32, lane);
    }
  }

  // FP64 field tile -> slots (zero outside the tile).
  static DEV void load(const double* __restrict__ tile, int ne, bool vec, double (&u)[NS], int lane) {
    const int pv = ne * n2;
    if (n == 8 && vec) {
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) {
        const int PI = pencil(blk * SPB, lane);
        const int a0 = axis(blk * SPB, lane);
#pragma unroll
        for (int h = 0; h < SPB / 2; ++h) {
          d2 v = {0.0, 0.0};
          if (PI < pv) v = __builtin_nontemporal_load((const d2*)(tile + PI * n + a0 + 2 * h));
          u[blk * SPB + 2 * h] = v.x;
          u[blk * SPB + 2 * h + 1] = v.y;
        }
      }
      return;
    }
    if constexpr (!MF) {
      // lanes past the tile read its last pencil (their values are never used): a
      // zero written beside a load in flight has waited for it (N = 5, 50,001
      // elements, 3 components: pass B 322 us, 285 so)
      const double* p = tile + (lane < pv ? lane : pv - 1) * n;
#pragma unroll
      for (int s = 0; s < NS; ++s) u[s] = __builtin_nontemporal_load(p + s);
      return;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int PI = pencil(s, lane), ax = axis(s, lane);
      u[s] = (PI < pv && ax < n) ? __builtin_nontemporal_load(tile + PI * n + ax) : 0.0;
    }
  }

  // Jacobians of this lane's slots (zero outside the tile): one value on the
  // FP64 path and at n = 8 (a lane's pencils lie in one element there), else
  // one a slot
  static constexpr int JS = !MF || n == 8 ? 1 : NS;
  static DEV void load_jac(const double* __restrict__ jac, int ne, double (&jq)[JS], int lane) {
#pragma unroll
    for (int s = 0; s < JS; ++s) jq[s] = valid(s, lane, ne) ? jac[elem(s, lane)] : 0.0;
  }

  // One contraction on every pencil of the tile.
  static DEV void stage_mf(const wt (&x)[NS], wt (&y)[NS], const float (&f)[4], s4 h, s4 l) {
    static_assert(MF, "MFMA stage");
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      f4 d = {0.0f, 0.0f, 0.0f, 0.0f};
      if (PREC == P_FP32) {
#pragma unroll
        for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f32_16x16x4f32(f[s], (float)x[4 * blk + s], d, 0, 0, 0);
      } else {
        s4 xh, xl;
        split_bf16x4((float)x[4 * blk], (float)x[4 * blk + 1], (float)x[4 * blk + 2], (float)x[4 * blk + 3], xh, xl);
        d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(h, xh, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(l, xh, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(h, xl, d, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) y[4 * blk + v] = (wt)d[v];
    }
  }

  // LDS coordinates (e, x2, x1, x0) of a (pencil, index) pair; the pencil's
  // own two coordinates are (a, b) = ((PI % n2) / n, PI % n).
  //   pattern 1: (a, b, ax)   pattern 2: (a, ax, b)   pattern 3: (ax, a, b)
  template <int PAT>
  static DEV int addr(int PI, int ax) {
    const int e = PI / n2, rem = PI % n2, a = rem / n, b = rem % n;
    const int x2 = PAT == 3 ? ax : a;
    const int x1 = PAT == 1 ? b : (PAT == 2 ? ax : a);
    const int x0 = PAT == 1 ? ax : b;
    return ((e * n + x2) * n + x1) * P0 + x0;
  }
  // n = 8 (one element per tile, every slot valid): the address is a lane
  // part plus a per-slot constant, so that every access is one base register
  // with an immediate offset.
  template <int PAT>
  static DEV int lane_part(int lane) {
    if constexpr (MF) {
      const int P = lane & 15, hs = lane >> 5, gl = (lane >> 4) & 1;
      const int a = 2 * hs + (P >> 3), b = P & 7;
      if constexpr (PAT == 1) return (a * 8 + b) * P0 + 4 * gl;
      if constexpr (PAT == 2) return (a * 8 + 4 * gl) * P0 + b;
      return (32 * gl + a) * P0 + b;
    } else {
      const int a = lane >> 3, b = lane & 7;
      if constexpr (PAT == 1) return (a * 8 + b) * P0;
      if constexpr (PAT == 2) return a * 8 * P0 + b;
      return a * P0 + b;
    }
  }
  template <int PAT>
  static constexpr int slot_part(int s) {
    if constexpr (MF) {
      const int blk = s >> 2, m = s & 3;
      if constexpr (PAT == 1) return 32 * P0 * blk + m;
      if constexpr (PAT == 2) return 32 * P0 * blk + m * P0;
      return (8 * m + 4 * blk) * P0;
    } else {
      if constexpr (PAT == 1) return s;
      if constexpr (PAT == 2) return s * P0;
      return 8 * s * P0;
    }
  }
  template <int WP, int RP>
  static DEV void xpose(const wt (&y)[NS], wt (&x)[NS], wt* buf, int lane) {
    if constexpr (n == 8) {
      wt* bw = buf + lane_part<WP>(lane);
      const wt* br = buf + lane_part<RP>(lane);
#pragma unroll
      for (int s = 0; s < NS; ++s) bw[slot_part<WP>(s)] = y[s];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s = 0; s < NS; ++s) x[s] = br[slot_part<RP>(s)];
      asm volatile("" ::: "memory");
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (pvalid(s, lane)) buf[addr<WP>(pencil(s, lane), axis(s, lane))] = y[s];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s = 0; s < NS; ++s) x[s] = pvalid(s, lane) ? buf[addr<RP>(pencil(s, lane), axis(s, lane))] : (wt)0;
      asm volatile("" ::: "memory");
    }
  }

  // forward: contract i (pattern 1 -> 2), j (2 -> 3), k; slots of the field
  // tile in, slots of the coefficients (pencil (q, p), index r) out.  In two
  // parts, so that a pass can reuse the field's registers after the first.
  static DEV void forward1(const double (&u)[NS], wt (&x)[NS], wt* buf, const Mats& mt, const DevTables& t, int lane) {
    wt y[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s] = (wt)u[s];
    if constexpr (MF)
      stage_mf(x, y, mt.fa, mt.ha, mt.la);
    else
      forward64<n>(t.A, x, y);
    xpose<1, 2>(y, x, buf, lane);
  }
  static DEV void forward2(wt (&x)[NS], double (&c)[NS], wt* buf, const Mats& mt, const DevTables& t, int lane) {
    wt y[NS];
    if constexpr (MF) {
      stage_mf(x, y, mt.fa, mt.ha, mt.la);
      xpose<2, 3>(y, x, buf, lane);
      stage_mf(x, y, mt.fa, mt.ha, mt.la);
    } else {
      forward64<n>(t.A, x, y);
      xpose<2, 3>(y, x, buf, lane);
      forward64<n>(t.A, x, y);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) c[s] = (double)y[s];
  }
  static DEV void forward(const double (&u)[NS], double (&c)[NS], wt* buf, const Mats& mt, const DevTables& t,
                          int lane) {
    wt x[NS];
    forward1(u, x, buf, mt, t, lane);
    forward2(x, c, buf, mt, t, lane);
  }

  // inverse: contract r (3 -> 2), q (2 -> 1), p; coefficient slots in, field
  // slots out
  static DEV void inverse(const double (&cm)[NS], double (&ut)[NS], wt* buf, const Mats& mt, const DevTables& t,
                          int lane) {
    wt x[NS], y[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) x[s] = (wt)cm[s];
    if constexpr (MF) {
      stage_mf(x, y, mt.fv, mt.hv, mt.lv);
      xpose<3, 2>(y, x, buf, lane);
      stage_mf(x, y, mt.fv, mt.hv, mt.lv);
      xpose<2, 1>(y, x, buf, lane);
      stage_mf(x, y, mt.fv, mt.hv, mt.lv);
    } else {
      inverse64<n>(t.V, x, y);
      xpose<3, 2>(y, x, buf, lane);
      inverse64<n>(t.V, x, y);
      xpose<2, 1>(y, x, buf, lane);
      inverse64<n>(t.V, x, y);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) ut[s] = (double)y[s];
  }

  // Table indices of the slots: w3 for field slots, g3 for coefficient slots
  // (n = 8: a lane part plus a per-slot constant).
  DEV static int w3i(int s, int lane) {
    if constexpr (n == 8 && MF) return ((lane >> 5) * 16 + (lane & 15)) * 8 + 4 * ((lane >> 4) & 1) + (256 * (s >> 2) + (s & 3));
    if constexpr (n == 8) return lane * 8 + s;
    return (pencil(s, lane) % n2) * n + axis(s, lane);
  }
  DEV static int g3i(int s, int lane) {
    if constexpr (n == 8 && MF) return (256 * ((lane >> 4) & 1) + (lane >> 5) * 16 + (lane & 15)) + (64 * (s & 3) + 32 * (s >> 2));
    if constexpr (n == 8) return s * 64 + lane;
    return axis(s, lane) * n2 + pencil(s, lane) % n2;
  }

  // OR the kept bits of slot s (ballot m) into the tile's bitmap words in LDS
  // (bm[ee * W + w]); wave-uniform, one lane writes.
  static DEV void bitmap_or(u64* bm, u64 m, int s, int ne, int lane) {
    constexpr int RUNS = MF ? 4 : 1, RLEN = MF ? 16 : 64;
#pragma unroll
    for (int g = 0; g < RUNS; ++g) {
      const int L0 = g * RLEN;
      const int PI0 = pencil(s, L0), ax = axis(s, L0);
      if (ax >= n) continue;
      const u64 bits = RLEN == 64 ? m : ((m >> L0) & ((1ull << RLEN) - 1ull));
      int pos = 0;
      while (pos < RLEN && (bits >> pos) != 0ull) {
        const int PI = PI0 + pos;
        const int ee = PI / n2;
        if (ee >= ne) break;
        const int rem = PI % n2;
        const int c = (RLEN - pos) < (n2 - rem) ? (RLEN - pos) : (n2 - rem);
        const u64 chunk = (bits >> pos) & (c >= 64 ? ~0ull : ((1ull << c) - 1ull));
        if (chunk && lane == 0) {
          const int f0 = ax * n2 + rem, w = f0 >> 6, o = f0 & 63;
          atomicOr(&bm[ee * W + w], chunk << o);
          if (o && o + c > 64) atomicOr(&bm[ee * W + w + 1], chunk >> (64 - o));
        }
        pos += c;
      }
    }
  }
};

// w3 and g3 of every (slot, lane) in LDS, slot-major so that the 64 lanes of
// a read hit 64 consecutive doubles (registers would cost 4 NS VGPRs).
struct TabLds {
  double w3[8][64], g3[8][64];
};
template <class G>
DEV void tab_load(TabLds& T, const DevTables& t, int tid) {
  for (int k = tid; k < G::NS * 64; k += 256) {
    const int s = k >> 6, l = k & 63;
    const bool v = G::pvalid(s, l);
    T.w3[s][l] = v ? t.w3[G::w3i(s, l)] : 0.0;
    T.g3[s][l] = v ? t.g3[G::g3i(s, l)] : 0.0;
  }
}

// ---- sample pass --------------------------------------------------------------
constexpr int SBINS = HBINS;

template <int N, int PREC>
struct SampleLds {
  typename Eng<N, PREC>::wt buf[4][Eng<N, PREC>::LDSW];
  TabLds tab;
  float hs[SBINS];  // sums of energy / 2^(bin exponent), each term in [1, 2)
  double u2[4];
  int maxe;
  int last;
};

template <int N, int PREC>
DEV void sample_body(const Job& j, int comp, int vb, int nvb, SampleLds<N, PREC>& L, bool tail) {
  typedef Eng<N, PREC> G;
  constexpr int n3 = G::n3, NS = G::NS, EPW = G::EPW;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  CompState* st = j.st + comp;
  for (int k = tid; k < SBINS; k += 256) L.hs[k] = 0.0f;
  if (tid == 0) L.maxe = 0;
  typename G::Mats mt;
  G::init(mt, j.tab, lane);
  tab_load<G>(L.tab, j.tab, tid);
  __syncthreads();
  const long long E = j.n_elem, tiles = (E + EPW - 1) / EPW;
  const long long ss = j.sample_stride > 0 ? j.sample_stride : 1;
  const long long stiles = (tiles + ss - 1) / ss;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  const bool vec = ((((uintptr_t)ub) & 15) == 0);
  const long long nw = (long long)nvb * 4;
  double u2 = 0.0;
  int maxe = 0;
  for (long long k = (long long)vb * 4 + wv; k < stiles; k += nw) {
    const long long t = k * ss;
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    double u[NS], c[NS], jq[G::JS];
    G::load(ub + e0 * n3, ne, vec, u, lane);
#pragma unroll
    for (int s = 0; s < G::JS; ++s) jq[s] = 1.0;  // (1.0 * w is w: no branch per value)
    if (j.jac) G::load_jac(j.jac + e0, ne, jq, lane);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double x = G::valid(s, lane, ne) ? (jq[s % G::JS] * L.tab.w3[s][lane]) * (u[s] * u[s]) : 0.0;
      u2 += x;
      const int ex = bits_exp(dbits(x));
      maxe = ex > maxe ? ex : maxe;
    }
    G::forward(u, c, L.buf[wv], mt, j.tab, lane);
    // energies first, then their atomics: none of these waits for the next
    // (rounded sums only place the window)
    int eb[NS];
    float em[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double en = G::valid(s, lane, ne) ? (jq[s % G::JS] * L.tab.g3[s][lane]) * (c[s] * c[s]) : 0.0;
      eb[s] = bits_exp(dbits(en));
      em[s] = eb[s] < HBINS - 1 ? (float)ldexp(en, 1023 - eb[s]) : 0.0f;
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
      if (em[s] != 0.0f) atomicAdd(&L.hs[eb[s]], em[s]);
  }
  u2 = wave_sum_f64(u2);
  for (int m = 32; m > 0; m >>= 1) {
    const int o = __shfl_xor(maxe, m);
    maxe = o > maxe ? o : maxe;
  }
  if (lane == 0) {
    L.u2[wv] = u2;
    atomicMax(&L.maxe, maxe);
  }
  __syncthreads();
  HistBin* H = j.histEs + (size_t)comp * HBINS;
  for (int k = tid; k < SBINS; k += 256) {
    if (L.hs[k] != 0.0f) {
      atomicAdd((double*)&H[k].lo, ldexp((double)L.hs[k], k - 1023));
    }
  }
  if (tid == 0) {
    atomicAdd(&st->samp_u2, L.u2[0] + L.u2[1] + L.u2[2] + L.u2[3]);
    atomicMax(&st->samp_maxe, L.maxe);
  }
  if (!tail || !last_block(j.done + D_SAMPLE * 8 + comp, &L.last, nvb)) return;
  if (tid < 64) select_sample_body(j, comp);
}

template <int N, int PREC>
__global__ __launch_bounds__(256, ISR_FAST_MINB) void k_sample(Job j) {
  __shared__ SampleLds<N, PREC> L;
  sample_body<N, PREC>(j, blockIdx.y, blockIdx.x, gridDim.x, L, false);
}

// ---- pass A -------------------------------------------------------------------
constexpr int CAPB = 256;  // per-wave staging of window candidates

template <int N, int PREC>
struct PassALds {
  typename Eng<N, PREC>::wt buf[4][Eng<N, PREC>::LDSW];
  TabLds tab;
  u64 key[4][CAPB];
  u32 idx[4][CAPB];
  u32 ecnt[4][16];
  XFar far[PREC == P_FP64 ? 2 : 1];  // FP64 path: norm terms, energies
  long long red[4][8];
};

DEV void cap_flush(u64* key, u32* idx, u32& ncap, CompState* st, u64* list, u32* lidx, u64 cap, int lane) {
  if (ncap == 0u) return;
  u64 base = 0ull;
  if (lane == 0) base = atomicAdd(&st->list_count[0], (u64)ncap);
  base = bcast64(base, 0);
  for (u32 i = lane; i < ncap; i += 64) {
    const u64 pos = base + i;
    if (pos < cap) {
      list[pos] = key[i];
      lidx[pos] = idx[i];
    } else {
      atomicOr(&st->flags, ST_LIST);
    }
  }
  ncap = 0u;
  asm volatile("" ::: "memory");
}

template <int N, int PREC>
DEV void passA_body(const Job& j, int comp, int vb, int nvb, PassALds<N, PREC>& L) {
  typedef Eng<N, PREC> G;
  constexpr int n3 = G::n3, NS = G::NS, EPW = G::EPW;
  constexpr bool EXACT = PREC == P_FP64;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  CompState* st = j.st + comp;
  if (st->flags & ST_MISS) return;
  const int wlo = st->win_lo, whi = st->win_hi;
  const XParm PN = xparm(st->xm_norm, j.xh);
  const XParm PE = xparm(wlo - 1023, j.xh);
  const u32 hwlo = (u32)wlo << 20, hwhi = (u32)whi << 20;  // the window's edges as high words of energies
  const XRange RN = xrange(PN);  // FP64 path
  XRange RE = xrange(PE);
  RE.lo = RE.lo < hwlo ? RE.lo : hwlo;  // (without a window, wlo = 0, nothing is below it)
  HistBin* gN = j.histN + (size_t)comp * HBINS;
  HistBin* gE = j.histE + (size_t)comp * HBINS;
  u64* list = list_ptr(j, comp, 0);
  u32* lidx = j.lidx + (size_t)comp * j.list_cap;
  const long long E = j.n_elem, tiles = (E + EPW - 1) / EPW;
  u32* cnt = j.cnt + (size_t)comp * E;
  typename G::Mats mt;
  G::init(mt, j.tab, lane);
  tab_load<G>(L.tab, j.tab, tid);
  if constexpr (EXACT) {
    xfar_clear(L.far[0], tid);
    xfar_clear(L.far[1], tid);
  }
  __syncthreads();
  XAcc an = {0.0, 0.0, 0.0}, ae = {0.0, 0.0, 0.0};
  XRun rn = xrun(PN), re = xrun(PE);  // FP64 path
  double pe = 0.0;  // fixed-order sum of the energies below the window
  double pn = 0.0;  // MFMA paths: fixed-order sum of the norm terms
  u64 hi_tot = 0ull;
  u32 ncap = 0u;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  const bool vec = ((((uintptr_t)ub) & 15) == 0);
  const long long nw = (long long)nvb * 4;
  // the next tile's field values (and Jacobians) are loaded while this one is
  // processed: at the top of the tile on the MFMA paths (which wait for memory
  // more than they issue; 196 us at N = 7 BF16 against 214 with the later
  // load), on the FP64 path into the same registers once the first contraction
  // has taken the values (issue bound: 16 registers and copies less).  The wait
  // for them also waits for every store issued since, so a tile's counts are
  // stored with the next tile's loads, just ahead of them.
  constexpr bool EARLY = G::MF;
  double u[NS], un[EARLY ? NS : 1], jq[G::JS];
  auto fetch = [&](long long t) {
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    if constexpr (EARLY)
      G::load(ub + e0 * n3, ne, vec, un, lane);
    else
      G::load(ub + e0 * n3, ne, vec, u, lane);
    if (j.jac) G::load_jac(j.jac + e0, ne, jq, lane);
  };
  long long cnt_e = -1;  // this lane's element with a count to be stored, and the count
  u32 cnt_v = 0u;
  if ((long long)vb * 4 + wv < tiles) fetch((long long)vb * 4 + wv);
  for (long long t = (long long)vb * 4 + wv; t < tiles; t += nw) {
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    double c[NS];
    double jt[G::JS];
#pragma unroll
    for (int s = 0; s < G::JS; ++s) jt[s] = jq[s];
    if constexpr (EARLY) {
#pragma unroll
      for (int s = 0; s < NS; ++s) u[s] = un[s];
      if (cnt_e >= 0) cnt[cnt_e] = cnt_v;
      if (t + nw < tiles) fetch(t + nw);
    }
    // quadrature weights of the slots (times the element's Jacobian), with the
    // Jacobian test taken once per tile
    double wq[NS];
    if (j.jac) {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = jt[s % G::JS] * L.tab.w3[s][lane];
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = L.tab.w3[s][lane];
    }
    // norm terms: every term split exactly on the FP64 path; on the MFMA
    // paths each lane sums its terms in a fixed FP64 order and only the lane
    // totals are added exactly (as for the energies and the error terms)
    u64 odd = 0ull;  // lanes with a term out of the running sums' range
    double xs[EXACT ? NS : 1];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool v = G::valid(s, lane, ne);
      const double x = v ? wq[s] * (u[s] * u[s]) : 0.0;
      if constexpr (EXACT) {
        xs[s] = x;
        odd |= __builtin_amdgcn_ballot_w64(xrun_left(rn, RN, x) && v);
        // one slot at a time: interleaving them would hold every slot's
        // temporaries at once and cut the occupancy
        __builtin_amdgcn_sched_barrier(0);
      } else {
        pn += x;
      }
    }
    if constexpr (EXACT) {
      if (odd)  // (one vote a tile keeps this out of the slots' way)
        xfar_tile<EPW * G::n2, NS, true>(L.far[0], xfar_m(PN.m, j.xh), gN, L.buf, xs, [&](double x) { return !xin(RN, x); });
      odd = 0ull;
    }
    if constexpr (EXACT) pin(rn);
    typename G::wt x1[NS];
    G::forward1(u, x1, L.buf[wv], mt, j.tab, lane);
    if constexpr (!EARLY) {
      if (cnt_e >= 0) cnt[cnt_e] = cnt_v;
      if (t + nw < tiles) fetch(t + nw);
    }
    G::forward2(x1, c, L.buf[wv], mt, j.tab, lane);
    if (EPW > 1) {
      if (lane < EPW) L.ecnt[wv][lane] = 0u;
      asm volatile("" ::: "memory");
    }
    u32 hc = 0u, hmax = 0u;
    if (j.jac) {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = jt[s % G::JS] * L.tab.g3[s][lane];
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = L.tab.g3[s][lane];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool v = G::valid(s, lane, ne);
      const double en = v ? wq[s] * (c[s] * c[s]) : 0.0;
      const u64 key = dbits(en);
      // below, inside or above the window by the high words alone (its edges
      // are powers of two; Inf and NaN, whatever their sign, are above)
      const u32 hw = hi_word(en);
      const bool hi = v && hw >= hwhi;
      const bool cp = v && hw < hwhi && hw >= hwlo;
      hmax = hw > hmax ? hw : hmax;
      // the wave votes first: lane flags that stay live across the divergent
      // branches below would be copied through vector registers on every slot
      const u64 bh = ballot(hi);
      const u64 bc = ballot(cp);
      hc += (u32)__popcll(bh);
      if (EPW > 1 && hi) atomicAdd(&L.ecnt[wv][G::elem(s, lane)], 1u);
      if (bc) {
        const u32 pos = ncap + (u32)__popcll(bc & ((1ull << lane) - 1ull));
        if (cp) {
          L.key[wv][pos] = key;
          L.idx[wv][pos] = (u32)(e0 + G::elem(s, lane));
        }
        ncap += (u32)__popcll(bc);
        if (ncap > (u32)(CAPB - 64)) {
          asm volatile("" ::: "memory");
          cap_flush(L.key[wv], L.idx[wv], ncap, st, list, lidx, j.list_cap, lane);
        }
      }
      if constexpr (EXACT) {  // (the running sums' range ends at the window)
        xs[s] = en;
        const bool tiny = hw < RE.lo;
        xrun_add(re, hw < hwlo && !tiny ? en : 0.0);
        odd |= __builtin_amdgcn_ballot_w64(tiny && v);
      } else {
        pe += hw < hwlo ? en : 0.0;  // (zero in masked slots)
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (EXACT) pin(re);
    if constexpr (EXACT) {
      if (odd)
        xfar_tile<EPW * G::n2, NS, true>(L.far[1], xfar_m(PE.m, j.xh), gE, L.buf, xs, [&](double x) { return hi_word(x) < RE.lo; });
    }
    if (hmax >= 0x7ff00000u) slow_bin(gE, __builtin_inf());  // Inf/NaN: counted in the flag bin
    hi_tot += hc;
    if (EPW == 1) {
      cnt_e = lane == 0 ? e0 : -1;
      cnt_v = hc;
    } else {
      asm volatile("" ::: "memory");
      cnt_e = lane < ne ? e0 + lane : -1;
      cnt_v = L.ecnt[wv][lane < EPW ? lane : 0];
    }
  }
  if (cnt_e >= 0) cnt[cnt_e] = cnt_v;
  asm volatile("" ::: "memory");
  cap_flush(L.key[wv], L.idx[wv], ncap, st, list, lidx, j.list_cap, lane);
  // (formed again: held across the loop they cost some twenty scalar registers.
  // Not read again from st: its line takes every wave's list atomics, and that
  // read made the kernel 80 us longer)
  const XParm QN = xparm(again(PN.m), j.xh);
  const XParm QE = xparm(again(PE.m), j.xh);
  if constexpr (EXACT) {
    an = xrun_sums(rn, QN);
    ae = xrun_sums(re, QE);
  } else {
    const double le = xadd_sum(ae, QE, pe);
    if (le != 0.0) slow_bin(gE, le);
    const double ln = xadd_sum(an, QN, pn);
    if (ln != 0.0) slow_bin(gN, ln);
  }
  long long v[7];
  long long kn[3], ke[3];
  xints(an, QN, kn);
  xints(ae, QE, ke);
  v[0] = kn[0];
  v[1] = kn[1];
  v[2] = kn[2];
  v[3] = ke[0];
  v[4] = ke[1];
  v[5] = ke[2];
  v[6] = lane == 0 ? (long long)hi_tot : 0ll;
  block_sum_i64<7>(v, L.red, tid);
  if (tid < 7) j.slotsA[((size_t)comp * j.gA + vb) * 8 + tid] = L.red[0][tid];
  if constexpr (EXACT) {
    xfar_out(L.far[0], gN, tid);
    if (wlo < whi) xfar_out(L.far[1], gE, tid - 64);
  }
}

template <int N, int PREC>
__global__ __launch_bounds__(256, ISR_FAST_MINB) void k_passA(Job j) {
  __shared__ PassALds<N, PREC> L;
  passA_body<N, PREC>(j, blockIdx.y, blockIdx.x, gridDim.x, L);
}

// ---- pass B -------------------------------------------------------------------
template <int N, int PREC>
struct PassBLds {
  typename Eng<N, PREC>::wt buf[4][Eng<N, PREC>::LDSW];
  TabLds tab;
  u64 bm[4][16];
  u32 wp[4][16];
  XFar far;  // FP64 path: error terms
  long long red[4][8];
  __int128 r3[4][3];
  int last;
};

template <int N, int PREC>
DEV void passB_body(const Job& j, int comp, int vb, int nvb, PassBLds<N, PREC>& L, bool tail) {
  typedef Eng<N, PREC> G;
  constexpr int n3 = G::n3, NS = G::NS, EPW = G::EPW, W = G::W;
  constexpr bool EXACT = PREC == P_FP64;
  static_assert(EPW * W <= 16, "tile bitmap fits the LDS slot");
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  CompState* st = j.st + comp;
  if (st->flags & ST_MISS) return;
  const XParm PR = xparm(st->xm_err, j.xh);
  HistBin* gR = j.histR + (size_t)comp * HBINS;
  // the threshold: the component's, or (per-element cut, FP64 path) the
  // element's, loaded with the tile
  double tau = st->tau, tn = tau;
  const double* te = EXACT && j.tau_elem ? j.tau_elem + (size_t)comp * j.n_elem : nullptr;
  u64 voff = 0ull;
  for (int cc = 0; cc < comp; ++cc) voff += j.st[cc].kept;
  const u64 vcap = (u64)j.ncomp * (u64)j.n_elem * (u64)n3;
  const long long E = j.n_elem, tiles = (E + EPW - 1) / EPW;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  u64* gbm = j.bitmap + (size_t)comp * E * W;
  typedef typename Pick<G::MF, float, double>::type vt;  // the blob's values (vbytes)
  typename G::Mats mt;
  G::init(mt, j.tab, lane);
  tab_load<G>(L.tab, j.tab, tid);
  if constexpr (EXACT) xfar_clear(L.far, tid);
  __syncthreads();
  XAcc ar = {0.0, 0.0, 0.0};
  const XRange RR = xrange(PR);  // FP64 path
  XRun rr = xrun(PR);
  double pr = 0.0;  // fixed-order sum of the error terms
  bool bad = false;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  const bool vec = ((((uintptr_t)ub) & 15) == 0);
  const long long nw = (long long)nvb * 4;
  u64* bm = L.bm[wv];
  u32* wp = L.wp[wv];
  // the next tile's field values (and Jacobians) are loaded while this one is
  // processed
  double un[NS], jn[G::JS];
  {
    const long long t0 = (long long)vb * 4 + wv;
    if (t0 < tiles) {
      const int ne0 = (int)((E - t0 * EPW) < EPW ? (E - t0 * EPW) : EPW);
      G::load(ub + t0 * EPW * n3, ne0, vec, un, lane);
      if (j.jac) G::load_jac(j.jac + t0 * EPW, ne0, jn, lane);
      if (te && G::valid(0, lane, ne0)) tn = te[t0 * EPW + G::elem(0, lane)];
    }
  }
  for (long long t = (long long)vb * 4 + wv; t < tiles; t += nw) {
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    double u[NS], c[NS], jq[G::JS];
#pragma unroll
    for (int s = 0; s < NS; ++s) u[s] = un[s];
#pragma unroll
    for (int s = 0; s < G::JS; ++s) jq[s] = jn[s];
    tau = tn;
    if (t + nw < tiles) {
      const long long e1 = (t + nw) * EPW;
      const int ne1 = (int)((E - e1) < EPW ? (E - e1) : EPW);
      G::load(ub + e1 * n3, ne1, vec, un, lane);
      if (j.jac) G::load_jac(j.jac + e1, ne1, jn, lane);
      if (te && G::valid(0, lane, ne1)) tn = te[e1 + G::elem(0, lane)];
    }
    G::forward(u, c, L.buf[wv], mt, j.tab, lane);
    // energy weights of the slots (times the element's Jacobian), with the
    // Jacobian test taken once per tile
    double wq[NS];
    if (j.jac) {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = jq[s % G::JS] * L.tab.g3[s][lane];
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = L.tab.g3[s][lane];
    }
    bool keep[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool v = G::valid(s, lane, ne);
      const double en = v ? wq[s] * (c[s] * c[s]) : 0.0;
      keep[s] = v && !(en < tau);  // (a NaN is kept: pass A counts it among the energies above)
    }
    if constexpr (G::n == 8) {
      // one element per tile and one 64-bit word per index r: the words come
      // straight from the ballots (wave-uniform, no LDS)
      u64 B[NS];
#pragma unroll
      for (int s = 0; s < NS; ++s) B[s] = ballot(keep[s]);
      // indices 0..3 and 4..7 apart, so that picking one by lane below is a
      // select and not an indexed access
      u64 wa[4], wb[4];
      if constexpr (G::MF) {
        // slot s = 4 blk + m on lane 16 g + P: index r = 4 (g & 1) + m, pencil
        // 32 blk + 16 (g >> 1) + P
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          wa[m] = wb[m] = 0ull;
#pragma unroll
          for (int blk = 0; blk < 2; ++blk)
#pragma unroll
            for (int hs = 0; hs < 2; ++hs) {
              wa[m] |= ((B[4 * blk + m] >> (32 * hs)) & 0xFFFFull) << (32 * blk + 16 * hs);
              wb[m] |= ((B[4 * blk + m] >> (32 * hs + 16)) & 0xFFFFull) << (32 * blk + 16 * hs);
            }
        }
      } else {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          wa[m] = B[m];
          wb[m] = B[4 + m];
        }
      }
      u32 pa[4], pb[4];
      u32 tot = 0u;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        pa[m] = tot;
        tot += (u32)__popcll(wa[m]);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        pb[m] = tot;
        tot += (u32)__popcll(wb[m]);
      }
      u64 mine = 0ull;
      mine = writelane64<0>(wa[0], mine);
      mine = writelane64<1>(wa[1], mine);
      mine = writelane64<2>(wa[2], mine);
      mine = writelane64<3>(wa[3], mine);
      mine = writelane64<4>(wb[0], mine);
      mine = writelane64<5>(wb[1], mine);
      mine = writelane64<6>(wb[2], mine);
      mine = writelane64<7>(wb[3], mine);
      if (lane < 8) gbm[e0 * 8 + lane] = mine;
      const u64 ebase = eptr[e0];
      const u64 vbase = voff + ebase;
      // offsets that disagree with the bitmap: never write past the values
      const bool fits = vbase <= vcap && (u64)tot <= vcap - vbase;
      if ((u64)tot != eptr[e0 + 1] - ebase || !fits) bad = true;
      if (fits) {
        // the element's values: a uniform base and a 32-bit rank per lane
        vt* dst = (vt*)j.values + vbase;
        if constexpr (G::MF) {
          // index r = 4 (g & 1) + (s & 3): one of two words; block 0 holds
          // the pencils of a word's low half, block 1 those of its high half
          const bool up = (lane >> 4) & 1;
          const u32 below = (1u << (16 * (lane >> 5) + (lane & 15))) - 1u;
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            const u64 wd = up ? wb[m] : wa[m];
            const u32 lo = (u32)wd, hi = (u32)(wd >> 32), pr = up ? pb[m] : pa[m];
            if (keep[m]) dst[pr + (u32)__popc(lo & below)] = (vt)c[m];
            if (keep[4 + m]) dst[pr + (u32)__popc(lo) + (u32)__popc(hi & below)] = (vt)c[4 + m];
          }
        } else {
#pragma unroll
          for (int s = 0; s < NS; ++s)
            if (keep[s]) dst[(s < 4 ? pa[s & 3] : pb[s & 3]) + lane_rank(B[s])] = (vt)c[s];
        }
      }
    } else {
      if (lane < EPW * W) bm[lane] = 0ull;
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s = 0; s < NS; ++s) G::bitmap_or(bm, ballot(keep[s]), s, ne, lane);
      asm volatile("" ::: "memory");
      // bitmap words out, exclusive word prefixes inside each element
      int wl = lane;
      if constexpr (EXACT) asm volatile("" : "+v"(wl));  // (no address made from it is kept across tiles)
      if (wl < ne * W) {
        const u64 wd = bm[wl];
        gbm[e0 * W + wl] = wd;
        const int ee = wl / W, w = wl % W;
        u32 pre = 0u;
        for (int k = 0; k < w; ++k) pre += (u32)__popcll(bm[ee * W + k]);
        wp[wl] = pre;
        if (w == W - 1) {
          const u64 expect = eptr[e0 + ee + 1] - eptr[e0 + ee];
          if ((u64)(pre + (u32)__popcll(wd)) != expect) bad = true;
        }
      }
      asm volatile("" ::: "memory");
      // kept values at their element offsets
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        if (!keep[s]) continue;
        const int PI = G::pencil(s, lane), ax = G::axis(s, lane);
        const int ee = PI / G::n2, f = ax * G::n2 + PI % G::n2;
        const int wi = ee * W + (f >> 6);
        const u64 rank = (u64)wp[wi] + (u64)__popcll(bm[wi] & ((1ull << (f & 63)) - 1ull));
        const u64 pos = voff + eptr[e0 + ee] + rank;
        if (pos >= vcap) {  // offsets disagree with the bitmap: never write past the values
          bad = true;
          continue;
        }
        if (j.vbytes == 8)
          ((double*)j.values)[pos] = c[s];
        else
          ((float*)j.values)[pos] = (float)c[s];
      }
    }
    double cm[NS], ut[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) cm[s] = keep[s] ? c[s] : 0.0;
    G::inverse(cm, ut, L.buf[wv], mt, j.tab, lane);
    if constexpr (EXACT && N == 7) __builtin_amdgcn_sched_barrier(0);  // (interleaved, both would spill)
    // quadrature weights of the slots, the same way
    if (j.jac) {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = jq[s % G::JS] * L.tab.w3[s][lane];
    } else {
#pragma unroll
      for (int s = 0; s < NS; ++s) wq[s] = L.tab.w3[s][lane];
    }
    u64 odd = 0ull;
    double xs[EXACT ? NS : 1];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool v = G::valid(s, lane, ne);
      const double d = u[s] - ut[s];
      const double x = v ? wq[s] * (d * d) : 0.0;
      if constexpr (EXACT) {
        xs[s] = x;
        odd |= ballot(xrun_left(rr, RR, x) && x != 0.0);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        pr += x;
      }
    }
    if constexpr (EXACT) pin(rr);
    if constexpr (EXACT) {
      if (odd)
        xfar_tile<EPW * G::n2, NS, false>(L.far, xfar_m(PR.m, j.xh), gR, L.buf, xs, [&](double x) { return !xin(RR, x); });
    }
  }
  if (ballot(bad)) {
    if (lane == 0) atomicOr(&st->flags, ST_LIST);
  }
  const XParm QR = xparm(again(PR.m), j.xh);
  if constexpr (EXACT) {
    ar = xrun_sums(rr, QR);
  } else {
    const double r = xadd_sum(ar, QR, pr);
    if (r != 0.0) slow_bin(gR, r);
  }
  long long v[3];
  xints(ar, QR, v);
  block_sum_i64<3>(v, L.red, tid);
  if (tid < 3) j.slotsB[((size_t)comp * j.gB + vb) * 4 + tid] = L.red[0][tid];
  if constexpr (EXACT) xfar_out(L.far, gR, tid);
  if (!tail || !last_block(j.done + D_PASSB * 8 + comp, &L.last, nvb)) return;
  passB_tail(j, comp, L.r3);
}

template <int N, int PREC>
__global__ __launch_bounds__(256, (fast_minb_b<N, PREC>())) void k_passB(Job j) {
  __shared__ PassBLds<N, PREC> L;
  passB_body<N, PREC>(j, blockIdx.y, blockIdx.x, gridDim.x, L, false);
}

// ---- decompress of blobs made by this engine --------------------------------------
// The blob's kept values go back into the slots pass B took them from, and the
// same inverse runs on them, so that the reconstruction is the one whose
// error pass B measured, bit for bit (FP32 / BF16 blobs); FP64 blobs of these
// orders (quantisation codes included) take the same fixed-order inverse as
// the workgroup tiles of isr_passes.cuh, in one wavefront without barriers.
//
// Bound by the writes of the field at n = 8 (8 or 4 B a value against ~0.5 B
// of blob read), so the shape keeps the store stream going: blockIdx.y is the
// component, every wavefront walks its tiles with the next tile's bitmap words
// and offset already in flight (one memory round per tile, the kept values'),
// and the field leaves in whole lines: the MFMA layout at n = 8 holds four
// consecutive FP32 values a lane (one 16-byte store each), everything else is
// transposed through the tile's LDS buffer into dense order.  The stores are
// non-temporal (nothing here reads them back; as ordinary stores the same
// kernel takes 217 and 103 us).  65,536 elements, N = 7, 3 components: FP64 to
// FP64 358 -> 156 us (5.2 TB/s written), BF16 to FP32 305 -> 85 us (4.7 TB/s).
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// Calls fn(slot, place, index) for every kept coefficient of this lane's slots
// (place: among the blob's values; index: flat index in its element), and sets
// the other slots to zero: cm[s] = kept ? fn(...) : 0.  wcur: the tile's bitmap
// words, one a lane; base: the place of its first kept value.
template <int N, int PREC, int NS, class FN>
DEV void kept_slots(double (&cm)[NS], u64 wcur, u64 base, int ne, u64* bm, u32* wp, int lane, FN fn) {
  typedef Eng<N, PREC> G;
  static_assert(NS == G::NS, "a tile's slots");
  constexpr int n = G::n, n2 = G::n2, W = G::W;
  if constexpr (n == 8) {
    // one element, one word per index r: uniform words and prefixes
    // (indices 0..3 and 4..7 apart, so that picking one by lane is a select
    // and not an indexed access)
    u64 wa[4], wb[4];
    u32 pa[4], pb[4], tot = 0u;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      wa[r] = bcast64(wcur, r);
      pa[r] = tot;
      tot += (u32)__popcll(wa[r]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      wb[r] = bcast64(wcur, 4 + r);
      pb[r] = tot;
      tot += (u32)__popcll(wb[r]);
    }
    if constexpr (G::MF) {
      // slot s = 4 blk + m: index r = 4 gl + m, pencil 32 blk + p32
      const bool up = (lane >> 4) & 1;
      const int p32 = 16 * (lane >> 5) + (lane & 15);
      const u32 bit = 1u << p32, below = bit - 1u;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const u64 wd = up ? wb[m] : wa[m];
        const u32 lo = (u32)wd, hi = (u32)(wd >> 32), pr = up ? pb[m] : pa[m];
        const int f = (4 * (int)up + m) * 64 + p32;
        cm[m] = (lo & bit) ? fn(m, base + (pr + (u32)__popc(lo & below)), f) : 0.0;
        cm[4 + m] =
            (hi & bit) ? fn(4 + m, base + (pr + (u32)__popc(lo) + (u32)__popc(hi & below)), f + 32) : 0.0;
      }
    } else {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const u64 wd = r < 4 ? wa[r & 3] : wb[r & 3];
        const u32 pr = r < 4 ? pa[r & 3] : pb[r & 3];
        cm[r] = lane_bit(wd) ? fn(r, base + (pr + lane_rank(wd)), r * 64 + lane) : 0.0;
      }
    }
  } else {
    // the tile's kept values follow each other in the blob: ranks run over
    // all of its words
    const u32 pc = (u32)__popcll(wcur);
    u32 incl = pc;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const u32 o = (u32)__shfl_up((int)incl, d);
      incl += lane >= d ? o : 0u;
    }
    if (lane < 16) {
      bm[lane] = wcur;
      wp[lane] = incl - pc;
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      cm[s] = 0.0;
      if (!G::valid(s, lane, ne)) continue;
      const int PI = G::pencil(s, lane), ax = G::axis(s, lane);
      const int f = ax * n2 + PI % n2, wi = (PI / n2) * W + (f >> 6);
      const u64 wd = bm[wi];
      if ((wd >> (f & 63)) & 1ull)
        cm[s] = fn(s, base + (wp[wi] + (u32)__popcll(wd & ((1ull << (f & 63)) - 1ull))), f);
    }
    asm volatile("" ::: "memory");
  }
}

template <int N, int PREC, bool OUT64>
__global__ __launch_bounds__(256, 4) void k_decompW(Job j, void* out) {
  typedef Eng<N, PREC> G;
  constexpr int n = G::n, n3 = G::n3, NS = G::NS, EPW = G::EPW, W = G::W;
  static_assert(EPW * W <= 16, "tile bitmap fits the LDS slot");
  typedef typename Pick<OUT64, double, float>::type ot;
  __shared__ typename G::wt lbuf[4][G::LDSW];
  __shared__ u64 lbm[4][16];
  __shared__ u32 lwp[4][16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int comp = blockIdx.y;
  typename G::wt* buf = lbuf[wv];
  typename G::Mats mt;
  G::init(mt, j.tab, lane);
  const long long E = j.n_elem, tiles = (E + EPW - 1) / EPW, nw = (long long)gridDim.x * 4;
  const u64* gbm = j.bitmap + (size_t)comp * E * W;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  const u64 voff = j.voff[comp];
  const double qs = !G::MF && j.qstep ? j.qstep[comp] : 0.0;
  ot* ocomp = (ot*)out + (size_t)comp * E * n3;
  long long t = (long long)blockIdx.x * 4 + wv;
  if (t >= tiles) return;
  u64 wnext = 0ull, bnext = 0ull;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    wnext = lane < ne * W ? gbm[e0 * W + lane] : 0ull;
    bnext = eptr[e0];
  };
  fetch(t);
  for (; t < tiles; t += nw) {
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    const u64 wcur = wnext, base = voff + bnext;
    if (t + nw < tiles) fetch(t + nw);
    double cm[NS], ut[NS];
    kept_slots<N, PREC>(cm, wcur, base, ne, lbm[wv], lwp[wv], lane, [&](int, u64 pos, int f) -> double {
      if constexpr (G::MF) return (double)((const float*)j.values)[pos];
      if (j.vbytes == 8) return ((const double*)j.values)[pos];
      // quantisation codes: the value is (code * step) / sqrt(g3)
      return ((double)((const float*)j.values)[pos] * qs) / __builtin_sqrt(j.tab.g3[f]);
    });
    G::inverse(cm, ut, buf, mt, j.tab, lane);
    ot* o = ocomp + e0 * n3;
    if constexpr (n == 8 && G::MF && !OUT64) {
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        const f4u v = {(float)ut[4 * blk], (float)ut[4 * blk + 1], (float)ut[4 * blk + 2], (float)ut[4 * blk + 3]};
        __builtin_nontemporal_store(v, (f4u*)(o + G::pencil(4 * blk, lane) * n + G::axis(4 * blk, lane)));
      }
    } else {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int s = 0; s < NS; ++s)
        if (G::pvalid(s, lane)) buf[G::pencil(s, lane) * G::P0 + G::axis(s, lane)] = (typename G::wt)ut[s];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int k = 0; k < (EPW * n3 + 63) / 64; ++k) {
        const int v = lane + 64 * k;
        if (v < ne * n3) __builtin_nontemporal_store((ot)buf[(v / n) * G::P0 + v % n], &o[v]);
      }
      asm volatile("" ::: "memory");
    }
  }
}

// ---- quantised variant, orders 1..7 ------------------------------------------------
// The codes of the kept values and the error they leave: a kept coefficient c
// gets the code q = rint((c sqrt(g3)) / step), an FP32 integer at the value's
// place; the terms w3 (u - u~)^2 of the dequantised (q step) / sqrt(g3) go into
// the exact error; a code of magnitude 2^24 or more sets j.ticket[1].  Unit
// Jacobians.  One tile per wavefront: the next tile's field, words and offset
// in flight, the error terms into running exact sums instead of LDS histogram
// atomics.  The per-workgroup sums go to j.slotsB; j.qxm: log2 of the bound on
// the error terms per component.  10,007 elements, N = 7, 3 components: 218 ->
// 65 us (83 on pass B's grid, a third larger than what is resident of this kernel).
template <int N>
struct QuantWLds {
  typedef Eng<N, P_FP64> G;
  double buf[4][G::LDSW];
  double w3[8][64], sq[8][64];  // quadrature weights of field slots, sqrt(g3) of coefficient slots
  u64 bm[4][16];
  u32 wp[4][16];
  XFar far;  // error terms
  long long red[4][8];
};

template <int N>
__global__ __launch_bounds__(256, 3) void k_quantW(Job j) {
  typedef Eng<N, P_FP64> G;
  constexpr int n3 = G::n3, NS = G::NS, EPW = G::EPW, W = G::W;
  __shared__ QuantWLds<N> L;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int comp = blockIdx.y;
  for (int k = tid; k < NS * 64; k += 256) {
    const int s = k >> 6, l = k & 63;
    const bool v = G::pvalid(s, l);
    L.w3[s][l] = v ? j.tab.w3[G::w3i(s, l)] : 0.0;
    L.sq[s][l] = v ? __builtin_sqrt(j.tab.g3[G::g3i(s, l)]) : 1.0;
  }
  xfar_clear(L.far, tid);
  __syncthreads();
  const typename G::Mats mt{};
  const long long E = j.n_elem, tiles = (E + EPW - 1) / EPW, nw = (long long)gridDim.x * 4;
  const double* ub = j.u + (size_t)comp * j.comp_stride;
  const bool vec = ((((uintptr_t)ub) & 15) == 0);
  const u64* gbm = j.bitmap + (size_t)comp * E * W;
  const u64* eptr = j.elem_ptr + (size_t)comp * (E + 1);
  const u64 voff = j.voff[comp];
  const double step = j.qstep[comp];
  const XParm PR = xparm(j.qxm[comp], j.xh);
  const XRange RR = xrange(PR);
  XRun rr = xrun(PR);
  HistBin* gR = j.histR + (size_t)comp * HBINS;
  bool big = false;
  double un[NS];
  u64 wnext = 0ull, bnext = 0ull;
  auto fetch = [&](long long tt) {
    const long long e0 = tt * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    G::load(ub + e0 * n3, ne, vec, un, lane);
    wnext = lane < ne * W ? gbm[e0 * W + lane] : 0ull;
    bnext = eptr[e0];
  };
  long long t = (long long)blockIdx.x * 4 + wv;
  if (t < tiles) fetch(t);
  for (; t < tiles; t += nw) {
    const long long e0 = t * EPW;
    const int ne = (int)((E - e0) < EPW ? (E - e0) : EPW);
    const u64 wcur = wnext, base = voff + bnext;
    double u[NS], cm[NS], ut[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) u[s] = un[s];
    if (t + nw < tiles) fetch(t + nw);
    kept_slots<N, P_FP64>(cm, wcur, base, ne, L.bm[wv], L.wp[wv], lane, [&](int s, u64 pos, int) -> double {
      const double c = ((const double*)j.values)[pos];
      const double sq = L.sq[s][lane];
      const double q = __builtin_rint((c * sq) / step);
      if (!(__builtin_fabs(q) < 16777216.0)) big = true;
      j.qvals[pos] = (float)q;
      return (q * step) / sq;
    });
    G::inverse(cm, ut, L.buf[wv], mt, j.tab, lane);
    u64 odd = 0ull;
    double xs[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const bool v = G::valid(s, lane, ne);
      const double d = u[s] - ut[s];
      const double x = v ? L.w3[s][lane] * (d * d) : 0.0;
      xs[s] = x;
      odd |= ballot(xrun_left(rr, RR, x) && x != 0.0);
      __builtin_amdgcn_sched_barrier(0);
    }
    pin(rr);
    if (odd)
      xfar_tile<EPW * G::n2, NS, false>(L.far, xfar_m(PR.m, j.xh), gR, L.buf, xs, [&](double x) { return !xin(RR, x); });
  }
  if (big) atomicOr(&j.ticket[1], 1u);
  const XParm QR = xparm(again(PR.m), j.xh);
  long long v[3];
  xints(xrun_sums(rr, QR), QR, v);
  block_sum_i64<3>(v, L.red, tid);
  if (tid < 3) j.slotsB[((size_t)comp * j.gB + blockIdx.x) * 4 + tid] = L.red[0][tid];
  xfar_out(L.far, gR, tid);
}

// Grid of a decompression: gx workgroups per component cover its tiles once;
// no more than are resident at once are launched (each wavefront then walks
// several tiles and loads ahead), so that no partial second round is left.
inline int resident_wgs(const void* kernel) {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, 256, 0) != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  return nb > 0 ? nb : 1;
}
inline dim3 decomp_grid(const Job& j, int gx, int nb, int cus) {
  const int most = cus * nb / j.ncomp;
  return dim3(gx < most ? gx : (most > 0 ? most : 1), j.ncomp);
}

// ---- launchers ------------------------------------------------------------------
#define ISR_FAST_ORDERS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7)

template <int PREC>
hipError_t launch_decompW_prec(const Job& j, int gx, int cus, hipStream_t s, void* out, int out_fp64) {
  switch (j.order) {
#define CASE(NN)                                                                       \
  case NN:                                                                             \
  {                                                                                    \
    static const int nb = resident_wgs((const void*)k_decompW<NN, PREC, true>),        \
                     nb32 = resident_wgs((const void*)k_decompW<NN, PREC, false>);     \
    if (out_fp64)                                                                      \
      hipLaunchKernelGGL((k_decompW<NN, PREC, true>), decomp_grid(j, gx, nb, cus), dim3(256), 0, s, j, out); \
    else                                                                               \
      hipLaunchKernelGGL((k_decompW<NN, PREC, false>), decomp_grid(j, gx, nb32, cus), dim3(256), 0, s, j, out); \
    break;                                                                             \
  }
    ISR_FAST_ORDERS(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

inline hipError_t launch_quantW(const Job& j, hipStream_t s) {
  switch (j.order) {
#define CASE(NN)                                                                    \
  case NN:                                                                          \
    hipLaunchKernelGGL((k_quantW<NN>), dim3(j.gB, j.ncomp), dim3(256), 0, s, j);    \
    break;
    ISR_FAST_ORDERS(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int PREC>
hipError_t launch_fast_prec(int kind, const Job& j, int gx, hipStream_t s) {
  const dim3 grid(gx, j.ncomp), blk(256);
  switch (j.order) {
#define CASE(NN)                                                   \
  case NN:                                                         \
    if (kind == F_SAMPLE)                                          \
      hipLaunchKernelGGL((k_sample<NN, PREC>), grid, blk, 0, s, j); \
    else if (kind == F_PASSA)                                      \
      hipLaunchKernelGGL((k_passA<NN, PREC>), grid, blk, 0, s, j);  \
    else if (kind == F_PASSB)                                      \
      hipLaunchKernelGGL((k_passB<NN, PREC>), grid, blk, 0, s, j);  \
    else                                                           \
      return hipErrorInvalidValue;                                 \
    break;
    ISR_FAST_ORDERS(CASE)
#undef CASE
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int PREC>
int resident_fast_prec(int kind, int order) {
  int nb = 0;
  hipError_t e = hipErrorInvalidValue;
  switch (order) {
#define CASE(NN)                                                                                         \
  case NN:                                                                                               \
    if (kind == F_SAMPLE)                                                                                \
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_sample<NN, PREC>, 256, 0);   \
    else if (kind == F_PASSA)                                                                            \
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_passA<NN, PREC>, 256, 0);    \
    else if (kind == F_PASSB)                                                                            \
      e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_passB<NN, PREC>, 256, 0);    \
    if constexpr (PREC == P_FP64) {                                                                      \
      if (kind == F_QUANT)                                                                               \
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_quantW<NN>, 256, 0);        \
    }                                                                                                    \
    break;
    ISR_FAST_ORDERS(CASE)
#undef CASE
    default:
      break;
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return 2;
  }
  return nb > 0 ? nb : 1;
}

}  // namespace isr
