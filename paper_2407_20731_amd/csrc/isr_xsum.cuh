// Exact sums without atomics on the hot path, shared by the streaming
// passes (isr_engine.cuh) and the order-independent kernels (isr_select.hip).
//
// Every lane splits each non-negative term x <= M = 2^m into three parts on
// fixed grids by error-free extraction against powers of two (Rump, Ogita and
// Oishi, "Accurate floating-point summation part I", SIAM J. Sci. Comput.
// 31(1), 2008, Alg. 3.2) and keeps three FP64 running sums, which stay exact
// while a lane adds at most 2^(h-1) terms.  Terms far below M are summed by
// themselves (XFar); terms above it go to the global exponent bins.
// Workgroups publish the three sums as integers; the consumer adds them up
// as 128-bit integers and writes the exact total into exponent bins.  On the
// FP64 path every term is split this way; on the MFMA paths a lane first adds
// its terms in a fixed FP64 order and only that total is split (xadd_sum).
#pragma once

#include "isr_common.cuh"

namespace isr {

typedef double d2 __attribute__((ext_vector_type(2)));

// ---- exact sums by error-free extraction -------------------------------------
constexpr int XM_MIN = -876;  // keeps every extraction unit a normal number
constexpr int XM_MAX = 800;   // keeps the three 64-bit words of a total below bin 2047
constexpr int XH_MIN = 7, XH_MAX = 20;

// Units (exponents of 2) of the three parts: u1 = m + h - 52, u2 = m + 2h - 106,
// u3 = m + 3h - 159.  A lane may add at most 2^(h-1) terms.
struct XParm {
  double S1, S2, S3, u3, M;
  int m, h;
};

// 2^k for a normal exponent k, built from its bits (scalar instructions, so the
// parameters stay in scalar registers)
DEV double pow2(int k) { return __longlong_as_double((long long)(k + 1023) << 52); }

DEV XParm xparm(int m, int h) {
  XParm P;
  P.m = m;
  P.h = h;
  P.M = pow2(m);
  P.S1 = pow2(m + h);
  P.S2 = pow2(m + 2 * h - 53);
  P.S3 = pow2(m + 3 * h - 106);
  P.u3 = pow2(m + 3 * h - 159);
  return P;
}

// A uniform value hidden from the compiler, so that what is formed from it is
// formed here and not kept from an earlier place.
DEV int again(int m) {
  m = __builtin_amdgcn_readfirstlane(m);
  asm volatile("" : "+s"(m));
  return m;
}

struct XAcc {
  double a1, a2, a3;
};

// One term straight into the exact global exponent bins.
DEV void slow_bin(HistBin* g, double v) {
  const u64 bits = dbits(v);
  if (bits == 0ull) return;
  const int E = bits_exp(bits);
  u64 sig = (bits & M52) | (E ? (1ull << 52) : 0ull);
  if (E == 2047) sig = 0ull;
  global_bin_add(g, E, 1ull, sig & M21, sig >> 21);
}

// Running form of the three sums, for terms in [2^(m+3h-107), 2^m) (and exact
// zeros): the first two are held in accumulators biased to the middle of a
// binade, so that adding a term rounds it to the accumulator's own grid and
// the rounded part is the accumulator's change (three operations a level
// instead of the four of extracting against a fixed power of two and adding);
// what is left after two levels is a multiple of u3 for every term of that
// range, so the third sum takes it as it is.  At most 2^(h-1) terms: the
// accumulators stay in their binades (a1 in [2^(m+h), 1.5 2^(m+h)], grid u1;
// a2 within 2^(m+2h-54) of 1.5 2^(m+2h-53), grid 2 u2) and |a3| stays within
// 2^52 u3.  Terms outside the range (at h = 12 those below 2^-71 of the bound)
// are left to XFar: next to none of a noisy field's, a quarter to three quarters of
// a smooth field's energies.  N = 7, 65,536 elements, FP64: pass A 517 -> 342 us,
// pass B 517 -> 441 us, with the registers that the shorter sums free.
struct XRun {
  double a1, a2, a3;
};

DEV XRun xrun(const XParm& P) { return {P.S1, 1.5 * P.S2, 0.0}; }

// The range test on the high words alone (both ends have zero low words):
// false for zero, tiny, large and negative terms, Inf and NaN.
struct XRange {
  u32 lo, span;
};
DEV u32 hi_word(double x) { return (u32)((u64)__double_as_longlong(x) >> 32); }
DEV XRange xrange(const XParm& P) {
  const u32 lo = hi_word(pow2(P.m + 3 * P.h - 107));
  return {lo, hi_word(P.M) - lo};
}
DEV bool xin(const XRange& R, double x) { return hi_word(x) - R.lo < R.span; }

// y in range, or zero
DEV void xrun_add(XRun& A, double y) {
  const double t1 = A.a1 + y;
  const double r1 = y - (t1 - A.a1);
  A.a1 = t1;
  const double t2 = A.a2 + r1;
  A.a3 = A.a3 + (r1 - (t2 - A.a2));
  A.a2 = t2;
}

// Keeps a tile's additions where they stand: the compiler otherwise sinks them
// to the end of the loop and holds every slot's operands until there.  (On the
// MFMA paths, one add a term, that is the better order: 196 us against 216.)
DEV void pin(XRun& A) { asm volatile("" : "+v"(A.a1), "+v"(A.a2), "+v"(A.a3)); }

// Adds x when it is in range; otherwise true: unless it is zero, x belongs in the
// sums below (XFar) or, too large, in the exact bins.
DEV bool xrun_left(XRun& A, const XRange& R, double x) {
  const bool in = xin(R, x);
  xrun_add(A, in ? x : 0.0);
  return !in;
}

DEV XAcc xrun_sums(const XRun& A, const XParm& P) { return {A.a1 - P.S1, A.a2 - 1.5 * P.S2, A.a3}; }

// A lane's fixed-order FP64 sum s of at most 2^(h-1) terms in [0, M] (so
// s <= 2^(m+h-1)) added to the three sums, exactly down to u3; returns what
// is left for the global bins: the part below u3 (0 <= r < 2 u3), or s itself
// when it is out of that range (Inf and NaN included).
DEV double xadd_sum(XAcc& A, const XParm& P, double s) {
  const bool in = s >= 0.0 && s <= 0.5 * P.S1;
  const double y = in ? s : 0.0;
  const double q1 = (P.S1 + y) - P.S1;
  const double r1 = y - q1;
  const double q2 = (P.S2 + r1) - P.S2;
  const double r2 = r1 - q2;
  const double t3 = (P.S3 + r2) - P.S3;
  const double q3 = t3 > r2 ? t3 - P.u3 : t3;
  A.a1 = A.a1 + q1;
  A.a2 = A.a2 + q2;
  A.a3 = A.a3 + q3;
  return in ? r2 - q3 : s;
}

// The three sums as integers in their units (exact: |sum| < 2^53 units).
DEV void xints(const XAcc& A, const XParm& P, long long (&k)[3]) {
  k[0] = (long long)ldexp(A.a1, -(P.m + P.h - 52));
  k[1] = (long long)ldexp(A.a2, -(P.m + 2 * P.h - 106));
  k[2] = (long long)ldexp(A.a3, -(P.m + 3 * P.h - 159));
}

// 192-bit two's complement integer.
struct I192 {
  u64 w[3];
};

DEV void i192_add_shl(I192& z, __int128 v, int sh) {  // z += v << sh, 0 <= sh < 128
  const unsigned __int128 uv = (unsigned __int128)v;
  u64 a[3] = {(u64)uv, (u64)(uv >> 64), v < 0 ? ~0ull : 0ull};
  while (sh >= 64) {
    a[2] = a[1];
    a[1] = a[0];
    a[0] = 0ull;
    sh -= 64;
  }
  if (sh) {
    a[2] = (a[2] << sh) | (a[1] >> (64 - sh));
    a[1] = (a[1] << sh) | (a[0] >> (64 - sh));
    a[0] = a[0] << sh;
  }
  u64 c = 0;
  for (int k = 0; k < 3; ++k) {
    const u64 s = z.w[k] + a[k];
    const u64 c1 = s < z.w[k];
    const u64 s2 = s + c;
    const u64 c2 = s2 < s;
    z.w[k] = s2;
    c = c1 | c2;
  }
}

// Adds v (< 2^85) units of bin b to the global bins.  The bin also counts
// one term: readers skip bins whose count is zero (the counts of these bins,
// all below the boundary bin, are never used otherwise).
DEV void add_piece(HistBin* g, int b, unsigned __int128 v) {
  if (v == 0) return;
  const u64 lo = (u64)v & M21;
  const u64 hi = (u64)(v >> 21);
  atomicAdd(&g[b].cnt, 1ull);
  if (lo) atomicAdd(&g[b].lo, lo);
  if (hi) atomicAdd(&g[b].hi, hi);
}

// Exact total of three integer sums (units u1, u2, u3 of XParm(m, h)) as bins.
// btop < 0: three 64-bit words at the bins of u3, u3 * 2^64, u3 * 2^128;
// btop >= 0: all of it in bins <= btop (the part above bit btop - b3 in btop).
DEV void emit_total(HistBin* g, const __int128 (&K)[3], int m, int h, int btop) {
  I192 z = {{0ull, 0ull, 0ull}};
  i192_add_shl(z, K[0], 107 - 2 * h);
  i192_add_shl(z, K[1], 53 - h);
  i192_add_shl(z, K[2], 0);
  const int b3 = m + 3 * h + 916;  // bin whose unit is u3
  if (btop < 0) {
    for (int k = 0; k < 3; ++k) add_piece(g, b3 + 64 * k, z.w[k]);
    return;
  }
  const int d = btop - b3;  // 46..85 for the window placements used
  const unsigned __int128 lo128 = ((unsigned __int128)z.w[1] << 64) | z.w[0];
  const unsigned __int128 mask = d >= 128 ? ~(unsigned __int128)0 : (((unsigned __int128)1 << d) - 1);
  add_piece(g, b3, lo128 & mask);
  // z >> d (fits 85 bits: the total is below 2^32 terms of at most M each)
  unsigned __int128 hi128;
  if (d < 64)
    hi128 = (lo128 >> d) | ((unsigned __int128)z.w[2] << (128 - d));
  else
    hi128 = (((unsigned __int128)z.w[2] << 64) | z.w[1]) >> (d - 64);
  add_piece(g, btop, hi128);
}

// Wave sums over data-parallel lane moves (six steps of a few cycles each;
// the LDS permutes of a shuffle wait some hundred cycles a step), the same
// value in every lane.  Row shifts sum the rows of 16 into their last lanes,
// the row broadcasts carry those on to lane 63.
template <int CTRL, int ROWS>
DEV u64 dpp64(u64 v) {
  const u32 lo = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)v, CTRL, ROWS, 0xf, false);
  const u32 hi = (u32)__builtin_amdgcn_update_dpp(0, (int)(u32)(v >> 32), CTRL, ROWS, 0xf, false);
  return ((u64)hi << 32) | lo;
}
template <class OP>
DEV u64 wave_reduce_dpp(u64 v, OP op) {  // op(x, 0) == x
  v = op(v, dpp64<0x111, 0xf>(v));  // row_shr 1, 2, 4, 8
  v = op(v, dpp64<0x112, 0xf>(v));
  v = op(v, dpp64<0x114, 0xf>(v));
  v = op(v, dpp64<0x118, 0xf>(v));
  v = op(v, dpp64<0x142, 0xa>(v));  // row_bcast 15 into rows 1 and 3
  v = op(v, dpp64<0x143, 0xc>(v));  // row_bcast 31 into rows 2 and 3
  return bcast64(v, 63);
}
DEV double wave_sum_dpp(double v) {
  return __longlong_as_double((long long)wave_reduce_dpp(dbits(v), [](u64 a, u64 b) {
    return dbits(__longlong_as_double((long long)a) + __longlong_as_double((long long)b));
  }));
}
DEV u64 wave_sum_dpp(u64 v) {
  return wave_reduce_dpp(v, [](u64 a, u64 b) { return a + b; });
}
DEV u64 wave_max_dpp(u64 v) {
  return wave_reduce_dpp(v, [](u64 a, u64 b) { return a > b ? a : b; });
}

// The same total as a wave-distributed big integer (X units of 2^-1075), from
// sums that every lane holds.
DEV u64 total_words(const __int128 (&K)[3], int m, int h) {
  I192 z = {{0ull, 0ull, 0ull}};
  i192_add_shl(z, K[0], 107 - 2 * h);
  i192_add_shl(z, K[1], 53 - h);
  i192_add_shl(z, K[2], 0);
  const int sh = m + 3 * h + 916;  // u3 in X units: at least 2^61
  u64 w = part_at(z.w[0], z.w[1], sh);
  wb_add(w, part_at(z.w[2], 0ull, sh + 128));
  return w;
}

// Terms below the running sums' range, a tile's at a time: three sums as above, over
// the whole wave, take those within 77 binades of the range's end; if terms are left,
// the largest of them sets the bound of the next three, and so on.  Each total goes
// into 32-bit digits in LDS, of the workgroup, which cover all exponents.
// Smooth fields live on this (energies that are rounding noise, and the noise of the
// noise where the field does not vary along an axis; errors of elements that keep
// everything): a global atomic or three each into the exact bins, on a few dozen
// of them, made the request 164 ms at N = 9, 32,768 elements, Taylor-Green, FP64, 3
// components, where it takes 2.15 ms so (noisy field: 1.53); N = 7, 65,536 elements
// 72.4 -> 1.38 ms (0.92).  One second set of three sums alone took 1.95 and 1.33 ms,
// but left what is far below that range too to the bins: 393 elements of N = 10,
// Taylor-Green in a plane, 1235 us where it takes 221 (noisy 190); 719 of N = 8,
// noisy X 1e-150, per-element cut 26.3 ms where it takes 0.17.
constexpr int XF_H = 10;    // at most 2^9 terms: eight a lane
constexpr int XF_DIG = 62;  // terms below 2^XM_MAX

DEV int xfar_m(int m, int h) { return m + 3 * h - 107; }

struct XFar {
  u64 d[XF_DIG];  // digit k counts 2^(32 k) X units of 2^-1075 (room for 2^32 carries)
};

// (by the whole workgroup, ahead of a barrier)
DEV void xfar_clear(XFar& F, int tid) {
  if (tid < XF_DIG) F.d[tid] = 0ull;
}

// The thread's number hidden from the compiler (no address made from it is kept
// across tiles).
DEV int again_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// The k slots of terms in the wave's LDS buffer (the first LANES lanes; zero in the
// others), those with out(x), by the whole wave; m: the running sums take from 2^m on.
template <int LANES, class OUT>
DEV void xfar_sum(XFar& F, HistBin* g, const double* buf, int k, int lane, int m, OUT out) {
  auto term = [&](int s) {
    const double v = LANES == 64 || lane < LANES ? buf[LANES * s + lane] : 0.0;
    return out(v) ? v : 0.0;
  };
  u64 limit = dbits(pow2(m));  // terms not yet taken are below
#pragma unroll 1
  for (bool first = true;; first = false) {
    const int up = m < XM_MIN ? 256 : 0;  // (scaled, exactly, so that every unit is normal)
    const XParm P = xparm(m + up, XF_H);
    const XRange R = xrange(P);
    const double scale = pow2(up);
    XRun A = xrun(P);
    bool rest = false;
#pragma unroll 1
    for (int s = 0; s < k; ++s) {
      const double v = term(s);
      const u64 b = dbits(v);
      if (first && b >= limit) slow_bin(g, v);  // (above the running sums' range, Inf, NaN)
      const double y = b < limit ? v * scale : 0.0;
      const bool in = xin(R, y);
      xrun_add(A, in ? y : 0.0);
      rest = (!in && y != 0.0) || rest;
    }
    // multiples of a unit, below 2^53 of it: the wave's sums are exact too
    const XAcc S = xrun_sums(A, P);
    const XAcc T = {wave_sum_dpp(S.a1), wave_sum_dpp(S.a2), wave_sum_dpp(S.a3)};
    long long K[3];
    xints(T, P, K);
    I192 z = {{0ull, 0ull, 0ull}};
    i192_add_shl(z, (__int128)K[0], 107 - 2 * XF_H);
    i192_add_shl(z, (__int128)K[1], 53 - XF_H);
    i192_add_shl(z, (__int128)K[2], 0);
    int at = m + 3 * XF_H + 916;  // u3 in X units; z has no bits below the first of those
    for (; at < 0; ++at) {
      z.w[0] = (z.w[0] >> 1) | (z.w[1] << 63);
      z.w[1] = (z.w[1] >> 1) | (z.w[2] << 63);
      z.w[2] >>= 1;
    }
    const int r = at & 63;
    const u64 w0 = z.w[0] << r, w1 = r ? (z.w[1] << r) | (z.w[0] >> (64 - r)) : z.w[1],
              w2 = r ? (z.w[2] << r) | (z.w[1] >> (64 - r)) : z.w[2], w3 = r ? z.w[2] >> (64 - r) : 0ull;
    const u64 w = lane < 4 ? (lane < 2 ? w0 : w1) : (lane < 6 ? w2 : w3);
    const u64 digit = lane & 1 ? w >> 32 : w & 0xffffffffull;
    if (lane < 8 && digit) atomicAdd((unsigned long long*)&F.d[2 * (at >> 6) + lane], (unsigned long long)digit);
    if (!ballot(rest)) return;
    limit = dbits(ldexp(1.0, m + 3 * XF_H - 107));
    u64 mk = 0ull;
#pragma unroll 1
    for (int s = 0; s < k; ++s) {
      const u64 b = dbits(term(s));
      mk = b < limit && b > mk ? b : mk;
    }
    m = (int)(wave_max_dpp(mk) >> 52) - 1022;  // every term left is below 2^m
  }
}

// One tile's terms x of the first LANES lanes (zero in the others), those with
// out(x).  m: xfar_m of the running sums.  ZEROS: called for tiles that only have
// exact zeros there too.  By way of the wave's LDS buffer, CH slots at a time, and
// in rolled loops: unrolled on registers this branch took the prefetched tile's
// (N = 7, 65,536 elements, noisy field: the request 911 us without the branch, 1217
// with it unrolled, 917 so).
template <int LANES, int CH, bool ZEROS, int CNT, int LDSW, class OUT>
DEV void xfar_tile(XFar& F, int m, HistBin* g, double (*bufs)[LDSW], const double (&x)[CNT], OUT out) {
  static_assert(CH * LANES <= LDSW, "the terms fit the wave's buffer");
  static_assert(CH * 64 <= 1 << (XF_H - 1), "the wave's sums are exact");
  if constexpr (ZEROS) {
    bool any = false;
#pragma unroll
    for (int s = 0; s < CNT; ++s) any = (out(x[s]) && x[s] != 0.0) || any;
    if (!ballot(any)) return;
  }
  const int tid = again_tid(), lane = tid & 63;
  double* buf = bufs[tid >> 6];
#pragma unroll
  for (int c = 0; c < CNT; c += CH) {
    const int k = CNT - c < CH ? CNT - c : CH;
#pragma unroll
    for (int s = 0; s < k; ++s)
      if (LANES == 64 || lane < LANES) buf[LANES * s + lane] = x[c + s];
    asm volatile("" ::: "memory");
    xfar_sum<LANES>(F, g, buf, k, lane, again(m), out);
    asm volatile("" ::: "memory");
  }
}

// The workgroup's digits into the exact bins, each in a bin below its own magnitude
// (by the whole workgroup, behind a barrier).
DEV void xfar_out(const XFar& F, HistBin* g, int tid) {
  if ((u32)tid >= (u32)XF_DIG) return;
  const u64 v = F.d[tid];
  if (tid == 0)
    add_piece(g, 1, v >> 1);
  else
    add_piece(g, 32 * tid - 20, (unsigned __int128)v << 20);
}

DEV long long wave_sum_i64(long long v) { return (long long)wave_sum64((u64)v); }

DEV double wave_sum_f64(double v) {
  for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m);
  return v;
}

// Workgroup of 256: sums `cnt` signed 64-bit values per thread into out[k]
// (thread 0 holds the totals afterwards in red[0][k]).
template <int CNT>
DEV void block_sum_i64(long long (&v)[CNT], long long (*red)[8], int tid) {
  const int lane = tid & 63, wv = tid >> 6;
#pragma unroll
  for (int k = 0; k < CNT; ++k) {
    const long long s = wave_sum_i64(v[k]);
    if (lane == 0) red[wv][k] = s;
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int k = 0; k < CNT; ++k) red[0][k] = red[0][k] + red[1][k] + red[2][k] + red[3][k];
  }
  __syncthreads();
}

DEV __int128 shfl_xor128(__int128 v, int m) {
  const unsigned __int128 u = (unsigned __int128)v;
  const u64 lo = shfl_xor64((u64)u, m), hi = shfl_xor64((u64)(u >> 64), m);
  return (__int128)(((unsigned __int128)hi << 64) | lo);
}

// Workgroup of 256: totals of fields 0..F-1 over `count` rows of `stride`
// 64-bit signed values starting at base (row r, field f at base[r * stride +
// f]), as 128-bit integers, in every thread.  Every field of a row is loaded
// at once, so the workgroup waits for memory once.  red: [4][F] of LDS.
template <int F>
DEV void block_totals(const long long* base, int count, int stride, __int128 (&tot)[F], __int128 (*red)[F], int tid) {
  const int lane = tid & 63, wv = tid >> 6;
  __int128 p[F];
#pragma unroll
  for (int f = 0; f < F; ++f) p[f] = 0;
  for (int r = tid; r < count; r += 256) {
    long long v[F];
#pragma unroll
    for (int f = 0; f < F; ++f) v[f] = base[(size_t)r * stride + f];
#pragma unroll
    for (int f = 0; f < F; ++f) p[f] += (__int128)v[f];
  }
#pragma unroll
  for (int f = 0; f < F; ++f)
    for (int m = 32; m > 0; m >>= 1) p[f] += shfl_xor128(p[f], m);
  if (lane == 0)
#pragma unroll
    for (int f = 0; f < F; ++f) red[wv][f] = p[f];
  __syncthreads();
#pragma unroll
  for (int f = 0; f < F; ++f) tot[f] = red[0][f] + red[1][f] + red[2][f] + red[3][f];
  __syncthreads();
}

// Last workgroup of a component to finish (returns true in every thread of
// that workgroup, after an acquire fence).
DEV bool last_block(u32* counter, int* flag_lds, int nblocks) {
  __threadfence();
  __syncthreads();
  if (threadIdx.x == 0) *flag_lds = atomicAdd(counter, 1u) == (u32)(nblocks - 1);
  __syncthreads();
  const bool last = *flag_lds != 0;
  if (last) __threadfence();
  return last;
}

}  // namespace isr
