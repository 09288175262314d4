// Device building blocks shared by the kernels: shapes, exact-sum histograms,
// wave-distributed big integers, and the FP64 fixed-order contractions.
#pragma once

#include "isr_internal.h"

namespace isr {

#define DEV __device__ __forceinline__

constexpr u64 M52 = (1ull << 52) - 1;
constexpr u64 M21 = (1ull << 21) - 1;
constexpr u64 M43 = (1ull << 43) - 1;
constexpr u64 M62 = (1ull << 62) - 1;
typedef unsigned __int128 u128;

// ---- element tile shapes --------------------------------------------------
// A workgroup works on EPI elements at a time; one thread per (element,
// pencil) with n^2 pencils per element.
template <int N>
struct Shape {
  static constexpr int n = N + 1, n2 = n * n, n3 = n2 * n;
  static constexpr int EPI = (256 / n2) > 0 ? (256 / n2) : 1;
  static constexpr int ACT = EPI * n2;
  static constexpr int THREADS = ((ACT + 63) / 64) * 64;
  static constexpr int TILE = EPI * n3;
  static constexpr int W = (n3 + 63) / 64;
};

DEV u64 dbits(double v) { return (u64)__double_as_longlong(v); }
DEV int lane_id() { return (int)__lane_id(); }

// ---- wave helpers -----------------------------------------------------------
DEV u64 ballot(bool p) { return (u64)__ballot(p); }
// this lane's bit of a wave mask, and the set bits below it
DEV bool lane_bit(u64 m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
DEV u32 lane_rank(u64 m) { return __builtin_amdgcn_mbcnt_hi((u32)(m >> 32), __builtin_amdgcn_mbcnt_lo((u32)m, 0u)); }
DEV u64 bcast64(u64 v, int src) {
  u32 lo = (u32)__builtin_amdgcn_readlane((int)(u32)v, src);
  u32 hi = (u32)__builtin_amdgcn_readlane((int)(u32)(v >> 32), src);
  return ((u64)hi << 32) | lo;
}
// v with lane DST's value replaced by the uniform s.  The compiler puts two wait
// states between a vector instruction that writes a scalar register (a compare, a
// lane read) and one that reads it, but does not look into inline assembly.
template <int DST>
DEV u64 writelane64(u64 s, u64 v) {
  u32 lo = (u32)v, hi = (u32)(v >> 32);
  const u32 slo = (u32)__builtin_amdgcn_readfirstlane((int)(u32)s);
  const u32 shi = (u32)__builtin_amdgcn_readfirstlane((int)(u32)(s >> 32));
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
      : "+v"(lo), "+v"(hi)
      : "s"(slo), "s"(shi), "n"(DST));
  return ((u64)hi << 32) | lo;
}
DEV u64 shfl_xor64(u64 v, int m) {
  u32 lo = (u32)__shfl_xor((int)(u32)v, m);
  u32 hi = (u32)__shfl_xor((int)(u32)(v >> 32), m);
  return ((u64)hi << 32) | lo;
}
DEV u64 shfl_up64(u64 v, int d) {
  u32 lo = (u32)__shfl_up((int)(u32)v, d);
  u32 hi = (u32)__shfl_up((int)(u32)(v >> 32), d);
  return ((u64)hi << 32) | lo;
}
DEV u64 wave_sum64(u64 v) {
  for (int m = 32; m > 0; m >>= 1) v += shfl_xor64(v, m);
  return v;
}

// ---- wave-distributed big integers ----------------------------------------
// Lane l holds 64-bit word l of a 4096-bit two's complement integer.  Sums of
// energies live in "X units" of 2^-1075, needing at most ~2150 bits, so the
// top lanes are sign extension.  Carries/borrows resolve in O(1) wave steps:
// with G = lanes that generate and P = lanes that propagate, the carry into
// every lane is ((G + (G|P)) ^ G ^ (G|P)).
DEV u64 carry_in(u64 G, u64 P) {
  u64 Y = G | P;
  return (G + Y) ^ G ^ Y;
}
DEV void wb_add(u64& w, u64 part) {
  u64 s = w + part;
  u64 c = carry_in(ballot(s < w), ballot(s == ~0ull));
  w = s + ((c >> lane_id()) & 1ull);
}
DEV void wb_sub(u64& w, u64 part) {
  u64 d = w - part;
  u64 c = carry_in(ballot(w < part), ballot(d == 0ull));
  w = d - ((c >> lane_id()) & 1ull);
}
// This lane's share of the 128-bit value (lo, hi) shifted left by s bits.
DEV u64 part_at(u64 lo, u64 hi, int s) {
  int q = s >> 6, r = s & 63, l = lane_id();
  if (l == q) return lo << r;
  if (l == q + 1) return r ? ((lo >> (64 - r)) | (hi << r)) : hi;
  if (l == q + 2) return r ? (hi >> (64 - r)) : 0ull;
  return 0ull;
}
DEV bool wb_neg(u64 w) { return (bcast64(w, 63) >> 63) != 0; }

// Round a non-negative big integer in X units to the nearest double (ties to
// even).
DEV double wb_round(u64 w) {
  u64 nz = ballot(w != 0);
  if (!nz) return 0.0;
  int L = 63 - __clzll((long long)nz);
  u64 top = bcast64(w, L);
  int t = 64 * L + 63 - __clzll((long long)top);  // highest set bit
  int lsb = t - 52 > 1 ? t - 52 : 1;              // X-unit weight of the result's ulp
  int q = lsb >> 6, r = lsb & 63;
  u64 a = bcast64(w, q);
  u64 b = (q + 1 < 64) ? bcast64(w, q + 1) : 0ull;
  u64 m = r ? ((a >> r) | (b << (64 - r))) : a;   // at most 53 significant bits
  int rb_pos = lsb - 1;
  int rq = rb_pos >> 6, rr = rb_pos & 63;
  u64 rw = bcast64(w, rq);
  u64 rbit = (rw >> rr) & 1ull;
  bool sticky = ((rw & ((1ull << rr) - 1ull)) != 0ull) || (ballot(w != 0 && lane_id() < rq) != 0ull);
  if (rbit && (sticky || (m & 1ull))) m += 1ull;
  return ldexp((double)m, lsb - 1075);
}

// 128 bits of the big integer starting at bit s; sat = bits above them exist.
DEV void wb_extract128(u64 w, int s, u64& lo, u64& hi, bool& sat) {
  int q = s >> 6, r = s & 63;
  u64 a = bcast64(w, q), b = bcast64(w, q + 1), c = bcast64(w, q + 2);
  lo = r ? ((a >> r) | (b << (64 - r))) : a;
  hi = r ? ((b >> r) | (c << (64 - r))) : b;
  u64 rest = r ? (c >> r) : c;
  sat = rest != 0ull || ballot(w != 0 && lane_id() > q + 2) != 0ull;
}

// Significand sum of one exponent bin as a 128-bit integer.
DEV u128 bin_sum(const HistBin& h) { return ((u128)h.hi << 21) + (u128)h.lo; }

// Walks over a histogram's non-empty bins in ascending order, by one wave.
// The bins' counts are loaded first, 64 neighbouring bins a load and all loads
// in flight at once; a round of 64 bins is looked at again only when one of its
// counts is set (two or three of the 32 rounds: exponents sit together).  The
// code is short on purpose: these walks run once per kernel, on a cold
// instruction cache, and their unrolled forms (32 bins a lane, 128-bit shifts
// per bin) spent most of their ~20 us fetching instructions.
constexpr int HROUNDS = HBINS / 64;

// Lane l's counts of bins 64 k + l; bin 2047 (non-finite) is excluded.
DEV void hist_counts(const HistBin* H, u64 (&c)[HROUNDS]) {
#pragma unroll
  for (int k = 0; k < HROUNDS; ++k) {
    const int b = 64 * k + lane_id();
    c[k] = H[b].cnt;  // (HBINS bins: always inside)
  }
  // all of the loads before the first use (left to itself the compiler waits
  // for each in turn)
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int k = 0; k < HROUNDS; k += 8)
    asm volatile("" : "+v"(c[k]), "+v"(c[k + 1]), "+v"(c[k + 2]), "+v"(c[k + 3]), "+v"(c[k + 4]), "+v"(c[k + 5]),
                      "+v"(c[k + 6]), "+v"(c[k + 7]));
  if (lane_id() == 63) c[HROUNDS - 1] = 0ull;  // bin 2047
}
// Bit k: round k has a non-empty bin.
DEV u32 hist_rounds(const u64 (&c)[HROUNDS]) {
  u32 r = 0u;
#pragma unroll
  for (int k = 0; k < HROUNDS; ++k) r |= ballot(c[k] != 0ull) ? (1u << k) : 0u;
  return r;
}
// fn(bin, lo, hi, count) for every non-empty bin, ascending, with the bin's
// significand sum (lo, hi) and count in every lane; stops when fn is false.
template <class FN>
DEV void hist_walk(const HistBin* H, u32 rounds, FN fn) {
  while (rounds) {
    const int k = __ffs((int)rounds) - 1;
    rounds &= rounds - 1u;
    const int b = 64 * k + lane_id();
    const HistBin h = b < HBINS - 1 ? H[b] : HistBin{0ull, 0ull, 0ull};
    const u128 s = bin_sum(h);
    u64 m = ballot(h.cnt != 0ull);
    while (m) {
      const int l = __ffsll((long long)m) - 1;
      m &= m - 1ull;
      if (!fn(64 * k + l, bcast64((u64)s, l), bcast64((u64)(s >> 64), l), bcast64(h.cnt, l))) return;
    }
  }
}

// Exact total of a histogram as a wave-distributed big integer.
DEV u64 hist_sum(const HistBin* H, u32 rounds) {
  u64 acc = 0;
  hist_walk(H, rounds, [&](int bin, u64 lo, u64 hi, u64) {
    wb_add(acc, part_at(lo, hi, bin > 1 ? bin : 1));
    return true;
  });
  return acc;
}
DEV u64 hist_total(const HistBin* H) {
  u64 c[HROUNDS];
  hist_counts(H, c);
  return hist_sum(H, hist_rounds(c));
}

// ---- LDS histogram window of one workgroup ----------------------------------
// HC copies of every bin (lane parity picks the copy) halve same-address
// atomic conflicts inside a wave.
constexpr int HC = 2;
struct LdsHist {
  u64 w[WIN][HC][2];  // [0] = (count << 43) + sum(sig & (2^21-1)), [1] = sum(sig >> 21)
  u32 zero;           // exact zeros
  int lo;             // exponent of w[0]
  int maxE;
  int pad;
};

DEV void lh_init(LdsHist& h, int tid, int nthr) {
  u64* p = &h.w[0][0][0];
  for (int k = tid; k < WIN * HC * 2; k += nthr) p[k] = 0ull;
  if (tid == 0) {
    h.zero = 0u;
    h.maxE = 0;
    h.lo = 0;
  }
}

DEV void global_bin_add(HistBin* g, int E, u64 cnt, u64 lo, u64 hi) {
  if (cnt) atomicAdd(&g[E].cnt, cnt);
  if (lo) atomicAdd(&g[E].lo, lo);
  if (hi) atomicAdd(&g[E].hi, hi);
}

DEV int bits_exp(u64 bits) {
  return (bits >> 63) ? 2047 : (int)(bits >> 52);  // negative = only NaN here
}

DEV void lh_insert(LdsHist& h, HistBin* g, double v) {
  u64 bits = dbits(v);
  if (bits == 0ull) {
    atomicAdd(&h.zero, 1u);
    return;
  }
  int E = bits_exp(bits);
  u64 sig = (bits & M52) | (E ? (1ull << 52) : 0ull);
  if (E == 2047) sig = 0;
  int b = E - h.lo;
  if ((unsigned)b < (unsigned)WIN) {
    const int cp = lane_id() & (HC - 1);
    atomicAdd(&h.w[b][cp][0], (1ull << 43) + (sig & M21));
    atomicAdd(&h.w[b][cp][1], sig >> 21);
  } else {
    global_bin_add(g, E, 1ull, sig & M21, sig >> 21);
  }
}

// Window placement from the largest exponent seen in the first tile.
DEV void lh_note_max(LdsHist& h, double v) {
  int E = bits_exp(dbits(v));
  if (E > 0 && E < 2047) atomicMax(&h.maxE, E);
}
DEV void lh_place(LdsHist& h) { h.lo = h.maxE + WIN_HEAD - WIN + 1; }

DEV void lh_flush(LdsHist& h, HistBin* g, int tid, int nthr) {
  for (int b = tid; b < WIN; b += nthr) {
    u64 cnt = 0, lo = 0, hi = 0;
    for (int cp = 0; cp < HC; ++cp) {
      const u64 w0 = h.w[b][cp][0];
      cnt += w0 >> 43;
      lo += w0 & M43;
      hi += h.w[b][cp][1];
    }
    if (cnt | lo | hi) global_bin_add(g, h.lo + b, cnt, lo, hi);
  }
  if (tid == 0 && h.zero) atomicAdd(&g[0].cnt, (u64)h.zero);
}

// ---- candidate lists -------------------------------------------------------------
// List 0 of every component (the candidates, capacity list_cap), then list 1 of
// every component: the members of the threshold's sub-bin, once they are few
// enough to be sorted (at most CAP, and never more than there are candidates).
DEV u64 list_capk(const Job& j, int k) { return k == 0 || j.list_cap < (u64)CAP ? j.list_cap : (u64)CAP; }
DEV u64* list_ptr(const Job& j, int comp, int k) {
  return j.lists + (size_t)(k * j.ncomp) * j.list_cap + (size_t)comp * list_capk(j, k);
}

// ---- decoupled look-back --------------------------------------------------------
// Descriptor per tile: flag << 62 | value; flag 1 = aggregate, 2 = inclusive
// prefix.  publish() posts the tile's aggregate (tile 0 posts its prefix);
// wait() reads 64 predecessors at a time (lane i: tile base - i) until one
// carries an inclusive prefix, then posts the tile's own prefix.  Both run on
// one whole wave.
DEV u64 lb_load(const u64* p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT); }
DEV void lb_store(u64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT); }

DEV u64 tile_agg(const u32* cntl, int ne) {
  u64 agg = 0;
  for (int k = 0; k < ne; ++k) agg += cntl[k];
  return agg;
}

DEV void lookback_publish(u64* lb, long long t, const u32* cntl, int ne, u64* excl_out) {
  if (lane_id() != 0) return;
  const u64 agg = tile_agg(cntl, ne);
  if (t == 0) {
    lb_store(&lb[0], (2ull << 62) | agg);
    *excl_out = 0ull;
  } else {
    lb_store(&lb[t], (1ull << 62) | agg);
  }
}

constexpr int SPIN_LIMIT = 1 << 24;

DEV void lookback_wait(u64* lb, long long t, const u32* cntl, int ne, int* flags, u64* excl_out) {
  if (t == 0) return;
  const int lane = lane_id();
  u64 ex = 0;
  long long base = t - 1;
  for (;;) {
    const long long idx = base - lane;
    u64 sv = 2ull << 62;  // before tile 0: an inclusive prefix of 0
    if (idx >= 0) {
      int spins = 0;
      for (;;) {
        sv = lb_load(&lb[idx]);
        if ((sv >> 62) != 0ull || ++spins >= SPIN_LIMIT) break;
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (ballot((sv >> 62) == 0ull)) {  // a predecessor never published (cannot happen)
      if (lane == 0) atomicOr(flags, ST_SPIN);
      break;
    }
    const u64 pm = ballot((sv >> 62) == 2ull);
    const int stop = pm ? (__ffsll((long long)pm) - 1) : 63;
    ex += wave_sum64(lane <= stop ? (sv & M62) : 0ull);
    if (pm) break;
    base -= 64;
  }
  if (lane == 0) {
    lb_store(&lb[t], (2ull << 62) | (ex + tile_agg(cntl, ne)));
    *excl_out = ex;
  }
}

// ---- FP64 fixed-order contraction ---------------------------------------------
// y[a] = M[a][0]*x[0] + M[a][1]*x[1] + ... left to right, every product and
// sum rounded separately (the library is built with -ffp-contract=off).
//
// The matrix entries are read through the scalar cache into scalar registers
// (the multiplies take them as their scalar operand), so a contraction issues
// no vector or LDS load of its own.  Broadcast vector loads of the entries
// cost 16 L1 cycles per two of them (n = 8: 96 such loads a forward transform,
// which alone was the passes' time), broadcast LDS reads 8 cycles.  N = 7,
// 65,536 elements, 3 components: pass A 866 -> 517 us, pass B 1231 -> 517 us.
//
// The tables are symmetric about the element's middle, bit for bit (a CPU
// test checks every order):
//   A[p][n-1-i] = (-1)^p A[p][i]      V[n-1-i][k] = (-1)^k V[i][k]
// so only half of the entries are read, and in the inverse the products of
// the mirrored rows i and n-1-i are the same up to the sign and are formed
// once.  Negation is exact and IEEE subtraction is the addition of the
// negated operand: the results are those of the full matrices, bit for bit.
typedef __attribute__((address_space(4))) const double sdouble;

// Base of a group of table rows, opaque to the compiler: the rows of a group
// are loaded here, instead of every row of every stage being held (or
// spilled) across the whole transform.
DEV sdouble* table_rows(const double* M) {
  // (the pointer is the same in every lane; in the batch kernel it comes from
  // memory, so the compiler has to be told)
  const uintptr_t m = (uintptr_t)M;
  uintptr_t p = (uintptr_t)(u32)__builtin_amdgcn_readfirstlane((int)(u32)m) |
                ((uintptr_t)(u32)__builtin_amdgcn_readfirstlane((int)(u32)(m >> 32)) << 32);
  asm volatile("" : "+s"(p));
  return (sdouble*)p;
}

constexpr int SROWS = 16;  // table entries in flight (32 of the ~100 scalar registers)

// y = A x
template <int n>
DEV void forward64(const double* A, const double (&x)[n], double (&y)[n]) {
  constexpr int H = (n + 1) / 2;
  constexpr int G = SROWS / H < n ? SROWS / H : n;  // rows per group
#pragma unroll
  for (int a0 = 0; a0 < n; a0 += G) {
    sdouble* M = table_rows(A + a0 * n);
#pragma unroll
    for (int a = a0; a < (a0 + G < n ? a0 + G : n); ++a) {
      double acc = M[(a - a0) * n] * x[0];
#pragma unroll
      for (int b = 1; b < n; ++b) {
        const double t = M[(a - a0) * n + (b < H ? b : n - 1 - b)] * x[b];
        acc = b >= H && (a & 1) ? acc - t : acc + t;
      }
      y[a] = acc;
    }
  }
}

// y = V x
template <int n>
DEV void inverse64(const double* V, const double (&x)[n], double (&y)[n]) {
  constexpr int H = (n + 1) / 2;
  constexpr int G = SROWS / n < H ? SROWS / n : H;
#pragma unroll
  for (int a0 = 0; a0 < H; a0 += G) {
    sdouble* M = table_rows(V + a0 * n);
#pragma unroll
    for (int a = a0; a < (a0 + G < H ? a0 + G : H); ++a) {
      double t = M[(a - a0) * n] * x[0];
      double acc = t, mir = t;
#pragma unroll
      for (int b = 1; b < n; ++b) {
        t = M[(a - a0) * n + b] * x[b];
        acc = acc + t;
        mir = b & 1 ? mir - t : mir + t;
      }
      y[a] = acc;
      if (n - 1 - a != a) y[n - 1 - a] = mir;
    }
  }
}

}  // namespace isr
