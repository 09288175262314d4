// Threshold-selection bodies (device functions), shared by the per-phase
// kernels (isr_select.hip) and the persistent batch kernel (isr_batch.cuh).
// The threshold rule (arXiv 2407.20731, Sec. IV-B reading): tau is the largest
// energy value v whose dropped energy S(v) = RN(exact sum of energies < v)
// does not exceed B = (tol*tol)*U2.
#pragma once

#include "isr.h"
#include "isr_common.cuh"

namespace isr {

// --------------------------------------------------------------------------
// select, level 1 (one wave per component): U2, B, the slack integer
// Tint = largest X-unit sum whose round-to-nearest is <= B, and the boundary
// exponent bin b*: the last non-empty bin whose exclusive prefix sum is <= Tint.

// With sample = 1 the same walk runs on the histograms of the sampled tiles
// and only records the window of exponent bins [b - 1, b + 2) that pass 1
// then copies to the candidate list; with sample = 0 it decides whether the
// true boundary bin fell inside that window (else the candidate pass runs).
// Run by one whole wave.
DEV void select1_body(const Job& j, int comp, int sample) {
  const int lane = lane_id();
  CompState* st = j.st + comp;
  const HistBin* HN = (sample ? j.histNs : j.histN) + (size_t)comp * HBINS;
  const HistBin* HE = (sample ? j.histEs : j.histE) + (size_t)comp * HBINS;
  const double tol = j.tol;
  int flags = 0;
  // both histograms' counts in flight before either is used
  u64 cE[HROUNDS];
  u32 rN;
  {
    u64 cN[HROUNDS];
    hist_counts(HN, cN);
    hist_counts(HE, cE);
    rN = hist_rounds(cN);
  }
  if (HN[HBINS - 1].cnt) flags |= ST_NONFINITE;
  if (HE[HBINS - 1].cnt) flags |= ST_OVERFLOW;
  const double U2 = wb_round(hist_sum(HN, rN));
  if (sample) {
    if (tol < 0.0) return;
  } else if (lane == 0) {
    const int nn = j.order + 1;
    st->U2 = U2;
    st->tol = tol;
    st->n_values = (u64)j.n_elem * (u64)(nn * nn * nn);
    st->flags |= flags;
  }
  if (tol < 0.0) {  // keep everything
    if (lane == 0) {
      st->B = 0.0;
      st->tau = 0.0;
      st->kept = st->n_values;
      st->dropped = 0.0;
      st->bstar = -1;
      st->resolved = 1;
      st->level = 1;
    }
    return;
  }
  double B = (tol * tol) * U2;
  if (j.cut_scale != 1.0) B = B * j.cut_scale;  // a share of the budget left to a later stage
  // MFMA paths: the measured error differs from the dropped energy by the
  // transform error (about 1e-5 relative in FP32-split BF16 at tol 1e-3), so
  // they select against a budget that much smaller and rarely need a repair
  if (j.precision == ISR_PREC_BF16)
    B = B * (1.0 - 0x1p-10);
  else if (j.precision == ISR_PREC_FP32)
    B = B * (1.0 - 0x1p-17);
  if (!sample && comp < 8 && j.Bov[comp] >= 0.0) B = j.Bov[comp];
  // Tint = X(B) + half ulp(B) - (sig(B) odd)
  const u64 bb = dbits(B);
  const int EB = (int)(bb >> 52);
  const u64 sigB = (bb & M52) | (EB ? (1ull << 52) : 0ull);
  const int sB = EB > 1 ? EB : 1;
  u64 Tw = 0;
  const bool Binf = EB == 2047;
  if (!Binf) {
    wb_add(Tw, part_at(sigB, 0ull, sB));
    wb_add(Tw, part_at(1ull, 0ull, sB - 1));
    if (sigB & 1ull) wb_sub(Tw, part_at(1ull, 0ull, 0));
  }
  // walk the energy bins up to the one whose sum no longer fits
  u64 R = Tw, P = 0ull;
  int bstar = -1;
  u64 bcnt = 0ull;
  bool found = false;
  if (!Binf) {
    hist_walk(HE, hist_rounds(cE), [&](int bin, u64 lo, u64 hi, u64 cnt) {
      const u64 part = part_at(lo, hi, bin > 1 ? bin : 1);
      u64 tmp = R;
      wb_sub(tmp, part);
      if (wb_neg(tmp)) {
        bstar = bin;
        bcnt = cnt;
        found = true;
        return false;
      }
      R = tmp;
      wb_add(P, part);
      return true;
    });
  }
  if (!sample && st->win_mode) {
    // the streaming pass kept exact sums only inside the window: a boundary
    // outside it (or none at all) sends the request to the general pipeline
    const bool hit = found && bstar >= st->win_lo && bstar < st->win_hi;
    if (!hit) {
      if (lane == 0) {
        st->flags |= ST_MISS;
        st->resolved = 1;
      }
      return;
    }
  }
  if (sample) {
    if (lane == 0 && found) {
      st->win_lo = bstar > 0 ? bstar - 1 : 0;
      st->win_hi = bstar + 2 < HBINS - 1 ? bstar + 2 : HBINS - 1;
    }
    return;
  }
  if (!found) {  // every energy can be dropped: tau = +inf
    double dropped = 0.0;
    if (Binf) {
      u64 tot = hist_total(HE);
      dropped = wb_round(tot);
    } else {
      dropped = wb_round(P);
    }
    if (lane == 0) {
      st->B = B;
      st->tau = __builtin_inf();
      st->kept = 0ull;
      st->dropped = dropped;
      st->bstar = -1;
      st->resolved = 1;
      st->level = 1;
    }
    return;
  }
  // counts above b*
  u64 above = 0ull;
#pragma unroll
  for (int k = 0; k < HROUNDS; ++k) above += 64 * k + lane > bstar ? cE[k] : 0ull;
  above = wave_sum64(above);
  const int s = bstar > 1 ? bstar : 1;
  u64 rlo, rhi;
  bool sat;
  wb_extract128(R, s, rlo, rhi, sat);
  if (sat) rlo = rhi = ~0ull;
  st->P1[lane] = P;
  if (lane == 0) {
    st->B = B;
    st->bstar = bstar;
    st->kept_above = above;
    st->cur_count = bcnt;
    st->key_prefix = (u64)bstar << 52;
    st->key_mask = 0x7FFull << 52;
    st->r_lo = rlo;
    st->r_hi = rhi;
    st->w_lo = 0ull;
    st->w_hi = 0ull;
    st->level = 1;
    st->resolved = 0;
    // pass 1 captured the window [win_lo, win_hi); outside it, pass 2 gathers
    // the boundary bin into a fresh list 0
    const bool hit = bstar >= st->win_lo && bstar < st->win_hi;
    st->need_pass2 = hit ? 0 : 1;
    st->list0_exact = hit ? 0 : 1;
    if (!hit) st->list_count[0] = 0ull;
  }
}

// --------------------------------------------------------------------------
// refine, level L in 2..6: histogram of the next fraction bits of the listed
// energies that match the current prefix, or, once a sub-bin has at most CAP
// members (L >= 3), those members in a list of their own for the selection of
// the same level to sort.

// List 0 (the candidates of the boundary bin or window) is only read, by every
// level, so that it stays whole for the per-element kept counts; the members
// go to list 1, which the selection of the same level resolves (one list is
// enough: no level reads another's).
DEV int list_members(int L) { return L == 2 ? 0 : 1; }

// Worker `item` of `nitems` handles list entries item*256 + tid + k*nitems*256
// (blockDim must be 256).
DEV void refine_body(const Job& j, int comp, int L, u64 (*h)[2], u64 item, u64 nitems) {
  const int tid = threadIdx.x;
  CompState* st = j.st + comp;
  if (st->resolved) return;
  __syncthreads();
  const int nb = 1 << level_bits(L), sh = level_shift(L);
  const u64 fmask = (u64)(nb - 1);
  // A sub-bin that the selection will sort (at most CAP members) needs no
  // histogram: its members are collected in the same LDS (which holds CAP of
  // them) and appended with one global atomic per workgroup.
  static_assert(2 * RBINS >= CAP, "the histogram's LDS holds the members");
  __shared__ u32 nst;
  __shared__ u64 gbase;
  const bool gather = L >= 3 && st->cur_count <= (u64)CAP;
  u64* stage = &h[0][0];
  if (tid == 0) nst = 0u;
  if (!gather)
    for (int k = tid; k < nb; k += 256) h[k][0] = h[k][1] = 0ull;
  __syncthreads();
  const u64* in = list_ptr(j, comp, 0);
  const u64 nin = st->list_count[0] < list_capk(j, 0) ? st->list_count[0] : list_capk(j, 0);
  const u64 prefix = st->key_prefix, mask = st->key_mask;
  const int bstar = st->bstar;
  const u64 implicit = bstar ? (1ull << 52) : 0ull;
  const int lo_idx = list_members(L);
  u64* out = list_ptr(j, comp, lo_idx);
  const u64 stride = nitems * 256;
  // sixteen entries per lane per step, loaded before any is used (the lists
  // run to millions of entries: more loads in flight per lane)
  constexpr int U = 16;
  HistBin* g = j.histL + ((size_t)(L - 2) * j.ncomp + comp) * RBINS;
  // at most 2^20 entries of a worker between two flushes: a bin's count has 21
  // bits in LDS
  const u64 seg = nitems << 20;
  for (u64 s0 = 0; s0 < nin; s0 += seg) {
    const u64 end = nin - s0 < seg ? nin : s0 + seg;
    for (u64 i0 = s0 + item * 256 + tid; i0 < end; i0 += U * stride) {
      u64 keys[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u64 i = i0 + u * stride;
        keys[u] = i < end ? in[i] : 0ull;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u64 i = i0 + u * stride;
        const u64 key = keys[u];
        const bool m = i < end && (key & mask) == prefix;
        if (gather) {
          if (m) {  // (the bin's count bounds this; a list that disagrees with it is flagged below)
            const u32 pos = atomicAdd(&nst, 1u);
            if (pos < (u32)CAP) stage[pos] = key;
          }
          continue;
        }
        if (m) {
          const u64 sig = (key & M52) | implicit;
          const int sb = (int)((key >> sh) & fmask);
          atomicAdd(&h[sb][0], (1ull << 43) + (sig & M21));
          atomicAdd(&h[sb][1], sig >> 21);
        }
      }
    }
    if (gather) continue;
    __syncthreads();
    for (int k = tid; k < nb; k += 256) {
      const u64 w0 = h[k][0], w1 = h[k][1];
      if (w0 | w1) {
        global_bin_add(g, k, w0 >> 43, w0 & M43, w1);
        h[k][0] = h[k][1] = 0ull;
      }
    }
    __syncthreads();
  }
  __syncthreads();
  if (gather) {
    const u32 k = nst < (u32)CAP ? nst : (u32)CAP;
    if (tid == 0) {
      gbase = k ? atomicAdd(&st->list_count[lo_idx], (u64)nst) : 0ull;
      if (nst > (u32)CAP) atomicOr(&st->flags, ST_LIST);
    }
    __syncthreads();
    for (u32 i = tid; i < k; i += 256) {
      if (gbase + i < list_capk(j, lo_idx))
        out[gbase + i] = stage[i];
      else
        atomicOr(&st->flags, ST_LIST);
    }
    __syncthreads();
  }
}


// Resolve tau among <= CAP listed members of the current sub-bin: narrowed in
// LDS by eight fraction bits at a time (exact sums of 256 bins, scanned by the
// workgroup) until few are left, which are sorted and scanned in ascending
// order.  (Sorting some 1500 members took 60 us: 66 bitonic steps of 8 LDS
// round trips a thread each; narrowing takes ~3 us a step.)
constexpr int SORT_MAX = 64;

// Inclusive scan of one 128-bit value per thread (Hillis-Steele in LDS).
DEV u128 block_incl_scan128(u128 v, u64* slo, u64* shi, int tid) {
  u128 incl = v;
  for (int d = 1; d < 256; d <<= 1) {
    slo[tid] = (u64)incl;
    shi[tid] = (u64)(incl >> 64);
    __syncthreads();
    u128 add = 0;
    if (tid >= d) add = ((u128)shi[tid - d] << 64) | slo[tid - d];
    __syncthreads();
    incl += add;
  }
  return incl;
}

struct SelLds {
  u64 keys[CAP];
  u64 slo[256], shi[256];
  u64 hist[256][2];  // (count << 43) + sum of the low 21 significand bits, sum of the rest
  int best;
  u32 n, above;
  u64 exlo, exhi;
};

DEV void resolve_sorted(const Job& j, CompState* st, int comp, int ml, int L, SelLds& S) {
  const int tid = threadIdx.x;
  u64* keys = S.keys;
  const u64* list = list_ptr(j, comp, ml);
  const u64 lc = st->list_count[ml];
  int cnt = (int)(lc < (u64)CAP ? lc : (u64)CAP);  // == cur_count unless a list overflowed
  const u64 implicit = st->bstar ? (1ull << 52) : 0ull;
  u128 r = ((u128)st->r_hi << 64) | st->r_lo;
  u128 w = ((u128)st->w_hi << 64) | st->w_lo;
  u64 kept_above = st->kept_above;
  int fixed = L == 2 ? 52 : level_shift(L - 1);  // fraction bits below this one are still open
  for (int i = tid; i < cnt; i += 256) keys[i] = list[i];
  __syncthreads();
  while (cnt > SORT_MAX && fixed > 0) {
    const int sh = fixed > 8 ? fixed - 8 : 0;
    const u64 fmask = (1ull << (fixed - sh)) - 1ull;
    S.hist[tid][0] = S.hist[tid][1] = 0ull;
    if (tid == 0) {
      S.n = S.above = 0u;
      S.best = -1;
    }
    __syncthreads();
    for (int i = tid; i < cnt; i += 256) {
      const u64 sig = (keys[i] & M52) | implicit;
      const int sb = (int)((keys[i] >> sh) & fmask);
      atomicAdd(&S.hist[sb][0], (1ull << 43) + (sig & M21));
      atomicAdd(&S.hist[sb][1], sig >> 21);
    }
    __syncthreads();
    const u64 w0 = S.hist[tid][0], w1 = S.hist[tid][1];
    const u128 sum = ((u128)w1 << 21) + (u128)(w0 & M43);
    const u128 incl = block_incl_scan128(sum, S.slo, S.shi, tid);
    // the boundary: the first bin whose inclusive sum no longer fits
    if (incl > r && incl - sum <= r) {
      S.best = tid;
      S.exlo = (u64)(incl - sum);
      S.exhi = (u64)((incl - sum) >> 64);
    }
    __syncthreads();
    const int sb = S.best;
    if (sb < 0) break;  // everything fits (a list that disagrees with its counts: flagged below)
    if (tid > sb && w0) atomicAdd(&S.above, (u32)(w0 >> 43));
    // the boundary bin's members to the front (all read before any is written)
    u64 mine[CAP / 256];
#pragma unroll
    for (int k = 0; k < CAP / 256; ++k) {
      const int i = tid + 256 * k;
      mine[k] = i < cnt ? keys[i] : 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < CAP / 256; ++k)
      if (tid + 256 * k < cnt && (int)((mine[k] >> sh) & fmask) == sb) keys[atomicAdd(&S.n, 1u)] = mine[k];
    __syncthreads();
    const u128 ex = ((u128)S.exhi << 64) | S.exlo;
    r -= ex;
    w += ex;
    kept_above += S.above;
    cnt = (int)S.n;
    fixed = sh;
    __syncthreads();
  }
  __syncthreads();  // (a wave may still be reading S.best)
  if (tid == 0) S.best = 0;
  // (with no bit open the members are one value: any order is sorted)
  int np = 1;
  if (fixed > 0)
    while (np < cnt) np <<= 1;
  for (int i = cnt + tid; i < np; i += 256) keys[i] = ~0ull;
  __syncthreads();
  for (int k = 2; k <= np; k <<= 1) {
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
      for (int i = tid; i < np; i += 256) {
        const int ixj = i ^ jj;
        if (ixj > i) {
          const u64 x = keys[i], y = keys[ixj];
          const bool asc = (i & k) == 0;
          if ((x > y) == asc) {
            keys[i] = y;
            keys[ixj] = x;
          }
        }
      }
      __syncthreads();
    }
  }
  const int per = (cnt + 255) / 256;
  const int i0 = tid * per;
  u128 run = 0;
  for (int k = 0; k < per; ++k) {
    const int i = i0 + k;
    if (i < cnt) run += (u128)((keys[i] & M52) | implicit);
  }
  u128 ex = block_incl_scan128(run, S.slo, S.shi, tid) - run;
  int mybest = -1;
  u128 myex = 0;
  for (int k = 0; k < per; ++k) {
    const int i = i0 + k;
    if (i >= cnt) break;
    const bool first = i == 0 || keys[i] != keys[i - 1];
    if (first && ex <= r) {
      mybest = i;
      myex = ex;
    }
    ex += (u128)((keys[i] & M52) | implicit);
  }
  if (mybest >= 0) atomicMax(&S.best, mybest);
  __syncthreads();
  const int bi = S.best;
  if (mybest >= 0 && mybest == bi) {
    w += myex;
    st->w_lo = (u64)w;
    st->w_hi = (u64)(w >> 64);
    st->tau = __longlong_as_double((long long)keys[bi]);
    st->kept = kept_above + (u64)(cnt - bi);
    st->resolved = 1;
    st->level = L;
    if (lc != st->cur_count) st->flags |= ST_LIST;
  }
}

// blockDim must be 256; the sub-bin walk runs on wave 0.
// One wave walks the NB = 64 PER sub-bins of level L: lane l sums sub-bins
// [PER l, PER l + PER), a 128-bit scan finds the lane whose chunk crosses the
// remaining budget, and that chunk's sub-bins are loaded one per lane and
// walked in registers.  Every load of a step is issued before any is used.
template <int PER>
DEV void select_walk(const Job& j, CompState* st, int comp, int L) {
  const int nb = 1 << level_bits(L), sh = level_shift(L);
  const HistBin* H = j.histL + ((size_t)(L - 2) * j.ncomp + comp) * RBINS;
  const int lane = lane_id();
  u128 cs = 0;
#pragma unroll 8
  for (int k = 0; k < PER; ++k) {
    const int sb = lane * PER + k;
    if (sb < nb) cs += bin_sum(H[sb]);
  }
  // inclusive scan of the lane chunk sums
  u64 ilo = (u64)cs, ihi = (u64)(cs >> 64);
  for (int d = 1; d < 64; d <<= 1) {
    const u64 olo = shfl_up64(ilo, d), ohi = shfl_up64(ihi, d);
    if (lane >= d) {
      const u128 v = (((u128)ihi << 64) | ilo) + (((u128)ohi << 64) | olo);
      ilo = (u64)v;
      ihi = (u64)(v >> 64);
    }
  }
  const u128 r = ((u128)st->r_hi << 64) | st->r_lo;
  const u128 incl = ((u128)ihi << 64) | ilo;
  const u64 over = ballot(incl > r);
  if (over == 0ull) {  // cannot happen: the current bin's total exceeds r
    if (lane == 0) {
      st->flags |= ST_LIST;
      st->tau = __builtin_nan("");
      st->resolved = 1;
    }
    return;
  }
  const int fl = __ffsll((long long)over) - 1;
  u128 excl = 0;
  {
    const u128 myex = incl - cs;
    const u64 elo = bcast64((u64)myex, fl), ehi = bcast64((u64)(myex >> 64), fl);
    excl = ((u128)ehi << 64) | elo;
  }
  // the crossing chunk, one sub-bin per lane, then walked in registers
  const int msb = fl * PER + lane;
  const HistBin mine = (lane < PER && msb < nb) ? H[msb] : HistBin{0ull, 0ull, 0ull};
  int chosen = -1;
  u64 ccnt = 0ull;
  for (int k = 0; k < PER; ++k) {
    const u64 c = bcast64(mine.cnt, k);
    if (c == 0ull) continue;
    const u128 s = (((u128)bcast64(mine.hi, k)) << 21) + (u128)bcast64(mine.lo, k);
    chosen = fl * PER + k;
    ccnt = c;
    if (excl + s > r) break;
    excl += s;
  }
  if (chosen < 0) {  // cannot happen: the crossing chunk is non-empty
    if (lane == 0) {
      st->flags |= ST_LIST;
      st->tau = __builtin_nan("");
      st->resolved = 1;
    }
    return;
  }
  u64 above = 0;
#pragma unroll 8
  for (int k = 0; k < PER; ++k) {
    const int sb = lane * PER + k;
    if (sb < nb && sb > chosen) above += H[sb].cnt;
  }
  above = wave_sum64(above);
  if (lane == 0) {
    const u128 rn = r - excl;
    st->r_lo = (u64)rn;
    st->r_hi = (u64)(rn >> 64);
    const u128 w = (((u128)st->w_hi << 64) | st->w_lo) + excl;
    st->w_lo = (u64)w;
    st->w_hi = (u64)(w >> 64);
    st->kept_above += above;
    st->cur_count = ccnt;
    st->key_prefix |= (u64)chosen << sh;
    st->key_mask |= ((u64)nb - 1ull) << sh;
    st->level = L;
    if (L == NLEV) {  // every bit fixed: the sub-bin is the single value tau
      st->tau = __longlong_as_double((long long)st->key_prefix);
      st->kept = st->kept_above + st->cur_count;
      st->resolved = 1;
    } else {
      st->list_count[1] = 0ull;
    }
  }
}

DEV void select_body(const Job& j, int comp, int L, SelLds& S) {
  const int tid = threadIdx.x;
  CompState* st = j.st + comp;
  // (read by every wave before the walk below may change them)
  const bool done = st->resolved != 0;
  const bool few = st->cur_count <= (u64)CAP && (L > 2 || st->list0_exact);
  const int ml = list_members(L);
  __syncthreads();
  if (done) return;
  if (few) {
    resolve_sorted(j, st, comp, ml, L, S);
    return;
  }
  if (tid >= 64) return;
  // walk the level-L sub-bins with one wave
  if (level_bits(L) == 11)
    select_walk<(1 << 11) / 64>(j, st, comp, L);
  else
    select_walk<((1 << 8) + 63) / 64>(j, st, comp, L);
}

// --------------------------------------------------------------------------
// finalize (one wave per component): err2, rel, dropped energy.

// Run by one whole wave.  more: what the error sum holds beside the bins (a
// wave-distributed big integer).
DEV void finalize_body(const Job& j, int comp, u64 more = 0ull) {
  const int lane = lane_id();
  CompState* st = j.st + comp;
  u64 er = hist_total(j.histR + (size_t)comp * HBINS);
  wb_add(er, more);
  const double err2 = wb_round(er);
  const double U2 = st->U2;
  const double rel = U2 > 0.0 ? __builtin_sqrt(err2 / U2) : 0.0;
  double dropped = st->dropped;
  if (st->resolved && st->bstar >= 0) {
    u64 P = st->P1[lane];
    const int s = st->bstar > 1 ? st->bstar : 1;
    wb_add(P, part_at(st->w_lo, st->w_hi, s));
    dropped = wb_round(P);
  }
  if (lane == 0) {
    st->err2 = err2;
    st->rel = rel;
    st->dropped = dropped;
    if (!st->resolved) st->flags |= ST_SPIN;
    u64 vo = 0;
    for (int cc = 0; cc < comp; ++cc) vo += j.st[cc].kept;
    j.voff[comp] = vo;
  }
}

}  // namespace isr
