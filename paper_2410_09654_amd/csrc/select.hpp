// Top-M selection and output compaction, driven from the device.
//
// After the merge every bucket b holds its surviving strings (length cap and
// coefficient threshold applied; keys as order keys) at U slots
// [b_ubase[b], b_ubase[b] + b_slots[b]), with per-bucket counts of survivors and keep-set survivors and
// a replicated level-0 histogram of |c|^2 (its top 13 bits) over the non-keep survivors.  The
// kernels below decide, without a host round trip, whether a threshold is
// needed (the keep set is always kept and counts toward M; ties are broken by
// ascending key), find it by a two-level radix select over the composite
// ordering key (|c|^2 bits, then the complemented key words), and write the
// kept strings in bucket order.
//
// Flow (one stream, no host synchronisation in between):
//   k_plan  k_sel_pass1  k_sel_narrow  k_write_out
// The serial step behind each of the first three (the select mode and the
// level-0 bin; the digit-1 bin; the threshold and the output bases) is taken by
// the kernel's last block (last_block).  As kernels of their own those steps
// took 3.5 to 18 us each and a small call launched seven kernels here.
// Candidate lists live per bucket in the bucket's own U slot range, so no
// pass appends through a single global counter except the final list of at
// most FINISH_CAP entries.
// The select kernels return at once unless the plan chose S_THRESHOLD.  When
// more than FINISH_CAP candidates share the first two digits (large groups of
// exactly equal |c|), k_sel_pass1 sets ctl->deep, the later kernels stand
// down and the host finishes the call with the multi-level select.
#pragma once
#include "kernels.hpp"

namespace pauli {

constexpr int SEL_CHUNK = 4;       // buckets per 256-thread block (one wave per bucket)
constexpr int SEL_BLOCKS = 512;    // blocks of the select passes (1024 threads, one wave per
                                   // bucket at a time; one ticket per block)

// Bin holding the K-th largest entry of hist[0..nbins) (bins ordered from the
// top): one block of 1024 threads; every thread gets the bin, the rank of the
// K-th entry inside it (1-based) and the bin's count.  K must lie in
// [1, sum(hist)].  tmp: 19 words of shared memory.
DEV void pick_bin(const uint32_t* hist, int nbins, unsigned long long K,
                  unsigned long long* tmp, unsigned int* out_digit,
                  unsigned long long* out_krem, unsigned long long* out_count) {
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int per = nbins / 1024;  // 2 or 4
  const int hiB = nbins - t * per;
  if (t == 0) {
    tmp[16] = 0ull;
    tmp[17] = 0ull;
    tmp[18] = 0ull;
  }
  unsigned int hv[4] = {0u, 0u, 0u, 0u};
  unsigned long long s = 0;
  for (int q = 1; q <= per; q++) {
    hv[q - 1] = hist[hiB - q];
    s += hv[q - 1];
  }
  unsigned long long x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    unsigned long long y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) tmp[wv] = x;
  __syncthreads();
  unsigned long long w = lane < 16 ? tmp[lane] : 0ull;
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    unsigned long long y = __shfl_up(w, d, 64);
    if (lane >= d) w += y;
  }
  const unsigned long long before = wv > 0 ? __shfl(w, wv - 1, 64) : 0ull;
  __syncthreads();
  unsigned long long cum = before + x - s;  // entries in the bins above this thread's
  for (int q = 1; q <= per; q++) {
    const unsigned long long h = hv[q - 1];
    if (cum < K && K <= cum + h) {
      tmp[16] = (unsigned long long)(hiB - q);
      tmp[17] = K - cum;
      tmp[18] = h;
    }
    cum += h;
  }
  __syncthreads();
  *out_digit = (unsigned int)tmp[16];
  *out_krem = tmp[17];
  *out_count = tmp[18];
}

struct PlanArgs {
  const uint32_t* b_slots;
  const uint32_t* b_surv;
  const uint32_t* b_keep;
  const uint32_t* b_unique;  // nullable: leave ctl->u_unique as it is
  uint32_t nbk;
  int want_select;
  long long max_strings;
  const uint32_t* hist0;     // HREP replicas of the level-0 |c|^2 histogram (SEL0_BINS each)
  uint32_t* hist1;           // digit-1 histogram replicas, cleared here (nullable)
  unsigned long long* psum;  // [PLAN_PARTS][4] partial counter sums
  uint32_t* h0sum;           // [SEL0_BINS] the level-0 histogram, replicas summed
  uint32_t* b_obase;         // output bases, written here when there is nothing to select
  Ctl* ctl;
  Ctl* hctl;                 // the host's copy (nullable: the host reads ctl itself)
};

// Eight consecutive words p[b0 .. b0 + 8) (zero past nb), as two 16-byte
// loads when the eight lie inside the array (b0 is a multiple of 8 and the
// arena aligns the tables to 256 bytes).
DEV void load8(const uint32_t* p, uint32_t b0, uint32_t nb, uint32_t* v) {
  if (b0 + 8 <= nb) {
    const uint4 a = *reinterpret_cast<const uint4*>(p + b0);
    const uint4 c = *reinterpret_cast<const uint4*>(p + b0 + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
  } else {
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = b0 + k < nb ? p[b0 + k] : 0u;
  }
}

// Output bases: survivors kept per bucket (by the select mode), exclusive
// scan over the buckets in tiles of 8192 (one block; thread t owns eight
// consecutive buckets, read and written as 16-byte vectors).
DEV void scan_out(const uint32_t* b_surv, const uint32_t* b_keep, const uint32_t* b_abv,
                  const uint32_t* b_bcnt, uint32_t nb, int mode, uint32_t* b_obase, Ctl* ctl) {
  constexpr int PER = 8, TILE = 1024 * PER;
  __shared__ unsigned long long tmp[17];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  unsigned long long carry = 0;
  for (uint32_t base = 0; base < nb; base += TILE) {
    const uint32_t b0 = base + (uint32_t)t * PER;
    uint32_t loc[PER];
    if (mode == S_ALL) {
      load8(b_surv, b0, nb, loc);
    } else if (mode == S_KEEP_ONLY) {
      load8(b_keep, b0, nb, loc);
    } else {
      uint32_t a[PER], c[PER];
      load8(b_keep, b0, nb, loc);
      load8(b_abv, b0, nb, a);
      load8(b_bcnt, b0, nb, c);
#pragma unroll
      for (int k = 0; k < PER; k++) loc[k] += a[k] + c[k];
    }
    unsigned long long s = 0;
#pragma unroll
    for (int k = 0; k < PER; k++) s += loc[k];
    unsigned long long x = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      unsigned long long y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) tmp[wv] = x;
    __syncthreads();
    unsigned long long w = lane < 16 ? tmp[lane] : 0ull;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      unsigned long long y = __shfl_up(w, d, 64);
      if (lane >= d) w += y;
    }
    const unsigned long long before = wv > 0 ? __shfl(w, wv - 1, 64) : 0ull;
    const unsigned long long tile_total = __shfl(w, 15, 64);
    unsigned long long pre = carry + before + x - s;
    uint32_t o[PER];
#pragma unroll
    for (int k = 0; k < PER; k++) {
      o[k] = (uint32_t)pre;
      pre += loc[k];
    }
    if (b0 + PER <= nb) {
      *reinterpret_cast<uint4*>(b_obase + b0) = make_uint4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<uint4*>(b_obase + b0 + 4) = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
#pragma unroll
      for (int k = 0; k < PER; k++)
        if (b0 + k < nb) b_obase[b0 + k] = o[k];
    }
    carry += tile_total;
    __syncthreads();  // tmp is rewritten by the next tile
  }
  if (t == 0) ctl->out_total = carry;
}

// Totals of the per-bucket counters, the select mode, and the level-0 bin of
// the threshold.  Blocks [0, P) sum the four per-bucket counters over a P-th of the
// buckets each, blocks [P, 2P) sum the HREP replicas of SEL0_BINS / P bins
// of the level-0 histogram each, blocks [2P, 3P) clear a P-th of the digit-1
// replicas; the last block adds up and decides.
constexpr int PLAN_PARTS = 16;
constexpr uint32_t PLAN_ONE = 8192;  // buckets that one block plans alone (nothing to select)
static_assert(SEL0_BINS == PLAN_PARTS * 256 && HREP % 4 == 0 &&
                  HREP * SEL_BINS == PLAN_PARTS * 4096,
              "k_plan: 256 level-0 bins and 4096 digit-1 words per block");
__global__ __launch_bounds__(1024) void k_plan(PlanArgs a) {
  __shared__ unsigned long long red[4][16];
  __shared__ uint32_t hr[4][256];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int blk = blockIdx.x;
  if (gridDim.x == 1) {
    // few buckets and nothing to select: one block does it all
    unsigned long long v[4] = {0, 0, 0, 0};
    for (uint32_t b = t; b < a.nbk; b += 1024) {
      v[0] += a.b_slots[b];
      v[1] += a.b_surv[b];
      v[2] += a.b_keep[b];
      if (a.b_unique) v[3] += a.b_unique[b];
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      for (int d = 32; d >= 1; d >>= 1) v[q] += __shfl_down(v[q], d, 64);
      if (lane == 0) red[q][wv] = v[q];
    }
    __syncthreads();
    if (t < 4) {
      unsigned long long s = 0;
#pragma unroll
      for (int w = 0; w < 16; w++) s += red[t][w];
      if (t == 0) a.ctl->u_slots = s;
      if (t == 1) a.ctl->surv_total = s;
      if (t == 2) a.ctl->keep_total = s;
      if (t == 3 && a.b_unique) a.ctl->u_unique = s;
      if (t == 0) a.ctl->sel_mode = S_ALL;
    }
    scan_out(a.b_surv, a.b_keep, nullptr, nullptr, a.nbk, S_ALL, a.b_obase, a.ctl);
    publish(a.ctl, a.hctl);
    return;
  }
  if (blk < PLAN_PARTS) {
    const uint32_t chunk = (a.nbk + PLAN_PARTS - 1) / PLAN_PARTS;
    const uint32_t b0 = min(a.nbk, blk * chunk), b1 = min(a.nbk, b0 + chunk);
    unsigned long long v[4] = {0, 0, 0, 0};
    for (uint32_t b = b0 + t; b < b1; b += 1024) {
      v[0] += a.b_slots[b];
      v[1] += a.b_surv[b];
      v[2] += a.b_keep[b];
      if (a.b_unique) v[3] += a.b_unique[b];
    }
#pragma unroll
    for (int q = 0; q < 4; q++) {
      unsigned long long x = v[q];
      for (int d = 32; d >= 1; d >>= 1) x += __shfl_down(x, d, 64);
      if (lane == 0) red[q][wv] = x;
    }
    __syncthreads();
    if (t < 4) {
      unsigned long long s = 0;
      for (int w = 0; w < 16; w++) s += red[t][w];
      st_agent(&a.psum[blk * 4 + t], s);
    }
  } else if (blk < 2 * PLAN_PARTS) {
    const int bin = (blk - PLAN_PARTS) * 256 + (t & 255), g = t >> 8;
    uint32_t s = 0;
#pragma unroll
    for (int r = g; r < HREP; r += 4) s += a.hist0[(size_t)r * SEL0_BINS + bin];
    hr[g][t & 255] = s;
    __syncthreads();
    if (t < 256) st_agent(&a.h0sum[bin], hr[0][t] + hr[1][t] + hr[2][t] + hr[3][t]);
  } else if (a.hist1) {
    uint4* z = reinterpret_cast<uint4*>(a.hist1) + (size_t)(blk - 2 * PLAN_PARTS) * 1024;
    z[t] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (!last_block(&a.ctl->ticket[2])) return;
  __shared__ unsigned long long tmp[19];
  __shared__ uint32_t hs[SEL0_BINS];
  __shared__ unsigned long long s_K;
  __shared__ int s_mode;
  constexpr int BPT0 = SEL0_BINS / 1024;
#pragma unroll
  for (int k = 0; k < BPT0; k++) hs[k * 1024 + t] = a.h0sum[k * 1024 + t];
  if (t < 4) {
    unsigned long long tot = 0;
#pragma unroll
    for (int p = 0; p < PLAN_PARTS; p++) tot += a.psum[p * 4 + t];
    tmp[t] = tot;
  }
  __syncthreads();
  if (t == 0) {
    a.ctl->u_slots = tmp[0];
    a.ctl->surv_total = tmp[1];
    a.ctl->keep_total = tmp[2];
    if (a.b_unique) a.ctl->u_unique = tmp[3];
    const unsigned long long surv = tmp[1], fk = tmp[2];
    int mode = S_ALL;
    unsigned long long K = 0;
    if (a.want_select) {
      const long long budget = a.max_strings - (long long)fk;
      const unsigned long long nonkeep = surv - fk;
      if (budget <= 0) mode = fk == surv ? S_ALL : S_KEEP_ONLY;
      else if ((unsigned long long)budget >= nonkeep) mode = S_ALL;
      else {
        mode = S_THRESHOLD;
        K = (unsigned long long)budget;
      }
    }
    s_mode = mode;
    s_K = K;
    a.ctl->sel_mode = mode;
  }
  __syncthreads();
  if (!a.want_select) {
    scan_out(a.b_surv, a.b_keep, nullptr, nullptr, a.nbk, S_ALL, a.b_obase, a.ctl);
    publish(a.ctl, a.hctl);
    return;
  }
  if (s_mode != S_THRESHOLD) return;
  unsigned int d0;
  unsigned long long krem, cnt;
  pick_bin(hs, SEL0_BINS, s_K, tmp, &d0, &krem, &cnt);
  if (t == 0) {
    a.ctl->sel_d0 = d0;
    a.ctl->sel_K = krem;
    a.ctl->sel_count = cnt;
    a.ctl->fin_level = cnt <= (unsigned long long)FINISH_CAP ? 0u : 1u;
  }
}

struct Sel2Args {
  const uint32_t* b_ubase;
  const uint32_t* b_slots;
  uint32_t* b_abv;
  uint32_t* b_bcnt;
  const void* uk;
  const double2* uc;
  const void* keep_mk;
  int n_keep;
  uint32_t nbk;
  uint32_t* list0;   // level-1 candidates of bucket b at [b_ubase[b], b_ubase[b] + cc0[b])
  uint32_t* cc0;
  uint32_t* listf;   // candidates of the final bin (<= FINISH_CAP) ...
  uint32_t* listfb;  // ... and their buckets
  uint32_t* hist1;   // HREP replicas of the digit-1 histogram
  const uint32_t* b_surv;
  const uint32_t* b_keep;
  uint32_t* b_obase;
  Ctl* ctl;
  Ctl* hctl;
};

// Wave-aggregated append: lanes with `take` get consecutive slots of a
// list whose length lives in *counter.  Call with the whole wave.
DEV uint32_t wave_append(bool take, unsigned long long* counter) {
  const uint64_t m = __ballot(take);
  unsigned long long base = 0;
  if (m) {
    if ((threadIdx.x & 63) == 0) base = atomicAdd(counter, (unsigned long long)__popcll(m));
    base = __shfl(base, 0, 64);
  }
  return (uint32_t)base + mbcnt64(m);
}

// Level 1 over all survivors, one wave per bucket: counts per bucket the
// non-keep survivors whose level-0 digit is above the threshold bin, lists
// those inside it and histograms their digit 1 (when the bin is too large to
// finish directly).  The last block then picks the digit-1 bin.
template <int W>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_sel_pass1(Sel2Args a) {
  constexpr int NW = 1 + 2 * W;
  if (a.ctl->sel_mode != S_THRESHOLD) return;
  const uint32_t D0 = a.ctl->sel_d0;
  const bool lvl1 = a.ctl->fin_level == 1u;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  uint32_t* hrep = a.hist1 + (size_t)(blockIdx.x % HREP) * SEL_BINS;
  WaveBuckets wb(a.b_ubase, a.b_slots, blockIdx.x * 16 + wv, gridDim.x * 16, a.nbk);
  for (uint32_t b, ub, ns; wb.next(b, ub, ns);) {
    uint32_t abv = 0, nc = 0;
    // keys are read only in buckets that hold a string of the keep set
    const int n_keep = a.n_keep && a.b_keep[b] ? a.n_keep : 0;
    // SB loads in flight per lane
    constexpr int SB = 4;
    for (uint32_t i00 = 0; i00 < ns; i00 += 64 * SB) {
      double2 vv[SB];
#pragma unroll
      for (int u = 0; u < SB; u++) {
        const uint32_t i = i00 + 64 * u + lane;
        vv[u] = i < ns ? a.uc[ub + i] : make_double2(0.0, 0.0);
      }
#pragma unroll
      for (int u = 0; u < SB; u++) {
        const uint32_t i = i00 + 64 * u + lane;
        const double2 v = vv[u];
        bool cand = false;
        if (!is_zero(v)) {
          bool isk = false;
          if (n_keep) isk = keep_lookup<W>(keep, n_keep, ukb[ub + i]);
          if (!isk) {
            const uint32_t d0 = (uint32_t)((uint64_t)__double_as_longlong(weight2(v)) >> SEL0_SHIFT);
            if (d0 > D0) {
              abv++;
            } else if (d0 == D0) {
              cand = true;
              if (lvl1) {
                // digit 1: the 12 bits of |c|^2 after the level-0 bits (the
                // string words of the composite do not reach it)
                uint64_t c[NW] = {};
                c[0] = (uint64_t)__double_as_longlong(weight2(v));
                atomicAdd(&hrep[comp_digit<W>(c, 1)], 1u);
              }
            }
          }
        }
        const uint64_t m = __ballot(cand);
        if (cand) a.list0[ub + nc + mbcnt64(m)] = ub + i;
        nc += (uint32_t)__popcll(m);
      }
    }
    for (int d = 32; d >= 1; d >>= 1) abv += __shfl_down(abv, d, 64);
    if (lane == 0) {
      a.b_abv[b] = abv;
      a.cc0[b] = nc;
    }
  }
  if (!lvl1 || !last_block(&a.ctl->ticket[3])) return;
  __shared__ unsigned long long tmp[19];
  __shared__ uint32_t hs[SEL_BINS];
  const unsigned long long K = a.ctl->sel_K;
  constexpr int BPT = SEL_BINS / 1024;
  uint32_t h[BPT];
#pragma unroll
  for (int k = 0; k < BPT; k++) {
    h[k] = 0;
#pragma unroll 4
    for (int r = 0; r < HREP; r++) h[k] += a.hist1[(size_t)r * SEL_BINS + k * 1024 + threadIdx.x];
  }
#pragma unroll
  for (int k = 0; k < BPT; k++) hs[k * 1024 + threadIdx.x] = h[k];
  __syncthreads();
  unsigned int d1;
  unsigned long long krem, cnt;
  pick_bin(hs, SEL_BINS, K, tmp, &d1, &krem, &cnt);
  if (threadIdx.x == 0) {
    a.ctl->sel_d1 = d1;
    a.ctl->sel_K = krem;
    a.ctl->sel_count = cnt;
    if (cnt > (unsigned long long)FINISH_CAP) a.ctl->deep = 1u;
  }
}

// Threshold: the K-th largest composite among the final candidates (one block
// of 1024 threads, two candidates per thread in registers): 12-bit digits of
// the composite are histogrammed in LDS until at most 64 candidates share the
// K-th one's, then one wave ranks those.  The K entries at or above the
// threshold are counted into their buckets.  A bitonic sort of up to 2048
// entries in LDS (66 steps with a barrier each) took 17.5 us at 2048.
template <int W>
DEV bool sel_finish(const Sel2Args& a) {
  constexpr int NW = 1 + 2 * W, PER = FINISH_CAP / 1024;
  static_assert(FINISH_CAP % 1024 == 0, "whole candidates per thread");
  __shared__ uint32_t hs[SEL_BINS];
  __shared__ unsigned long long tmp[19];
  __shared__ uint64_t cs[64][NW];
  __shared__ uint64_t sT[NW];
  __shared__ unsigned int s_m;
  const int t = threadIdx.x;
  const unsigned long long n = a.ctl->cand_n[1];
  unsigned long long K = a.ctl->sel_K;
  if (n > (unsigned long long)FINISH_CAP || K < 1 || K > n) {
    if (t == 0) a.ctl->deep = 1u;
    return false;
  }
  const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
  uint64_t c[PER][NW];
  uint32_t bk[PER];
  int in[PER];  // 1: shares the K-th one's digits so far, 2: above them, 0: below
#pragma unroll
  for (int q = 0; q < PER; q++) {
    const uint32_t i = t + q * 1024;
    in[q] = i < (uint32_t)n ? 1 : 0;
    if (in[q]) {
      const uint32_t ui = a.listf[i];
      bk[q] = a.listfb[i];
      composite<W>(a.uc[ui], unmix_key<W>(ukb[ui]), c[q]);
    }
  }
  unsigned long long cnt = n;
  // (distinct strings have distinct composites: the digits separate them)
  for (int level = a.ctl->fin_level == 1u ? 2 : 1; cnt > 64; level++) {
#pragma unroll
    for (int k = 0; k < SEL_BINS / 1024; k++) hs[k * 1024 + t] = 0u;
    __syncthreads();
    uint32_t dg[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
      dg[q] = 0u;
      if (in[q] == 1) {
        dg[q] = comp_digit<W>(c[q], level);
        atomicAdd(&hs[dg[q]], 1u);
      }
    }
    __syncthreads();
    unsigned int d;
    unsigned long long krem, m;
    pick_bin(hs, SEL_BINS, K, tmp, &d, &krem, &m);
#pragma unroll
    for (int q = 0; q < PER; q++)
      if (in[q] == 1 && dg[q] != d) in[q] = dg[q] > d ? 2 : 0;
    K = krem;
    cnt = m;
  }
  if (t == 0) s_m = 0u;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; q++)
    if (in[q] == 1) {
      const unsigned int p = atomicAdd(&s_m, 1u);
#pragma unroll
      for (int w = 0; w < NW; w++) cs[p][w] = c[q][w];
    }
  __syncthreads();
  if (t < (int)cnt) {
    uint64_t me[NW];
#pragma unroll
    for (int w = 0; w < NW; w++) me[w] = cs[t][w];
    unsigned int rank = 0;
    for (int k = 0; k < (int)cnt; k++) rank += comp_cmp<W>(cs[k], me) > 0 ? 1u : 0u;
    if ((unsigned long long)rank + 1 == K) {
#pragma unroll
      for (int w = 0; w < NW; w++) {
        sT[w] = me[w];
        a.ctl->T[w] = me[w];
      }
      a.ctl->t_found = 1u;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; q++)
    if (in[q] == 2 || (in[q] == 1 && comp_cmp<W>(c[q], sT) >= 0)) atomicAdd(&a.b_bcnt[bk[q]], 1u);
  return true;
}

// The final candidates, gathered into one list: the level-1 candidates
// inside the digit-1 bin, or all of them when the level-0 bin is small.
// Also counts per bucket the candidates above the digit-1 bin.  One wave per
// bucket.  The last block then finds the threshold and the output bases (the
// latter also when there is no threshold to find).
template <int W>
__global__ __launch_bounds__(1024) void k_sel_narrow(Sel2Args a) {
  constexpr int NW = 1 + 2 * W;
  const int mode = a.ctl->sel_mode;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const bool deep = a.ctl->deep != 0u;
  if (mode == S_THRESHOLD && !deep) {
    const bool l1 = a.ctl->fin_level == 1u;
    const uint32_t D1 = a.ctl->sel_d1;
    WaveBuckets wb(a.b_ubase, a.cc0, blockIdx.x * 16 + wv, gridDim.x * 16, a.nbk);
    for (uint32_t b, ub, n; wb.next(b, ub, n);) {
      uint32_t above = 0;
      for (uint32_t i0 = 0; i0 < n; i0 += 64) {
        const uint32_t i = i0 + lane;
        bool take = false;
        uint32_t ui = 0;
        if (i < n) {
          ui = a.list0[ub + i];
          take = true;
          if (l1) {
            // the digit-1 bin holds the 12 bits of |c|^2 after the level-0 bits:
            // the string words of the composite do not reach it
            uint64_t c[NW] = {};
            c[0] = (uint64_t)__double_as_longlong(weight2(a.uc[ui]));
            const uint32_t d1 = comp_digit<W>(c, 1);
            take = d1 == D1;
            above += d1 > D1 ? 1u : 0u;
          }
        }
        const uint32_t pos = wave_append(take, &a.ctl->cand_n[1]);
        if (take && pos < (uint32_t)FINISH_CAP) {
          st_agent(&a.listf[pos], ui);
          st_agent(&a.listfb[pos], b);
        }
      }
      // candidates above the final bin are above the threshold; sel_finish
      // adds those of the final bin at or above it
      for (int d = 32; d >= 1; d >>= 1) above += __shfl_down(above, d, 64);
      if (lane == 0) st_agent(&a.b_bcnt[b], above);
    }
    if (!last_block(&a.ctl->ticket[3])) return;
  } else if (blockIdx.x != 0) {
    return;  // nothing to gather: one block finishes
  }
  bool ok = !deep;
  if (ok && mode == S_THRESHOLD) {
    ok = sel_finish<W>(a);
    // the counts just added are read below
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
  if (ok) scan_out(a.b_surv, a.b_keep, a.b_abv, a.b_bcnt, a.nbk, mode, a.b_obase, a.ctl);
  publish(a.ctl, a.hctl);
}

// Kept strings in bucket order, one wave per bucket, WB strings per lane at a
// time (13 M one-word strings, all kept: 278 -> 250 us).  Writes nothing when the
// output does not fit (the host reports the size).
template <int W>
__global__ __launch_bounds__(256) void k_write_out(WriteArgs a, uint32_t nbk) {
  constexpr int NW = 1 + 2 * W, WB = W == 1 ? 4 : 2;
  if (a.ctl->deep || a.ctl->out_total > (unsigned long long)a.ocap) return;
  const int mode = a.ctl->sel_mode;
  uint64_t T[NW];
  if (mode == S_THRESHOLD)
#pragma unroll
    for (int q = 0; q < NW; q++) T[q] = a.ctl->T[q];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  const uint32_t b = blockIdx.x * SEL_CHUNK + wv;
  if (b >= nbk) return;
  const uint32_t ub = a.b_ubase[b], ns = a.b_slots[b];
  const int n_keep = a.n_keep && a.b_keep[b] ? a.n_keep : 0;
  uint32_t obase = a.b_obase[b];
  for (uint32_t i0 = lane; i0 < ns + lane; i0 += 64 * WB) {
    // WB values, then the keys of those that are kept, in flight per lane
    double2 v[WB];
    bool s[WB];
    Key<W> mk[WB];
#pragma unroll
    for (int u = 0; u < WB; u++)
      v[u] = i0 + 64 * u < ns ? a.uc[ub + i0 + 64 * u] : make_double2(0.0, 0.0);
    if (mode == S_ALL) {
#pragma unroll
      for (int u = 0; u < WB; u++) {
        s[u] = !is_zero(v[u]);
        if (s[u]) mk[u] = ukb[ub + i0 + 64 * u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < WB; u++) {
        const uint32_t i = i0 + 64 * u;
        s[u] = false;
        if (!is_zero(v[u])) {
          if (n_keep && keep_lookup<W>(keep, n_keep, ukb[ub + i])) {
            s[u] = true;
          } else if (mode == S_THRESHOLD) {
            // |c|^2 bits decide unless they equal the threshold's
            const uint64_t m2 = (uint64_t)__double_as_longlong(weight2(v[u]));
            if (m2 != T[0]) {
              s[u] = m2 > T[0];
            } else {
              uint64_t c[NW];
              composite<W>(v[u], unmix_key<W>(ukb[ub + i]), c);
              s[u] = comp_cmp<W>(c, T) >= 0;
            }
          }
        }
      }
#pragma unroll
      for (int u = 0; u < WB; u++)
        if (s[u]) mk[u] = ukb[ub + i0 + 64 * u];
    }
#pragma unroll
    for (int u = 0; u < WB; u++) {
      const uint64_t m = __ballot(s[u]);
      if (s[u]) {
        const Key<W> raw = unmix_key<W>(mk[u]);
        const size_t o = (size_t)obase + mbcnt64(m);
#pragma unroll
        for (int w = 0; w < W; w++) {
          a.ox[(size_t)w * a.ocap + o] = raw.w[w];
          a.oz[(size_t)w * a.ocap + o] = raw.w[W + w];
        }
        if (a.out_f32)
          reinterpret_cast<float2*>(a.oc)[o] = make_float2((float)v[u].x, (float)v[u].y);
        else
          reinterpret_cast<double2*>(a.oc)[o] = v[u];
      }
      obase += (uint32_t)__popcll(m);
    }
  }
}

}  // namespace pauli
