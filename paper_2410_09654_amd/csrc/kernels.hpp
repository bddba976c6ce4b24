// HIP kernels of the Pauli-string engine (gfx950, wave64).
//
// Data flow of one engine call (commutator, linear combination, truncation,
// canonicalisation all use it):
//   k_emit<COUNT>   pair loop over (H string, O string) -> for every
//                   anticommuting pair the product string's mixed key picks a
//                   hash bin; per-workgroup bin histograms (LDS) -> counts
//                   matrix [rows][NBINS]; operator terms are binned the same way
//   k_scan          column prefix of the counts matrix, bin bases, bucket sizes
//   k_emit<SCATTER> the same pair loop, writing records (mixed key, value,
//                   source id) at their bin's cursor
//   k_merge         one workgroup per bucket of bins: records -> LDS, counting
//                   sort on the next 11 key bits + insertion sort per thread
//                   range, then every run of equal keys is folded in ascending
//                   source id (the canonical summation order), filtered, and
//                   written compactly; level-0 histogram of |c|^2 for top-M
//   k_norm, k_scale_filter
//                   Lanczos steps: b_n from the merged strings, division, filters
//   k_select / k_level1 / k_cand_level / k_finish / k_count_boundary
//                   exact radix select of the M-th largest (|c|^2, key) pair
//   k_scan_buckets / k_write
//                   bucket output bases, stable compaction into the caller's
//                   word-major output
#pragma once
#include <type_traits>

#include "device_common.hpp"

namespace pauli {

enum GroupKind : int { G_TERM = 0, G_SUM = 1, G_SUM_KAHAN32 = 2 };
enum AlphaKind : int { A_GENERAL = 0, A_ONE = 1, A_I = 2, A_DIV = 3 };  // A_DIV: v / alpha.x
enum MergeMode : int { M_PLAIN = 0, M_LANCZOS = 1 };
constexpr int MAX_GROUPS = 8;
constexpr int MAX_TERMS = 6;

struct Ctl {
  unsigned long long pe_total;   // records emitted in this pass
  unsigned int maxg[8];          // max records over aligned groups of 2^k bins
  unsigned int overflow;         // a bucket exceeded MERGE_CAP / u32 overflow
  unsigned int bad_keep;         // keep set not canonical
  unsigned long long u_slots;    // U slots written by the merges
  unsigned long long u_unique;   // distinct strings with nonzero merged value
  unsigned long long surv_total; // survivors after filters (incl. keep)
  unsigned long long keep_total; // keep-set survivors
  unsigned long long cand_n[3];  // candidate list sizes
  unsigned long long sel_K;      // records still needed inside the chosen bin
  unsigned long long sel_count;  // records in the chosen bin
  unsigned int sel_digit;
  unsigned int t_found;
  unsigned long long T[8];       // threshold composite (m2 bits, ~key words)
  unsigned long long out_total;
  double norm_hi, norm_lo;
  double inner[4];
  int sel_mode;                  // SelMode chosen on the device
  unsigned int fin_level;        // 0: finish on the level-1 list, 1: after digit 1
  unsigned int deep;             // the device select stopped: the host finishes it
  unsigned int sel_d0, sel_d1;   // threshold digits 0 and 1
  unsigned long long part_total; // records in all partitions (several-pass calls)
  unsigned int ndefer;           // buckets deferred to the full-size merge (this pass)
  unsigned int unsorted;         // a term of a direct merge is not in canonical order
  unsigned int spec_fail;        // a scatter launched before the count was read stands down
  unsigned int ticket[4];        // last_block: scan, norm, plan, select
};

struct EmitArgs {
  // commutator group: H packed [nH][2W] raw words in ascending order of their
  // lowest site (k_prep), with each entry's index in the caller's H and the
  // first entry whose lowest site is >= s (hstart[s], s = 0 .. 64W + 1);
  // O word-major
  const uint64_t* Hk;
  const uint32_t* Hidx;
  const uint32_t* hstart;
  const int* hspan;    // largest highest-minus-lowest site over H (device)
  const double2* Hc;
  int nH;
  int has_comm;
  int product;  // plain product A B (every pair, i^e h_a c_b) instead of [A, B]
  int ts_n;     // > 0: translation-symmetric operators on ts_n periodic sites; every
                // emitted string is replaced by its orbit representative
  int comm_rows;  // tile_rows x hseg
  int hseg;       // workgroups that share a tile, each every hseg-th entry of H
  int windows;    // tiles sorted by lowest site, H pruned to each wave's window
  uint32_t comm_group;
  const uint64_t* Ox;
  const uint64_t* Oz;
  int64_t Ocap;
  int64_t nO;
  const void* Oc;
  // operator terms
  int n_terms;
  int term_rows;
  const uint64_t* tx[MAX_TERMS];
  const uint64_t* tz[MAX_TERMS];
  int64_t tcap[MAX_TERMS];
  const void* tc[MAX_TERMS];
  int tf32[MAX_TERMS];
  uint32_t tgroup[MAX_TERMS];
  int tlist[MAX_TERMS];
  int64_t tstart[MAX_TERMS + 1];
  // strings longer than this are not emitted (plain mode; 0: no cap): the
  // length cap depends on the key alone, so it can act before the merge
  int max_len;
  // partition mode: the bin is the top pass_bits bits of the order key
  // (2^pass_bits partitions); records are written as the binning of a pass
  // will store them (source id in the top part_F bits of the key), the top
  // 32 bits of the order key go to ptop, and the source ids to psrc when they
  // are kept aside (wide)
  int part;
  int part_F;
  uint32_t* ptop;
  uint32_t* psrc;
  // binning
  int pass_bits;
  uint32_t pass_id;
  uint32_t* counts;
  const uint32_t* bin_base;
  void* recs;          // Rec<W, F32>[records]
  uint32_t* rsrc_wide; // source ids when they do not fit the folded bits
  int wide;
  const unsigned int* skip;  // scatter: nothing to do when *skip != 0 (nullable)
  // append mode (small calls, no count pass): bucket b (top append_F key bits)
  // holds up to append_cap records from b append_cap on, taken in any order by
  // atomics on cursor[b CURSOR_STRIDE], which counts on beyond append_cap; wide
  // ids
  uint32_t* cursor;
  int append_F;
  uint32_t append_cap;
  // wide bins: counts as bytes [rows][2^17], and the row prefixes k_scan_wide
  // makes of them
  uint8_t* counts8;
  const uint16_t* pre16;
  Ctl* ctl;
};

template <bool F32>
using RecV = typename std::conditional<F32, float2, double2>::type;

// One emitted record: the mixed key and the value.  The leading
// NBINS_LOG + pass_bits bits of the key are implied by the record's bin and
// pass, so they carry the source id instead: group in the top 3 bits, then
// the index inside the group (H index; 0 for operator terms).  Calls whose
// ids do not fit (canonicalisation of long lists) keep them in a side array.
// FP64 records of two-word keys (48 bytes) are padded to 64: the pass binning
// of the N = 128 precision-split step took 7 % less time.  Padding the FP32
// records (24 -> 32 and 40 -> 64 bytes) made their calls 3-6 % slower.
template <int W, bool F32>
constexpr int rec_pad_words() {
  return F32 ? 0 : (int)((32 - (sizeof(Key<W>) + sizeof(RecV<F32>)) % 32) % 32 / 8);
}
template <int W, bool F32, int PAD = rec_pad_words<W, F32>()>
struct Rec {
  Key<W> k;
  RecV<F32> v;
  uint64_t pad[PAD];  // written as zeros
};
template <int W, bool F32>
struct Rec<W, F32, 0> {
  Key<W> k;
  RecV<F32> v;
};
template <int W, bool F32>
DEV Rec<W, F32> make_rec(const Key<W>& k, RecV<F32> v) {
  Rec<W, F32> r;
  r.k = k;
  r.v = v;
  if constexpr (rec_pad_words<W, F32>() > 0)
#pragma unroll
    for (int i = 0; i < rec_pad_words<W, F32>(); i++) r.pad[i] = 0ull;
  return r;
}

// Row of the count matrix (and so the place of a workgroup's records inside
// every bin) for workgroup b of a grid of n: workgroups go to the eight XCDs
// round robin (b mod 8), so this numbering gives each XCD a contiguous range
// of rows.  Its partial cache lines in a bin then fill up inside its own L2
// instead of reaching memory as separate partial writes.
__device__ __forceinline__ uint32_t layout_row(uint32_t b, uint32_t n) {
  const uint32_t n8 = n & ~7u;
  return b < n8 ? (b & 7u) * (n8 >> 3) + (b >> 3) : b;
}

// TS: translation-symmetric operators (a.ts_n > 0), a kernel of its own because the search for
// the representative takes registers that the plain pair loop needs.
template <int W, bool F32, bool SCATTER, int NBL, bool TS>
// Eight waves per SIMD (two workgroups per CU) where registers and LDS allow;
// two-word strings need more than 64 registers per lane in the pair loop and
// 2^15 bins fill the LDS of a CU, so those aim at four.
__global__ __launch_bounds__(EMIT_THREADS)
__attribute__((amdgpu_waves_per_eu(W == 1 && NBL <= 14 ? 8 : 4))) void k_emit(EmitArgs a) {
  constexpr int NB = 1 << NBL;  // hash bins of this call
  // wide bins: one byte per bin (a workgroup rarely puts more than a few
  // records into one of 2^17; more than 255 send the call to the partitions).
  // The scatter takes a record's place from the bin's start, the row's prefix
  // in the bin (both from memory) and the byte.
  constexpr bool BYTES = NBL == NBINS_LOG_WIDE;
  using V = RecV<F32>;
  __shared__ uint32_t hist[BYTES ? NB / 4 : NB];
  __shared__ uint32_t queue[EMIT_THREADS / 64][128];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int row = blockIdx.x;
  const uint32_t lrow = layout_row(blockIdx.x, gridDim.x);
  if (SCATTER && a.skip && *a.skip) return;
  constexpr bool append = SCATTER && NBL == NBL_APPEND;
  if (BYTES) {
    for (int i = tid; i < NB / 4; i += EMIT_THREADS) hist[i] = 0u;
  } else if (SCATTER) {
    if (!append) {
      const uint32_t* crow = a.counts + (size_t)lrow * NB;
      for (int i = tid; i < NB; i += EMIT_THREADS) hist[i] = a.bin_base[i] + crow[i];
    }
  } else {
    for (int i = tid; i < NB; i += EMIT_THREADS) hist[i] = 0u;
  }
  __syncthreads();
  Rec<W, F32>* recs = reinterpret_cast<Rec<W, F32>*>(a.recs);
  const int F = NBL + a.pass_bits;

  auto deposit = [&](const Key<W>& raw, V val, uint32_t group, uint32_t index) {
    if (a.max_len > 0 && key_length<W>(raw) > a.max_len) return;
    Key<W> mk = mix_key<W>(raw);
    if constexpr (append) {
      const int AF = a.append_F;
      const uint32_t b = (uint32_t)(mk.w[0] >> (64 - AF));
      const uint32_t at = atomicAdd(&a.cursor[b * CURSOR_STRIDE], 1u);
      if (at < a.append_cap) {
        const size_t pos = (size_t)b * a.append_cap + at;
        mk.w[0] &= ~0ull >> AF;
        recs[pos] = make_rec<W, F32>(mk, val);
        a.rsrc_wide[pos] = (group << GROUP_SHIFT) | index;
      }
      return;
    }
    if (a.part) {
      const uint32_t pid = (uint32_t)(mk.w[0] >> (64 - a.pass_bits));
      const uint32_t pos = atomicAdd(&hist[pid], 1u);
      if (SCATTER) {
        const int PF = a.part_F;
        a.ptop[pos] = (uint32_t)(mk.w[0] >> 32);
        const uint64_t small = a.wide ? 0ull : (((uint64_t)group << (PF - 3)) | index);
        mk.w[0] = (small << (64 - PF)) | (mk.w[0] & (~0ull >> PF));
        recs[pos] = make_rec<W, F32>(mk, val);
        if (a.wide) a.psrc[pos] = (group << GROUP_SHIFT) | index;
      }
      return;
    }
    uint64_t top = mk.w[0];
    if (a.pass_bits) {
      if ((uint32_t)(top >> (64 - a.pass_bits)) != a.pass_id) return;
      top <<= a.pass_bits;
    }
    const uint32_t bin = (uint32_t)(top >> (64 - NBL));
    uint32_t pos;
    if constexpr (BYTES) {
      const uint32_t sh = (bin & 3u) * 8u;
      const uint32_t old = (atomicAdd(&hist[bin >> 2], 1u << sh) >> sh) & 255u;
      if constexpr (SCATTER) {
        pos = a.bin_base[bin] + a.pre16[(size_t)lrow * NB + bin] + old;
      } else if (old == 255u) {
        atomicOr(&a.ctl->overflow, 4u);
      }
    } else {
      pos = atomicAdd(&hist[bin], 1u);
    }
    if (SCATTER) {
      const uint64_t small = a.wide ? 0ull : (((uint64_t)group << (F - 3)) | index);
      mk.w[0] = (small << (64 - F)) | (mk.w[0] & (~0ull >> F));
      recs[pos] = make_rec<W, F32>(mk, val);
      if (a.wide) a.rsrc_wide[pos] = (group << GROUP_SHIFT) | index;
    }
  };

  if (a.has_comm && row < a.comm_rows) {
    // Each tile of EMIT_THREADS strings is put in ascending order of lowest
    // site, so a wave holds strings of nearby support and loops only over the
    // H strings whose sites can overlap its window [wlo, whi].  A pair whose
    // supports do not overlap commutes, so skipping it changes nothing.
    // Operators of few tiles are shared out over H too (hseg workgroups per
    // tile, each every hseg-th entry): see plan_rows
    constexpr int SITES = 64 * W;
    constexpr int HB = TS ? 1 : 4;  // entries of H per step (the representative search leaves no registers)
    __shared__ uint32_t scnt[SITES + 2];
    __shared__ uint16_t sperm[EMIT_THREADS];
    const V* Oc = reinterpret_cast<const V*>(a.Oc);
    const int64_t ntiles = (a.nO + EMIT_THREADS - 1) / EMIT_THREADS;
    const int tile_rows = a.comm_rows / a.hseg, seg = row % a.hseg;
    for (int64_t tile = row / a.hseg; tile < ntiles; tile += tile_rows) {
      int64_t i = tile * EMIT_THREADS + tid;
      if (a.windows) {
      // lowest and highest site of this thread's string (empty or padding
      // strings sort last, with site SITES)
      int lo = SITES, hi = -1;
      if (i < a.nO) {
#pragma unroll
        for (int w = W - 1; w >= 0; w--) {
          const uint64_t s = a.Ox[(size_t)w * a.Ocap + i] | a.Oz[(size_t)w * a.Ocap + i];
          if (s) {
            lo = 64 * w + __builtin_ctzll(s);
            if (hi < 0) hi = 64 * w + 63 - __builtin_clzll(s);
          }
        }
      }
      for (int q = tid; q < SITES + 2; q += EMIT_THREADS) scnt[q] = 0u;
      __syncthreads();
      const uint32_t rk = atomicAdd(&scnt[lo], 1u);
      __syncthreads();
      if (tid < 64) {  // exclusive scan of the SITES + 1 site counts (one wave)
        constexpr int PERL = (SITES + 1 + 63) / 64;
        uint32_t c[PERL], sum = 0;
#pragma unroll
        for (int q = 0; q < PERL; q++) {
          const int sidx = tid * PERL + q;
          c[q] = sidx <= SITES ? scnt[sidx] : 0u;
          sum += c[q];
        }
        uint32_t x = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t y = __shfl_up(x, d, 64);
          if (tid >= d) x += y;
        }
        uint32_t pre = x - sum;
#pragma unroll
        for (int q = 0; q < PERL; q++) {
          const int sidx = tid * PERL + q;
          if (sidx <= SITES) scnt[sidx] = pre;
          pre += c[q];
        }
      }
      __syncthreads();
      sperm[scnt[lo] + rk] = (uint16_t)tid;
      __syncthreads();
      i = tile * EMIT_THREADS + sperm[tid];
      __syncthreads();  // scnt / sperm are rewritten by the next tile
      }
      const bool valid = i < a.nO;
      uint64_t xb[W], zb[W];
      V cb;
#pragma unroll
      for (int w = 0; w < W; w++) {
        xb[w] = valid ? a.Ox[(size_t)w * a.Ocap + i] : 0ull;
        zb[w] = valid ? a.Oz[(size_t)w * a.Ocap + i] : 0ull;
      }
      if (valid) cb = Oc[i];
      else { cb.x = 0; cb.y = 0; }
      int hfirst = 0, hend = a.nH;
      if (a.windows) {
      // the wave's site window
      int slo = SITES, shi = -1;
#pragma unroll
      for (int w = W - 1; w >= 0; w--) {
        const uint64_t s = xb[w] | zb[w];
        if (s) {
          slo = 64 * w + __builtin_ctzll(s);
          if (shi < 0) shi = 64 * w + 63 - __builtin_clzll(s);
        }
      }
      int wlo = slo, whi = shi;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        wlo = min(wlo, __shfl_xor(wlo, d, 64));
        whi = max(whi, __shfl_xor(whi, d, 64));
      }
      if (whi < 0) continue;  // nothing but empty strings: all commute
      hfirst = (int)a.hstart[max(wlo - *a.hspan, 0)];
      hend = (int)a.hstart[whi + 1];
      }
      // this workgroup's entries: positions congruent to seg modulo hseg (which
      // strings share a wave, and so its window, differs between workgroups)
      hfirst += (seg + a.hseg - hfirst % a.hseg) % a.hseg;

      // Handle one queued (lane, H position) pair per lane.
      auto process = [&](uint32_t entry, bool active) {
        const int src_lane = (int)(entry & 63u);
        const int h = (int)(entry >> 6);
        uint64_t bx[W], bz[W];
#pragma unroll
        for (int w = 0; w < W; w++) {
          bx[w] = __shfl(xb[w], src_lane, 64);
          bz[w] = __shfl(zb[w], src_lane, 64);
        }
        V bc;
        bc.x = __shfl(cb.x, src_lane, 64);
        bc.y = __shfl(cb.y, src_lane, 64);
        if (!active) return;
        const uint64_t* hk = a.Hk + (size_t)h * (2 * W);
        Key<W> c;
        int pa = 0, pb = 0, pz = 0, pc = 0;
#pragma unroll
        for (int w = 0; w < W; w++) {
          const uint64_t ax = hk[w], az = hk[W + w];
          c.w[w] = ax ^ bx[w];
          c.w[W + w] = az ^ bz[w];
          pa += __popcll(ax & az);
          pb += __popcll(bx[w] & bz[w]);
          pz += __popcll(az & bx[w]);
          pc += __popcll(c.w[w] & c.w[W + w]);
        }
        // P_a P_b = i^(pa + pb + 2 pop(z_a & x_b) - pc) P_c; anticommuting
        // pairs contribute 2 i^e h_a c_b to [P_a, P_b] h_a c_b, every pair
        // i^e h_a c_b to the product.
        const int e = (pa + pb + 2 * pz - pc) & 3;
        // translation symmetry: several O strings can meet the same H entry
        // in one orbit; (H entry, rotation) orders their contributions
        int rot = 0;
        if constexpr (TS) rot = ts_representative<W>(c.w, a.ts_n);
        const uint32_t horig = a.Hidx[h];
        const double2 hd = a.Hc[horig];
        // FP32 records: the product of the FP64 H coefficient and the stored
        // FP32 coefficient is formed in FP64 and rounded once to FP32
        V prod;
        if constexpr (F32) {
          const double2 pd = cmul(hd, make_double2((double)bc.x, (double)bc.y));
          prod = make_float2((float)pd.x, (float)pd.y);
        } else {
          prod = cmul(hd, bc);
        }
        deposit(c, a.product ? times_ie(prod, e) : times_2ie(prod, e), a.comm_group,
                TS ? horig * 256u + (uint32_t)rot : horig);
      };

      // the range is the same for the whole wave: scalar loop counter and loads
      hfirst = __builtin_amdgcn_readfirstlane(hfirst);
      hend = __builtin_amdgcn_readfirstlane(hend);
      uint32_t qn = 0;  // wave-uniform queue fill
      for (int h0 = hfirst; h0 < hend; h0 += HB * a.hseg) {
       // parities of HB entries, whose loads are issued together
       uint32_t par[HB];
#pragma unroll
       for (int u = 0; u < HB; u++) {
        const uint64_t* hk = a.Hk + (size_t)min(h0 + u * a.hseg, hend - 1) * (2 * W);
        par[u] = 0;
#pragma unroll
        for (int w = 0; w < W; w++) par[u] += __popcll((hk[w] & zb[w]) ^ (hk[W + w] & xb[w]));
       }
#pragma unroll
       for (int u = 0; u < HB; u++) {
        const int h = h0 + u * a.hseg;
        const bool emit = valid && h < hend && (a.product || (par[u] & 1u));
        const uint64_t m = __ballot(emit);
        if (m) {
          const uint32_t pos = qn + mbcnt64(m);
          if (emit) queue[wv][pos] = (uint32_t)lane | ((uint32_t)h << 6);
          qn += (uint32_t)__popcll(m);
          if (qn >= 64) {
            wave_sync();
            process(queue[wv][lane], true);
            const uint32_t rem = qn - 64;
            const uint32_t mv = (uint32_t)lane < rem ? queue[wv][64 + lane] : 0u;
            wave_sync();
            if ((uint32_t)lane < rem) queue[wv][lane] = mv;
            wave_sync();
            qn = rem;
          }
        }
       }
      }
      if (qn) {
        wave_sync();
        process(queue[wv][lane], (uint32_t)lane < qn);
        wave_sync();
      }
    }
  } else if (a.n_terms > 0) {
    const int trow = row - (a.has_comm ? a.comm_rows : 0);
    const int64_t total = a.tstart[a.n_terms];
    const int64_t ntiles = (total + EMIT_THREADS - 1) / EMIT_THREADS;
    for (int64_t tile = trow; tile < ntiles; tile += a.term_rows) {
      const int64_t v = tile * EMIT_THREADS + tid;
      if (v < total) {
        int t = 0;
        while (t + 1 < a.n_terms && v >= a.tstart[t + 1]) t++;
        const int64_t k = v - a.tstart[t];
        Key<W> raw;
#pragma unroll
        for (int w = 0; w < W; w++) {
          raw.w[w] = a.tx[t][(size_t)w * a.tcap[t] + k];
          raw.w[W + w] = a.tz[t][(size_t)w * a.tcap[t] + k];
        }
        if constexpr (TS) (void)ts_representative<W>(raw.w, a.ts_n);
        V val;
        if (a.tf32[t]) {
          const float2 f = reinterpret_cast<const float2*>(a.tc[t])[k];
          val.x = f.x;
          val.y = f.y;
        } else {
          const double2 d = reinterpret_cast<const double2*>(a.tc[t])[k];
          val.x = d.x;
          val.y = d.y;
        }
        deposit(raw, val, a.tgroup[t], a.tlist[t] ? (uint32_t)k : 0u);
      }
    }
  }
  __syncthreads();
  if (!SCATTER) {
    uint32_t* crow = BYTES ? reinterpret_cast<uint32_t*>(a.counts8 + (size_t)lrow * NB)
                           : a.counts + (size_t)lrow * NB;
    for (int i = tid; i < (BYTES ? NB / 4 : NB); i += EMIT_THREADS) crow[i] = hist[i];
  }
}

// One partition of a several-pass call, binned for the merge: block r of the
// grid takes the r-th contiguous share of partition `part` (records as the
// merge reads them, from the partition-mode emission, and the top 32 bits of
// each order key in ptop), histograms the NBL key bits after the pass bits
// (COUNT: from ptop alone, into row r of the counts matrix) or copies each
// record to its bin cursor (SCATTER), with its source id when it is kept
// aside (wide).
struct SplitArgs {
  const void* precs;
  const uint32_t* ptop;
  const uint32_t* psrc;
  const uint32_t* pbase;  // partition starts [2^pass_bits + 1]
  uint32_t part;
  int pass_bits;
  int wide;
  uint32_t* counts;        // [gridDim.x][2^NBL]
  const uint32_t* bin_base;
  void* recs;
  uint32_t* rsrc_wide;
};

template <int W, bool F32, bool SCATTER, int NBL>
__global__ __launch_bounds__(1024) void k_split(SplitArgs a) {
  constexpr int NB = 1 << NBL;
  __shared__ uint32_t hist[NB];
  const int tid = threadIdx.x;
  // count-matrix row of this block: rows grouped by XCD, as in the emission
  const uint32_t lrow = layout_row(blockIdx.x, gridDim.x);
  const uint32_t* crow = a.counts + (size_t)lrow * NB;
  if (SCATTER)
    for (int i = tid; i < NB; i += 1024) hist[i] = a.bin_base[i] + crow[i];
  else
    for (int i = tid; i < NB; i += 1024) hist[i] = 0u;
  __syncthreads();
  const uint32_t lo = a.pbase[a.part], n = a.pbase[a.part + 1] - lo;
  const uint32_t chunk = (n + gridDim.x - 1) / gridDim.x;
  const uint32_t r0 = lo + min(n, blockIdx.x * chunk);
  const uint32_t r1 = lo + min(n, (blockIdx.x + 1) * chunk);
  // records moved as 64-bit words (word 0 is the key's leading word)
  constexpr int RW = (int)(sizeof(Rec<W, F32>) / 8);
  static_assert(sizeof(Rec<W, F32>) % 8 == 0, "records are whole 64-bit words");
  const uint64_t* in = reinterpret_cast<const uint64_t*>(a.precs);
  uint64_t* out = reinterpret_cast<uint64_t*>(a.recs);
  // SB records per thread and step, all loaded before any is binned, so that
  // each wave keeps SB loads in flight (COUNT: 4 bytes per record)
  constexpr int SB = SCATTER ? 4 : 8;
  for (uint32_t i0 = r0 + tid; i0 < r1; i0 += SB * 1024) {
    uint64_t rw[SCATTER ? SB : 1][RW];
    uint32_t top[SB], src[SB];
#pragma unroll
    for (int u = 0; u < SB; u++) {
      const uint32_t i = i0 + u * 1024;
      if (i < r1) {
        top[u] = a.ptop[i];
        if constexpr (SCATTER) {
#pragma unroll
          for (int q = 0; q < RW; q++) rw[u][q] = in[(size_t)i * RW + q];
          if (a.wide) src[u] = a.psrc[i];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < SB; u++) {
      const uint32_t i = i0 + u * 1024;
      if (i >= r1) break;
      const uint32_t bin = (top[u] << a.pass_bits) >> (32 - NBL);
      const uint32_t pos = atomicAdd(&hist[bin], 1u);
      if constexpr (SCATTER) {
#pragma unroll
        for (int q = 0; q < RW; q++) out[(size_t)pos * RW + q] = rw[u][q];
        if (a.wide) a.rsrc_wide[pos] = src[u];
      }
    }
  }
  if (!SCATTER) {
    __syncthreads();
    uint32_t* w = a.counts + (size_t)lrow * NB;
    for (int i = tid; i < NB; i += 1024) w[i] = hist[i];
  }
}

// Exclusive scan of the partition totals (one block of 1024 threads, at most
// 4096 partitions): pbase[p] for p < np, pbase[p] = total beyond.
__global__ __launch_bounds__(1024) void k_scan_part(const uint32_t* total, int np, uint32_t* pbase,
                                                    int nbase, Ctl* ctl) {
  __shared__ uint32_t scan_tmp[1024 / 64 + 1];
  const int t = threadIdx.x;
  uint32_t v[4], s = 0;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int p = t * 4 + k;
    v[k] = p < np ? total[p] : 0u;
    s += v[k];
  }
  uint32_t tot;
  uint32_t pre = block_exclusive_scan(s, scan_tmp, &tot);
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int p = t * 4 + k;
    if (p < np) pbase[p] = pre;
    pre += v[k];
  }
  for (int p = np + t; p < nbase; p += 1024) pbase[p] = tot;
  if (t == 0) ctl->part_total = tot;
}

// Partition prefixes from the first count pass, which binned every record by
// the top NBINS_LOG bits of its order key and left, per bin, the exclusive
// prefix over rows and the total.  A partition (top pass_bits bits) is an
// aligned group of 2^(NBINS_LOG - pass_bits) bins, so its prefixes and total
// are the sums of theirs.  Block r < rows reduces row r into row r of pc
// (ncol columns, those at and above 2^pass_bits zero); block `rows` reduces
// the bin totals and replaces the first 2^pass_bits of them in place (all
// read before any is written).  Each thread sums 16 consecutive bins, then a
// tree in LDS combines the 2^(10 - pass_bits) threads of a partition.
// pass_bits <= 10; the caller guarantees fewer than 2^32 records, so no sum
// wraps.
__global__ __launch_bounds__(1024) void k_part_from_bins(const uint32_t* counts, int rows,
                                                         int pass_bits, int ncol, uint32_t* pc,
                                                         uint32_t* total) {
  static_assert(NBINS == 16 * 1024, "one thread per 16 bins");
  __shared__ uint32_t part[1024];
  const int r = blockIdx.x, t = threadIdx.x;
  const int np = 1 << pass_bits, g = 1024 >> pass_bits;  // threads per partition
  const uint32_t* src = r < rows ? counts + (size_t)r * NBINS : total;
  const uint4* s4 = reinterpret_cast<const uint4*>(src) + 4 * t;
  uint32_t v = 0u;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const uint4 u = s4[q];
    v += u.x + u.y + u.z + u.w;
  }
  part[t] = v;
  __syncthreads();
  for (int d = 1; d < g; d <<= 1) {
    if ((t & (2 * d - 1)) == 0) part[t] += part[t + d];
    __syncthreads();
  }
  if (r < rows) {
    for (int p = t; p < ncol; p += 1024) pc[(size_t)r * ncol + p] = p < np ? part[p * g] : 0u;
  } else if (t < np) {
    total[t] = part[t * g];
  }
}

// Column-wise exclusive prefix of the counts matrix (rows x nbins, row
// major) and the bin totals.  A block of SC_NSEG x SC_COLS threads covers
// SC_COLS columns: thread (segment g, column b) loads rows
// [SC_SEG g, SC_SEG g + SC_SEG) of column b all at once, the segment sums of
// a column are combined in LDS, and each thread writes its rows' prefixes.
// rows <= SC_NSEG * SC_SEG.  Totals above 32 bits set *overflow |= 2.
constexpr int SC_COLS = 32, SC_SEG = 36, SC_NSEG = 32;
constexpr int SC_ROWS_MAX = SC_SEG * SC_NSEG;
DEV void scan_cols(uint32_t* counts, int rows, uint32_t* bin_total, Ctl* ctl, int nbins) {
  __shared__ unsigned long long ssum[SC_NSEG][SC_COLS];
  const int col = threadIdx.x % SC_COLS, seg = threadIdx.x / SC_COLS;
  const int b = blockIdx.x * SC_COLS + col;
  const int r0 = seg * SC_SEG;
  const bool on = b < nbins;
  uint32_t c[SC_SEG];
#pragma unroll
  for (int q = 0; q < SC_SEG; q++)
    c[q] = (on && r0 + q < rows) ? counts[(size_t)(r0 + q) * nbins + b] : 0u;
  unsigned long long s = 0;
#pragma unroll
  for (int q = 0; q < SC_SEG; q++) s += c[q];
  ssum[seg][col] = s;
  __syncthreads();
  const int last = (rows - 1) / SC_SEG;  // last segment that holds rows
  unsigned long long run = 0;
  if (seg <= last)
    for (int g = 0; g < seg; g++) run += ssum[g][col];
#pragma unroll
  for (int q = 0; q < SC_SEG; q++) {
    if (on && r0 + q < rows) counts[(size_t)(r0 + q) * nbins + b] = (uint32_t)run;
    run += c[q];
  }
  if (on && seg == last) {  // the last segment's running sum is the column total
    if (run > 0xFFFFFFFFull) atomicOr(&ctl->overflow, 2u);
    st_agent(&bin_total[b], (uint32_t)run);
  }
}
__global__ __launch_bounds__(SC_COLS * SC_NSEG) void k_scan_cols(uint32_t* counts, int rows,
                                                                 uint32_t* bin_total, Ctl* ctl,
                                                                 int nbins) {
  scan_cols(counts, rows, bin_total, ctl, nbins);
}

// Both scans of a count pass: every block turns its columns into row prefixes
// (scan_cols), then the last block scans the 2^NBL bin totals into bin bases
// and takes the largest totals over aligned groups of 1, 2, 4, 8, 16 bins:
// thread t owns the BPT consecutive bins from t BPT; groups wider than BPT are
// combined in LDS.
template <int NBL>
__global__ __launch_bounds__(1024) void k_scan(uint32_t* counts, int rows, uint32_t* bin_total,
                                               uint32_t* bin_base, Ctl* ctl,
                                               unsigned long long* look,
                                               unsigned long long spec_cap,
                                               unsigned int merge_cap) {
  static_assert(SC_COLS * SC_NSEG == 1024, "one block size for both parts");
  constexpr int NB = 1 << NBL;
  constexpr int BPT = NB / 1024;
  static_assert(BPT * 1024 == NB, "every thread owns whole bins");
  // clears a look-back state per bin, for merges that follow (nullable)
  if (look && threadIdx.x < SC_COLS) look[blockIdx.x * SC_COLS + threadIdx.x] = 0ull;
  scan_cols(counts, rows, bin_total, ctl, NB);
  if (!last_block(&ctl->ticket[0])) return;
  __shared__ unsigned long long tmp[17];
  __shared__ unsigned int gmax[5];
  __shared__ uint32_t gsum[1024];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  if (t < 5) gmax[t] = 0u;
  uint32_t v[BPT];
  if constexpr (BPT >= 4) {
    const uint4* src = reinterpret_cast<const uint4*>(bin_total) + (size_t)t * (BPT / 4);
#pragma unroll
    for (int q = 0; q < BPT / 4; q++) {
      const uint4 c = src[q];
      v[4 * q] = c.x;
      v[4 * q + 1] = c.y;
      v[4 * q + 2] = c.z;
      v[4 * q + 3] = c.w;
    }
  } else {
#pragma unroll
    for (int q = 0; q < BPT; q++) v[q] = bin_total[t * BPT + q];
  }
  unsigned long long s = 0;
#pragma unroll
  for (int k = 0; k < BPT; k++) s += v[k];
  gsum[t] = s > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)s;
  // block exclusive scan (u64); its barriers also publish gsum and gmax
  unsigned long long x = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) tmp[wv] = x;
  __syncthreads();
  unsigned long long w = lane < 16 ? tmp[lane] : 0ull;
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    const unsigned long long y = __shfl_up(w, d, 64);
    if (lane >= d) w += y;
  }
  const unsigned long long before = wv > 0 ? __shfl(w, wv - 1, 64) : 0ull;
  const unsigned long long total = __shfl(w, 15, 64);
  unsigned long long pre = before + x - s;
  uint32_t o[BPT];
#pragma unroll
  for (int q = 0; q < BPT; q++) {
    o[q] = (uint32_t)pre;
    pre += v[q];
  }
  if constexpr (BPT >= 4) {
    uint4* dst = reinterpret_cast<uint4*>(bin_base) + (size_t)t * (BPT / 4);
#pragma unroll
    for (int q = 0; q < BPT / 4; q++)
      dst[q] = make_uint4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
  } else {
#pragma unroll
    for (int q = 0; q < BPT; q++) bin_base[t * BPT + q] = o[q];
  }
#pragma unroll
  for (int lg = 0; lg < 5; lg++) {
    const int g = 1 << lg;
    unsigned int best = 0;
    if (g <= BPT) {
#pragma unroll
      for (int k = 0; k < BPT; k += g) {
        unsigned long long acc = 0;
#pragma unroll
        for (int q = 0; q < (g <= BPT ? g : 1); q++) acc += v[k + q];
        best = max(best, acc > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned int)acc);
      }
    } else if ((t & (g / BPT - 1)) == 0) {
      unsigned long long acc = 0;
      for (int q = 0; q < g / BPT; q++) acc += gsum[t + q];
      best = acc > 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned int)acc;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) best = max(best, (unsigned int)__shfl_xor((int)best, d, 64));
    if (lane == 0) atomicMax(&gmax[lg], best);
  }
  __syncthreads();
  if (t == 0) {
    bin_base[NB] = (uint32_t)total;
    ctl->pe_total = total;
    ctl->ndefer = 0u;
    if (total > 0xFFFFFFFFull) ctl->overflow |= 2u;
    for (int lg = 0; lg < 5; lg++) ctl->maxg[lg] = gmax[lg];
    // a scatter already launched for a single pass laid out for spec_cap
    // records stands down unless the records fit and every bin fits a bucket
    if (spec_cap) ctl->spec_fail = (total > spec_cap || gmax[0] > merge_cap) ? 1u : 0u;
  }
}

// The scans of a wide count: row prefixes (16 bits; a bin whose total exceeds
// merge_cap sends the call to the partitions, so no prefix that is used wraps)
// from the byte counts, four bins per thread and row, and the bin totals; the
// last block scans those into bin bases, 16384 bins at a time, as k_scan does.
constexpr int SW_SEG = 20, SW_ROWS_MAX = SW_SEG * 32;
__global__ __launch_bounds__(1024) void k_scan_wide(const uint8_t* counts8, int rows,
                                                    uint16_t* pre16, uint32_t* bin_total,
                                                    uint32_t* bin_base, Ctl* ctl,
                                                    unsigned long long* look) {
  constexpr int NB = NBINS_WIDE;
  __shared__ uint4 ssum[32][32];
  const int t = threadIdx.x, col = t & 31, seg = t >> 5, lane = t & 63, wv = t >> 6;
  const int word = blockIdx.x * 32 + col;  // bins 4 word .. 4 word + 3
  if (t < 128) look[blockIdx.x * 128 + t] = 0ull;
  {
    const int r0 = seg * SW_SEG;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(counts8) + word;
    uint32_t c[SW_SEG];
#pragma unroll
    for (int q = 0; q < SW_SEG; q++) c[q] = r0 + q < rows ? src[(size_t)(r0 + q) * (NB / 4)] : 0u;
    uint4 s = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int q = 0; q < SW_SEG; q++) {
      s.x += c[q] & 255u;
      s.y += (c[q] >> 8) & 255u;
      s.z += (c[q] >> 16) & 255u;
      s.w += c[q] >> 24;
    }
    ssum[seg][col] = s;
    __syncthreads();
    const int last = (rows - 1) / SW_SEG;
    uint4 run = make_uint4(0u, 0u, 0u, 0u);
    if (seg <= last)
      for (int g = 0; g < seg; g++) {
        const uint4 o = ssum[g][col];
        run.x += o.x;
        run.y += o.y;
        run.z += o.z;
        run.w += o.w;
      }
    uint2* dst = reinterpret_cast<uint2*>(pre16) + word;
#pragma unroll
    for (int q = 0; q < SW_SEG; q++) {
      if (r0 + q < rows)
        dst[(size_t)(r0 + q) * (NB / 4)] =
            make_uint2((run.x & 0xFFFFu) | (run.y << 16), (run.z & 0xFFFFu) | (run.w << 16));
      run.x += c[q] & 255u;
      run.y += (c[q] >> 8) & 255u;
      run.z += (c[q] >> 16) & 255u;
      run.w += c[q] >> 24;
    }
    if (seg == last) {
      st_agent(&bin_total[4 * word], run.x);
      st_agent(&bin_total[4 * word + 1], run.y);
      st_agent(&bin_total[4 * word + 2], run.z);
      st_agent(&bin_total[4 * word + 3], run.w);
    }
  }
  if (!last_block(&ctl->ticket[0])) return;
  __shared__ unsigned long long tmp[17];
  __shared__ unsigned int gmax[5];
  if (t < 5) gmax[t] = 0u;
  unsigned long long carry = 0;
  unsigned int best[5] = {0u, 0u, 0u, 0u, 0u};
  for (int b0 = 0; b0 < NB; b0 += 16 * 1024) {
    const uint4* src = reinterpret_cast<const uint4*>(bin_total + b0) + 4 * t;
    uint32_t v[16];
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const uint4 c = src[q];
      v[4 * q] = c.x;
      v[4 * q + 1] = c.y;
      v[4 * q + 2] = c.z;
      v[4 * q + 3] = c.w;
    }
    unsigned long long s = 0;
#pragma unroll
    for (int k = 0; k < 16; k++) s += v[k];
#pragma unroll
    for (int lg = 0; lg < 5; lg++)
#pragma unroll
      for (int k = 0; k < 16; k += 1 << lg) {
        unsigned int acc = 0;  // (at most 16 x 640 x 255)
#pragma unroll
        for (int q = 0; q < (1 << lg); q++) acc += v[k + q];
        best[lg] = max(best[lg], acc);
      }
    unsigned long long x = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) tmp[wv] = x;
    __syncthreads();
    unsigned long long w = lane < 16 ? tmp[lane] : 0ull;
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
      const unsigned long long y = __shfl_up(w, d, 64);
      if (lane >= d) w += y;
    }
    const unsigned long long before = wv > 0 ? __shfl(w, wv - 1, 64) : 0ull;
    unsigned long long pre = carry + before + x - s;
    carry += __shfl(w, 15, 64);
    uint4* dst = reinterpret_cast<uint4*>(bin_base + b0) + 4 * t;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      uint4 o;
      o.x = (uint32_t)pre;
      pre += v[4 * q];
      o.y = (uint32_t)pre;
      pre += v[4 * q + 1];
      o.z = (uint32_t)pre;
      pre += v[4 * q + 2];
      o.w = (uint32_t)pre;
      pre += v[4 * q + 3];
      dst[q] = o;
    }
    __syncthreads();  // tmp is rewritten by the next bins
  }
#pragma unroll
  for (int lg = 0; lg < 5; lg++) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1)
      best[lg] = max(best[lg], (unsigned int)__shfl_xor((int)best[lg], d, 64));
    if (lane == 0) atomicMax(&gmax[lg], best[lg]);
  }
  __syncthreads();
  if (t == 0) {
    bin_base[NB] = (uint32_t)carry;
    ctl->pe_total = carry;
    ctl->ndefer = 0u;
    if (carry > 0xFFFFFFFFull) ctl->overflow |= 2u;
    for (int lg = 0; lg < 5; lg++) ctl->maxg[lg] = gmax[lg];
  }
}

// ---------------------------------------------------------------------------
// Linear combinations of canonical operators, merged without emission.  A
// term in canonical order (ascending mixed key, distinct strings) holds the
// strings of hash bucket b (the top F bits of the mixed key) as one
// contiguous run, so the merge can read each bucket straight from the terms:
// k_term_stream and k_term_bounds find the runs, the former also confirms the
// order of terms the engine did not write itself.
// ---------------------------------------------------------------------------
struct TermView {
  int n_terms;
  int F;  // 2^F buckets
  const uint64_t* tx[MAX_TERMS];
  const uint64_t* tz[MAX_TERMS];
  int64_t tcap[MAX_TERMS];
  int64_t tn[MAX_TERMS];
  const void* tc[MAX_TERMS];
  int tf32[MAX_TERMS];
  uint32_t tgroup[MAX_TERMS];
  const uint32_t* bounds;  // [n_terms][2^F + 1]: strings of term t in buckets below b
};

template <int W>
DEV Key<W> load_raw(const uint64_t* x, const uint64_t* z, int64_t cap, int64_t i) {
  Key<W> raw;
#pragma unroll
  for (int w = 0; w < W; w++) {
    raw.w[w] = x[(size_t)w * cap + i];
    raw.w[W + w] = z[(size_t)w * cap + i];
  }
  return raw;
}

// Bucket bounds of terms by one pass over them (each thread one string):
// string i starts every bucket after string i - 1's up to its own.  Sets
// *flag when mixed keys do not strictly ascend (bounds are then not used).
// Used for terms the engine did not write, which have to be read to check
// their order in any case, and for short ones, whose binary search below is a
// chain of dependent loads (9 us for 16384 strings, and 2 us for the check as
// a kernel of its own; 3.9 us here).
// More than STREAM_GAP buckets between two strings (short terms beside a long
// one, the ends of a term) are filled by the whole wave: a thread for each gap
// took 147 us for 4 M one-word strings plus one, now 35.  A wave that sees a
// descent, or the flag of one that did, fills nothing: with every string
// filling the gap to its predecessor, two terms of 2^20 shuffled strings took
// 3.2 ms, now 16 us.
constexpr int STREAM_GAP = 8;
template <int W>
__global__ __launch_bounds__(256) void k_term_stream(TermView v, uint32_t mask, uint32_t* bounds,
                                                     unsigned int* flag) {
  const uint32_t nb = 1u << v.F;
  const int lane = threadIdx.x & 63;
  int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  bool bad = false;
  const bool known =
      __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
#pragma unroll
  for (int t = 0; t < MAX_TERMS; t++) {
    if (t >= v.n_terms || !((mask >> t) & 1u)) continue;
    const int64_t n = v.tn[t];
    int64_t from = 0, to = -1;  // bounds [from, to] are id
    if (id >= 0 && id <= n) {
      to = nb;
      if (id > 0) {
        const Key<W> p = mix_key<W>(load_raw<W>(v.tx[t], v.tz[t], v.tcap[t], id - 1));
        from = (v.F ? (int64_t)(p.w[0] >> (64 - v.F)) : 0) + 1;
        if (id < n) {
          const Key<W> m = mix_key<W>(load_raw<W>(v.tx[t], v.tz[t], v.tcap[t], id));
          bad = bad || key_cmp<W>(p, m) >= 0;
          to = v.F ? (int64_t)(m.w[0] >> (64 - v.F)) : 0;
        }
      } else if (n > 0) {
        const Key<W> m = mix_key<W>(load_raw<W>(v.tx[t], v.tz[t], v.tcap[t], 0));
        to = v.F ? (int64_t)(m.w[0] >> (64 - v.F)) : 0;
      }
    }
    if (!known && !__ballot(bad)) {
      uint32_t* bt = bounds + (size_t)t * (nb + 1);
      const bool wide = to - from >= STREAM_GAP;
      if (!wide)
        for (int64_t b = from; b <= to; b++) bt[b] = (uint32_t)id;
      for (uint64_t m = __ballot(wide); m; m &= m - 1) {
        const int l = __builtin_ctzll(m);
        const uint32_t b0 = __shfl((uint32_t)from, l, 64), b1 = __shfl((uint32_t)to, l, 64);
        const uint32_t first = __shfl((uint32_t)id, l, 64);
        for (uint32_t b = b0 + lane; b <= b1; b += 64) bt[b] = first;
      }
    }
    id -= n + 1;
  }
  // one store a block, and none when it is there already: an atomic from every
  // wave in flight queued up for 0.1 ms
  if (__syncthreads_or(bad ? 1 : 0) && threadIdx.x == 0 &&
      __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u)
    st_agent(flag, 1u);
}

// bounds[t][b], b = 0 .. 2^F: the first string of term t whose bucket is at
// least b (binary search over the canonical order; one thread per entry).
template <int W>
__global__ __launch_bounds__(256) void k_term_bounds(TermView v, uint32_t mask, uint32_t* bounds) {
  const int64_t nb1 = ((int64_t)1 << v.F) + 1;
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= nb1 * v.n_terms) return;
  const int t = (int)(id / nb1);
  if (!((mask >> t) & 1u)) return;
  const uint64_t b = (uint64_t)(id - (int64_t)t * nb1);
  int64_t lo = 0, hi = v.tn[t];
  if (v.F == 0) {
    lo = b ? hi : 0;
  } else {
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      const Key<W> m = mix_key<W>(load_raw<W>(v.tx[t], v.tz[t], v.tcap[t], mid));
      if ((m.w[0] >> (64 - v.F)) < b) lo = mid + 1;
      else hi = mid;
    }
  }
  bounds[id] = (uint32_t)lo;
}

struct MergeArgs {
  const uint32_t* bin_base;
  const uint32_t* bin_count;  // append mode: the cursors (bucket j lies from j append_cap on)
  uint32_t append_cap;
  int nbins_log;  // hash bins of the call: 2^nbins_log per pass
  int g_log;
  int digit_shift;
  int pass_bits;
  uint32_t pass_id;
  int wide;
  const void* recs;
  const uint32_t* rsrc_wide;
  double2 alpha[MAX_GROUPS];
  int alpha_kind[MAX_GROUPS];
  int gkind[MAX_GROUPS];
  int mode;
  int single;  // one group, not Kahan: runs fold as plain sums
  int round32;
  int max_len;
  int use_eps;
  double eps2;
  const void* keep_mk;
  int n_keep;
  unsigned long long u_off;
  void* uk;
  double2* uc;
  uint32_t bucket_off;
  uint32_t* b_ubase;
  uint32_t* b_slots;
  uint32_t* b_surv;
  uint32_t* b_keep;
  uint32_t* b_unique;
  uint32_t* hist0;
  uint32_t* defer;  // buckets above the small variant's capacity (nullptr: none deferred)
  Ctl* ctl;
  TermView tv;      // direct merges: the canonical terms and their bucket runs
  // final merges (nothing to select): the output operator, the look-back
  // states of this launch's buckets (zero at the start), and the host's copy of
  // the control block, written by the last launch of the call
  unsigned long long* look;
  uint64_t* ox;
  uint64_t* oz;
  void* oc;
  int64_t ocap;
  int out_f32;
  Ctl* hctl;
};

// Look-back: the number of output rows before bucket j of a launch, from the
// states of the buckets below it.  A state is 0 until the bucket has counted
// its rows, then LB_SUM | rows (set by the caller), and LB_TOTAL | (rows up to and including the
// bucket) once its own look-back is done; bucket 0 starts from `base`.  Buckets
// are numbered in the order in which their blocks draw them, so every bucket
// waited for belongs to a block that is already running, and no block waits
// before it has published its own count: the lowest unfinished bucket waits
// for nothing, and every wait ends.  Called by one whole wave.
constexpr unsigned long long LB_SUM = 1ull << 62, LB_TOTAL = 2ull << 62, LB_VALUE = LB_SUM - 1ull;
DEV unsigned long long look_back(unsigned long long* look, uint32_t j, uint32_t rows,
                                 unsigned long long base) {
  const int lane = threadIdx.x & 63;
  unsigned long long before = j == 0 ? base : 0ull;
  for (int64_t hi = (int64_t)j - 1; hi >= 0; hi -= 64) {
    const int64_t i = hi - lane;
    unsigned long long w = i >= 0 ? 0ull : LB_TOTAL;  // (below bucket 0)
    uint64_t m;
    for (;;) {
      if (w == 0ull) w = __hip_atomic_load(&look[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t none = __ballot(w == 0ull);
      m = __ballot((w & LB_TOTAL) != 0ull);
      // every bucket down to the nearest total has published
      if (!(none & (m ? (m & (~m + 1ull)) - 1ull : ~0ull))) break;
      __builtin_amdgcn_s_sleep(8);
    }
    const int last = m ? __builtin_ctzll(m) : 63;
    unsigned long long v = lane <= last ? (w & LB_VALUE) : 0ull;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    before += v;
    if (m) break;
  }
  if (lane == 0) st_agent(&look[j], LB_TOTAL | (before + rows));
  return before;
}
// The control block to the host's pinned copy: the host reads it after it has
// waited for the stream, with no copy of its own.  Called by a whole block, all
// of whose writes to the block lie before it.
DEV void publish(const Ctl* ctl, Ctl* hctl) {
  __syncthreads();
  if (!hctl) return;
  const uint32_t* src = reinterpret_cast<const uint32_t*>(ctl);
  uint32_t* dst = reinterpret_cast<uint32_t*>(hctl);
  for (uint32_t i = threadIdx.x; i < sizeof(Ctl) / 4; i += blockDim.x) dst[i] = src[i];
}

template <int W>
DEV bool keep_lookup(const Key<W>* keep, int n, const Key<W>& mk) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    const int c = key_cmp<W>(keep[mid], mk);
    if (c == 0) return true;
    if (c < 0) lo = mid + 1;
    else hi = mid;
  }
  return false;
}

DEV double2 apply_alpha(int kind, double2 alpha, double2 v) {
  if (kind == A_ONE) return v;
  if (kind == A_I) return make_double2(-v.y, v.x);
  if (kind == A_DIV) return make_double2(v.x / alpha.x, v.y / alpha.x);
  return cmul(alpha, v);
}

DEV double round_to_f32(double v) { return (double)(float)v; }

// The DIGIT_BITS + 32 bits of a mixed key that follow its first `shift`
// bits (0 <= shift < 64): the in-bucket digit on top, then 32 sort bits.
template <int W>
DEV uint64_t key_window(const Key<W>& m, int shift) {
  const uint64_t hi = shift ? ((m.w[0] << shift) | (m.w[1] >> (64 - shift))) : m.w[0];
  return hi >> (64 - DIGIT_BITS - 32);
}

// Rank of every record of the block inside its digit group by full
// (mixed key, source id) comparison, used when two distinct keys of a group
// share their 32 sort bits.  On entry mk/sx hold the n records grouped by
// digit (ascending) and id their source ids; on return mk/sx are in (key,
// source id) order.
template <int W, int THREADS, int CAP>
DEV void merge_full_rank(Key<W>* mk, uint32_t* sx, const uint32_t* id, uint32_t n, int shift) {
  constexpr int PER = (CAP + THREADS - 1) / THREADS;
  Key<W> k[PER];
  uint32_t x[PER], pos[PER];
#pragma unroll
  for (int q = 0; q < PER; q++) {
    const uint32_t p = threadIdx.x + q * THREADS;
    pos[q] = p;
    if (p < n) {
      k[q] = mk[p];
      x[q] = sx[p];
      const uint32_t me = id[p];
      const uint32_t d = (uint32_t)(key_window<W>(k[q], shift) >> 32);
      // digit group [s0, s1): binary searches on the (ascending) digits
      uint32_t lo = 0, hi = p;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint32_t)(key_window<W>(mk[mid], shift) >> 32) < d) lo = mid + 1;
        else hi = mid;
      }
      const uint32_t s0 = lo;
      lo = p + 1;
      hi = n;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if ((uint32_t)(key_window<W>(mk[mid], shift) >> 32) <= d) lo = mid + 1;
        else hi = mid;
      }
      const uint32_t s1 = lo;
      uint32_t rank = 0;
      for (uint32_t r = s0; r < s1; r++) rank += key_src_less<W>(mk[r], id[r], k[q], me) ? 1u : 0u;
      pos[q] = s0 + rank;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; q++) {
    const uint32_t p = threadIdx.x + q * THREADS;
    if (p < n) {
      mk[pos[q]] = k[q];
      sx[pos[q]] = x[q];
    }
  }
  __syncthreads();
}

// THREADS threads merge one bucket of at most CAP records.  MODE
// MERGE_GRID: block j merges bucket j; MERGE_SMALL: the same, but a bucket
// above CAP goes to the list a.defer instead (the small-bucket variant, 512
// threads, three blocks per CU by LDS); MERGE_LIST: the blocks merge the
// listed buckets.
enum MergeKind : int { MERGE_GRID = 0, MERGE_SMALL = 1, MERGE_LIST = 2 };
// DIRECT: the records of bucket j are the j-th runs of the canonical terms
// of a.tv (g_log = 0, no pass bits), read in place; source id = term group.
// OUT: nothing is selected afterwards, so every survivor is an output row and
// the block writes its strings to the output itself, at the row that the
// look-back over the earlier buckets gives (no merged copy, no second pass to
// move it: 19 M records into 13 M strings 386 + 278 -> 504 us). Not with MERGE_LIST, and MERGE_SMALL only where every
// bucket fits.
template <int W, bool F32, int THREADS, int CAP, int MODE, bool DIRECT = false, bool OUT = false>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(MODE == MERGE_SMALL ? 6 : 8))) void k_merge(MergeArgs a) {
  constexpr bool SMALL = MODE == MERGE_SMALL;
  using V = RecV<F32>;
  constexpr int PER = (CAP + THREADS - 1) / THREADS;
  constexpr int DPT = NDIGITS / THREADS;
  static_assert(CAP <= NDIGITS, "the source ids of a bucket fit the digit table");
  static_assert(SEL0_BINS == 2 * NDIGITS,
                "digit counts and the |c|^2 histogram (16-bit counters, two per word) share LDS");
  // Sort: a counting sort on the DIGIT_BITS key bits after the bucket bits,
  // then the rank of every record inside its digit group by a 64-bit sort
  // word (the next 32 key bits, then the source id), read from `swd` (which
  // aliases mk until the keys are written).  mk / sx then hold the keys and
  // SX words (group, position in the bucket) in sorted order; the values stay
  // in sv where their records lie in the bucket, so a one-word record is read
  // from memory once, key and value together.  (Values written in sorted order were
  // read a second time for it: 7 us of a block's 33 us, and in direct merges,
  // whose values lie in arrays of their own, from memory: 4.82 -> 3.59 ms for
  // 137 M term strings, with the terms' pointers in LDS.)  Two-word records are
  // read twice in any case, the value with the second read (with the first
  // one the merge of 27 M of them took 0.84 ms, so 0.79).  dh holds the digit counts and starts, then the
  // level-0 histogram of |c|^2.  Two distinct keys of one digit group with
  // equal sort bits show up as adjacent entries with equal windows but
  // different keys; the block then ranks by full keys (merge_full_rank).
  __shared__ Key<W> mk[CAP];
  __shared__ __align__(16) V sv[CAP];
  static_assert(sizeof(Key<W>) >= sizeof(uint64_t), "sort words alias the keys");
  uint64_t* const swd = reinterpret_cast<uint64_t*>(mk);
  // SX word: source group on top, a flag for strings above the length cap
  // (direct merges), the record's position in the bucket
  constexpr uint32_t SX_LONG = 1u << (GROUP_SHIFT - 1), SX_POS = SX_LONG - 1u;
  __shared__ uint32_t sx[CAP];
  __shared__ int s_collide;
  __shared__ uint32_t s_pk;
  __shared__ uint32_t dh[NDIGITS];
  uint32_t* const h0 = dh;
  __shared__ uint32_t scan_tmp[THREADS / 64 + 1];
  __shared__ int s_gk[MAX_GROUPS], s_ak[MAX_GROUPS];
  __shared__ double2 s_al[MAX_GROUPS];
  __shared__ uint32_t sbb[17];
  __shared__ int s_kr[2];
  constexpr int NHW = (CAP + 63) / 64;
  __shared__ uint64_t hmask[NHW];  // bit p: sorted position p starts a run of equal keys

  const int tid = threadIdx.x;
  struct TermDesc {
    const uint64_t *x, *z;
    const void* c;
    int64_t cap;
    uint32_t group;
    int f32;
  };
  __shared__ TermDesc s_term[DIRECT ? MAX_TERMS : 1];
  if constexpr (DIRECT) {
    if (tid < a.tv.n_terms) {
      TermDesc d;
      d.x = a.tv.tx[tid];
      d.z = a.tv.tz[tid];
      d.c = a.tv.tc[tid];
      d.cap = a.tv.tcap[tid];
      d.group = a.tv.tgroup[tid];
      d.f32 = a.tv.tf32[tid];
      s_term[tid] = d;
    }
    __syncthreads();
  }
  // OUT: the first output row of bucket j with `rows` rows; the last bucket's
  // block also writes the total and, when asked, the host's control block
  __shared__ unsigned long long s_row;
  auto finish = [&](const uint32_t j, const uint32_t rows) -> unsigned long long {
    if constexpr (OUT) {
      if (tid < 64) {
        const unsigned long long r = look_back(a.look, j, rows, a.ctl->out_total);
        if (tid == 0) {
          s_row = r;
          if (j == gridDim.x - 1) {
            a.ctl->out_total = r + rows;
            a.ctl->surv_total = r + rows;
            if (!a.use_eps) a.ctl->u_unique = r + rows;
            a.ctl->sel_mode = 0;  // S_ALL
            st_agent(&a.ctl->ticket[2], 0u);
          }
        }
      }
      __syncthreads();
      if (j == gridDim.x - 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        publish(a.ctl, a.hctl);
      }
      return s_row;
    }
    return 0ull;
  };
  auto bucket = [&](const uint32_t j) {
  const uint32_t gb = a.bucket_off + j;
  uint32_t b0, b1;
  // direct merges: start of the bucket's run in each term and the run's
  // first position in the bucket (tpre, ascending over the terms)
  uint32_t tst[DIRECT ? MAX_TERMS : 1], tpre[DIRECT ? MAX_TERMS : 1];
  if constexpr (DIRECT) {
    // (all bounds loaded before any is used: a load per term and branch made a
    // chain of up to six reads)
    const uint32_t stride = (1u << a.tv.F) + 1u;
    uint32_t s0[MAX_TERMS], s1[MAX_TERMS];
#pragma unroll
    for (int t = 0; t < MAX_TERMS; t++) {
      const uint32_t* bt = a.tv.bounds + (size_t)min(t, a.tv.n_terms - 1) * stride + j;
      s0[t] = bt[0];
      s1[t] = bt[1];
    }
    b0 = 0u;
    b1 = 0u;
#pragma unroll
    for (int t = 0; t < MAX_TERMS; t++) {
      tst[t] = 0u;
      tpre[t] = 0xFFFFFFFFu;
      if (t < a.tv.n_terms) {
        tst[t] = s0[t];
        tpre[t] = b1 - b0;
        b0 += s0[t];
        b1 += s1[t];
      }
    }
    if (a.ctl->unsorted) b0 = b1 = 0u;  // the call is redone by emission
  } else if (MODE == MERGE_GRID && a.bin_count) {
    const uint32_t cnt = a.bin_count[j * CURSOR_STRIDE];
    b0 = j * a.append_cap;
    // records beyond the bucket's room were not written: the call is redone
    b1 = b0 + (cnt > a.append_cap ? (uint32_t)CAP + 1u : cnt);
    if (tid == 0) atomicAdd(&a.ctl->pe_total, (unsigned long long)cnt);
  } else {
    b0 = a.bin_base[j << a.g_log];
    b1 = a.bin_base[(j + 1) << a.g_log];
  }
  const uint32_t n = b1 - b0;
  const unsigned long long ub = a.u_off + b0;
  // direct merges: where the string at bucket position i lies (in the last
  // term whose run starts at or before i; empty runs are passed over), from the
  // terms' copies in LDS (indexed by lane, the kernel arguments would be read
  // from memory before the string)
  struct TermPos {
    const uint64_t *x, *z;
    const void* c;
    int64_t cap, e;
    uint32_t group;
    int f32;
  };
  auto term_pos = [&](uint32_t i) -> TermPos {
    int t = 0;
    int64_t e = 0;
#pragma unroll
    for (int u = 0; u < (DIRECT ? MAX_TERMS : 1); u++)
      if (i >= tpre[u]) {
        t = u;
        e = (int64_t)tst[u] + (int64_t)(i - tpre[u]);
      }
    const TermDesc& d = s_term[t];
    return TermPos{d.x, d.z, d.c, d.cap, e, d.group, d.f32};
  };
  // direct merges apply the length cap here (emission applies it to records
  // before they reach a bucket)
  const int cap_len = DIRECT && a.mode == M_PLAIN ? a.max_len : 0;
  auto term_src = [&](uint32_t group, const Key<W>& raw) -> uint32_t {
    const uint32_t g = group << GROUP_SHIFT;
    return cap_len > 0 && key_length<W>(raw) > cap_len ? g | SX_LONG : g;
  };
  auto term_raw = [&](const TermPos& q) -> Key<W> { return load_raw<W>(q.x, q.z, q.cap, q.e); };
  auto term_val = [&](const TermPos& q) -> V {
    V v;
    if (F32 || q.f32) {
      const float2 f = reinterpret_cast<const float2*>(q.c)[q.e];
      v.x = f.x;
      v.y = f.y;
    } else {
      const double2 d = reinterpret_cast<const double2*>(q.c)[q.e];
      v.x = d.x;
      v.y = d.y;
    }
    return v;
  };
  if constexpr (OUT) {
    if (n > (uint32_t)CAP) {
      if (tid == 0) {
        atomicOr(&a.ctl->overflow, 1u);
        __builtin_amdgcn_s_waitcnt(0);
        if (j > 0) st_agent(&a.look[j], LB_SUM);
      }
      finish(j, 0u);
      return;
    }
  }
  if (n > (uint32_t)CAP) {
    if (SMALL) {  // left to the full-size variant
      if (tid == 0) a.defer[atomicAdd(&a.ctl->ndefer, 1u)] = j;
      return;
    }
    if (tid == 0) {
      atomicOr(&a.ctl->overflow, 1u);
      a.b_ubase[gb] = (uint32_t)ub;
      a.b_slots[gb] = 0;
      a.b_surv[gb] = 0;
      a.b_keep[gb] = 0;
      a.b_unique[gb] = 0;
    }
    return;
  }
  const Rec<W, F32>* recs = reinterpret_cast<const Rec<W, F32>*>(a.recs);
  const int F = a.nbins_log + a.pass_bits;
  const uint32_t ibits = (uint32_t)(F - 3);
  // Per record the digit, its rank among the digit's records, the source id
  // and the 32 sort bits stay in registers, and at W = 1 the order key; a
  // wider key is read a second time, from cache, for the sorted write, which
  // keeps the kernel spill-free at 8 waves per SIMD.
  constexpr bool HOLD_KEY = W == 1;
  uint32_t dig[PER], rnk[PER], rsx[PER], swl[PER];
  uint64_t rkw[HOLD_KEY ? 2 * W : 1][PER];
  typename std::conditional<F32, float, double>::type rvx[HOLD_KEY ? PER : 1],
      rvy[HOLD_KEY ? PER : 1];
  // one-word keys: the record loads are issued before the shared-memory
  // set-up, so that their latency overlaps it
  if constexpr (HOLD_KEY) {
#pragma unroll
    for (int k = 0; k < PER; k++) {
      const uint32_t i = tid + k * THREADS;
      rsx[k] = 0;
      if (i < n) {
        Key<W> m;
        if constexpr (DIRECT) {
          const TermPos q = term_pos(i);
          m = term_raw(q);  // (mixed below, when it has arrived)
          rsx[k] = q.group;
          const V v = term_val(q);
          rvx[k] = v.x;
          rvy[k] = v.y;
        } else {
          m = recs[b0 + i].k;
          const V v = recs[b0 + i].v;
          rvx[k] = v.x;
          rvy[k] = v.y;
          if (a.wide) rsx[k] = a.rsrc_wide[b0 + i];
        }
#pragma unroll
        for (int q = 0; q < 2 * W; q++) rkw[q][k] = m.w[q];
      }
    }
  }
  for (int i = tid; i < NDIGITS; i += THREADS) dh[i] = 0u;
  if (tid < MAX_GROUPS) {
    s_gk[tid] = a.gkind[tid];
    s_ak[tid] = a.alpha_kind[tid];
    s_al[tid] = a.alpha[tid];
  }
  const int G = 1 << a.g_log;
  if (!DIRECT && tid <= G && G > 1) sbb[tid] = a.bin_base[(j << a.g_log) + tid];
  if (tid == 0) {
    s_collide = 0;
    s_pk = 0u;
  }
  // the keep keys of this bucket: [s_kr[0], s_kr[1]) of the sorted keep set
  // (mostly none, and then no string looks its key up)
  if (!OUT && tid < 2 && a.n_keep) {
    const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
    const uint64_t first = ((uint64_t)a.pass_id << a.nbins_log) | ((uint64_t)j << a.g_log);
    const uint64_t bound = first + (tid ? (1ull << a.g_log) : 0ull);
    int lo = 0, hi = a.n_keep;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((F ? keep[mid].w[0] >> (64 - F) : 0ull) < bound) lo = mid + 1;
      else hi = mid;
    }
    s_kr[tid] = lo;
  }
  __syncthreads();

  // the record's order key: the bin bits that the source id displaced restored
  auto order_key = [&](uint32_t pos, const Key<W>& rk) -> Key<W> {
    int kb = 0;
    while (kb + 1 < G && sbb[kb + 1] <= pos) kb++;
    const uint64_t T = ((uint64_t)a.pass_id << a.nbins_log) | (uint64_t)((j << a.g_log) + kb);
    Key<W> m = rk;
    m.w[0] = (T << (64 - F)) | (rk.w[0] & (~0ull >> F));
    return m;
  };
  // sort word of record k: the 32 key bits after the digit, then the source id
  auto sort_word = [&](int k) -> uint64_t { return ((uint64_t)swl[k] << 32) | rsx[k]; };
#pragma unroll
  for (int k = 0; k < PER; k++) {
    const uint32_t i = tid + k * THREADS;
    dig[k] = 0;
    rnk[k] = 0;
    swl[k] = 0;
    if (!HOLD_KEY) rsx[k] = 0;
    if (i < n) {
      const uint32_t pos = b0 + i;
      Key<W> m;
      if constexpr (HOLD_KEY) {
#pragma unroll
        for (int q = 0; q < 2 * W; q++) m.w[q] = rkw[q][k];
        sv[i].x = rvx[k];
        sv[i].y = rvy[k];
        if constexpr (DIRECT) {
          rsx[k] = term_src(rsx[k], m);
          m = mix_key<W>(m);
#pragma unroll
          for (int q = 0; q < 2 * W; q++) rkw[q][k] = m.w[q];
        }
      } else if constexpr (DIRECT) {
        const TermPos q = term_pos(i);
        sv[i] = term_val(q);
        m = term_raw(q);
        rsx[k] = term_src(q.group, m);
        m = mix_key<W>(m);
      } else {
        m = recs[pos].k;
        if (a.wide) rsx[k] = a.rsrc_wide[pos];
      }
      if constexpr (!DIRECT) {
        // the source id from the key's top bits, then the order key
        const uint32_t small = (uint32_t)(m.w[0] >> (64 - F));
        if (!a.wide) rsx[k] = ((small >> ibits) << GROUP_SHIFT) | (small & ((1u << ibits) - 1u));
        m = order_key(pos, m);
        if constexpr (HOLD_KEY) {
#pragma unroll
          for (int q = 0; q < 2 * W; q++) rkw[q][k] = m.w[q];
        }
      }
      const uint64_t win = key_window<W>(m, a.digit_shift);
      dig[k] = (uint32_t)(win >> 32);
      swl[k] = (uint32_t)win;
      rnk[k] = atomicAdd(&dh[dig[k]], 1u);
    }
  }
  __syncthreads();
  // digit starts (exclusive scan of the digit counts)
  {
    uint32_t loc[DPT], s = 0;
#pragma unroll
    for (int q = 0; q < DPT; q++) {
      loc[q] = dh[tid * DPT + q];
      s += loc[q];
    }
    uint32_t tot;
    uint32_t pre = block_exclusive_scan(s, scan_tmp, &tot);
#pragma unroll
    for (int q = 0; q < DPT; q++) {
      dh[tid * DPT + q] = pre;
      pre += loc[q];
    }
  }
  __syncthreads();
  // sort words in digit-group order
#pragma unroll
  for (int k = 0; k < PER; k++) {
    const uint32_t i = tid + k * THREADS;
    if (i < n) swd[dh[dig[k]] + rnk[k]] = sort_word(k);
  }
  __syncthreads();
  // Final position of every record: its digit group's start plus the number of
  // group members with a smaller sort word (equal words: earlier entry first).
  uint32_t fpos[PER];
#pragma unroll
  for (int k = 0; k < PER; k++) {
    const uint32_t i = tid + k * THREADS;
    fpos[k] = 0;
    if (i < n) {
      const uint32_t s0 = dh[dig[k]];
      const uint32_t s1 = dig[k] + 1 < (uint32_t)NDIGITS ? dh[dig[k] + 1] : n;
      const uint32_t me = s0 + rnk[k];
      const uint64_t w = sort_word(k);
      uint32_t rank = 0;
      uint32_t p = s0;
      for (; p + 4 <= s1; p += 4) {
        const uint64_t w0 = swd[p], w1 = swd[p + 1], w2 = swd[p + 2], w3 = swd[p + 3];
        rank += ((w0 < w) | ((w0 == w) & (p < me))) ? 1u : 0u;
        rank += ((w1 < w) | ((w1 == w) & (p + 1 < me))) ? 1u : 0u;
        rank += ((w2 < w) | ((w2 == w) & (p + 2 < me))) ? 1u : 0u;
        rank += ((w3 < w) | ((w3 == w) & (p + 3 < me))) ? 1u : 0u;
      }
      for (; p < s1; p++) {
        const uint64_t w0 = swd[p];
        rank += ((w0 < w) | ((w0 == w) & (p < me))) ? 1u : 0u;
      }
      fpos[k] = s0 + rank;
    }
  }
  __syncthreads();
  // keys and SX words in sorted order; the digit counts become the
  // level-0 |c|^2 histogram (16-bit counters, two per word)
  if (!OUT && a.mode == M_PLAIN)
    for (int i = tid; i < NDIGITS; i += THREADS) h0[i] = 0u;
#pragma unroll
  for (int k = 0; k < PER; k++) {
    const uint32_t i = tid + k * THREADS;
    if (i < n) {
      if constexpr (HOLD_KEY) {
        Key<W> m;
#pragma unroll
        for (int q = 0; q < 2 * W; q++) m.w[q] = rkw[q][k];
        mk[fpos[k]] = m;
      } else if constexpr (DIRECT) {
        mk[fpos[k]] = mix_key<W>(term_raw(term_pos(i)));  // second read (cache)
      } else {
        const Rec<W, F32> r = recs[b0 + i];  // second read (cache)
        mk[fpos[k]] = order_key(b0 + i, r.k);
        sv[i] = r.v;
      }
      sx[fpos[k]] = (rsx[k] & ~SX_POS & ~(DIRECT ? 0u : SX_LONG)) | i;
    }
  }
  __syncthreads();

  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  const int kr0 = !OUT && a.n_keep ? s_kr[0] : 0, kr1 = !OUT && a.n_keep ? s_kr[1] : 0;
  // Fold the run [p, q) of equal keys: groups in ascending id, a SUM group
  // adds its contributions in ascending source index, then
  // acc = g0, acc = fl(acc + g1), ... after scaling each group by its alpha.
  auto val = [&](uint32_t r) -> V { return sv[sx[r] & SX_POS]; };
  auto fold = [&](uint32_t p, uint32_t q, double2& out) -> bool {
    if constexpr (DIRECT) {
      // every entry of the run is a group of its own
      double2 acc = make_double2(0.0, 0.0);
      for (uint32_t r = p; r < q; r++) {
        const uint32_t x = sx[r];
        const int g = (int)(x >> GROUP_SHIFT);
        const V v = sv[x & SX_POS];
        const double2 gv = apply_alpha(s_ak[g], s_al[g], make_double2((double)v.x, (double)v.y));
        acc = r == p ? gv : make_double2(acc.x + gv.x, acc.y + gv.y);
      }
      if (a.round32) acc = make_double2(round_to_f32(acc.x), round_to_f32(acc.y));
      out = acc;
      return !is_zero(acc);
    }
    if (a.single) {
      // one group: the sequential sum of the run, then the group's alpha
      const int g = (int)(sx[p] >> GROUP_SHIFT);
      const V v0 = val(p);
      double sr = (double)v0.x, si = (double)v0.y;
      uint32_t r = p + 1;
      for (; r + 4 <= q; r += 4) {
        const V v1 = val(r), v2 = val(r + 1), v3 = val(r + 2), v4 = val(r + 3);
        sr = sr + (double)v1.x;
        si = si + (double)v1.y;
        sr = sr + (double)v2.x;
        si = si + (double)v2.y;
        sr = sr + (double)v3.x;
        si = si + (double)v3.y;
        sr = sr + (double)v4.x;
        si = si + (double)v4.y;
      }
      for (; r < q; r++) {
        const V v1 = val(r);
        sr = sr + (double)v1.x;
        si = si + (double)v1.y;
      }
      double2 acc = apply_alpha(s_ak[g], s_al[g], make_double2(sr, si));
      if (a.round32) acc = make_double2(round_to_f32(acc.x), round_to_f32(acc.y));
      out = acc;
      return !is_zero(acc);
    }
    bool present = false;
    double2 acc = make_double2(0.0, 0.0);
    int cur = -1;
    double2 gs = make_double2(0.0, 0.0);
    float kr = 0.f, kcr = 0.f, ki = 0.f, kci = 0.f;  // Kahan state (FP32 records only)
    auto finish = [&]() {
      double2 gv = gs;
      if constexpr (F32) {
        if (s_gk[cur] == G_SUM_KAHAN32)
          gv = make_double2((double)kr - (double)kcr, (double)ki - (double)kci);
      }
      gv = apply_alpha(s_ak[cur], s_al[cur], gv);
      if (!present) acc = gv;
      else acc = make_double2(acc.x + gv.x, acc.y + gv.y);
      present = true;
    };
    constexpr int FU = 2;  // run entries loaded per step (LDS loads issued together)
    for (uint32_t r0 = p; r0 < q; r0 += FU) {
     uint32_t gx[FU];
     V vv[FU];
#pragma unroll
     for (int u = 0; u < FU; u++)
       if (r0 + u < q) {
         gx[u] = sx[r0 + u];
         vv[u] = sv[gx[u] & SX_POS];
       }
#pragma unroll
     for (int u = 0; u < FU; u++) {
      if (r0 + u >= q) break;
      const int g = (int)(gx[u] >> GROUP_SHIFT);
      const V v = vv[u];
      const bool kahan = F32 && s_gk[g] == G_SUM_KAHAN32;
      if (g != cur) {
        if (cur >= 0) finish();
        cur = g;
        if (kahan) {
          kr = 0.f; kcr = 0.f; ki = 0.f; kci = 0.f;
          kahan_add(kr, kcr, (float)v.x);
          kahan_add(ki, kci, (float)v.y);
        } else {
          gs = make_double2((double)v.x, (double)v.y);
        }
      } else {
        if (kahan) {
          kahan_add(kr, kcr, (float)v.x);
          kahan_add(ki, kci, (float)v.y);
        } else {
          gs = make_double2(gs.x + (double)v.x, gs.y + (double)v.y);
        }
      }
     }
    }
    if (cur >= 0) finish();
    if (a.round32) acc = make_double2(round_to_f32(acc.x), round_to_f32(acc.y));
    out = acc;
    return !is_zero(acc);
  };

  // Head bits of the sorted positions (a position starts a run of equal keys).
  Key<W>* uk = reinterpret_cast<Key<W>*>(a.uk) + ub;
  double2* uc = a.uc + ub;
  uint32_t kc = 0, nzu = 0;
  const uint32_t nround = (n + THREADS - 1) / THREADS;
  const uint32_t nwords = (n + 63) / 64;
  // the window (digit and sort bits) as masks of the first two key words:
  // two keys share it when their XOR has none of the masked bits
  constexpr int WB = DIGIT_BITS + 32;
  const int wsh = a.digit_shift;
  const uint64_t wm0 = wsh + WB <= 64 ? (((1ull << WB) - 1ull) << (64 - wsh - WB)) : (~0ull >> wsh);
  const uint64_t wm1 = wsh + WB <= 64 ? 0ull : ~(~0ull >> (wsh + WB - 64));
  for (uint32_t r = 0; r < nround; r++) {
    const uint32_t p = r * THREADS + tid;
    bool head = false;
    if (p < n) {
      head = p == 0;
      if (p > 0) {
        const Key<W> k0 = mk[p - 1], k1 = mk[p];
        head = !key_eq<W>(k0, k1);
        if (head && ((k0.w[0] ^ k1.w[0]) & wm0) == 0 && ((k0.w[1] ^ k1.w[1]) & wm1) == 0)
          s_collide = 1;
      }
    }
    const uint64_t m = __ballot(head);
    if ((tid & 63) == 0 && (p >> 6) < (uint32_t)NHW) hmask[p >> 6] = m;
  }
  __syncthreads();
  if (s_collide) {
    // rare: distinct keys with equal sort bits; rank again by full keys
    // (their source ids, from the records, in dh for the time being)
    for (uint32_t p = tid; p < n; p += THREADS) {
      const uint32_t i = sx[p] & SX_POS;
      uint32_t id = sx[p] & ~SX_POS;
      if constexpr (!DIRECT) {
        if (a.wide) {
          id = a.rsrc_wide[b0 + i];
        } else {
          const uint32_t small = (uint32_t)(recs[b0 + i].k.w[0] >> (64 - F));
          id = ((small >> ibits) << GROUP_SHIFT) | (small & ((1u << ibits) - 1u));
        }
      }
      dh[p] = id;
    }
    __syncthreads();
    merge_full_rank<W, THREADS, CAP>(mk, sx, dh, n, a.digit_shift);
    for (int i = tid; i < NDIGITS; i += THREADS) dh[i] = 0u;
    for (uint32_t r = 0; r < nround; r++) {
      const uint32_t p = r * THREADS + tid;
      const bool head = p < n && (p == 0 || !key_eq<W>(mk[p - 1], mk[p]));
      const uint64_t m = __ballot(head);
      if ((tid & 63) == 0 && (p >> 6) < (uint32_t)NHW) hmask[p >> 6] = m;
    }
    __syncthreads();
  }
  // Thread t owns the `per` consecutive sorted positions [per t, per t + per)
  // (per = ceil(n / threads) <= PER, so the work spreads over all waves): it
  // folds the runs that start there (a run may reach into the next threads'
  // positions), applies the filters (plain mode), and one block scan places
  // every survivor in sorted order.
  static_assert(PER * THREADS >= CAP, "every position has an owner");
  const uint32_t per = (n + THREADS - 1) / THREADS;
  double2 fv[PER];
  uint32_t smask = 0;
#pragma unroll
  for (int k = 0; k < PER; k++) {
    const uint32_t p = tid * per + k;
    fv[k] = make_double2(0.0, 0.0);
    if ((uint32_t)k < per && p < n && ((hmask[p >> 6] >> (p & 63)) & 1ull)) {
      // end of the run: the next head bit after p (or n)
      uint32_t q = n;
      const uint32_t w = p >> 6, bp = p & 63;
      const uint64_t rest = bp == 63 ? 0ull : (hmask[w] >> (bp + 1));
      if (rest) {
        q = p + 1 + (uint32_t)__builtin_ctzll(rest);
      } else {
        for (uint32_t ww = w + 1; ww < nwords; ww++)
          if (hmask[ww]) {
            q = ww * 64 + (uint32_t)__builtin_ctzll(hmask[ww]);
            break;
          }
      }
      if (q > n) q = n;
      double2 v;
      const bool too_long = DIRECT && (sx[p] & SX_LONG);
      if (!too_long && fold(p, q, v)) {
        nzu++;
        bool surv = true;
        if (a.mode != M_LANCZOS) {
          // the length cap was applied when the records were emitted
          if (a.use_eps && !(weight2(v) >= a.eps2)) surv = false;
          if (!OUT && surv) {
            const bool isk = kr1 > kr0 && keep_lookup<W>(keep + kr0, kr1 - kr0, mk[p]);
            if (isk) kc++;
            else {
              // 16-bit counters (a bucket holds < 2^16 records), two per word
              const uint32_t hb = (uint32_t)((uint64_t)__double_as_longlong(weight2(v)) >> SEL0_SHIFT);
              atomicAdd(&h0[hb >> 1], 1u << ((hb & 1u) << 4));
            }
          }
        }
        if (surv) {
          fv[k] = v;
          smask |= 1u << k;
        }
      }
    }
  }
  // block totals of the keep count and the nonzero count (both <= CAP: one
  // packed word), added per wave before the scan's barriers
  {
    uint32_t pk = (kc << 16) | nzu;
    for (int d = 32; d >= 1; d >>= 1) pk += __shfl_down(pk, d, 64);
    if ((tid & 63) == 0) atomicAdd(&s_pk, pk);
  }
  uint32_t tot_cnt;
  {
    uint32_t o = block_exclusive_scan((uint32_t)__popc(smask), scan_tmp, &tot_cnt);
    // OUT, FP64: the survivors' values and sorted positions go to LDS in output
    // order (sv and sx have been read), so that neighbouring threads write
    // neighbouring strings: 612 -> 579 us for 13 M strings (merged copies,
    // written as whole records, gain nothing by it)
    constexpr bool STAGE = OUT && !F32;
    if constexpr (OUT) {
      if (tid == 0) {
        if (a.use_eps && (s_pk & 0xFFFFu))
          atomicAdd(&a.ctl->u_unique, (unsigned long long)(s_pk & 0xFFFFu));
        __builtin_amdgcn_s_waitcnt(0);  // counted before the bucket is known to be
        if (j > 0) st_agent(&a.look[j], LB_SUM | (unsigned long long)tot_cnt);
      }
    }
    if constexpr (STAGE) {
#pragma unroll
      for (int k = 0; k < PER; k++)
        if ((smask >> k) & 1u) {
          sv[o].x = fv[k].x;
          sv[o].y = fv[k].y;
          sx[o] = tid * per + k;
          o++;
        }
    }
    auto each = [&](auto&& put) {
      if constexpr (STAGE) {
        __syncthreads();
        for (uint32_t r = tid; r < tot_cnt; r += THREADS)
          put(r, mk[sx[r]], make_double2((double)sv[r].x, (double)sv[r].y));
      } else {
#pragma unroll
        for (int k = 0; k < PER; k++)
          if ((smask >> k) & 1u) put(o++, mk[tid * per + k], fv[k]);
      }
    };
    if constexpr (OUT) {
      const unsigned long long row = finish(j, tot_cnt);
      if (row + tot_cnt > (unsigned long long)a.ocap) return;  // the host reports the size
      each([&](uint32_t q, const Key<W>& k, double2 v) {
        const size_t r = (size_t)row + q;
        const Key<W> raw = unmix_key<W>(k);
#pragma unroll
        for (int w = 0; w < W; w++) {
          a.ox[(size_t)w * a.ocap + r] = raw.w[w];
          a.oz[(size_t)w * a.ocap + r] = raw.w[W + w];
        }
        if (a.out_f32)
          reinterpret_cast<float2*>(a.oc)[r] = make_float2((float)v.x, (float)v.y);
        else
          reinterpret_cast<double2*>(a.oc)[r] = v;
      });
      return;
    }
    // U keeps order keys; raw strings are restored where needed
    each([&](uint32_t q, const Key<W>& k, double2 v) {
      uk[q] = k;
      uc[q] = v;
    });
  }
  // the scan's barriers have ordered every histogram and s_pk update
  const uint32_t tot_kc = s_pk >> 16, tot_nzu = s_pk & 0xFFFFu;
  if (a.mode == M_PLAIN) {
    // word i of the LDS histogram holds bins 2i (low half) and 2i + 1
    uint32_t* hrep = a.hist0 + (size_t)(j % HREP) * SEL0_BINS;
    for (int i = tid; i < NDIGITS; i += THREADS) {
      const uint32_t w = h0[i];
      if (w & 0xFFFFu) atomicAdd(&hrep[2 * i], w & 0xFFFFu);
      if (w >> 16) atomicAdd(&hrep[2 * i + 1], w >> 16);
    }
  }
  if (tid == 0) {
    a.b_ubase[gb] = (uint32_t)ub;
    a.b_slots[gb] = tot_cnt;
    a.b_surv[gb] = tot_cnt;
    a.b_keep[gb] = tot_kc;
    a.b_unique[gb] = tot_nzu;
  }
  };
  if constexpr (OUT) {
    static_assert(MODE != MERGE_LIST, "buckets are numbered as they are drawn");
    __shared__ uint32_t s_j;
    if (tid == 0)
      s_j = __hip_atomic_fetch_add(&a.ctl->ticket[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    bucket(s_j);
  } else if constexpr (MODE != MERGE_LIST) {
    bucket(blockIdx.x);
  } else {
    const uint32_t nd = *reinterpret_cast<volatile unsigned int*>(&a.ctl->ndefer);
    for (uint32_t it = blockIdx.x; it < nd; it += gridDim.x) {
      bucket(a.defer[it]);
      __syncthreads();  // the next bucket reuses the shared arrays
    }
  }
}

// Coefficient of the identity string (all mask words zero) of an operator
// with distinct strings: Tr(A)/2^N.  `res` (two doubles, pinned) starts at
// zero; at most one thread writes it.
template <int W>
__global__ __launch_bounds__(256) void k_trace(const uint64_t* x, const uint64_t* z, int64_t cap,
                                               int64_t n, const void* coef, int f32, double* res) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    uint64_t s = 0;
#pragma unroll
    for (int w = 0; w < W; w++) s |= x[(size_t)w * cap + i] | z[(size_t)w * cap + i];
    if (s == 0) {
      const double2 v = f32 ? make_double2((double)reinterpret_cast<const float2*>(coef)[i].x,
                                           (double)reinterpret_cast<const float2*>(coef)[i].y)
                            : reinterpret_cast<const double2*>(coef)[i];
      res[0] = v.x;
      res[1] = v.y;
    }
  }
}

// The buckets first, first + step, ... of one wave, with the next one's start
// and length loaded while the current one is worked on.
struct WaveBuckets {
  const uint32_t *start, *len;
  uint32_t b, step, nbk, ub, ns;
  DEV WaveBuckets(const uint32_t* s, const uint32_t* l, uint32_t first, uint32_t st, uint32_t n)
      : start(s), len(l), b(first), step(st), nbk(n), ub(0), ns(0) {
    if (b < nbk) load();
  }
  DEV void load() {
    ub = start[b];
    ns = len[b];
  }
  DEV bool next(uint32_t& cb, uint32_t& cu, uint32_t& cn) {
    if (b >= nbk) return false;
    cb = b;
    cu = ub;
    cn = ns;
    b += step;
    if (b < nbk) load();
    return true;
  }
};

// Lanczos: sum |c|^2 of the merged, untruncated O'_n in double-double, in a
// fixed order: one wave per bucket, block partials (at most NORM_BLOCKS), and
// the last block adds them into ctl->norm_hi, norm_lo.  TS: each merged string
// weighted by its stabilizer count (the norm of sum_k T_k(A) over N).
constexpr int NORM_BLOCKS = 1024;
DEV dd dd_block_sum(dd s, double* rh, double* rl) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int d = 32; d >= 1; d >>= 1) {
    dd o;
    o.hi = __shfl_down(s.hi, d, 64);
    o.lo = __shfl_down(s.lo, d, 64);
    if (lane < d) s = dd_add(s, o);
  }
  if (lane == 0) {
    rh[wv] = s.hi;
    rl[wv] = s.lo;
  }
  __syncthreads();
  dd t = {rh[0], rl[0]};
  for (int w = 1; w < 4; w++) t = dd_add(t, dd{rh[w], rl[w]});
  return t;
}
template <int W, bool TS>
__global__ __launch_bounds__(256) void k_norm(const uint32_t* b_ubase, const uint32_t* b_slots,
                                              const void* uk_, const double2* uc, int N, TsTop top,
                                              uint32_t nbk, double2* part, Ctl* ctl) {
  __shared__ double rh[4], rl[4];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const Key<W>* uk = reinterpret_cast<const Key<W>*>(uk_);
  dd s = dd_zero();
  WaveBuckets wb(b_ubase, b_slots, blockIdx.x * 4 + wv, gridDim.x * 4, nbk);
  for (uint32_t b, ub, ns; wb.next(b, ub, ns);) {
    for (uint32_t i0 = lane; i0 < ns; i0 += 256) {
      double w2[4];
#pragma unroll
      for (int q = 0; q < 4; q++) w2[q] = i0 + 64 * q < ns ? weight2(uc[ub + i0 + 64 * q]) : 0.0;
#pragma unroll
      for (int q = 0; q < 4; q++) {
        int st = 1;
        if constexpr (TS) {
          if (i0 + 64 * q < ns) {
            const Key<W> raw = unmix_key<W>(uk[ub + i0 + 64 * q]);
            st = ts_stabilizers<W>(raw.w, raw.w + W, N, top);
          }
        }
        for (int r = 0; r < st; r++) s = dd_add(s, w2[q]);
      }
    }
  }
  const dd t = dd_block_sum(s, rh, rl);
  if (tid == 0) st_agent(&part[blockIdx.x], make_double2(t.hi, t.lo));
  if (!last_block(&ctl->ticket[1])) return;
  dd u = dd_zero();
  for (uint32_t i = tid; i < gridDim.x; i += 256) u = dd_add(u, dd{part[i].x, part[i].y});
  __syncthreads();  // rh, rl are reused
  const dd v = dd_block_sum(u, rh, rl);
  if (tid == 0) {
    ctl->norm_hi = v.hi;
    ctl->norm_lo = v.lo;
  }
}

// Lanczos: divide the merged O'_n by b_n (IEEE division), then apply the
// plain-mode filters on the FP64 quotient (FP32 outputs are rounded when
// written); dropped strings become exact zeros in place.
struct ScaleArgs {
  const uint32_t* b_ubase;
  const uint32_t* b_slots;
  uint32_t* b_surv;
  uint32_t* b_keep;
  uint32_t nbk;
  void* uk;
  double2* uc;
  const double* norm2;  // ||O'_n||^2, written by the norm reduction
  double floor_b;       // b_n at or below this is a breakdown: nothing survives
  int round32;
  int max_len;
  int use_eps;
  double eps2;
  const void* keep_mk;
  int n_keep;
  uint32_t* hist0;
  Ctl* ctl;
};

// One wave per bucket, SCALE_BLOCKS blocks at most, so that the 4096-bin
// histogram in LDS is cleared and added to memory once per block and not once
// per bucket: over 131072 buckets of 560 two-word strings 1.06 -> 0.50 ms (4.7
// TB/s of values read and written).
constexpr int SCALE_BLOCKS = 1024;
template <int W>
__global__ __launch_bounds__(512) void k_scale_filter(ScaleArgs a) {
  __shared__ uint32_t h0[SEL0_BINS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < SEL0_BINS; i += 512) h0[i] = 0u;
  __syncthreads();
  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  // b_n = sqrt(||O'_n||^2), correctly rounded as on the host, which reads the
  // same norm with the output size and reports the breakdown
  const double bn = sqrt(*a.norm2);
  const bool brk = !(bn > a.floor_b);
  WaveBuckets wb(a.b_ubase, a.b_slots, blockIdx.x * 8 + wv, gridDim.x * 8, a.nbk);
  for (uint32_t b, ub, ns; wb.next(b, ub, ns);) {
    const Key<W>* uk = reinterpret_cast<const Key<W>*>(a.uk) + ub;
    double2* uc = a.uc + ub;
    uint32_t surv = 0, kc = 0;
    for (uint32_t i0 = lane; i0 < ns; i0 += 256) {
      double2 vv[4];
#pragma unroll
      for (int q = 0; q < 4; q++)
        if (i0 + 64 * q < ns) vv[q] = uc[i0 + 64 * q];
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const uint32_t i = i0 + 64 * q;
        if (i >= ns) break;
        double2 v = make_double2(vv[q].x / bn, vv[q].y / bn);
        // FP32 storage: a string whose stored value would be an exact zero is
        // dropped; every other decision (cutoff, top-M) is taken on the FP64
        // quotient, which the output write rounds to FP32
        bool ok = !brk && (a.round32 ? !is_zero(make_double2(round_to_f32(v.x), round_to_f32(v.y)))
                                     : !is_zero(v));
        if (ok && a.max_len > 0 && key_length<W>(unmix_key<W>(uk[i])) > a.max_len) ok = false;
        if (ok && a.use_eps && !(weight2(v) >= a.eps2)) ok = false;
        if (ok) {
          surv++;
          bool isk = a.n_keep ? keep_lookup<W>(keep, a.n_keep, uk[i]) : false;
          if (isk) kc++;
          else atomicAdd(&h0[(uint32_t)((uint64_t)__double_as_longlong(weight2(v)) >> SEL0_SHIFT)], 1u);
        } else {
          v = make_double2(0.0, 0.0);
        }
        uc[i] = v;
      }
    }
    for (int d = 32; d >= 1; d >>= 1) {
      surv += __shfl_down(surv, d, 64);
      kc += __shfl_down(kc, d, 64);
    }
    if (lane == 0) {
      a.b_surv[b] = surv;
      a.b_keep[b] = kc;
    }
  }
  __syncthreads();
  uint32_t* hrep = a.hist0 + (size_t)(blockIdx.x % HREP) * SEL0_BINS;
  for (int i = tid; i < SEL0_BINS; i += 512)
    if (h0[i]) atomicAdd(&hrep[i], h0[i]);
}

// ---------------------------------------------------------------------------
// Top-M selection: exact radix select over the composite ordering key
// (|c|^2 bits, then the complemented key words x[W-1]..x[0], z[W-1]..z[0]):
// larger composite = kept first.  Digit 0 = the top 13 bits of |c|^2 (sign,
// always 0, the 11 exponent bits and the first mantissa bit: 4096 bins),
// digit L >= 1 = the 12 bits at position 12L + 1 of the composite bit string.
// ---------------------------------------------------------------------------
template <int W>
DEV void composite(double2 v, const Key<W>& raw, uint64_t* c) {
  c[0] = (uint64_t)__double_as_longlong(weight2(v));
#pragma unroll
  for (int i = 0; i < W; i++) {
    c[1 + i] = ~raw.w[W - 1 - i];
    c[1 + W + i] = ~raw.w[2 * W - 1 - i];
  }
}

template <int W>
DEV uint32_t comp_digit(const uint64_t* c, int level) {
  if (level == 0) return (uint32_t)(c[0] >> SEL0_SHIFT);
  const int p = 12 * level + (64 - SEL0_SHIFT - 12);  // 12-bit digits after the level-0 bits
  const int wi = p >> 6, off = p & 63;
  constexpr int NW = 1 + 2 * W;
  const uint64_t hi = wi < NW ? c[wi] : 0ull;
  const uint64_t lo = wi + 1 < NW ? c[wi + 1] : 0ull;
  const uint64_t v = off ? ((hi << off) | (lo >> (64 - off))) : hi;
  return (uint32_t)(v >> 52);
}

template <int W>
DEV int comp_cmp(const uint64_t* a, const uint64_t* b) {
#pragma unroll
  for (int i = 0; i < 1 + 2 * W; i++)
    if (a[i] != b[i]) return a[i] < b[i] ? -1 : 1;
  return 0;
}

// Sum of the HREP replicas of a select histogram.
__global__ void k_hist_reduce(const uint32_t* rep, int nbins, uint32_t* sum) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbins) return;
  uint32_t s = 0;
#pragma unroll 8
  for (int r = 0; r < HREP; r++) s += rep[(size_t)r * nbins + b];
  sum[b] = s;
}

// Pick the bin holding the K-th largest: K from ctl->sel_K (1-based).
__global__ __launch_bounds__(1024) void k_select(const uint32_t* hist, int nbins, Ctl* ctl) {
  __shared__ unsigned long long tmp[17];
  __shared__ unsigned long long Ks;
  const int t = threadIdx.x;
  if (t == 0) Ks = ctl->sel_K;
  const int per = nbins / 1024;  // nbins is 2048 or 4096
  // thread t owns bins [nbins - (t+1)*per, nbins - t*per), scanned high to low
  const int hiB = nbins - t * per;
  unsigned int hv[4] = {0u, 0u, 0u, 0u};
  for (int q = 1; q <= per; q++) hv[q - 1] = hist[hiB - q];
  unsigned long long s = 0;
  for (int q = 1; q <= per; q++) s += hv[q - 1];
  const int lane = t & 63, wv = t >> 6;
  unsigned long long x = s;
  for (int d = 1; d < 64; d <<= 1) {
    unsigned long long y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) tmp[wv] = x;
  __syncthreads();
  if (t == 0) {
    unsigned long long run = 0;
    for (int i = 0; i < 16; i++) {
      unsigned long long q = tmp[i];
      tmp[i] = run;
      run += q;
    }
  }
  __syncthreads();
  const unsigned long long K = Ks;
  unsigned long long cum = tmp[wv] + x - s;  // records in bins above this thread's
  for (int q = 1; q <= per; q++) {
    const int b = hiB - q;
    const unsigned long long h = hv[q - 1];
    if (cum < K && K <= cum + h) {
      ctl->sel_digit = (unsigned int)b;
      ctl->sel_K = K - cum;
      ctl->sel_count = h;
    }
    cum += h;
  }
}

struct SelArgs {
  const uint32_t* b_ubase;
  const uint32_t* b_slots;
  uint32_t* b_abv;
  uint32_t* b_bcnt;
  const void* uk;
  const double2* uc;
  const void* keep_mk;
  int n_keep;
  uint32_t nbk;
  // candidate lists: the entries of bucket b sit at [b_ubase[b], b_ubase[b] + cc[b])
  const uint32_t* list_in;
  const uint32_t* cc_in;
  uint32_t* list_out;
  uint32_t* cc_out;
  int level;
  uint32_t* hist;  // histogram of the next digit (nullable)
  Ctl* ctl;
};

// Level 1: one block per bucket, full pass over its U slots.  Counts the
// non-keep survivors whose digit 0 is above the chosen bin, collects the
// chosen bin's records (in bucket order) and histograms their digit 1.
template <int W>
__global__ __launch_bounds__(256) void k_level1(SelArgs a) {
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t ra[4];
  __shared__ uint32_t scan_tmp[256 / 64 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint32_t b = blockIdx.x;
  for (int i = tid; i < SEL_BINS; i += 256) h[i] = 0u;
  __syncthreads();
  const uint32_t D = a.ctl->sel_digit;
  const uint32_t ub = a.b_ubase[b], ns = a.b_slots[b];
  const Key<W>* uk = reinterpret_cast<const Key<W>*>(a.uk) + ub;
  const double2* uc = a.uc + ub;
  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  uint32_t abv = 0, nout = 0;
  const uint32_t nround = (ns + 255) / 256;
  for (uint32_t r = 0; r < nround; r++) {
    const uint32_t i = r * 256 + tid;
    bool cand = false;
    uint64_t c[1 + 2 * W];
    if (i < ns) {
      const double2 v = uc[i];
      if (!is_zero(v)) {
        const Key<W> mk = uk[i];
        const bool isk = a.n_keep ? keep_lookup<W>(keep, a.n_keep, mk) : false;
        if (!isk) {
          composite<W>(v, unmix_key<W>(mk), c);
          const uint32_t d0 = comp_digit<W>(c, 0);
          if (d0 > D) abv++;
          else if (d0 == D) cand = true;
        }
      }
    }
    uint32_t tot;
    const uint32_t pos = block_exclusive_scan(cand ? 1u : 0u, scan_tmp, &tot);
    if (cand) {
      a.list_out[ub + nout + pos] = ub + i;
      atomicAdd(&h[comp_digit<W>(c, 1)], 1u);
    }
    nout += tot;
  }
  for (int d = 32; d >= 1; d >>= 1) abv += __shfl_down(abv, d, 64);
  if (lane == 0) ra[wv] = abv;
  __syncthreads();
  uint32_t* hrep = a.hist + (size_t)(b % HREP) * SEL_BINS;
  for (int i = tid; i < SEL_BINS; i += 256)
    if (h[i]) atomicAdd(&hrep[i], h[i]);
  if (tid == 0) {
    a.b_abv[b] = ra[0] + ra[1] + ra[2] + ra[3];
    a.cc_out[b] = nout;
  }
}

// Level L >= 1, one block per bucket over its candidates: keep those whose
// digit L equals the chosen bin, histogram their digit L+1 (if hist given).
template <int W>
__global__ __launch_bounds__(256) void k_cand_level(SelArgs a) {
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t scan_tmp[256 / 64 + 1];
  const int tid = threadIdx.x;
  const uint32_t b = blockIdx.x;
  const uint32_t n = a.cc_in[b];
  if (n == 0) {
    if (tid == 0) a.cc_out[b] = 0;
    return;
  }
  const bool with_hist = a.hist != nullptr;
  if (with_hist)
    for (int i = tid; i < SEL_BINS; i += 256) h[i] = 0u;
  __syncthreads();
  const uint32_t D = a.ctl->sel_digit;
  const uint32_t ub = a.b_ubase[b];
  const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
  uint32_t nout = 0;
  const uint32_t nround = (n + 255) / 256;
  for (uint32_t r = 0; r < nround; r++) {
    const uint32_t i = r * 256 + tid;
    bool keepit = false;
    uint64_t c[1 + 2 * W];
    uint32_t ui = 0;
    if (i < n) {
      ui = a.list_in[ub + i];
      composite<W>(a.uc[ui], unmix_key<W>(ukb[ui]), c);
      keepit = comp_digit<W>(c, a.level) == D;
    }
    uint32_t tot;
    const uint32_t pos = block_exclusive_scan(keepit ? 1u : 0u, scan_tmp, &tot);
    if (keepit) {
      a.list_out[ub + nout + pos] = ui;
      if (with_hist) atomicAdd(&h[comp_digit<W>(c, a.level + 1)], 1u);
    }
    nout += tot;
  }
  __syncthreads();
  if (with_hist) {
    uint32_t* hrep = a.hist + (size_t)(b % HREP) * SEL_BINS;
    for (int i = tid; i < SEL_BINS; i += 256)
      if (h[i]) atomicAdd(&hrep[i], h[i]);
  }
  if (tid == 0) a.cc_out[b] = nout;
}

// Final level (one block): every entry of list_in belongs to the chosen bin
// and there are at most FINISH_CAP of them; the entry of rank K-1
// (descending composite) is the threshold T.
template <int W>
__global__ __launch_bounds__(1024) void k_finish(SelArgs a) {
  constexpr int NW = 1 + 2 * W;
  __shared__ uint64_t cs[FINISH_CAP][NW];
  __shared__ unsigned int m;
  const int tid = threadIdx.x;
  if (tid == 0) m = 0;
  __syncthreads();
  const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
  for (uint32_t b = tid; b < a.nbk; b += 1024) {
    const uint32_t n = a.cc_in[b];
    if (!n) continue;
    const uint32_t ub = a.b_ubase[b];
    for (uint32_t k = 0; k < n; k++) {
      const uint32_t ui = a.list_in[ub + k];
      uint64_t c[NW];
      composite<W>(a.uc[ui], unmix_key<W>(ukb[ui]), c);
      const unsigned int p = atomicAdd(&m, 1u);
      if (p < FINISH_CAP)
        for (int q = 0; q < NW; q++) cs[p][q] = c[q];
    }
  }
  __syncthreads();
  const unsigned int mm = m < FINISH_CAP ? m : FINISH_CAP;
  const unsigned long long K = a.ctl->sel_K;
  for (unsigned int i = tid; i < mm; i += 1024) {
    unsigned int rank = 0;
    for (unsigned int k = 0; k < mm; k++) rank += comp_cmp<W>(cs[k], cs[i]) > 0 ? 1u : 0u;
    if ((unsigned long long)rank + 1 == K) {
      for (int q = 0; q < NW; q++) a.ctl->T[q] = cs[i][q];
      a.ctl->t_found = 1;
    }
  }
}

// Per bucket (one wave): level-1 candidates at or above the threshold.
template <int W>
__global__ __launch_bounds__(64) void k_count_boundary(SelArgs a) {
  constexpr int NW = 1 + 2 * W;
  const uint32_t b = blockIdx.x;
  const uint32_t n = a.cc_in[b];
  uint32_t cnt = 0;
  if (n) {
    uint64_t T[NW];
    for (int q = 0; q < NW; q++) T[q] = a.ctl->T[q];
    const uint32_t ub = a.b_ubase[b];
    const Key<W>* ukb = reinterpret_cast<const Key<W>*>(a.uk);
    for (uint32_t i = threadIdx.x; i < n; i += 64) {
      const uint32_t ui = a.list_in[ub + i];
      uint64_t c[NW];
      composite<W>(a.uc[ui], unmix_key<W>(ukb[ui]), c);
      if (comp_cmp<W>(c, T) >= 0) cnt++;
    }
    for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_down(cnt, d, 64);
  }
  if (threadIdx.x == 0) a.b_bcnt[b] = cnt;
}

// Output bases: survivors per bucket are counted according to the select
// mode; exclusive scan over the buckets (one block).
enum SelMode : int { S_ALL = 0, S_KEEP_ONLY = 1, S_THRESHOLD = 2 };

__global__ __launch_bounds__(1024) void k_scan_buckets(const uint32_t* b_surv,
                                                       const uint32_t* b_keep,
                                                       const uint32_t* b_abv,
                                                       const uint32_t* b_bcnt, uint32_t nb,
                                                       int sel_mode, uint32_t* b_obase, Ctl* ctl) {
  __shared__ unsigned long long tmp[17];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t per = (nb + 1023) / 1024;
  const uint32_t lo = t * per;
  unsigned long long s = 0;
  for (uint32_t k = 0; k < per; k++) {
    const uint32_t b = lo + k;
    if (b < nb) {
      uint32_t c = sel_mode == S_ALL ? b_surv[b]
                   : sel_mode == S_KEEP_ONLY ? b_keep[b]
                                             : b_keep[b] + b_abv[b] + b_bcnt[b];
      s += c;
    }
  }
  unsigned long long x = s;
  for (int d = 1; d < 64; d <<= 1) {
    unsigned long long y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) tmp[wv] = x;
  __syncthreads();
  if (t == 0) {
    unsigned long long run = 0;
    for (int i = 0; i < 16; i++) {
      unsigned long long q = tmp[i];
      tmp[i] = run;
      run += q;
    }
    tmp[16] = run;
  }
  __syncthreads();
  unsigned long long pre = tmp[wv] + x - s;
  for (uint32_t k = 0; k < per; k++) {
    const uint32_t b = lo + k;
    if (b < nb) {
      b_obase[b] = (uint32_t)pre;
      uint32_t c = sel_mode == S_ALL ? b_surv[b]
                   : sel_mode == S_KEEP_ONLY ? b_keep[b]
                                             : b_keep[b] + b_abv[b] + b_bcnt[b];
      pre += c;
    }
  }
  if (t == 0) ctl->out_total = tmp[16];
}

struct WriteArgs {
  const uint32_t* b_keep;
  const uint32_t* b_ubase;
  const uint32_t* b_slots;
  const uint32_t* b_obase;
  const void* uk;
  const double2* uc;
  const void* keep_mk;
  int n_keep;
  int sel_mode;
  const Ctl* ctl;
  uint64_t* ox;
  uint64_t* oz;
  void* oc;
  int64_t ocap;
  int out_f32;
};

template <int W>
__global__ __launch_bounds__(256) void k_write(WriteArgs a) {
  constexpr int NW = 1 + 2 * W;
  __shared__ uint32_t scan_tmp[256 / 64 + 1];
  const int tid = threadIdx.x;
  const uint32_t b = blockIdx.x;
  const uint32_t ub = a.b_ubase[b], ns = a.b_slots[b];
  uint32_t obase = a.b_obase[b];
  const Key<W>* uk = reinterpret_cast<const Key<W>*>(a.uk) + ub;
  const double2* uc = a.uc + ub;
  const Key<W>* keep = reinterpret_cast<const Key<W>*>(a.keep_mk);
  uint64_t T[NW];
  if (a.sel_mode == S_THRESHOLD)
    for (int q = 0; q < NW; q++) T[q] = a.ctl->T[q];
  const uint32_t nround = (ns + 255) / 256;
  for (uint32_t r = 0; r < nround; r++) {
    const uint32_t i = r * 256 + tid;
    bool s = false;
    Key<W> raw;
    double2 v = make_double2(0.0, 0.0);
    if (i < ns) {
      v = uc[i];
      if (!is_zero(v)) {
        raw = unmix_key<W>(uk[i]);
        if (a.sel_mode == S_ALL) {
          s = true;
        } else {
          const bool isk = a.n_keep ? keep_lookup<W>(keep, a.n_keep, uk[i]) : false;
          if (isk) s = true;
          else if (a.sel_mode == S_THRESHOLD) {
            uint64_t c[NW];
            composite<W>(v, raw, c);
            s = comp_cmp<W>(c, T) >= 0;
          }
        }
      }
    }
    uint32_t tot;
    const uint32_t pos = block_exclusive_scan(s ? 1u : 0u, scan_tmp, &tot);
    if (s) {
      const size_t o = (size_t)obase + pos;
#pragma unroll
      for (int w = 0; w < W; w++) {
        a.ox[(size_t)w * a.ocap + o] = raw.w[w];
        a.oz[(size_t)w * a.ocap + o] = raw.w[W + w];
      }
      if (a.out_f32) reinterpret_cast<float2*>(a.oc)[o] = make_float2((float)v.x, (float)v.y);
      else reinterpret_cast<double2*>(a.oc)[o] = v;
    }
    obase += tot;
  }
}

// ---------------------------------------------------------------------------
// Small helpers
// ---------------------------------------------------------------------------
// First kernel of an engine call, PREP_BLOCKS blocks of 1024 threads.  The
// blocks after the first clear the level-0 |c|^2 histogram `hist0`; the first
// clears the control block, takes the order keys of the keep set (n_keep <=
// KEEP_PREP; a larger one is left to k_mix_keys) and, for a commutator (n > 0,
// n <= 2047), lays out H: packed raw words [n][2W] in ascending order of lowest
// site, the index of each entry in the caller's H, hstart[s] = first entry with
// lowest site >= s (s = 0 .. 64W + 1; the empty string sorts as site 64W) and
// the largest highest-minus-lowest site.  The order among entries of one lowest
// site is not fixed: every entry carries its own index.
constexpr int PREP_BLOCKS = 1 + HREP, KEEP_PREP = 1024;
struct PrepArgs {
  const uint64_t* x;
  const uint64_t* z;
  int64_t cap;
  int n;
  uint64_t* packed;
  uint32_t* hidx;
  uint32_t* hstart;
  int* hspan;
  const uint64_t* kx;
  const uint64_t* kz;
  int64_t kcap;
  int n_keep;
  void* keep_mk;
  uint32_t* hist0;
  uint32_t* cursor;  // append mode: n_cursor <= 1024 bucket cursors to clear
  int n_cursor;
  unsigned long long* look;  // n_look <= 1024 look-back states to clear
  int n_look;
  Ctl* ctl;
};
template <int W>
__global__ __launch_bounds__(1024) void k_prep(PrepArgs a) {
  constexpr int SITES = 64 * W;
  static_assert(SEL0_BINS == 4 * 1024, "one replica per block, 16 bytes per thread");
  if (blockIdx.x > 0) {
    uint4* z = reinterpret_cast<uint4*>(a.hist0 + (size_t)(blockIdx.x - 1) * SEL0_BINS);
    z[threadIdx.x] = make_uint4(0u, 0u, 0u, 0u);
    return;
  }
  const uint64_t* x = a.x;
  const uint64_t* z = a.z;
  const int64_t cap = a.cap;
  const int n = a.n;
  __shared__ uint32_t cnt[SITES + 2];
  __shared__ int span;
  const int t = threadIdx.x;
  __shared__ int bad;
  for (uint32_t q = t; q < sizeof(Ctl) / 4; q += 1024) reinterpret_cast<uint32_t*>(a.ctl)[q] = 0u;
  for (int q = t; q < SITES + 2; q += 1024) cnt[q] = 0u;
  if (t < a.n_cursor) a.cursor[t * CURSOR_STRIDE] = 0u;
  if (t < a.n_look) a.look[t] = 0ull;
  if (t == 0) {
    span = 0;
    bad = 0;
  }
  __syncthreads();
  if (a.n_keep > 0) {
    Key<W>* mk = reinterpret_cast<Key<W>*>(a.keep_mk);
    if (t < a.n_keep) {
      const Key<W> m = mix_key<W>(load_raw<W>(a.kx, a.kz, a.kcap, t));
      mk[t] = m;
      if (t > 0 && key_cmp<W>(mix_key<W>(load_raw<W>(a.kx, a.kz, a.kcap, t - 1)), m) >= 0) bad = 1;
    }
    __syncthreads();
    if (t == 0 && bad) a.ctl->bad_keep = 1u;
  }
  if (n == 0) return;
  int lo[2], rk[2];
  for (int k = 0; k < 2; k++) {
    const int i = t + k * 1024;
    lo[k] = SITES;
    rk[k] = 0;
    if (i < n) {
      int hi = -1;
#pragma unroll
      for (int w = W - 1; w >= 0; w--) {
        const uint64_t s = x[(size_t)w * cap + i] | z[(size_t)w * cap + i];
        if (s) {
          lo[k] = 64 * w + __builtin_ctzll(s);
          if (hi < 0) hi = 64 * w + 63 - __builtin_clzll(s);
        }
      }
      if (hi >= 0) atomicMax(&span, hi - lo[k]);
      rk[k] = (int)atomicAdd(&cnt[lo[k]], 1u);
    }
  }
  __syncthreads();
  if (t == 0) {
    uint32_t run = 0;
    for (int q = 0; q <= SITES; q++) {
      const uint32_t c = cnt[q];
      cnt[q] = run;
      run += c;
    }
    cnt[SITES + 1] = run;
  }
  __syncthreads();
  for (int k = 0; k < 2; k++) {
    const int i = t + k * 1024;
    if (i < n) {
      const int p = (int)cnt[lo[k]] + rk[k];
#pragma unroll
      for (int w = 0; w < W; w++) {
        a.packed[(size_t)p * 2 * W + w] = x[(size_t)w * cap + i];
        a.packed[(size_t)p * 2 * W + W + w] = z[(size_t)w * cap + i];
      }
      a.hidx[p] = (uint32_t)i;
    }
  }
  for (int q = t; q < SITES + 2; q += 1024) a.hstart[q] = cnt[q];
  if (t == 0) *a.hspan = span;
}

// Mixed keys of a canonical operator; flags a violation of ascending order.
template <int W>
__global__ void k_mix_keys(const uint64_t* x, const uint64_t* z, int64_t cap, int64_t n,
                           Key<W>* out, unsigned int* bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Key<W> raw;
#pragma unroll
  for (int w = 0; w < W; w++) {
    raw.w[w] = x[(size_t)w * cap + i];
    raw.w[W + w] = z[(size_t)w * cap + i];
  }
  const Key<W> m = mix_key<W>(raw);
  out[i] = m;
  if (i > 0) {
    Key<W> rp;
#pragma unroll
    for (int w = 0; w < W; w++) {
      rp.w[w] = x[(size_t)w * cap + i - 1];
      rp.w[W + w] = z[(size_t)w * cap + i - 1];
    }
    if (key_cmp<W>(mix_key<W>(rp), m) >= 0) *bad = 1u;  // (may lie in host memory)
  }
}

// Depolarizing noise in place: c_k *= f[len_k], f[w] = exp(-lambda w)
// computed on the host (len = sites with x or z set).  FP32 coefficients are
// scaled in double and rounded once.
constexpr int NOISE_TABLE = 129;  // lengths 0..128
struct NoiseTable {
  double f[NOISE_TABLE];
};
template <int W>
__global__ __launch_bounds__(256) void k_add_noise(const uint64_t* x, const uint64_t* z,
                                                   int64_t cap, int64_t n, void* coef, int f32,
                                                   NoiseTable t) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    int len = 0;
#pragma unroll
    for (int w = 0; w < W; w++) len += __popcll(x[(size_t)w * cap + i] | z[(size_t)w * cap + i]);
    const double f = t.f[len];
    if (f32) {
      float2* c = reinterpret_cast<float2*>(coef) + i;
      const float2 v = *c;
      *c = make_float2((float)((double)v.x * f), (float)((double)v.y * f));
    } else {
      double2* c = reinterpret_cast<double2*>(coef) + i;
      const double2 v = *c;
      *c = make_double2(v.x * f, v.y * f);
    }
  }
}

// Adjoint in place: the imaginary part of every coefficient changes sign.
__global__ __launch_bounds__(256) void k_conj(void* coef, int64_t n, int f32) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    if (f32) {
      float2* c = reinterpret_cast<float2*>(coef) + i;
      c->y = -c->y;
    } else {
      double2* c = reinterpret_cast<double2*>(coef) + i;
      c->y = -c->y;
    }
  }
}

// Position of the order key m among n strings in canonical order (key(i): the
// order key of string i), or -1.  Order keys are spread evenly, so the
// position is interpolated between the keys seen so far: about four dependent
// reads where bisection takes log2(n); after eight, whatever the keys are,
// bisection finishes.
template <int W, typename F>
DEV int64_t find_key(const Key<W>& m, int64_t n, F key) {
  int64_t lo = 0, hi = n;
  uint64_t klo = 0ull, khi = ~0ull;  // leading words below lo and from hi on
  for (int step = 0; lo < hi; step++) {
    int64_t mid = (lo + hi) >> 1;
    if (step < 8 && khi > klo) {
      const double f = fmin((double)(m.w[0] - klo) / (double)(khi - klo), 1.0);
      mid = min(max(lo + (int64_t)(f * (double)(hi - lo)), lo), hi - 1);
    }
    const Key<W> k = key(mid);
    const int c = key_cmp<W>(k, m);
    if (c == 0) return mid;
    if (c < 0) {
      lo = mid + 1;
      klo = k.w[0];
    } else {
      hi = mid;
      khi = k.w[0];
    }
  }
  return -1;
}

DEV double2 load_coef(const void* c, int f32, int64_t i) {
  if (f32) {
    const float2 f = reinterpret_cast<const float2*>(c)[i];
    return make_double2((double)f.x, (double)f.y);
  }
  return reinterpret_cast<const double2*>(c)[i];
}

// Coefficients in A (canonical) of the strings of Q: out[q] = A's coefficient
// of Q's string q, or 0 when A lacks it.  A's keys are mixed where the search
// reads them: mixing all of A first took 3 of 10 us at 2^18 strings.
template <int W>
__global__ __launch_bounds__(64) void k_lookup(const uint64_t* ax, const uint64_t* az,
                                               int64_t acap, const void* acoef, int af32,
                                               int64_t na, const uint64_t* qx, const uint64_t* qz,
                                               int64_t qcap, int64_t nq, double2* out) {
  const int64_t q = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (q >= nq) return;
  const Key<W> mk = mix_key<W>(load_raw<W>(qx, qz, qcap, q));
  const int64_t i = find_key<W>(
      mk, na, [&](int64_t k) { return mix_key<W>(load_raw<W>(ax, az, acap, k)); });
  out[q] = i >= 0 ? load_coef(acoef, af32, i) : make_double2(0.0, 0.0);
}

// H = sum_k T_k(H0) listed as T_0(h_0), T_1(h_0), ..., T_{N-1}(h_0), T_0(h_1), ...
// (entry h N + k: h_h translated by k sites); out word-major with capacity
// nH0 N, FP64 coefficients.
template <int W>
__global__ __launch_bounds__(256) void k_ts_expand(const uint64_t* x, const uint64_t* z,
                                                   int64_t cap, const double2* c, int64_t nh,
                                                   int N, uint64_t* ox, uint64_t* oz,
                                                   double2* oc) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t n = nh * N;
  if (i >= n) return;
  const int64_t h = i / N;
  const int k = (int)(i % N);
  uint64_t vx[W], vz[W], tx[W], tz[W];
#pragma unroll
  for (int w = 0; w < W; w++) {
    vx[w] = x[(size_t)w * cap + h];
    vz[w] = z[(size_t)w * cap + h];
  }
  // translation by k = rotation down by (N - k) mod N
  const int r = k ? N - k : 0;
  ts_rot_down<W>(vx, N, r, tx);
  ts_rot_down<W>(vz, N, r, tz);
#pragma unroll
  for (int w = 0; w < W; w++) {
    ox[(size_t)w * n + i] = tx[w];
    oz[(size_t)w * n + i] = tz[w];
  }
  oc[i] = c[h];
}

// Reductions over an operator's strings: at most RED_BLOCKS blocks of
// RED_THREADS threads leave double-double partials in pinned host memory, which
// the host adds up after its one wait (a second kernel and a copy of its result
// took longer than the sum).  A block for every CU: with 128, half of them were
// idle, and the inner product of 2^22 one-word strings took 254 us, now 168
// (2^18: 48 and 43).
constexpr int RED_BLOCKS = 256, RED_THREADS = 1024;
DEV void red_part(dd s, double2* part) {
  __shared__ double rh[RED_THREADS / 64], rl[RED_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int d = 32; d >= 1; d >>= 1) {
    dd o;
    o.hi = __shfl_down(s.hi, d, 64);
    o.lo = __shfl_down(s.lo, d, 64);
    if (lane < d) s = dd_add(s, o);
  }
  __syncthreads();  // rh, rl of an earlier sum have been read
  if (lane == 0) {
    rh[wv] = s.hi;
    rl[wv] = s.lo;
  }
  __syncthreads();
  if (tid == 0) {
    dd t = {rh[0], rl[0]};
    for (int w = 1; w < RED_THREADS / 64; w++) t = dd_add(t, dd{rh[w], rl[w]});
    part[blockIdx.x] = make_double2(t.hi, t.lo);
  }
}

// sum_k stab(s_k) |c_k|^2: the norm of a translation-symmetric operator held
// as representatives, over N (stab = translations k in [0, N) that leave the
// string unchanged).
template <int W, bool F32>
__global__ __launch_bounds__(RED_THREADS) void k_norm_part_ts(const uint64_t* x, const uint64_t* z,
                                                              int64_t cap, const void* coef,
                                                              int64_t n, int N, TsTop top,
                                                              double2* part) {
  dd s = dd_zero();
  for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * RED_THREADS) {
    const double2 v = load_coef(coef, F32, i);
    const Key<W> raw = load_raw<W>(x, z, cap, i);
    const int st = ts_stabilizers<W>(raw.w, raw.w + W, N, top);
    const double w2 = weight2(v);
    for (int r = 0; r < st; r++) s = dd_add(s, w2);
  }
  red_part(s, part);
}

// Order keys of an operator's strings, and the strings of order keys.
template <int W>
__global__ void k_order_keys(const uint64_t* x, const uint64_t* z, int64_t cap, int64_t n,
                             Key<W>* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  Key<W> raw;
#pragma unroll
  for (int w = 0; w < W; w++) {
    raw.w[w] = x[(size_t)w * cap + i];
    raw.w[W + w] = z[(size_t)w * cap + i];
  }
  out[i] = mix_key<W>(raw);
}

template <int W>
__global__ void k_from_order_keys(const Key<W>* keys, int64_t n, uint64_t* x, uint64_t* z,
                                  int64_t cap) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Key<W> raw = unmix_key<W>(keys[i]);
#pragma unroll
  for (int w = 0; w < W; w++) {
    x[(size_t)w * cap + i] = raw.w[w];
    z[(size_t)w * cap + i] = raw.w[W + w];
  }
}

// sum |c|^2
template <bool F32>
__global__ __launch_bounds__(RED_THREADS) void k_norm_part(const void* coef, int64_t n,
                                                           double2* part) {
  dd s = dd_zero();
  const int64_t step = (int64_t)gridDim.x * RED_THREADS;
  for (int64_t i0 = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i0 < n; i0 += 4 * step) {
    double w2[4];
#pragma unroll
    for (int u = 0; u < 4; u++)
      w2[u] = i0 + u * step < n ? weight2(load_coef(coef, F32, i0 + u * step)) : 0.0;
#pragma unroll
    for (int u = 0; u < 4; u++) s = dd_add(s, w2[u]);
  }
  red_part(s, part);
}

// Inner product: every string of A is looked up in B's order keys.
template <int W>
__global__ __launch_bounds__(RED_THREADS) void k_inner_part(const uint64_t* ax, const uint64_t* az,
                                                            int64_t acap, int64_t na,
                                                            const void* acoef, int af32,
                                                            const Key<W>* bmk, int64_t nb,
                                                            const void* bcoef, int bf32,
                                                            double2* part_re, double2* part_im) {
  dd sr = dd_zero(), si = dd_zero();
  for (int64_t i = (int64_t)blockIdx.x * RED_THREADS + threadIdx.x; i < na;
       i += (int64_t)gridDim.x * RED_THREADS) {
    const Key<W> m = mix_key<W>(load_raw<W>(ax, az, acap, i));
    const int64_t found = find_key<W>(m, nb, [&](int64_t k) { return bmk[k]; });
    if (found >= 0) {
      const double2 av = load_coef(acoef, af32, i), bv = load_coef(bcoef, bf32, found);
      const double p1 = av.x * bv.x, p2 = av.y * bv.y, p3 = av.x * bv.y, p4 = av.y * bv.x;
      sr = dd_add(sr, p1);
      sr = dd_add(sr, p2);
      si = dd_add(si, p3);
      si = dd_add(si, -p4);
    }
  }
  red_part(sr, part_re);
  red_part(si, part_im);
}

__global__ void k_fill_u32(uint32_t* p, uint32_t v, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace pauli
