// Host orchestration and C ABI of the Pauli-string engine (see include/pauli.h).
//
// Every operation is one or more "engine calls": records from a commutator
// pair loop and/or from operator terms are binned by the leading bits of
// their mixed key, merged per bucket in LDS (summing each string's
// contributions in canonical order), filtered, reduced to the top-M by an
// exact radix select and compacted into the output.  The engine carves all
// of its scratch from the caller's workspace; intermediate operators of a
// Runge-Kutta step live at the top end of the same workspace.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <set>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/pauli.h"
#include "kernels.hpp"
#include "select.hpp"
#include "mlp.hpp"

using namespace pauli;

namespace {

thread_local std::string g_last_error;
thread_local pauli_stats g_stats;
thread_local pauli_totals g_totals;

// ---------------------------------------------------------------------------
// Optional kernel timing
// ---------------------------------------------------------------------------
struct Prof {
  std::mutex mu;
  bool on = false;
  std::set<std::string> only;  // kernel names to time; empty: every kernel
  struct Pending {
    const char* name;
    hipEvent_t a, b;
  };
  std::vector<Pending> pending;
  std::vector<hipEvent_t> pool;
  std::map<std::string, std::pair<long, double>> acc;

  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  void resolve() {  // call after the stream is synchronised
    std::lock_guard<std::mutex> g(mu);
    for (auto& p : pending) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, p.a, p.b) == hipSuccess) {
        auto& e = acc[p.name];
        e.first += 1;
        e.second += ms;
      }
      pool.push_back(p.a);
      pool.push_back(p.b);
    }
    pending.clear();
  }
};
Prof g_prof;

struct ProfScope {
  const char* name;
  hipStream_t s;
  hipEvent_t a = nullptr, b = nullptr;
  ProfScope(const char* n, hipStream_t st) : name(n), s(st) {
    if (!g_prof.on) return;
    std::lock_guard<std::mutex> g(g_prof.mu);
    if (!g_prof.only.empty() && !g_prof.only.count(n)) return;
    a = g_prof.get();
    b = g_prof.get();
    if (a) (void)hipEventRecord(a, s);
  }
  ~ProfScope() {
    if (!a || !b) return;
    (void)hipEventRecord(b, s);
    std::lock_guard<std::mutex> g(g_prof.mu);
    g_prof.pending.push_back({name, a, b});
  }
};

#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess) {                                                        \
      g_last_error = std::string(#expr) + ": " + hipGetErrorString(e_);           \
      return PAULI_EHIP;                                                           \
    }                                                                              \
  } while (0)

#define LAUNCH(name, kern, grid, block, ...)                                       \
  do {                                                                             \
    ProfScope ps_(name, stream);                                                   \
    hipLaunchKernelGGL(kern, dim3(grid), dim3(block), 0, stream, __VA_ARGS__);     \
    HIP_TRY(hipGetLastError());                                                    \
  } while (0)

// the emission kernel of the call (translation-symmetric or plain)
#define EMIT(name, scatter, nbl)                                                   \
  do {                                                                             \
    if (c.ts)                                                                      \
      LAUNCH(name, (k_emit<W, F32, scatter, nbl, true>), rows, EMIT_THREADS, ea);  \
    else                                                                           \
      LAUNCH(name, (k_emit<W, F32, scatter, nbl, false>), rows, EMIT_THREADS, ea); \
  } while (0)

// both scans of a count matrix over 2^nbl bins
#define SCAN(nbl, counts, rows, spec_cap, mcap)                                    \
  LAUNCH("k_scan", k_scan<nbl>, (1 << nbl) / SC_COLS, SC_COLS * SC_NSEG, counts,   \
         rows, bin_total, bin_base, dctl, look, spec_cap, mcap)

#define TRY(expr)                    \
  do {                               \
    int rc_ = (expr);                \
    if (rc_ != PAULI_OK) return rc_; \
  } while (0)

inline size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }
inline int words_of(int n_qubits) { return (n_qubits + 63) / 64; }

// Pinned host memory of a thread, written by the device: the final control
// block of an engine call, and the partials and results of the reductions.
constexpr int RED_SUMS = 6;  // sums of one reduction call
struct HostBlock {
  Ctl ctl;
  unsigned int bad;                          // an operand is not in canonical order
  double2 part[RED_SUMS * RED_BLOCKS];
};
static_assert(sizeof(HostBlock) < (32 << 10), "as the header says");
constexpr int64_t LOOKUP_PINNED = 768;  // results of a lookup that go straight to pinned memory
thread_local HostBlock* t_host = nullptr;
thread_local hipEvent_t t_ctl_event = nullptr, t_scan_event = nullptr;
thread_local hipStream_t t_side_stream = nullptr;  // on device t_side_dev
thread_local int t_side_dev = -1;
int host_block(HostBlock** out) {
  if (!t_host) HIP_TRY(hipHostMalloc((void**)&t_host, sizeof(HostBlock), hipHostMallocPortable));
  *out = t_host;
  return PAULI_OK;
}
int host_ctl(Ctl** out) {
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  *out = &h->ctl;
  return PAULI_OK;
}
// the sum of the first n partials of slot k, rounded once
double host_sum(const HostBlock* h, int k, int n) {
  dd s = {0.0, 0.0};
  for (int i = 0; i < n; i++) {
    const double2 p = h->part[k * RED_BLOCKS + i];
    s = dd_add(s, dd{p.x, p.y});
  }
  return s.hi;
}
inline int red_blocks(int64_t n) {
  return (int)std::min<int64_t>((n + RED_THREADS - 1) / RED_THREADS, RED_BLOCKS);
}

// ---------------------------------------------------------------------------
// Workspace arena: engine scratch grows from the bottom (reset per engine
// call), operators that outlive an engine call are taken from the top.
// ---------------------------------------------------------------------------
struct Arena {
  char* base = nullptr;
  size_t cap = 0;
  size_t bottom = 0;  // next free byte from the bottom
  size_t top = 0;     // bytes used at the top end
  size_t need = 0;    // largest bottom + top requested so far
  bool short_ = false;

  bool dry = false;    // size only (pauli_workspace_query): no memory behind it

  void* take(size_t bytes) {
    bottom = align256(bottom);
    const size_t at = bottom;
    bottom += align256(bytes);
    if (bottom + top > need) need = bottom + top;
    if (dry) return nullptr;
    if (bottom + top > cap) {
      short_ = true;
      return nullptr;
    }
    return base + at;
  }
  void* take_top(size_t bytes) {
    top += align256(bytes);
    if (bottom + top > need) need = bottom + top;
    if (dry) return nullptr;
    if (bottom + top > cap) {
      short_ = true;
      return nullptr;
    }
    return base + (cap - top);
  }
};

struct OpV {
  int W = 1;
  int f32 = 0;
  int canon = 0;  // written by the engine: canonical order known
  int64_t n = 0;
  int64_t cap = 0;
  const uint64_t* x = nullptr;
  const uint64_t* z = nullptr;
  const void* c = nullptr;
};

OpV view(const pauli_op* o) {
  OpV v;
  v.W = words_of(o->n_qubits);
  v.f32 = o->dtype == PAULI_C64K;
  v.n = o->size;
  v.cap = o->capacity;
  v.x = o->x;
  v.z = o->z;
  v.c = o->coef;
  return v;
}

int check_op(const pauli_op* o, bool output) {
  if (!o) return PAULI_EINVAL;
  if (o->n_qubits < 1 || o->n_qubits > 128) return PAULI_EINVAL;
  if (o->dtype != PAULI_C128 && o->dtype != PAULI_C64K) return PAULI_EINVAL;
  if (o->capacity < 0 || (!output && (o->size < 0 || o->size > o->capacity))) return PAULI_EINVAL;
  if (o->capacity > 0 && (!o->x || !o->z || !o->coef)) return PAULI_EINVAL;
  return PAULI_OK;
}

struct GroupSpec {
  int kind = G_TERM;
  double2 alpha = make_double2(1.0, 0.0);
  bool divide = false;  // the group's values are divided by alpha.x instead
};

struct OutSpec {
  pauli_op* user = nullptr;  // write into the caller's operator
  bool to_arena = false;     // or allocate at the top of the workspace
  OpV arena_op;              // filled when to_arena
  int f32 = 0;
};

struct Call {
  int W = 1;
  bool f32rec = false;  // FP32 record values (precision split)
  bool has_comm = false;
  bool product = false;  // A B instead of [A, B] (H = A, O = B)
  int ts = 0;  // > 0: translation-symmetric operators on ts periodic sites (Alg. 2)
  OpV H, O;
  int comm_group = 0;
  int n_terms = 0;
  OpV T[MAX_TERMS];
  int tgroup[MAX_TERMS] = {0};
  int tlist[MAX_TERMS] = {0};
  int n_groups = 0;
  GroupSpec groups[MAX_GROUPS];
  int mode = M_PLAIN;
  bool round32 = false;
  const pauli_trunc* trunc = nullptr;
  OutSpec out;
  // Lanczos
  double b_prev = 0.0;
  double* b_out = nullptr;
};

int alpha_kind(double2 a) {
  if (a.x == 1.0 && a.y == 0.0) return A_ONE;
  if (a.x == 0.0 && a.y == 1.0) return A_I;
  return A_GENERAL;
}

// rotations N/q, q the primes of N, as ts_stabilizers takes them
TsTop ts_top(int N) {
  TsTop t = {{0, 0}};
  int m = N;
  for (int q = 2; q <= m; q++)
    if (m % q == 0) {
      const int r = N / q - 1;
      if (N > 1) t.w[r >> 6] |= 1ull << (r & 63);
      while (m % q == 0) m /= q;
    }
  return t;
}

// ---------------------------------------------------------------------------
// Planning and scratch layout of one engine call, shared by the engine and
// pauli_workspace_query (which lays the same buffers out on an empty arena).
// ---------------------------------------------------------------------------
// at most 1024 commutator rows (one tile of EMIT_THREADS O strings each up
// to |O| = 2^20: more, shorter rows scatter faster, since twice as many
// workgroups fit a CU as there are CUs) and 128 rows of operator terms
constexpr int64_t COMM_ROWS_MAX = 1024, TERM_ROWS_MAX = (1 << 17) / EMIT_THREADS;
static_assert(COMM_ROWS_MAX + TERM_ROWS_MAX <= SC_ROWS_MAX, "k_scan_cols covers every count row");
// Above this many tiles the strings of a tile are sorted by support and H is
// pruned to each wave's window (2 to 3 times fewer pairs tested); below, the
// pair tests take about a microsecond and the sort's loads and barriers more.
constexpr int EMIT_WINDOW_TILES = 32;
// One-pass calls over 2^17 bins: strings whose pairs are counted for the
// estimate, and rows of O tiles (one workgroup to a CU by LDS, two rounds)
// (64 tiles took 130 us of a translation-symmetric call of 53 M two-word
// records, 8 take 42; the estimate's spread stays far inside its 5 % margin)
constexpr int64_t WIDE_SAMPLE = 8 * EMIT_THREADS, WIDE_TILE_ROWS = 512;
static_assert(WIDE_SAMPLE <= 7 * NBINS, "an O of the sample's length never makes such a call");
static_assert(WIDE_TILE_ROWS + TERM_ROWS_MAX <= SW_ROWS_MAX, "k_scan_wide covers every row");
constexpr int MAX_PASS_BITS = 12;
constexpr int DIRECT_MAX_F = 22;  // at most 2^22 buckets in a direct merge
constexpr int64_t STREAM_MAX = 1 << 20;  // canonical terms up to here are streamed for their bounds
constexpr uint32_t MERGE_ONE_WAVE = 512;  // buckets that the full-size merge takes at once (two
                                          // blocks on each of 256 CUs)
constexpr int PART_NBL = 12;  // at most 2^12 partitions (MAX_PASS_BITS)
// blocks binning one partition: 1024 (one per CU, LDS-bound, so four
// rounds) write shorter per-(block, bin) runs and beat 256 and 512
constexpr int SPLIT_ROWS = 1024;
static_assert(SPLIT_ROWS <= SC_ROWS_MAX, "k_scan_cols covers every split row");

// An operator of few tiles would leave most CUs idle: its tiles are shared out
// over H (*hseg workgroups each, at least HSEG_MIN entries of H per share), up
// to HSEG_ROWS rows with those of the operator terms, which the count matrix
// holds room for in any case.  Ten
// noisy steps at 2^14 strings (16 tiles, |H| = 180) spent 102 + 61 us per
// commutator in the scatter and the count on 16 of 256 CUs: 16.5 -> 11.7 ms;
// a commutator of 77,777 two-word strings 304 -> 229 us (2^12 bins below 2^22
// possible records are part of both).
constexpr int64_t HSEG_ROWS = 256, HSEG_MIN = 8;
inline void plan_rows(bool comm, int64_t nH, int64_t nO, int64_t nterm_rec, int* comm_rows,
                      int* term_rows, int* hseg) {
  const int64_t tiles = comm ? std::min<int64_t>((nO + EMIT_THREADS - 1) / EMIT_THREADS, COMM_ROWS_MAX) : 0;
  *term_rows = nterm_rec > 0
                   ? (int)std::min<int64_t>((nterm_rec + EMIT_THREADS - 1) / EMIT_THREADS, TERM_ROWS_MAX)
                   : 0;
  *hseg = 1;
  if (comm)
    *hseg = (int)std::max<int64_t>(
        1, std::min<int64_t>((HSEG_ROWS - *term_rows) / tiles, nH / HSEG_MIN));
  *comm_rows = (int)tiles * *hseg;
}

// Hash passes from the largest bin of the NBINS_LOG-bin count: one pass when
// every bin fits a merge bucket; otherwise NBINS_LOG_MP bins per pass, whose
// largest holds about half as many, and one more pass bit per halving.
template <int W>
int plan_pass_bits(unsigned long long mx, int* nbl) {
  int pass_bits = 0;
  *nbl = NBINS_LOG;
  if (mx > (unsigned long long)merge_cap<W>()) {
    *nbl = NBINS_LOG_MP;
    mx = (mx + 1) / 2;
    while (mx > (unsigned long long)(merge_cap<W>() * 3 / 4) && pass_bits < 10) {
      pass_bits++;
      mx = (mx + 1) / 2;
    }
  }
  return pass_bits;
}

// scratch taken before the count pass
template <int W>
struct Bufs1 {
  Ctl* dctl = nullptr;
  uint64_t* Hk = nullptr;
  uint32_t* Hidx = nullptr;
  uint32_t* hstart = nullptr;
  int* hspan = nullptr;
  Key<W>* keep_mk = nullptr;
  uint32_t *counts = nullptr, *bin_total = nullptr, *bin_base = nullptr, *hist0 = nullptr;
  uint32_t* histL[2] = {nullptr, nullptr};
  uint32_t *hsum = nullptr, *h0sum = nullptr;
  unsigned long long* psum = nullptr;
  uint32_t* defer = nullptr;  // buckets left to the full-size merge (per pass)
  unsigned long long* look = nullptr;  // look-back states of a pass's buckets
};
template <int W>
void take_bufs1(Arena& ar, bool comm, int64_t nH, int64_t n_keep, int rows, Bufs1<W>& b) {
  const size_t KB = sizeof(Key<W>);
  b.dctl = (Ctl*)ar.take(sizeof(Ctl));
  b.Hk = comm ? (uint64_t*)ar.take((size_t)nH * KB) : nullptr;
  b.Hidx = comm ? (uint32_t*)ar.take((size_t)nH * 4) : nullptr;
  b.hstart = comm ? (uint32_t*)ar.take((size_t)(64 * W + 2) * 4) : nullptr;
  b.hspan = comm ? (int*)ar.take(4) : nullptr;
  b.keep_mk = n_keep ? (Key<W>*)ar.take((size_t)n_keep * KB) : nullptr;
  // rows of the emission, or of the partition binning (256 blocks)
  b.counts = (uint32_t*)ar.take((size_t)std::max(rows, 256) * NBINS_MP * 4);
  b.bin_total = (uint32_t*)ar.take(NBINS_MP * 4);
  b.bin_base = (uint32_t*)ar.take((NBINS_MP + 1) * 4);
  b.hist0 = (uint32_t*)ar.take((size_t)HREP * SEL0_BINS * 4);
  b.histL[0] = (uint32_t*)ar.take((size_t)HREP * SEL_BINS * 4);
  b.histL[1] = (uint32_t*)ar.take((size_t)HREP * SEL_BINS * 4);
  b.hsum = (uint32_t*)ar.take(SEL_BINS * 4);
  b.h0sum = (uint32_t*)ar.take(SEL0_BINS * 4);
  b.psum = (unsigned long long*)ar.take(PLAN_PARTS * 4 * 8);
  b.defer = (uint32_t*)ar.take(NBINS_MP * 4);
  // look-back states are in use where nothing is selected, this histogram
  // (cleared before each use) where the host finishes a select
  static_assert((size_t)HREP * SEL_BINS * 4 >= (size_t)NBINS_MP * 8, "a state per bin");
  b.look = (unsigned long long*)b.histL[0];
}

// scratch taken after the count pass: records (and their partitions),
// merged strings, per-bucket tables, select candidate lists
struct Bufs2 {
  void* recs = nullptr;
  uint32_t* rsrc_wide = nullptr;
  void* precs = nullptr;
  uint32_t *ptop = nullptr, *psrc = nullptr, *pbase = nullptr, *scounts = nullptr;
  void* uk = nullptr;
  double2* uc = nullptr;
  uint32_t *b_ubase = nullptr, *b_slots = nullptr, *b_surv = nullptr, *b_keep = nullptr;
  uint32_t *b_unique = nullptr, *b_abv = nullptr, *b_bcnt = nullptr, *b_obase = nullptr;
  double2* norm_part = nullptr;
  uint32_t* cand[3] = {nullptr, nullptr, nullptr};
  uint32_t* ccnt[3] = {nullptr, nullptr, nullptr};
};
template <int W, bool F32>
void take_bufs2(Arena& ar, size_t ptot, bool wide, bool partitioned, uint32_t max_buckets,
                bool want_select, Bufs2& b, bool records = true) {
  const size_t KB = sizeof(Key<W>), RB = sizeof(Rec<W, F32>);
  b.recs = records ? ar.take(ptot * RB) : nullptr;
  b.rsrc_wide = wide ? (uint32_t*)ar.take(ptot * 4) : nullptr;
  // several passes: every record is emitted once into 2^pass_bits partitions
  // (the top 32 bits of its order key aside, and its source id when wide);
  // each pass bins one partition
  b.precs = partitioned ? ar.take(ptot * RB) : nullptr;
  b.ptop = partitioned ? (uint32_t*)ar.take(ptot * 4) : nullptr;
  b.psrc = partitioned && wide ? (uint32_t*)ar.take(ptot * 4) : nullptr;
  b.pbase = partitioned ? (uint32_t*)ar.take(((1u << PART_NBL) + 1) * 4) : nullptr;
  b.scounts = partitioned ? (uint32_t*)ar.take((size_t)SPLIT_ROWS * NBINS_MP * 4) : nullptr;
  b.uk = ar.take(ptot * KB);
  b.uc = (double2*)ar.take(ptot * sizeof(double2));
  uint32_t** tabs[8] = {&b.b_ubase, &b.b_slots, &b.b_surv,  &b.b_keep,
                        &b.b_unique, &b.b_abv,  &b.b_bcnt, &b.b_obase};
  for (auto t : tabs) *t = (uint32_t*)ar.take((size_t)max_buckets * 4);
  b.norm_part = (double2*)ar.take((size_t)NORM_BLOCKS * sizeof(double2));
  if (want_select)
    for (int k = 0; k < 3; k++) {
      b.cand[k] = (uint32_t*)ar.take(ptot * 4);
      b.ccnt[k] = (uint32_t*)ar.take((size_t)max_buckets * 4);
    }
}

// An append call (at most append_max possible records): 2^append_bits buckets whose mean stays
// within 1024 records, with room for append_cap each; the records lie where the count matrix would.
// Lists, which repeat strings and emit every record, get twice the buckets, and are counted above
// half the records: 100,000 entries of 1000 strings overflowed 2^7 buckets and were redone (112 us
// with the count over 2^10 bins before, 160 redone, 63 in 2^8), 200,000 of 2000 strings 2^8.
inline unsigned long long append_max(bool list) { return list ? APPEND_MAX / 2 : APPEND_MAX; }
inline int append_bits(unsigned long long rec_bound, bool list) {
  int F = 1;
  while (rec_bound > ((list ? 512ull : 1024ull) << F)) F++;
  return F;
}
template <int W, bool F32>
void take_append(Arena& ar, int F, bool want_select, Bufs2& b) {
  static_assert(((size_t)append_cap<W>() << 8) * sizeof(Rec<W, F32>) <= (size_t)256 * NBINS_MP * 4 &&
                    (1024ull << 8) == APPEND_MAX,
                "the records of the longest call fit the count matrix");
  take_bufs2<W, F32>(ar, (size_t)append_cap<W>() << F, true, false, 1u << F, want_select, b, false);
}

// rows of an output at the top of the workspace
struct OutRows {
  uint64_t *x, *z;
  void* c;
};
template <int W>
OutRows take_rows(Arena& ar, size_t n, int f32) {
  OutRows r;
  r.x = (uint64_t*)ar.take_top(n * 8 * W);
  r.z = (uint64_t*)ar.take_top(n * 8 * W);
  r.c = ar.take_top(n * (f32 ? 8 : 16));
  return r;
}

struct Engine {
  Arena* ar;
  hipStream_t stream;
  Ctl* dctl = nullptr;
  Ctl* hctl = nullptr;
  bool pinned = false;  // *hctl is pinned: the device writes the final control block there
  // the count's copy to the host beside the scatter (pinned control block only):
  // recorded after the scan on the call's stream, then on a side stream
  // after the copy
  hipEvent_t ctl_event = nullptr, scan_event = nullptr;
  hipStream_t side_stream = nullptr;
  bool run_emit = false;  // take the emission path even for canonical terms
  bool run_counted = false;  // read the count before planning, even for small calls

  int read_ctl() {
    g_stats.host_syncs++;
    HIP_TRY(hipMemcpyAsync(hctl, dctl, sizeof(Ctl), hipMemcpyDeviceToHost, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    g_prof.resolve();
    return PAULI_OK;
  }
  // waits for the stream; the device has written the control block to *hctl
  int wait_ctl() {
    g_stats.host_syncs++;
    HIP_TRY(hipStreamSynchronize(stream));
    g_prof.resolve();
    return PAULI_OK;
  }
  int zero_u32(void* p, size_t words) {
    if (!words) return PAULI_OK;
    const size_t blocks = (words + 255) / 256;
    LAUNCH("k_fill_u32", k_fill_u32, blocks, 256, (uint32_t*)p, 0u, words);
    return PAULI_OK;
  }
  int set_u64(unsigned long long* dst, unsigned long long v) {
    // small host->device update of the control block (not used under capture)
    g_stats.host_syncs++;
    HIP_TRY(hipMemcpyAsync(dst, &v, sizeof(v), hipMemcpyHostToDevice, stream));
    HIP_TRY(hipStreamSynchronize(stream));
    return PAULI_OK;
  }

  template <int W, bool F32>
  int run(Call& c);
};

int ws_short(Arena& ar, pauli_ws* ws) {
  ws->required = ar.need + (1 << 20);
  return PAULI_EWORKSPACE;
}

template <int W, bool F32>
int Engine::run(Call& c) {
  const size_t KB = sizeof(Key<W>);
  constexpr size_t RB = sizeof(Rec<W, F32>);
  ar->bottom = 0;
  const size_t top0 = ar->top;
  memset(&g_stats, 0, sizeof(g_stats));
  // translation-symmetric commutator: H = sum_k T_k(H0), H0 listed over its
  // N translations (entry h N + k), then the plain commutator with every
  // product string replaced by its orbit representative.  c.H stays the
  // caller's H0: a call that is redone (below) expands it again.
  OpV H = c.H;
  if (c.ts && c.has_comm && H.n > 0) {
    const int64_t nf = H.n * c.ts;
    uint64_t* hx = (uint64_t*)ar->take((size_t)nf * 8 * W);
    uint64_t* hz = (uint64_t*)ar->take((size_t)nf * 8 * W);
    double2* hc = (double2*)ar->take((size_t)nf * sizeof(double2));
    if (ar->short_) return PAULI_EWORKSPACE;
    LAUNCH("k_ts_expand", (k_ts_expand<W>), (nf + 255) / 256, 256, H.x, H.z, H.cap,
           (const double2*)H.c, H.n, c.ts, hx, hz, hc);
    H.x = hx;
    H.z = hz;
    H.c = hc;
    H.n = nf;
    H.cap = nf;
  }
  // ----- inputs --------------------------------------------------------------
  const bool comm = c.has_comm && H.n > 0 && c.O.n > 0;
  int64_t tstart[MAX_TERMS + 1];
  tstart[0] = 0;
  for (int t = 0; t < c.n_terms; t++) tstart[t + 1] = tstart[t] + c.T[t].n;
  const int64_t nterm_rec = tstart[c.n_terms];
  const pauli_trunc* tr = c.trunc;
  const pauli_op* keep = tr ? tr->keep : nullptr;
  const int64_t n_keep = keep ? keep->size : 0;
  if (n_keep > 65536) return PAULI_EINVAL;
  if (keep && words_of(keep->n_qubits) != W) return PAULI_EINVAL;

  // every string's contributions must fit one merge bucket
  if (comm && H.n + c.n_terms + 8 > merge_cap<W>()) {
    g_last_error = "H has more strings than one merge bucket holds";
    return PAULI_EINVAL;
  }
  int comm_rows = 0, term_rows = 0, hseg = 1;
  plan_rows(comm, H.n, c.O.n, nterm_rec, &comm_rows, &term_rows, &hseg);
  const int rows = comm_rows + term_rows;

  // canonical linear combinations are merged from their terms (below), calls
  // of at most 2^18 possible records append to fixed buckets
  bool direct = !run_emit && !comm && c.n_terms > 0 && !c.ts && !c.product &&
                nterm_rec < ((int64_t)1 << 31);
  for (int t = 0; t < c.n_terms && direct; t++) {
    direct = !c.tlist[t];
    for (int u = 0; u < t; u++) direct = direct && c.tgroup[u] != c.tgroup[t];
  }
  const bool want_select = tr && tr->max_strings > 0;
  const unsigned long long rec_bound =
      (comm ? (unsigned long long)H.n * (unsigned long long)c.O.n : 0ull) +
      (unsigned long long)nterm_rec;
  // rows of an output at the top of the workspace: it never exceeds the records
  // emitted, nor max(M, |keep|) when a top-M cut is asked for
  auto arena_rows = [&](unsigned long long records) -> size_t {
    unsigned long long bound = records;
    if (want_select)
      bound = std::min<unsigned long long>(
          bound, (unsigned long long)std::max<long long>((long long)tr->max_strings, n_keep));
    return (size_t)std::max<unsigned long long>(bound, 1);
  };
  bool list = false;
  for (int t = 0; t < c.n_terms; t++) list = list || c.tlist[t];
  bool append = !direct && !run_counted && rows > 0 && rec_bound <= append_max(list);
  const int append_F = append_bits(append ? rec_bound : 0, list);
  Bufs1<W> b1;
  Bufs2 b2;
  take_bufs1<W>(*ar, comm, H.n, n_keep, rows, b1);
  if (append && !ar->short_) {
    const size_t mark_bottom = ar->bottom, mark_need = ar->need;
    take_append<W, F32>(*ar, append_F, want_select, b2);
    b2.recs = b1.counts;
    if (c.out.to_arena) {  // room for the output rows as well (place_output takes them)
      const size_t mark_top = ar->top;
      take_rows<W>(*ar, arena_rows(rec_bound), c.out.f32);
      ar->top = mark_top;
    }
    if (ar->short_) {  // the workspace holds the counted layout only
      ar->bottom = mark_bottom;
      ar->need = mark_need;
      ar->short_ = false;
      append = false;
      b2 = Bufs2();
    }
  }
  dctl = b1.dctl;
  uint64_t* Hk = b1.Hk;
  uint32_t* Hidx = b1.Hidx;
  uint32_t* hstart = b1.hstart;
  int* hspan = b1.hspan;
  Key<W>* keep_mk = b1.keep_mk;
  uint32_t* counts = b1.counts;
  uint32_t* bin_total = b1.bin_total;
  uint32_t* bin_base = b1.bin_base;
  uint32_t* hist0 = b1.hist0;
  uint32_t* histL[2] = {b1.histL[0], b1.histL[1]};
  uint32_t* hsum = b1.hsum;
  uint32_t* h0sum = b1.h0sum;
  unsigned long long* psum = b1.psum;
  unsigned long long* look = b1.look;
  if (ar->short_) return PAULI_EWORKSPACE;
  if (!hctl) {
    TRY(host_ctl(&hctl));
    pinned = true;
  }

  auto write_empty = [&]() -> int {
    if (c.out.to_arena) {
      c.out.arena_op = OpV();
      c.out.arena_op.W = W;
      c.out.arena_op.f32 = c.out.f32;
    } else {
      c.out.user->size = 0;
    }
    return PAULI_OK;
  };
  if (rows == 0) {
    if (c.mode == M_LANCZOS) {
      if (c.b_out) *c.b_out = 0.0;
      write_empty();
      return PAULI_BREAKDOWN;
    }
    return write_empty();
  }
  {
    // clears the control block and the level-0 |c|^2 histogram, lays out H
    PrepArgs pr;
    memset(&pr, 0, sizeof(pr));
    if (comm) {
      pr.x = H.x;
      pr.z = H.z;
      pr.cap = H.cap;
      pr.n = (int)H.n;
    }
    pr.packed = Hk;
    pr.hidx = Hidx;
    pr.hstart = hstart;
    pr.hspan = hspan;
    if (n_keep && n_keep <= KEEP_PREP) {
      pr.kx = keep->x;
      pr.kz = keep->z;
      pr.kcap = keep->capacity;
      pr.n_keep = (int)n_keep;
      pr.keep_mk = keep_mk;
    }
    pr.hist0 = hist0;
    if (append) {
      pr.cursor = bin_base;
      pr.n_cursor = 1 << append_F;
    }
    pr.look = look;
    pr.n_look = MERGE_ONE_WAVE;
    pr.ctl = dctl;
    LAUNCH("k_prep", (k_prep<W>), PREP_BLOCKS, 1024, pr);
  }
  if (n_keep > KEEP_PREP) {
    LAUNCH("k_mix_keys", (k_mix_keys<W>), (n_keep + 255) / 256, 256, keep->x, keep->z,
           keep->capacity, n_keep, keep_mk, &dctl->bad_keep);
  }

  // ----- canonical terms: every bucket merged straight from its term runs ---
  // A linear combination with no commutator, no list term and one group per
  // term needs no emission when each term is in canonical order: the strings
  // of a hash bucket (top F bits of the mixed key) are one contiguous run of
  // every term.  Terms the engine wrote are canonical; the others are checked
  // on the device, and when one is out of order the merges leave every bucket
  // empty and the call is redone by emission (run_emit), as it is when strings
  // crowd one bucket beyond the merge's capacity.
  unsigned long long pe_all = 0;
  bool scattered = false;  // one pass over 2^14 bins scattered before the count was read
  MergeArgs ma;
  WriteArgs wa;
  memset(&wa, 0, sizeof(wa));
  wa.keep_mk = keep_mk;
  wa.n_keep = (int)n_keep;
  wa.ctl = dctl;
  wa.out_f32 = c.out.f32;
  // where the output goes: the caller's operator, or the top of the workspace
  auto place_output = [&](unsigned long long records) -> int {
    if (c.out.to_arena) {
      const size_t n = arena_rows(records);
      const OutRows rows = take_rows<W>(*ar, n, c.out.f32);
      if (ar->short_) return PAULI_EWORKSPACE;
      c.out.arena_op.W = W;
      c.out.arena_op.f32 = c.out.f32;
      c.out.arena_op.canon = 1;
      c.out.arena_op.n = 0;
      c.out.arena_op.cap = (int64_t)n;
      c.out.arena_op.x = rows.x;
      c.out.arena_op.z = rows.z;
      c.out.arena_op.c = rows.c;
      wa.ox = rows.x;
      wa.oz = rows.z;
      wa.oc = rows.c;
      wa.ocap = (int64_t)n;
    } else {
      pauli_op* o = c.out.user;
      wa.ox = o->x;
      wa.oz = o->z;
      wa.oc = o->coef;
      wa.ocap = o->capacity;
    }
    ma.ox = wa.ox;
    ma.oz = wa.oz;
    ma.oc = wa.oc;
    ma.ocap = wa.ocap;
    ma.out_f32 = wa.out_f32;
    return PAULI_OK;
  };
  // Nothing is selected after a plain merge without a top-M cut: it writes the
  // output itself (k_merge's OUT).  Direct merges of more buckets than run at
  // once keep the small variant with its deferral list.
  bool final_merge = !want_select && c.mode == M_PLAIN;
  uint32_t nbk = 0;  // buckets written so far
  int npass = 1;
  auto merge_common = [&]() {
    memset(&ma, 0, sizeof(ma));
    for (int g = 0; g < c.n_groups; g++) {
      ma.alpha[g] = c.groups[g].alpha;
      ma.alpha_kind[g] = c.groups[g].divide ? A_DIV : alpha_kind(c.groups[g].alpha);
      ma.gkind[g] = c.groups[g].kind;
    }
    ma.mode = c.mode;
    ma.single = (c.n_groups == 1 && c.groups[0].kind != G_SUM_KAHAN32) ? 1 : 0;
    ma.round32 = c.round32 ? 1 : 0;
    ma.max_len = tr ? tr->max_len : 0;
    ma.use_eps = (tr && tr->coef_eps > 0.0) ? 1 : 0;
    ma.eps2 = tr ? tr->coef_eps * tr->coef_eps : 0.0;
    ma.keep_mk = keep_mk;
    ma.n_keep = (int)n_keep;
    ma.uk = b2.uk;
    ma.uc = b2.uc;
    ma.b_ubase = b2.b_ubase;
    ma.b_slots = b2.b_slots;
    ma.b_surv = b2.b_surv;
    ma.b_keep = b2.b_keep;
    ma.b_unique = b2.b_unique;
    ma.hist0 = hist0;
    ma.ctl = dctl;
    ma.defer = nullptr;
  };
  if (direct) {
    // 2^F buckets of at most 0.85 of the small merge's capacity on average
    constexpr int SCAP = small_merge_cap<W, F32>();
    int F = 0;
    while (F < DIRECT_MAX_F && (double)nterm_rec > std::ldexp(0.85 * SCAP, F)) F++;
    const uint32_t nb = 1u << F;
    uint32_t* tbounds = (uint32_t*)ar->take((size_t)c.n_terms * (nb + 1) * 4);
    take_bufs2<W, F32>(*ar, (size_t)nterm_rec, false, false, nb, want_select, b2, false);
    if (ar->short_) return PAULI_EWORKSPACE;
    TermView tv;
    memset(&tv, 0, sizeof(tv));
    tv.n_terms = c.n_terms;
    tv.F = F;
    tv.bounds = tbounds;
    uint32_t streamed = 0;  // terms whose bounds come from one pass over them
    int64_t nstream = 0;
    for (int t = 0; t < c.n_terms; t++) {
      const OpV& T = c.T[t];
      tv.tx[t] = T.x;
      tv.tz[t] = T.z;
      tv.tcap[t] = T.cap;
      tv.tn[t] = T.n;
      tv.tc[t] = T.c;
      tv.tf32[t] = T.f32;
      tv.tgroup[t] = (uint32_t)c.tgroup[t];
      if (!T.canon || T.n <= STREAM_MAX) {
        streamed |= 1u << t;
        nstream += T.n + 1;
      }
    }
    if (streamed)
      LAUNCH("k_term_stream", (k_term_stream<W>), (nstream + 255) / 256, 256, tv, streamed, tbounds,
             &dctl->unsorted);
    const int64_t nbounds = (int64_t)c.n_terms * (nb + 1);
    const uint32_t search = ((1u << c.n_terms) - 1u) & ~streamed;
    if (search)
      LAUNCH("k_term_bounds", (k_term_bounds<W>), (nbounds + 255) / 256, 256, tv, search, tbounds);
    merge_common();
    ma.tv = tv;
    ma.nbins_log = F;
    ma.digit_shift = F;
    final_merge = final_merge && nb <= MERGE_ONE_WAVE;
    if (final_merge) {
      TRY(place_output((unsigned long long)nterm_rec));
      ma.look = look;
      ma.hctl = pinned ? hctl : nullptr;
      LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID, true, true>),
             nb, MERGE_THREADS, ma);
    } else if (nb <= MERGE_ONE_WAVE) {
      // every bucket has a CU: the full-size variant takes them all at once
      LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID, true>), nb,
             MERGE_THREADS, ma);
    } else {
      ma.defer = b1.defer;
      // buckets above the small variant's capacity go to the full-size one
      LAUNCH("k_merge_small", (k_merge<W, F32, MERGE_SMALL_THREADS, SCAP, MERGE_SMALL, true>), nb,
             MERGE_SMALL_THREADS, ma);
      LAUNCH("k_merge_deferred",
             (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_LIST, true>),
             std::min<uint32_t>(nb, 512), MERGE_THREADS, ma);
    }
    nbk = nb;
    pe_all = (unsigned long long)nterm_rec;
  }
  if (!direct) {
    EmitArgs ea;
    memset(&ea, 0, sizeof(ea));
    ea.Hk = Hk;
    ea.Hidx = Hidx;
    ea.hstart = hstart;
    ea.hspan = hspan;
    ea.Hc = comm ? (const double2*)H.c : nullptr;
    ea.nH = comm ? (int)H.n : 0;
    ea.has_comm = comm ? 1 : 0;
    ea.product = c.product ? 1 : 0;
    ea.ts_n = c.ts;
    ea.comm_rows = comm_rows;
    ea.hseg = hseg;
    ea.windows = !c.product && (int64_t)comm_rows / hseg > EMIT_WINDOW_TILES ? 1 : 0;
    ea.comm_group = (uint32_t)c.comm_group;
    if (comm) {
      ea.Ox = c.O.x;
      ea.Oz = c.O.z;
      ea.Ocap = c.O.cap;
      ea.nO = c.O.n;
      ea.Oc = c.O.c;
    }
    ea.n_terms = c.n_terms;
    ea.term_rows = term_rows;
    for (int t = 0; t < c.n_terms; t++) {
      ea.tx[t] = c.T[t].x;
      ea.tz[t] = c.T[t].z;
      ea.tcap[t] = c.T[t].cap;
      ea.tc[t] = c.T[t].c;
      ea.tf32[t] = c.T[t].f32;
      ea.tgroup[t] = (uint32_t)c.tgroup[t];
      ea.tlist[t] = c.tlist[t];
    }
    for (int t = 0; t <= c.n_terms; t++) ea.tstart[t] = tstart[t];
    ea.counts = counts;
    ea.ctl = dctl;
    ea.bin_base = bin_base;
    ea.max_len = (c.mode == M_PLAIN && tr) ? tr->max_len : 0;

    if (append) {
      // A call of at most 2^18 possible records needs no count: 2^append_F
      // buckets whose mean stays within 1024 even if every possible record is
      // emitted, records appended by atomics on the bucket cursors (the merge sorts them), every bucket merged at once.  A
      // bucket above the capacity sends the call round again with the count
      // read first.  Count, scan and the deferral list took 19 of the 59 us
      // that the kernels of a step of a few hundred strings took.
      ea.recs = b2.recs;
      ea.rsrc_wide = b2.rsrc_wide;
      ea.wide = 1;
      ea.cursor = bin_base;
      ea.append_F = append_F;
      ea.append_cap = (uint32_t)append_cap<W>();
      EMIT("k_emit_append", true, NBL_APPEND);
      merge_common();
      ma.bin_count = bin_base;
      ma.append_cap = ea.append_cap;
      ma.recs = b2.recs;
      ma.rsrc_wide = b2.rsrc_wide;
      ma.wide = 1;
      ma.nbins_log = append_F;
      ma.digit_shift = append_F;
      nbk = 1u << append_F;
      pe_all = rec_bound;
      if (final_merge) {
        TRY(place_output(pe_all));
        ma.look = look;
        ma.hctl = pinned ? hctl : nullptr;
        LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID, false, true>),
               nbk, MERGE_THREADS, ma);
      } else {
        LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID>), nbk,
               MERGE_THREADS, ma);
      }
    } else {
    // 2^nbl hash bins per pass: NBINS_LOG while the call fits one pass,
    // NBINS_LOG_WIDE while it fits one pass over those, else NBINS_LOG_MP
    // (twice the records per pass) when it needs several, and
    // NBINS_LOG_MID for calls of at most 2^22 records even if every pair emits
    // one (the per-call bin tables then cost a quarter)
    int nbl = NBINS_LOG;
    // wide bins: emission rows (0: not used), row prefixes, tables
    int wtiles = 0, wrows = 0;
    bool counted_mp = false;  // the count read was taken over NBINS_LOG_MP bins
    uint16_t* pre16 = nullptr;
    uint32_t *wtotal = nullptr, *wbase = nullptr;
    unsigned long long* wlook = nullptr;
    uint32_t* defer = b1.defer;
    // (an H index of 512 or more would need ids aside there, which
    // translation-symmetric calls keep in any case)
    if (rec_bound <= (1ull << (NBINS_LOG_MID + 10)) &&
        (!comm || c.ts || H.n < (1 << (NBINS_LOG_MID - 3))))
      nbl = NBINS_LOG_MID;
    auto count_pass = [&](int pass_bits, uint32_t pass_id, bool read = true,
                          unsigned long long spec_cap = 0ull) -> int {
      ea.pass_bits = pass_bits;
      ea.pass_id = pass_id;
      const unsigned int mcap = merge_cap<W>();
      if (nbl == NBINS_LOG_MID) {
        EMIT("k_emit_count", false, NBINS_LOG_MID);
        SCAN(NBINS_LOG_MID, counts, rows, spec_cap, mcap);
      } else if (nbl == NBINS_LOG) {
        EMIT("k_emit_count", false, NBINS_LOG);
        SCAN(NBINS_LOG, counts, rows, spec_cap, mcap);
      } else {
        EMIT("k_emit_count", false, NBINS_LOG_MP);
        SCAN(NBINS_LOG_MP, counts, rows, 0ull, mcap);
      }
      return read ? read_ctl() : PAULI_OK;
    };
    // source ids fold into the key bits implied by the bin unless an index
    // needs more than 11 bits (H above 2047 strings, canonicalisation lists)
    // (translation-symmetric calls carry (H entry, rotation) as the source id)
    // (9 bits over 2^12 bins)
    auto wide_for = [&](int bins_log) {
      const int64_t max_h = (1 << (std::min(bins_log, NBINS_LOG) - 3)) - 1;
      bool w = comm && (H.n > max_h || c.ts);
      for (int t = 0; t < c.n_terms; t++) w = w || c.tlist[t];
      return w;
    };
    // seven passes' worth of possible records: see below
    const unsigned long long few = 7ull * (1ull << NBINS_LOG) * (unsigned long long)merge_cap<W>();
    bool spec = ctl_event && rec_bound <= few;
    if (rec_bound > few) {
      // A call of more possible records than that: the number is estimated
      // from the pairs of the first WIDE_SAMPLE strings (12 us and a host wait),
      // and the bins chosen by it.  (With no more strings of O than the sample
      // takes, H, which is shorter than a bucket, cannot make that many
      // records: they are operator terms, and go to the partitions.)
      //  - One pass over 2^14 bins: as a call of fewer possible records (19 M
      //    two-word records 1.65 ms, over 2^15 bins 1.75).
      //  - One pass over 2^15 bins: counted over those at once (a count over
      //    2^14 bins first took 0.21 of 2.43 ms for 23 M two-word FP32 records).
      //  - More, up to one pass over 2^17: counted over those, in bytes (which
      //    is what LDS holds of them), and scattered straight to the buckets,
      //    where the partitions below write and read every record twice: 96 M
      //    two-word records 6.8 -> 5.0 ms with the binning, the step 11.9 ->
      //    10.3 ms.  Not below 2^15 bins' worth: the open lines of 2^15 bins
      //    fit an L2, those of 2^17 do not (23 M records 0.80 -> 1.19 ms).  Nor
      //    translation-symmetric calls, whose binning runs beside the search
      //    for the representatives on one workgroup per CU: a step of 102 M
      //    one-word records 11.9 ms by partitions, 13.2 ms so.  Nor one-word FP32
      //    records, 24 bytes that straddle the lines they are scattered to:
      //    top-M commutators of 60, 111 and 200 M 4.4, 8.2 and 14.2 ms by
      //    partitions, 4.9, 9.3 and 17.0 so.
      //  - Otherwise, and when a count does not fit after all: the count over
      //    2^14 bins, and partitions.
      const int64_t tiles = (c.O.n + EMIT_THREADS - 1) / EMIT_THREADS;
      if (comm && c.O.n > WIDE_SAMPLE) {
        const double room = 0.85 * merge_cap<W>();
        EmitArgs se = ea;
        se.nO = WIDE_SAMPLE;
        se.n_terms = 0;
        se.hseg = (int)std::max<int64_t>(
            1, std::min<int64_t>(HSEG_ROWS * EMIT_THREADS / WIDE_SAMPLE, H.n / HSEG_MIN));
        se.comm_rows = (int)(WIDE_SAMPLE / EMIT_THREADS) * se.hseg;
        {
          const EmitArgs& ea = se;
          const int rows = se.comm_rows;
          EMIT("k_emit_sample", false, NBINS_LOG_MID);
          SCAN(NBINS_LOG_MID, counts, rows, 0ull, 0u);
        }
        TRY(read_ctl());
        const double mean = (double)hctl->pe_total * ((double)c.O.n / (double)WIDE_SAMPLE) +
                            (double)nterm_rec;
        const double est = 1.05 * mean;
        // (the largest of 2^14 bins lies some 4.2 standard deviations above their mean)
        if (mean <= (merge_cap<W>() - 4.2 * std::sqrt((double)merge_cap<W>())) * NBINS) {
          spec = ctl_event != nullptr;
        } else if (est <= room * NBINS_MP) {
          nbl = NBINS_LOG_MP;
        } else if (!c.ts && !(W == 1 && F32) && est <= room * NBINS_WIDE) {
          wtiles = (int)std::min<int64_t>(tiles, WIDE_TILE_ROWS);
          wrows = wtiles * hseg + term_rows;
        }
      }
    }
    if (spec) {
      // A call that may fit one pass over 2^12 or 2^14 bins (at most seven passes'
      // worth of possible records, or estimated to fit) is laid out for as many
      // records as the workspace holds beside the rest of that pass, up to what
      // the bins can hold; the count's control
      // block goes to the host behind an event and the scatter is launched
      // at once, so the GPU does not wait for the host's plan.  The bin scan
      // makes the scatter stand down when the records do not fit the layout
      // or a bin exceeds the merge capacity; the host then plans from the
      // count it has read, as below.
      const bool w14 = wide_for(nbl);
      const uint32_t mb = 1u << nbl;
      const size_t per = RB + KB + sizeof(double2) + (w14 ? 4 : 0) + (want_select ? 12 : 0) +
                         (c.out.to_arena ? (size_t)(16 * W + 16) : 0);
      const size_t fixed = (size_t)mb * (9 * 4 + (want_select ? 12 : 0)) +
                           NORM_BLOCKS * sizeof(double2) + ((size_t)64 << 10);
      const size_t used = align256(ar->bottom) + ar->top;
      const size_t avail = ar->cap > used + fixed ? ar->cap - used - fixed : 0;
      const unsigned long long cap_rec =
          std::min<unsigned long long>({rec_bound, (unsigned long long)(avail / per),
                                        (unsigned long long)mb * merge_cap<W>()});
      const size_t mark_bottom = ar->bottom, mark_need = ar->need;
      if (cap_rec >= (1ull << 16))
        take_bufs2<W, F32>(*ar, (size_t)cap_rec, w14, false, mb, want_select, b2);
      if (cap_rec < (1ull << 16) || ar->short_) {
        ar->bottom = mark_bottom;
        ar->need = mark_need;
        ar->short_ = false;
        TRY(count_pass(0, 0));
      } else {
        TRY(count_pass(0, 0, false, cap_rec));
        // the copy runs on a side stream once the scan is done, beside the scatter
        HIP_TRY(hipEventRecord(scan_event, stream));
        HIP_TRY(hipStreamWaitEvent(side_stream, scan_event, 0));
        HIP_TRY(hipMemcpyAsync(hctl, dctl, sizeof(Ctl), hipMemcpyDeviceToHost, side_stream));
        HIP_TRY(hipEventRecord(ctl_event, side_stream));
        ea.recs = b2.recs;
        ea.rsrc_wide = b2.rsrc_wide;
        ea.wide = w14 ? 1 : 0;
        ea.skip = &dctl->spec_fail;
        if (nbl == NBINS_LOG_MID)
          EMIT("k_emit_scatter", true, NBINS_LOG_MID);
        else
          EMIT("k_emit_scatter", true, NBINS_LOG);
        ea.skip = nullptr;
        g_stats.host_syncs++;
        HIP_TRY(hipEventSynchronize(ctl_event));
        if (!hctl->spec_fail) {
          scattered = true;  // the pass stands: layout and records are in place
        } else {
          ar->bottom = mark_bottom;
          ar->need = mark_need;
        }
      }
    } else {
      const size_t mark_bottom = ar->bottom, mark_need = ar->need;
      if (wrows) {
        pre16 = (uint16_t*)ar->take((size_t)wrows * NBINS_WIDE * 2);
        wtotal = (uint32_t*)ar->take(NBINS_WIDE * 4);
        wbase = (uint32_t*)ar->take((NBINS_WIDE + 1) * 4);
        wlook = (unsigned long long*)ar->take(NBINS_WIDE * 8);
        if (ar->short_) wrows = 0;
      }
      if (wrows) {
        ea.comm_rows = wtiles * hseg;
        ea.counts8 = (uint8_t*)counts;
        ea.pre16 = pre16;
        LAUNCH("k_emit_count", (k_emit<W, F32, false, NBINS_LOG_WIDE, false>), wrows, EMIT_THREADS,
               ea);
        LAUNCH("k_scan_wide", k_scan_wide, NBINS_WIDE / 128, 1024, (const uint8_t*)counts, wrows,
               pre16, wtotal, wbase, dctl, wlook);
        TRY(read_ctl());
        if ((hctl->overflow & 4u) || hctl->maxg[0] > (unsigned int)merge_cap<W>()) {
          wrows = 0;
          ea.comm_rows = comm_rows;
          TRY(zero_u32(&dctl->overflow, 1));
        }
      }
      if (wrows) {
        nbl = NBINS_LOG_WIDE;
        bin_base = wbase;
        look = wlook;
        defer = (uint32_t*)wlook;
        ea.bin_base = wbase;
      } else {
        ar->bottom = mark_bottom;
        ar->need = mark_need;
        ar->short_ = false;
        TRY(count_pass(0, 0));
        counted_mp = nbl == NBINS_LOG_MP;
        if (counted_mp && hctl->maxg[0] > (unsigned int)merge_cap<W>()) {
          counted_mp = false;
          nbl = NBINS_LOG;
          TRY(count_pass(0, 0));
        }
      }
    }
    if (nbl < NBINS_LOG && hctl->maxg[0] > (unsigned int)merge_cap<W>()) {
      // records that crowd one bin of 2^12: count again over 2^14 bins
      nbl = NBINS_LOG;
      TRY(count_pass(0, 0));
    }
    if (hctl->bad_keep) return PAULI_EINVAL;
    if (hctl->overflow & 2u) {
      g_last_error = "more than 2^32 records in one pass";
      return PAULI_EINTERNAL;
    }
    pe_all = hctl->pe_total;
    // passes over disjoint hash ranges keep every bucket within the merge capacity; the
    // largest bin does not always halve with each extra pass bit (all records
    // of one string share a bin), so a pass that still overflows restarts the
    // loop with one more pass bit
    // the count pass measured every bin exactly
    int pass_bits = nbl < NBINS_LOG || wrows || counted_mp ? 0 : plan_pass_bits<W>(hctl->maxg[0], &nbl);
    // Several passes bin each partition over 2^14 instead of 2^15 bins when
    // the 2^14 bins are expected to stay within 0.8 of the merge's capacity
    // (the merge then takes single bins where it would take pairs of 2^15
    // bins): half the destinations and count rows for the pass binning, and
    // its 64 KB bin table lets two blocks share a CU.
    int pnbl = nbl;  // bins per pass of the merge (and of the pass binning)
    if (nbl == NBINS_LOG_MP && pass_bits > 0 &&
        (double)hctl->maxg[0] <= std::ldexp(0.8 * merge_cap<W>(), pass_bits))
      pnbl = NBINS_LOG;
    // tables for two more pass bits where a pass can still turn out too full; up
    // to 2^14 bins the count has measured the one pass there is
    const int table_bits = wrows || nbl < NBINS_LOG_MP ? 0 : std::min(pass_bits + 2, MAX_PASS_BITS);
    const size_t ptot = (size_t)std::max<unsigned long long>(pe_all, 1);
    const uint32_t max_buckets = (uint32_t)(1u << nbl) << table_bits;
    // ----- records, U, bucket tables, candidate lists -------------------------
    const bool wide = wide_for(nbl);
    const bool partitioned = nbl == NBINS_LOG_MP;
    if (!scattered) {
      take_bufs2<W, F32>(*ar, ptot, wide, partitioned, max_buckets, want_select, b2);
      if (ar->short_) return PAULI_EWORKSPACE;
    }
    void* recs = b2.recs;
    uint32_t* rsrc_wide = b2.rsrc_wide;
    void* precs = b2.precs;
    uint32_t* ptop = b2.ptop;
    uint32_t* psrc = b2.psrc;
    uint32_t* pbase = b2.pbase;
    uint32_t* scounts = b2.scounts;
    void* uk = b2.uk;
    double2* uc = b2.uc;
    uint32_t* b_ubase = b2.b_ubase;
    uint32_t* b_slots = b2.b_slots;
    uint32_t* b_surv = b2.b_surv;
    uint32_t* b_keep = b2.b_keep;
    uint32_t* b_unique = b2.b_unique;
    uint32_t* b_abv = b2.b_abv;
    uint32_t* b_bcnt = b2.b_bcnt;
    uint32_t* b_obase = b2.b_obase;
    uint32_t* const* cand = b2.cand;
    uint32_t* const* ccnt = b2.ccnt;

    merge_common();
    // Its blocks wait for the rows of the buckets before them, so one bucket
    // with long runs (strings that many pairs meet in) holds up all that run
    // beside it.  Such a call shows by a bucket far above the mean: records
    // that meet by ones and twos stay within 6 standard deviations, long-run
    // calls are 11 to 17 off (product of 120,320 strings of H^3, N = 32:
    // 1.53 ms with the output in the merge, 1.32 without; of N = 40, 5.5 and
    // 4.1; a Runge-Kutta step of the 8 x 8 lattice at 9: 36.5 and 37.9).  Nor
    // in several passes (product of 2.0e8 pairs 49.5 and 31.2 ms).  Buckets
    // that all run at once wait for little.
    if (final_merge) {
      int g = 4;
      while (g > 0 && hctl->maxg[g] > (unsigned int)merge_cap<W>()) g--;
      // (a call that plan_pass_bits has just moved to 2^15 bins was counted over 2^14:
      // commutators of 30, 35 and 41 M one-word records with the output in the merge
      // 1.98, 2.25 and 2.61 ms, without 2.16, 2.50 and 2.99)
      const int counted_log = nbl == NBINS_LOG_MP && !counted_mp ? NBINS_LOG : nbl;
      const double nb = std::ldexp(1.0, counted_log - g), mean = (double)pe_all / nb;
      final_merge = pass_bits == 0 && (nb <= MERGE_ONE_WAVE ||
                                       (double)hctl->maxg[g] <= mean + 10.0 * std::sqrt(mean) + 10.0);
    }
    if (final_merge) TRY(place_output(pe_all));
    ma.bin_base = bin_base;
    ma.recs = recs;
    ma.rsrc_wide = rsrc_wide;
    ma.wide = wide ? 1 : 0;

    ea.recs = recs;
    ea.rsrc_wide = rsrc_wide;
    ea.wide = wide ? 1 : 0;
    nbk = 0;  // buckets written so far
    npass = 1 << pass_bits;
    // the first count pass's prefixes (in `counts`) and bin totals (in
    // bin_total) serve the first partitioning only
    bool first_counts = pe_all < 0xFFFFFFFFull && !counted_mp;
    for (bool done = false; !done;) {
      done = true;
      nbk = 0;
      unsigned long long u_off = 0;  // U slots reserved by earlier passes
      npass = 1 << pass_bits;
      SplitArgs sp;
      memset(&sp, 0, sizeof(sp));
      if (pass_bits > 0) {
        // emit every record once, into the partitions of its top pass_bits bits
        ea.part = 1;
        ea.pass_bits = pass_bits;
        ea.pass_id = 0;
        ea.recs = precs;
        ea.ptop = ptop;
        ea.psrc = psrc;
        ea.part_F = pnbl + pass_bits;
        ea.bin_base = pbase;
        if (first_counts && pass_bits <= 10) {
          // partition prefixes summed from the first count pass's bins, kept
          // above its rows x NBINS entries: no second pass over the pairs
          uint32_t* pcounts = counts + (size_t)rows * NBINS;
          LAUNCH("k_part_from_bins", k_part_from_bins, rows + 1, 1024, counts, rows, pass_bits,
                 1 << PART_NBL, pcounts, bin_total);
          ea.counts = pcounts;
        } else {
          EMIT("k_emit_part_count", false, PART_NBL);
          LAUNCH("k_scan_cols", k_scan_cols, (1 << PART_NBL) / SC_COLS, SC_COLS * SC_NSEG, counts, rows, bin_total, dctl,
                 1 << PART_NBL);
        }
        LAUNCH("k_scan_part", k_scan_part, 1, 1024, bin_total, npass, pbase, (1 << PART_NBL) + 1,
               dctl);
        EMIT("k_emit_part_scatter", true, PART_NBL);
        ea.counts = counts;
        first_counts = false;  // bin_total now holds partition, then split, totals
        ea.part = 0;
        ea.recs = recs;
        ea.bin_base = bin_base;
        sp.precs = precs;
        sp.ptop = ptop;
        sp.psrc = psrc;
        sp.pbase = pbase;
        sp.pass_bits = pass_bits;
        sp.wide = wide ? 1 : 0;
        sp.counts = scounts;
        sp.bin_base = bin_base;
        sp.recs = recs;
        sp.rsrc_wide = rsrc_wide;
      }
      for (int p = 0; p < npass; p++) {
        if (pass_bits > 0) {
          // bin partition p: histogram, scans (and the host check below)
          sp.part = (uint32_t)p;
          if (pnbl == NBINS_LOG) {
            LAUNCH("k_split_count", (k_split<W, F32, false, NBINS_LOG>), SPLIT_ROWS, 1024, sp);
            SCAN(NBINS_LOG, scounts, SPLIT_ROWS, 0ull, 0u);
          } else {
            LAUNCH("k_split_count", (k_split<W, F32, false, NBINS_LOG_MP>), SPLIT_ROWS, 1024, sp);
            SCAN(NBINS_LOG_MP, scounts, SPLIT_ROWS, 0ull, 0u);
          }
          TRY(read_ctl());
        } else if (nbl == NBINS_LOG_MP && !counted_mp) {
          // one pass at NBINS_LOG_MP bins: count again at that bin count; this
          // overwrites the first count pass's NBINS_LOG-bin prefixes and totals
          TRY(count_pass(pass_bits, (uint32_t)p));
          first_counts = false;
        }
        if (pass_bits > 0 && p == 0 && hctl->part_total != pe_all) {
          char msg[160];
          snprintf(msg, sizeof(msg), "partitions hold %llu records, the count pass %llu",
                   (unsigned long long)hctl->part_total, pe_all);
          g_last_error = msg;
          return PAULI_EINTERNAL;
        }
        const unsigned long long pe = hctl->pe_total;
        if (hctl->maxg[0] > (unsigned int)merge_cap<W>()) {
          if (pass_bits >= table_bits) {
            char msg[256];
            snprintf(msg, sizeof(msg),
                     "hash bucket above merge capacity: pass %d of %d, largest bin %u, "
                     "records in pass %llu, records in all passes %llu",
                     p, npass, hctl->maxg[0], (unsigned long long)pe, pe_all);
            g_last_error = msg;
            return PAULI_EINTERNAL;
          }
          pass_bits++;
          counted_mp = false;
          done = false;
          if (final_merge) {  // nothing is merged yet: one pass only
            final_merge = false;
            ar->top = top0;
          }
          // the earlier passes' merges filled the histogram
          TRY(zero_u32(hist0, (size_t)HREP * SEL0_BINS));
          break;
        }
        int g_log = 4;
        while (g_log > 0 && hctl->maxg[g_log] > (unsigned int)merge_cap<W>()) g_log--;
        if (pe == 0) continue;
        if (pass_bits > 0 && pnbl == NBINS_LOG)
          LAUNCH("k_split_scatter", (k_split<W, F32, true, NBINS_LOG>), SPLIT_ROWS, 1024, sp);
        else if (pass_bits > 0)
          LAUNCH("k_split_scatter", (k_split<W, F32, true, NBINS_LOG_MP>), SPLIT_ROWS, 1024, sp);
        else if (scattered)
          ;  // launched before the count was read
        else if (nbl == NBINS_LOG_WIDE)
          LAUNCH("k_emit_scatter", (k_emit<W, F32, true, NBINS_LOG_WIDE, false>), wrows,
                 EMIT_THREADS, ea);
        else if (nbl == NBINS_LOG_MID)
          EMIT("k_emit_scatter", true, NBINS_LOG_MID);
        else if (nbl == NBINS_LOG)
          EMIT("k_emit_scatter", true, NBINS_LOG);
        else
          EMIT("k_emit_scatter", true, NBINS_LOG_MP);
        ma.g_log = g_log;
        ma.nbins_log = pnbl;
        ma.digit_shift = pass_bits + pnbl - g_log;
        ma.pass_bits = pass_bits;
        ma.pass_id = (uint32_t)p;
        ma.u_off = u_off;
        ma.bucket_off = nbk;
        const uint32_t nb_pass = (uint32_t)((1u << pnbl) >> g_log);
        // Buckets up to the small variant's capacity run three to a CU: all
        // of them when the largest bucket fits; when most do, the full-size
        // merge takes the others from a deferral list; else the full-size merge
        // takes every bucket, and also when there are so few that all run at
        // once (1024 threads end a bucket sooner than 512: the merge of a
        // 3001-string step 9.2 -> 8.2 us, of a commutator at 2^18 strings of
        // the N = 30 chain 26.2 -> 25.1 us).
        constexpr int SCAP = small_merge_cap<W, F32>();
        const unsigned int big = hctl->maxg[g_log];
        if (final_merge) {
          ma.look = look;
          ma.hctl = pinned ? hctl : nullptr;
          if (big <= (unsigned int)SCAP && nb_pass > MERGE_ONE_WAVE)
            LAUNCH("k_merge_small",
                   (k_merge<W, F32, MERGE_SMALL_THREADS, SCAP, MERGE_SMALL, false, true>), nb_pass,
                   MERGE_SMALL_THREADS, ma);
          else
            LAUNCH("k_merge",
                   (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID, false, true>),
                   nb_pass, MERGE_THREADS, ma);
          nbk += nb_pass;
          u_off += pe;
          continue;
        }
        ma.defer = defer;
        if (nb_pass <= MERGE_ONE_WAVE) {
          LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID>), nb_pass,
                 MERGE_THREADS, ma);
        } else if (big <= (unsigned int)SCAP) {
          LAUNCH("k_merge_small", (k_merge<W, F32, MERGE_SMALL_THREADS, SCAP, MERGE_SMALL>),
                 nb_pass, MERGE_SMALL_THREADS, ma);
        } else if (pe <= (unsigned long long)nb_pass * (SCAP * 9 / 10)) {
          LAUNCH("k_merge_small", (k_merge<W, F32, MERGE_SMALL_THREADS, SCAP, MERGE_SMALL>),
                 nb_pass, MERGE_SMALL_THREADS, ma);
          LAUNCH("k_merge_deferred", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_LIST>),
                 std::min<uint32_t>(nb_pass, 512), MERGE_THREADS, ma);
        } else {
          LAUNCH("k_merge", (k_merge<W, F32, MERGE_THREADS, merge_cap<W>(), MERGE_GRID>), nb_pass,
                 MERGE_THREADS, ma);
        }
        nbk += nb_pass;
        u_off += pe;
      }
    }
    }
  }
  void* uk = b2.uk;
  double2* uc = b2.uc;
  uint32_t* b_ubase = b2.b_ubase;
  uint32_t* b_slots = b2.b_slots;
  uint32_t* b_surv = b2.b_surv;
  uint32_t* b_keep = b2.b_keep;
  uint32_t* b_unique = b2.b_unique;
  uint32_t* b_abv = b2.b_abv;
  uint32_t* b_bcnt = b2.b_bcnt;
  uint32_t* b_obase = b2.b_obase;
  double2* norm_part = b2.norm_part;
  uint32_t* const* cand = b2.cand;
  uint32_t* const* ccnt = b2.ccnt;
  g_stats.emitted = (int64_t)pe_all;
  g_stats.passes = npass;
  g_stats.buckets = (int32_t)nbk;
  if (nbk == 0) {
    TRY(read_ctl());
    if (hctl->overflow) {
      g_last_error = "merge bucket overflow";
      return PAULI_EINTERNAL;
    }
    g_stats.unique = 0;
    g_stats.survivors = 0;
    g_stats.output = 0;
    if (c.mode == M_LANCZOS) {
      if (c.b_out) *c.b_out = 0.0;
      write_empty();
      return PAULI_BREAKDOWN;
    }
    return write_empty();
  }

  const int nchunk = (int)((nbk + SEL_CHUNK - 1) / SEL_CHUNK);
  const double lanczos_floor_b = 1e-13 * (c.b_prev > 1.0 ? c.b_prev : 1.0);
  if (final_merge) {
    TRY(ma.hctl ? wait_ctl() : read_ctl());
  } else {
  // ----- Lanczos: b_n from the untruncated sum, then divide and filter -------
  if (c.mode == M_LANCZOS) {
    const int nblk = (int)std::min<uint32_t>((nbk + 3) / 4, NORM_BLOCKS);
    if (c.ts)
      LAUNCH("k_norm", (k_norm<W, true>), nblk, 256, b_ubase, b_slots, uk, uc, c.ts, ts_top(c.ts),
             nbk, norm_part, dctl);
    else
      LAUNCH("k_norm", (k_norm<W, false>), nblk, 256, b_ubase, b_slots, uk, uc, 0, TsTop{{0, 0}},
             nbk, norm_part, dctl);
    // b_n and the breakdown test are taken on the device (no read here); a
    // breakdown leaves nothing to keep, and the host reports it with the
    // output size
    ScaleArgs sa;
    memset(&sa, 0, sizeof(sa));
    sa.b_ubase = b_ubase;
    sa.b_slots = b_slots;
    sa.b_surv = b_surv;
    sa.b_keep = b_keep;
    sa.nbk = nbk;
    sa.uk = uk;
    sa.uc = uc;
    sa.norm2 = &dctl->norm_hi;
    sa.floor_b = lanczos_floor_b;
    sa.round32 = c.out.f32;
    sa.max_len = ma.max_len;
    sa.use_eps = ma.use_eps;
    sa.eps2 = ma.eps2;
    sa.keep_mk = keep_mk;
    sa.n_keep = (int)n_keep;
    sa.hist0 = hist0;
    sa.ctl = dctl;
    LAUNCH("k_scale_filter", (k_scale_filter<W>),
           (int)std::min<uint32_t>((nbk + 7) / 8, SCALE_BLOCKS), 512, sa);
  }

  // ----- top-M threshold, output offsets and write, decided on the device ---
  Sel2Args s2;
  memset(&s2, 0, sizeof(s2));
  s2.b_ubase = b_ubase;
  s2.b_slots = b_slots;
  s2.b_abv = b_abv;
  s2.b_bcnt = b_bcnt;
  s2.uk = uk;
  s2.uc = uc;
  s2.keep_mk = keep_mk;
  s2.n_keep = (int)n_keep;
  s2.nbk = nbk;
  s2.b_surv = b_surv;
  s2.b_keep = b_keep;
  s2.b_obase = b_obase;
  s2.ctl = dctl;
  s2.hctl = pinned ? hctl : nullptr;
  if (want_select) {
    // the candidate lists of the multi-level select double as these lists
    s2.list0 = cand[1];
    s2.cc0 = ccnt[1];
    s2.listf = cand[0];
    s2.listfb = cand[2];
    s2.hist1 = histL[1];
  }
  PlanArgs pa;
  memset(&pa, 0, sizeof(pa));
  pa.b_slots = b_slots;
  pa.b_surv = b_surv;
  pa.b_keep = b_keep;
  pa.b_unique = b_unique;
  pa.nbk = nbk;
  pa.want_select = want_select ? 1 : 0;
  pa.max_strings = want_select ? (long long)tr->max_strings : 0;
  pa.hist0 = hist0;
  pa.hist1 = want_select ? histL[1] : nullptr;
  pa.psum = psum;
  pa.h0sum = h0sum;
  pa.b_obase = b_obase;
  pa.ctl = dctl;
  pa.hctl = pinned ? hctl : nullptr;
  LAUNCH("k_plan", k_plan, !want_select && nbk <= PLAN_ONE ? 1 : 3 * PLAN_PARTS, 1024, pa);
  if (want_select) {
    const int nsel = (int)std::min<uint32_t>((nbk + 15) / 16, SEL_BLOCKS);
    LAUNCH("k_sel_pass1", (k_sel_pass1<W>), nsel, 1024, s2);
    LAUNCH("k_sel_narrow", (k_sel_narrow<W>), nsel, 1024, s2);
  }

  wa.b_keep = b_keep;
  wa.b_ubase = b_ubase;
  wa.b_slots = b_slots;
  wa.b_obase = b_obase;
  wa.uk = uk;
  wa.uc = uc;
  TRY(place_output(pe_all));
  LAUNCH("k_write_out", (k_write_out<W>), nchunk, 256, wa, nbk);
  TRY(pinned ? wait_ctl() : read_ctl());
  }
  if (direct && (hctl->unsorted || hctl->overflow)) {
    // a term out of canonical order (the buckets were left empty), or strings
    // crowded into one bucket beyond the merge's capacity: redo by emission,
    // whose hash-range passes split them
    ar->top = top0;
    run_emit = true;
    return run<W, F32>(c);
  }
  if (append && hctl->overflow) {
    // strings crowded into one bucket: redo with the count read first, whose
    // plan splits them
    ar->top = top0;
    run_counted = true;
    return run<W, F32>(c);
  }
  if (append) {
    if (hctl->bad_keep) return PAULI_EINVAL;
    g_stats.emitted = (int64_t)hctl->pe_total;
  }
  if (direct && hctl->bad_keep) return PAULI_EINVAL;
  if (hctl->overflow) {
    g_last_error = "merge bucket overflow";
    return PAULI_EINTERNAL;
  }
  if (c.mode == M_LANCZOS) {
    const double b = std::sqrt(hctl->norm_hi);
    if (c.b_out) *c.b_out = b;
    if (!(b > lanczos_floor_b)) {
      write_empty();
      return PAULI_BREAKDOWN;
    }
  }
  g_stats.unique = (int64_t)hctl->u_unique;
  g_stats.survivors = (int64_t)hctl->surv_total;

  // Output size known: report it, or fall back to the host-driven multi-level
  // select when the device select stopped at a large group of equal |c|.
  auto finish_output = [&](unsigned long long nout) -> int {
    g_stats.output = (int64_t)nout;
    if ((unsigned long long)wa.ocap < nout) {
      if (c.out.to_arena) {
        g_last_error = "output above its bound";
        return PAULI_EINTERNAL;
      }
      c.out.user->size = (int64_t)nout;
      return PAULI_ECAPACITY;
    }
    if (c.out.to_arena) c.out.arena_op.n = (int64_t)nout;
    else c.out.user->size = (int64_t)nout;
    return PAULI_OK;
  };
  if (!hctl->deep) {
    if (hctl->sel_mode == S_THRESHOLD && !hctl->t_found) {
      g_last_error = "top-M threshold not found";
      return PAULI_EINTERNAL;
    }
    return finish_output(hctl->out_total);
  }

  // ----- fallback: threshold by as many 12-bit levels as the ties need ------
  const unsigned long long surv = hctl->surv_total, fk = hctl->keep_total;
  const unsigned long long nonkeep = surv - fk;
  int sel_mode = S_ALL;
  if (want_select) {
    const long long budget = (long long)tr->max_strings - (long long)fk;
    if (budget <= 0) sel_mode = fk == surv ? S_ALL : S_KEEP_ONLY;
    else if ((unsigned long long)budget >= nonkeep) sel_mode = S_ALL;
    else sel_mode = S_THRESHOLD;
    if (sel_mode == S_THRESHOLD) {
      SelArgs sa;
      memset(&sa, 0, sizeof(sa));
      sa.b_ubase = b_ubase;
      sa.b_slots = b_slots;
      sa.b_abv = b_abv;
      sa.b_bcnt = b_bcnt;
      sa.uk = uk;
      sa.uc = uc;
      sa.keep_mk = keep_mk;
      sa.n_keep = (int)n_keep;
      sa.nbk = nbk;
      sa.ctl = dctl;
      TRY(set_u64(&dctl->sel_K, (unsigned long long)budget));
      LAUNCH("k_hist_reduce", k_hist_reduce, SEL0_BINS / 256, 256, hist0, SEL0_BINS, hsum);
      LAUNCH("k_select", k_select, 1, 1024, hsum, SEL0_BINS, dctl);
      // level 1: full pass over U into list 0 (kept for the boundary count)
      TRY(zero_u32(histL[0], (size_t)HREP * SEL_BINS));
      sa.list_out = cand[0];
      sa.cc_out = ccnt[0];
      sa.hist = histL[0];
      LAUNCH("k_level1", (k_level1<W>), nbk, 256, sa);
      TRY(read_ctl());
      int in = 0;
      unsigned long long cnt = hctl->sel_count;
      if (cnt > FINISH_CAP) {
        int level = 1, hslot = 0;
        LAUNCH("k_hist_reduce", k_hist_reduce, SEL_BINS / 256, 256, histL[0], SEL_BINS, hsum);
        LAUNCH("k_select", k_select, 1, 1024, hsum, SEL_BINS, dctl);
        TRY(read_ctl());
        cnt = hctl->sel_count;
        while (cnt > FINISH_CAP) {
          if (level >= (64 + 128 * W) / 12) {
            g_last_error = "top-M select did not converge";
            return PAULI_EINTERNAL;
          }
          const int out = in == 1 ? 2 : 1;
          hslot ^= 1;
          TRY(zero_u32(histL[hslot], (size_t)HREP * SEL_BINS));
          sa.list_in = cand[in];
          sa.cc_in = ccnt[in];
          sa.list_out = cand[out];
          sa.cc_out = ccnt[out];
          sa.hist = histL[hslot];
          sa.level = level;
          LAUNCH("k_cand_level", (k_cand_level<W>), nbk, 256, sa);
          LAUNCH("k_hist_reduce", k_hist_reduce, SEL_BINS / 256, 256, histL[hslot], SEL_BINS,
                 hsum);
          LAUNCH("k_select", k_select, 1, 1024, hsum, SEL_BINS, dctl);
          TRY(read_ctl());
          cnt = hctl->sel_count;
          in = out;
          level++;
        }
        // narrow to the chosen bin of the last level
        const int out = in == 1 ? 2 : 1;
        sa.list_in = cand[in];
        sa.cc_in = ccnt[in];
        sa.list_out = cand[out];
        sa.cc_out = ccnt[out];
        sa.hist = nullptr;
        sa.level = level;
        LAUNCH("k_cand_level", (k_cand_level<W>), nbk, 256, sa);
        in = out;
      }
      sa.list_in = cand[in];
      sa.cc_in = ccnt[in];
      LAUNCH("k_finish", (k_finish<W>), 1, 1024, sa);
      sa.list_in = cand[0];
      sa.cc_in = ccnt[0];
      LAUNCH("k_count_boundary", (k_count_boundary<W>), nbk, 64, sa);
    }
  }
  LAUNCH("k_scan_buckets", k_scan_buckets, 1, 1024, b_surv, b_keep, b_abv, b_bcnt, nbk, sel_mode,
         b_obase, dctl);
  TRY(read_ctl());
  if (sel_mode == S_THRESHOLD && !hctl->t_found) {
    g_last_error = "top-M threshold not found";
    return PAULI_EINTERNAL;
  }
  const unsigned long long nout = hctl->out_total;
  if ((unsigned long long)wa.ocap >= nout && nout) {
    wa.sel_mode = sel_mode;
    LAUNCH("k_write", (k_write<W>), nbk, 256, wa);
    g_stats.host_syncs++;
    HIP_TRY(hipStreamSynchronize(stream));
    g_prof.resolve();
  }
  return finish_output(nout);
}

int dispatch(Engine& e, Call& c) {
  if (c.W == 1) return c.f32rec ? e.run<1, true>(c) : e.run<1, false>(c);
  if (c.W == 2) return c.f32rec ? e.run<2, true>(c) : e.run<2, false>(c);
  return PAULI_EINVAL;
}

// hctl: host copy of the control block (nullptr: this thread's pinned block)
int run_call(Arena& ar, pauli_ws* ws, void* stream, Call& c, Ctl* hctl = nullptr) {
  Engine e;
  e.ar = &ar;
  e.stream = (hipStream_t)stream;
  e.hctl = hctl;
  // the overlapped count read needs the pinned control block, two events and
  // a side stream (created once per thread, default priority); callers that
  // bring their own block get none of them
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (!hctl && (!t_side_stream || t_side_dev == dev)) {
    if (!t_side_stream) {
      HIP_TRY(hipEventCreateWithFlags(&t_ctl_event, hipEventDisableTiming));
      HIP_TRY(hipEventCreateWithFlags(&t_scan_event, hipEventDisableTiming));
      HIP_TRY(hipStreamCreateWithFlags(&t_side_stream, hipStreamNonBlocking));
      t_side_dev = dev;
    }
    e.ctl_event = t_ctl_event;
    e.scan_event = t_scan_event;
    e.side_stream = t_side_stream;
  }
  int rc = dispatch(e, c);
  if (rc == PAULI_EWORKSPACE || ar.short_) return ws_short(ar, ws);
  if (rc == PAULI_OK || rc == PAULI_BREAKDOWN) {
    // algorithmic bytes of the pass: inputs read, records written and read,
    // merged strings written and read, output written, at the record size
    int64_t inputs = (c.has_comm ? c.O.n : 0);
    for (int t = 0; t < c.n_terms; t++) inputs += c.T[t].n;
    const double rb = 16.0 * c.W + (c.f32rec ? 8.0 : 16.0);
    g_totals.calls++;
    g_totals.inputs += inputs;
    g_totals.emitted += g_stats.emitted;
    g_totals.unique += g_stats.unique;
    g_totals.output += g_stats.output;
    g_totals.alg_bytes += rb * (double)(inputs + 2 * g_stats.emitted + 2 * g_stats.unique +
                                        g_stats.output);
  }
  return rc;
}

Arena make_arena(pauli_ws* ws) {
  Arena a;
  a.base = (char*)ws->ptr;
  a.cap = ws->ptr ? ws->bytes : 0;
  return a;
}

OpV as_input(const OpV& v) { return v; }

// ---------------------------------------------------------------------------
// Workspace sizing without device work: the engine's own scratch layout on a
// dry arena, with the records at their bound from the sizes and bins assumed
// to fill evenly (largest bin at most 1.5 times the mean plus the records one
// string can collect).
// ---------------------------------------------------------------------------
struct DryCall {
  bool comm = false;
  int64_t nH = 0, nO = 0;   // commutator operands (nH after the translation expansion)
  int ts = 0;               // translation-symmetric sites (H0 listed over ts translates)
  int64_t nterm = 0;        // operator-term records
  int n_terms = 0;
  bool wide = false;        // source ids kept aside (long canonicalisation lists)
  int64_t n_keep = 0;
  bool select = false;
  int64_t out_arena = -1;   // >= 0: output rows taken from the top of the workspace
  bool out_f32 = false;
};

template <int W, bool F32>
void dry_call(Arena& ar, const DryCall& d, unsigned long long* pe_out) {
  ar.bottom = 0;
  int64_t nH = d.nH;
  if (d.ts && d.comm && d.nH > 0) {
    nH = d.nH * d.ts;
    ar.take((size_t)nH * 8 * W);
    ar.take((size_t)nH * 8 * W);
    ar.take((size_t)nH * sizeof(double2));
  }
  const bool comm = d.comm && nH > 0 && d.nO > 0;
  int comm_rows = 0, term_rows = 0, hseg = 1;
  plan_rows(comm, nH, d.nO, d.nterm, &comm_rows, &term_rows, &hseg);
  Bufs1<W> b1;
  take_bufs1<W>(ar, comm, nH, d.n_keep, comm_rows + term_rows, b1);
  const unsigned long long pe =
      (comm ? (unsigned long long)nH * (unsigned long long)d.nO : 0ull) + (unsigned long long)d.nterm;
  if (pe_out) *pe_out = pe;
  const unsigned long long mx = pe * 3 / (2 * NBINS) + 1 + (comm ? nH : 0) + d.n_terms;
  int nbl = NBINS_LOG;
  const int pass_bits = plan_pass_bits<W>(mx, &nbl);
  const int table_bits = std::min(pass_bits + 2, MAX_PASS_BITS);
  const uint32_t max_buckets = (uint32_t)(1u << nbl) << table_bits;
  Bufs2 b2;
  const size_t mark_bottom = ar.bottom;
  // source ids aside as the engine decides (wide_for)
  take_bufs2<W, F32>(ar, (size_t)std::max<unsigned long long>(pe, 1), d.wide || (comm && (nH > 2047 || d.ts)),
                     nbl == NBINS_LOG_MP, max_buckets, d.select, b2);
  if (d.out_arena >= 0) take_rows<W>(ar, (size_t)std::max<int64_t>(d.out_arena, 1), d.out_f32);
  if (pe <= append_max(d.wide)) {
    // the fixed buckets that such a call takes when they fit (up to 2.75 times the records)
    ar.bottom = mark_bottom;
    take_append<W, F32>(ar, append_bits(pe, d.wide), d.select, b2);
  }
}

void dry(int W, bool f32rec, Arena& ar, const DryCall& d, unsigned long long* pe) {
  if (W == 1) f32rec ? dry_call<1, true>(ar, d, pe) : dry_call<1, false>(ar, d, pe);
  else f32rec ? dry_call<2, true>(ar, d, pe) : dry_call<2, false>(ar, d, pe);
}

// the output bound of a call emitting `pe` records under truncation t
int64_t out_bound(unsigned long long pe, const pauli_trunc* t) {
  unsigned long long b = pe;
  if (t && t->max_strings > 0) {
    const long long k = t->keep ? t->keep->size : 0;
    b = std::min<unsigned long long>(b, (unsigned long long)std::max<long long>(t->max_strings, k));
  }
  return (int64_t)std::max<unsigned long long>(b, 1);
}

int workspace_query(int op, const pauli_op* A, const pauli_op* B, const pauli_op* C,
                    const pauli_trunc* t, size_t* ws_bytes, int64_t* out_cap) {
  auto sz = [](const pauli_op* o) -> int64_t { return o ? std::max<int64_t>(o->size, 0) : 0; };
  const pauli_op* any = B ? B : A;
  if (!any || any->n_qubits < 1 || any->n_qubits > 128) return PAULI_EINVAL;
  const int W = words_of(any->n_qubits);
  const bool f32 = any->dtype == PAULI_C64K;
  const int64_t n_keep = (t && t->keep) ? t->keep->size : 0;
  const bool select = t && t->max_strings > 0;
  Arena ar;
  ar.dry = true;
  ar.cap = ~(size_t)0;
  unsigned long long pe = 0;
  int64_t cap = 1;
  DryCall d;
  d.n_keep = n_keep;
  d.select = select;
  switch (op) {
    case PAULI_Q_COMMUTATOR:
    case PAULI_Q_MULTIPLY:
    case PAULI_Q_COMMUTATOR_TS1D: {
      if (!A || !B) return PAULI_EINVAL;
      d.comm = true;
      d.nH = sz(A);
      d.nO = sz(B);
      d.ts = op == PAULI_Q_COMMUTATOR_TS1D ? B->n_qubits : 0;
      dry(W, f32, ar, d, &pe);
      cap = out_bound(pe, t);
      break;
    }
    case PAULI_Q_ADD: {
      if (!A || !B) return PAULI_EINVAL;
      d.nterm = sz(A) + sz(B);
      d.n_terms = 2;
      dry(W, A->dtype == PAULI_C64K && B->dtype == PAULI_C64K, ar, d, &pe);
      cap = out_bound(pe, t);
      break;
    }
    case PAULI_Q_TRUNCATE:
    case PAULI_Q_CANONICALIZE:
    case PAULI_Q_CANONICALIZE_TS1D: {
      if (!B) return PAULI_EINVAL;
      d.nterm = sz(B);
      d.n_terms = 1;
      d.wide = op != PAULI_Q_TRUNCATE;
      d.select = op == PAULI_Q_TRUNCATE && select;
      dry(W, f32, ar, d, &pe);
      cap = op == PAULI_Q_TRUNCATE ? out_bound(pe, t) : out_bound(pe, nullptr);
      break;
    }
    case PAULI_Q_LANCZOS:
    case PAULI_Q_LANCZOS_TS1D: {
      if (!A || !B) return PAULI_EINVAL;
      d.comm = true;
      d.nH = sz(A);
      d.nO = sz(B);
      d.ts = op == PAULI_Q_LANCZOS_TS1D ? B->n_qubits : 0;
      d.nterm = sz(C);
      d.n_terms = C ? 1 : 0;
      dry(W, f32, ar, d, &pe);
      cap = out_bound(pe, t);
      break;
    }
    case PAULI_Q_LANCZOS_REORTH: {
      if (!A || !B) return PAULI_EINVAL;
      DryCall d1;
      d1.comm = true;
      d1.nH = sz(A);
      d1.nO = sz(B);
      d1.nterm = sz(C);
      d1.n_terms = C ? 1 : 0;
      unsigned long long pe1 = 0;
      // O' at the top of the workspace, a bound without truncation
      d1.out_arena = (int64_t)std::max<unsigned long long>(
          (unsigned long long)d1.nH * (unsigned long long)d1.nO + (unsigned long long)d1.nterm, 1);
      dry(W, f32, ar, d1, &pe1);
      // projections: order keys of O_cur / O_prev
      ar.bottom = 0;
      ar.take((size_t)std::max<int64_t>(std::max(sz(B), sz(C)), 1) * 16 * W);
      d.nterm = d1.out_arena + sz(B) + sz(C);
      d.n_terms = 3;
      dry(W, false, ar, d, &pe);
      cap = out_bound(pe, t);
      break;
    }
    case PAULI_Q_RK4: {
      if (!A || !B) return PAULI_EINVAL;
      const int64_t nO = sz(B), nH = sz(A);
      int64_t S = nO, ksum = 0;
      for (int stage = 0; stage < 4; stage++) {
        DryCall dk;  // k = i [H, S], untruncated, at the top
        dk.comm = true;
        dk.nH = nH;
        dk.nO = S;
        const int64_t k = (int64_t)std::max<int64_t>(nH * S, 1);
        dk.out_arena = k;
        dry(W, false, ar, dk, nullptr);
        ksum += k;
        if (stage < 3) {
          DryCall ds;  // S = trunc(O + h k), at the top
          ds.nterm = nO + k;
          ds.n_terms = 2;
          ds.n_keep = n_keep;
          ds.select = select;
          ds.out_arena = out_bound((unsigned long long)(nO + k), t);
          dry(W, false, ar, ds, nullptr);
          S = ds.out_arena;
        }
      }
      d.nterm = nO + ksum;
      d.n_terms = 5;
      dry(W, false, ar, d, &pe);
      cap = out_bound(pe, t);
      break;
    }
    case PAULI_Q_REDUCTION: {
      // inner, correlator: order keys; coefficients: results (fewer bytes a
      // string); the sums go to the thread's pinned block
      ar.take((size_t)std::max<int64_t>(std::max(sz(A), sz(B)), 1) * 16 * W);
      cap = 0;
      break;
    }
    default:
      return PAULI_EINVAL;
  }
  // the engine adds the same margin when it reports a shortfall
  if (ws_bytes) *ws_bytes = ar.need + (1 << 20);
  if (out_cap) *out_cap = cap;
  return PAULI_OK;
}

// ---------------------------------------------------------------------------
// Scratch that needs no allocation: a file-scope device array (one copy per
// GPU, held until the process ends) for callers that cannot allocate.  Host
// code never passes the array's name to a kernel (on the host it is only a
// stand-in for the symbol): its device address on each GPU comes from
// hipGetSymbolAddress, taken once per device with that device current.
// ---------------------------------------------------------------------------
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)256 << 20;
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[MAX_DEVICES] = {nullptr};
// host copy of the control block for these calls (pageable: no host allocation)
thread_local Ctl t_static_hctl;

}  // namespace

__device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

namespace {
int static_scratch(void** out) {
  int dev = -1;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= MAX_DEVICES) {
    g_last_error = "device ordinal beyond the static scratch table";
    return PAULI_EINVAL;
  }
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p || ((uintptr_t)p & 255)) {
      g_last_error = "static scratch address not 256-byte aligned";
      return PAULI_EINTERNAL;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return PAULI_OK;
}
}  // namespace

namespace {
// Launches of the reductions; their sums go to the slots of h->part.
int launch_norm(hipStream_t stream, const pauli_op* A, HostBlock* h, int slot) {
  const int blocks = red_blocks(A->size);
  if (A->dtype == PAULI_C64K)
    LAUNCH("k_norm_part", k_norm_part<true>, blocks, RED_THREADS, A->coef, A->size,
           h->part + slot * RED_BLOCKS);
  else
    LAUNCH("k_norm_part", k_norm_part<false>, blocks, RED_THREADS, A->coef, A->size,
           h->part + slot * RED_BLOCKS);
  return PAULI_OK;
}
// <A, B> by lookups of A's strings in B, whose order keys go to bmk (slots
// slot, slot + 1); h->bad = 1 when B is not in canonical order
template <int W>
int launch_inner(hipStream_t stream, const OpV& A, const pauli_op* B, void* bmk, HostBlock* h,
                 int slot) {
  LAUNCH("k_mix_keys", k_mix_keys<W>, (B->size + 255) / 256, 256, B->x, B->z, B->capacity, B->size,
         (Key<W>*)bmk, &h->bad);
  LAUNCH("k_inner_part", k_inner_part<W>, red_blocks(A.n), RED_THREADS, A.x, A.z, A.cap, A.n, A.c,
         A.f32, (const Key<W>*)bmk, B->size, B->coef, B->dtype == PAULI_C64K ? 1 : 0,
         h->part + slot * RED_BLOCKS, h->part + (slot + 1) * RED_BLOCKS);
  return PAULI_OK;
}
int launch_inner(hipStream_t stream, const OpV& A, const pauli_op* B, void* bmk, HostBlock* h,
                 int slot) {
  return A.W == 1 ? launch_inner<1>(stream, A, B, bmk, h, slot)
                  : launch_inner<2>(stream, A, B, bmk, h, slot);
}
// workspace of a reduction: `keys` bytes of order keys
int red_room(pauli_ws* ws, size_t keys, void** out = nullptr) {
  Arena ar = make_arena(ws);
  void* p = ar.take(std::max<size_t>(keys, 16));
  if (out) *out = p;
  return ar.short_ ? ws_short(ar, ws) : PAULI_OK;
}
}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* pauli_strerror(int status) {
  switch (status) {
    case PAULI_OK: return "ok";
    case PAULI_EINVAL: return "invalid argument";
    case PAULI_ECAPACITY: return "output capacity too small (size holds the requirement)";
    case PAULI_EWORKSPACE: return "workspace too small (ws->required holds the requirement)";
    case PAULI_BREAKDOWN: return "Lanczos breakdown: b_n is zero";
    case PAULI_EHIP: return "HIP runtime error";
    case PAULI_EINTERNAL: return "internal limit exceeded";
    default: return "unknown status";
  }
}

const char* pauli_last_error(void) { return g_last_error.c_str(); }

void pauli_last_stats(pauli_stats* out) {
  if (out) *out = g_stats;
}

void pauli_read_totals(pauli_totals* out, int reset) {
  if (out) *out = g_totals;
  if (reset) memset(&g_totals, 0, sizeof(g_totals));
}

void pauli_profile_enable(int on) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.on = on != 0;
  g_prof.acc.clear();
}

void pauli_profile_only(const char* names) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  g_prof.only.clear();
  if (!names) return;
  std::string cur;
  for (const char* q = names;; q++) {
    if (*q == ',' || *q == 0) {
      if (!cur.empty()) g_prof.only.insert(cur);
      cur.clear();
      if (*q == 0) break;
    } else {
      cur += *q;
    }
  }
}

size_t pauli_profile_read(char* buf, size_t len) {
  std::lock_guard<std::mutex> g(g_prof.mu);
  std::string s;
  char line[256];
  for (auto& kv : g_prof.acc) {
    snprintf(line, sizeof(line), "%s %ld %.9f\n", kv.first.c_str(), kv.second.first,
             kv.second.second);
    s += line;
  }
  if (buf && len) {
    size_t n = std::min(len - 1, s.size());
    memcpy(buf, s.data(), n);
    buf[n] = 0;
  }
  return s.size() + 1;
}

int pauli_commutator(const pauli_op* H, const pauli_op* O, const pauli_trunc* t, pauli_op* out,
                     pauli_ws* ws, void* stream) {
  if (!ws || check_op(H, false) || check_op(O, false) || check_op(out, true)) return PAULI_EINVAL;
  if (H->n_qubits != O->n_qubits || out->n_qubits != O->n_qubits) return PAULI_EINVAL;
  if (H->dtype != PAULI_C128 || out->dtype != O->dtype) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(O->n_qubits);
  c.f32rec = O->dtype == PAULI_C64K;
  c.has_comm = true;
  c.H = view(H);
  c.O = view(O);
  c.comm_group = 0;
  c.n_groups = 1;
  c.groups[0].kind = c.f32rec ? G_SUM_KAHAN32 : G_SUM;
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_commutator_noalloc(const pauli_op* H, const pauli_op* O, const pauli_trunc* t,
                             pauli_op* out, void* stream) {
  if (check_op(H, false) || check_op(O, false) || check_op(out, true)) return PAULI_EINVAL;
  if (H->n_qubits != O->n_qubits || out->n_qubits != O->n_qubits) return PAULI_EINVAL;
  if (H->dtype != PAULI_C128 || out->dtype != O->dtype) return PAULI_EINVAL;
  void* base = nullptr;
  TRY(static_scratch(&base));
  pauli_ws ws = {base, STATIC_SCRATCH_BYTES, 0};
  Arena ar = make_arena(&ws);
  Call c;
  c.W = words_of(O->n_qubits);
  c.f32rec = O->dtype == PAULI_C64K;
  c.has_comm = true;
  c.H = view(H);
  c.O = view(O);
  c.comm_group = 0;
  c.n_groups = 1;
  c.groups[0].kind = c.f32rec ? G_SUM_KAHAN32 : G_SUM;
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  const int rc = run_call(ar, &ws, stream, c, &t_static_hctl);
  if (rc == PAULI_EWORKSPACE) {
    char msg[200];
    snprintf(msg, sizeof(msg),
             "the call needs %zu bytes of scratch; the static scratch holds %zu",
             ws.required, STATIC_SCRATCH_BYTES);
    g_last_error = msg;
  }
  return rc;
}

int pauli_multiply(const pauli_op* A, const pauli_op* B, const pauli_trunc* t, pauli_op* out,
                   pauli_ws* ws, void* stream) {
  if (!ws || check_op(A, false) || check_op(B, false) || check_op(out, true)) return PAULI_EINVAL;
  if (A->n_qubits != B->n_qubits || out->n_qubits != B->n_qubits) return PAULI_EINVAL;
  if (A->dtype != PAULI_C128 || out->dtype != B->dtype) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(B->n_qubits);
  c.f32rec = B->dtype == PAULI_C64K;
  c.has_comm = true;
  c.product = true;
  c.H = view(A);
  c.O = view(B);
  c.comm_group = 0;
  c.n_groups = 1;
  c.groups[0].kind = c.f32rec ? G_SUM_KAHAN32 : G_SUM;
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_commutator_ts1d(const pauli_op* H0, const pauli_op* O, const pauli_trunc* t,
                          pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(H0, false) || check_op(O, false) || check_op(out, true)) return PAULI_EINVAL;
  if (H0->n_qubits != O->n_qubits || out->n_qubits != O->n_qubits) return PAULI_EINVAL;
  if (H0->dtype != PAULI_C128 || out->dtype != O->dtype) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(O->n_qubits);
  c.f32rec = O->dtype == PAULI_C64K;
  c.has_comm = true;
  c.ts = O->n_qubits;
  c.H = view(H0);
  c.O = view(O);
  c.comm_group = 0;
  c.n_groups = 1;
  c.groups[0].kind = c.f32rec ? G_SUM_KAHAN32 : G_SUM;
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_canonicalize_ts1d(const pauli_op* in, pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(in, false) || check_op(out, true)) return PAULI_EINVAL;
  if (out->n_qubits != in->n_qubits) return PAULI_EINVAL;
  if (in->size >= ((int64_t)1 << GROUP_SHIFT)) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(in->n_qubits);
  c.f32rec = in->dtype == PAULI_C64K;
  c.ts = in->n_qubits;
  c.n_terms = 1;
  c.T[0] = view(in);
  c.tlist[0] = 1;
  c.n_groups = 1;
  c.groups[0].kind = G_SUM;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_norm2_ts1d(const pauli_op* A, double* out, pauli_ws* ws, void* stream_) {
  if (!ws || !out || check_op(A, false)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  TRY(red_room(ws, 0));
  if (A->size == 0) {
    *out = 0.0;
    return PAULI_OK;
  }
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  const int blocks = red_blocks(A->size);
  const int W = words_of(A->n_qubits), N = A->n_qubits;
  const bool f32 = A->dtype == PAULI_C64K;
#define NORM_TS(W, F)                                                                        \
  LAUNCH("k_norm_part_ts", (k_norm_part_ts<W, F>), blocks, RED_THREADS, A->x, A->z,          \
         A->capacity, A->coef, A->size, N, ts_top(N), h->part)
  if (W == 1) {
    if (f32) NORM_TS(1, true);
    else NORM_TS(1, false);
  } else {
    if (f32) NORM_TS(2, true);
    else NORM_TS(2, false);
  }
#undef NORM_TS
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  *out = host_sum(h, 0, blocks);
  return PAULI_OK;
}

int pauli_trace(const pauli_op* A, double out[2], pauli_ws* ws, void* stream_) {
  if (!ws || !out || check_op(A, false)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  TRY(red_room(ws, 0));
  out[0] = 0.0;
  out[1] = 0.0;
  if (A->size == 0) return PAULI_OK;
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  h->part[0] = make_double2(0.0, 0.0);
  const int blocks = (int)std::min<int64_t>((A->size + 255) / 256, 4096);
  const int f32 = A->dtype == PAULI_C64K ? 1 : 0;
  if (words_of(A->n_qubits) == 1)
    LAUNCH("k_trace", k_trace<1>, blocks, 256, A->x, A->z, A->capacity, A->size, A->coef, f32,
           &h->part[0].x);
  else
    LAUNCH("k_trace", k_trace<2>, blocks, 256, A->x, A->z, A->capacity, A->size, A->coef, f32,
           &h->part[0].x);
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  out[0] = h->part[0].x;
  out[1] = h->part[0].y;
  return PAULI_OK;
}

int pauli_add(const pauli_op* A, double ar_, double ai, const pauli_op* B, double br, double bi,
              const pauli_trunc* t, pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(A, false) || check_op(B, false) || check_op(out, true)) return PAULI_EINVAL;
  if (A->n_qubits != B->n_qubits || out->n_qubits != A->n_qubits) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(A->n_qubits);
  c.f32rec = A->dtype == PAULI_C64K && B->dtype == PAULI_C64K;
  c.n_terms = 2;
  c.T[0] = view(A);
  c.T[1] = view(B);
  c.tgroup[0] = 0;
  c.tgroup[1] = 1;
  c.n_groups = 2;
  c.groups[0].alpha = make_double2(ar_, ai);
  c.groups[1].alpha = make_double2(br, bi);
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_truncate(const pauli_op* in, const pauli_trunc* t, pauli_op* out, pauli_ws* ws,
                   void* stream) {
  if (!ws || check_op(in, false) || check_op(out, true)) return PAULI_EINVAL;
  if (out->n_qubits != in->n_qubits) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(in->n_qubits);
  c.f32rec = in->dtype == PAULI_C64K;
  c.n_terms = 1;
  c.T[0] = view(in);
  c.n_groups = 1;
  c.trunc = t;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_divide(const pauli_op* in, double b, pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(in, false) || check_op(out, true)) return PAULI_EINVAL;
  if (out->n_qubits != in->n_qubits || !(std::isfinite(b) && b != 0.0)) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(in->n_qubits);
  c.f32rec = in->dtype == PAULI_C64K;
  c.n_terms = 1;
  c.T[0] = view(in);
  c.n_groups = 1;
  c.groups[0].alpha = make_double2(b, 0.0);
  c.groups[0].divide = true;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

int pauli_canonicalize(const pauli_op* in, pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(in, false) || check_op(out, true)) return PAULI_EINVAL;
  if (out->n_qubits != in->n_qubits) return PAULI_EINVAL;
  if (in->size >= ((int64_t)1 << GROUP_SHIFT)) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(in->n_qubits);
  c.f32rec = in->dtype == PAULI_C64K;
  c.n_terms = 1;
  c.T[0] = view(in);
  c.tlist[0] = 1;
  c.n_groups = 1;
  c.groups[0].kind = G_SUM;
  c.out.user = out;
  c.out.f32 = out->dtype == PAULI_C64K;
  c.round32 = c.out.f32;
  return run_call(ar, ws, stream, c);
}

// ts = N: translation-symmetric operators of the periodic chain (H holds H0,
// the operators orbit representatives), else 0.
static int lanczos_step(const pauli_op* H, const pauli_op* O_prev, const pauli_op* O_cur,
                        double b_prev, const pauli_trunc* t, int ts, pauli_op* O_next,
                        double* b_out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(H, false) || check_op(O_cur, false) || check_op(O_next, true))
    return PAULI_EINVAL;
  if (O_prev && check_op(O_prev, false)) return PAULI_EINVAL;
  if (H->dtype != PAULI_C128 || O_next->dtype != O_cur->dtype) return PAULI_EINVAL;
  if (O_prev && O_prev->dtype != O_cur->dtype) return PAULI_EINVAL;
  if (H->n_qubits != O_cur->n_qubits || O_next->n_qubits != O_cur->n_qubits ||
      (O_prev && O_prev->n_qubits != O_cur->n_qubits))
    return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  Call c;
  c.W = words_of(O_cur->n_qubits);
  c.f32rec = O_cur->dtype == PAULI_C64K;
  c.has_comm = true;
  c.ts = ts;
  c.H = view(H);
  c.O = view(O_cur);
  c.comm_group = 0;
  c.n_groups = 1;
  c.groups[0].kind = c.f32rec ? G_SUM_KAHAN32 : G_SUM;
  if (O_prev && O_prev->size > 0) {
    c.n_terms = 1;
    c.T[0] = view(O_prev);
    c.tgroup[0] = 1;
    c.n_groups = 2;
    c.groups[1].kind = G_TERM;
    c.groups[1].alpha = make_double2(-b_prev, 0.0);
  }
  c.mode = M_LANCZOS;
  c.trunc = t;
  c.out.user = O_next;
  c.out.f32 = O_next->dtype == PAULI_C64K;
  c.b_prev = b_prev;
  double b = 0.0;
  c.b_out = &b;
  int rc = run_call(ar, ws, stream, c);
  if (b_out) *b_out = b;
  return rc;
}

// Lanczos step with local re-orthogonalisation: O' = [H, O_cur] - b_prev O_prev
// (untruncated, FP64, at the top of the workspace), then
// O'' = O' - (<O_cur,O'>/<O_cur,O_cur>) O_cur - (<O_prev,O'>/<O_prev,O_prev>) O_prev
// with both coefficients taken from O' (inner products and norms summed in
// double-double, rounded once, divided in FP64), b_n = ||O''||,
// O_next = trunc(O'' / b_n).
static int lanczos_step_reorth(const pauli_op* H, const pauli_op* O_prev, const pauli_op* O_cur,
                               double b_prev, const pauli_trunc* t, pauli_op* O_next,
                               double* b_out, pauli_ws* ws, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  Arena ar = make_arena(ws);
  const int W = words_of(O_cur->n_qubits);
  const bool f32 = O_cur->dtype == PAULI_C64K;
  const bool has_prev = O_prev && O_prev->size > 0;
  double b = 0.0;
  // 1. O' in FP64 (the commutator in FP32 with compensated sums for PAULI_C64K)
  Call c1;
  c1.W = W;
  c1.f32rec = f32;
  c1.has_comm = true;
  c1.H = view(H);
  c1.O = view(O_cur);
  c1.n_groups = 1;
  c1.groups[0].kind = f32 ? G_SUM_KAHAN32 : G_SUM;
  if (has_prev) {
    c1.n_terms = 1;
    c1.T[0] = view(O_prev);
    c1.tgroup[0] = 1;
    c1.n_groups = 2;
    c1.groups[1].kind = G_TERM;
    c1.groups[1].alpha = make_double2(-b_prev, 0.0);
  }
  c1.out.to_arena = true;
  c1.out.f32 = 0;
  TRY(run_call(ar, ws, stream, c1));
  const OpV Op = c1.out.arena_op;
  // 2. projections of O' on O_cur and O_prev
  double2 alpha[2] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
  const pauli_op* V[2] = {O_cur, has_prev ? O_prev : nullptr};
  if (Op.n > 0) {
    ar.bottom = 0;
    int64_t nk = 0;
    for (int k = 0; k < 2; k++)
      if (V[k]) nk = std::max<int64_t>(nk, V[k]->size);
    void* vmk = ar.take((size_t)std::max<int64_t>(nk, 1) * 16 * W);
    if (ar.short_) return ws_short(ar, ws);
    HostBlock* hb = nullptr;
    TRY(host_block(&hb));
    hb->bad = 0;
    for (int k = 0; k < 2; k++) {
      const pauli_op* v = V[k];
      if (!v || v->size == 0) continue;
      // <O', V> = sum conj(o') v over common strings (V canonical), ||V||^2
      TRY(launch_inner(stream, Op, v, vmk, hb, 3 * k));
      TRY(launch_norm(stream, v, hb, 3 * k + 2));
    }
    HIP_TRY(hipStreamSynchronize(stream));
    g_prof.resolve();
    if (hb->bad) {
      g_last_error = "re-orthogonalisation needs canonical O_cur and O_prev";
      return PAULI_EINVAL;
    }
    double h[12] = {0.0};
    for (int k = 0; k < 2; k++) {
      if (!V[k] || V[k]->size == 0) continue;
      h[6 * k] = host_sum(hb, 3 * k, red_blocks(Op.n));
      h[6 * k + 2] = host_sum(hb, 3 * k + 1, red_blocks(Op.n));
      h[6 * k + 4] = host_sum(hb, 3 * k + 2, red_blocks(V[k]->size));
    }
    for (int k = 0; k < 2; k++) {
      if (!V[k] || V[k]->size == 0) continue;
      const double n2 = h[6 * k + 4];
      // <V, O'> = conj(<O', V>), divided by <V, V>
      if (n2 > 0.0) alpha[k] = make_double2(h[6 * k] / n2, -h[6 * k + 2] / n2);
    }
  }
  // 3. O'' = O' - alpha_0 O_cur - alpha_1 O_prev, b_n, divide, truncate
  Call c2;
  c2.W = W;
  c2.f32rec = false;
  c2.n_terms = 0;
  c2.n_groups = 0;
  // a term with a zero coefficient only adds exact zeros: left out
  auto add_term = [&](const OpV& v, double2 al) {
    if (v.n == 0 || (al.x == 0.0 && al.y == 0.0)) return;
    c2.T[c2.n_terms] = v;
    c2.tgroup[c2.n_terms] = c2.n_groups;
    c2.groups[c2.n_groups].kind = G_TERM;
    c2.groups[c2.n_groups].alpha = al;
    c2.n_terms++;
    c2.n_groups++;
  };
  add_term(Op, make_double2(1.0, 0.0));
  for (int k = 0; k < 2; k++)
    if (V[k]) add_term(view(V[k]), make_double2(-alpha[k].x, -alpha[k].y));
  c2.mode = M_LANCZOS;
  c2.trunc = t;
  c2.out.user = O_next;
  c2.out.f32 = f32;
  c2.b_prev = b_prev;
  c2.b_out = &b;
  const int rc = run_call(ar, ws, stream, c2);
  if (b_out) *b_out = b;
  return rc;
}

int pauli_lanczos_step(const pauli_op* H, const pauli_op* O_prev, const pauli_op* O_cur,
                       double b_prev, const pauli_trunc* t, uint32_t flags, pauli_op* O_next,
                       double* b_out, pauli_ws* ws, void* stream) {
  if (flags & ~(uint32_t)PAULI_REORTH_LOCAL) return PAULI_EINVAL;
  if (!(flags & PAULI_REORTH_LOCAL))
    return lanczos_step(H, O_prev, O_cur, b_prev, t, 0, O_next, b_out, ws, stream);
  if (!ws || check_op(H, false) || check_op(O_cur, false) || check_op(O_next, true))
    return PAULI_EINVAL;
  if (O_prev && check_op(O_prev, false)) return PAULI_EINVAL;
  if (H->dtype != PAULI_C128 || O_next->dtype != O_cur->dtype) return PAULI_EINVAL;
  if (O_prev && O_prev->dtype != O_cur->dtype) return PAULI_EINVAL;
  if (H->n_qubits != O_cur->n_qubits || O_next->n_qubits != O_cur->n_qubits ||
      (O_prev && O_prev->n_qubits != O_cur->n_qubits))
    return PAULI_EINVAL;
  return lanczos_step_reorth(H, O_prev, O_cur, b_prev, t, O_next, b_out, ws, stream);
}

int pauli_lanczos_step_ts1d(const pauli_op* H0, const pauli_op* O_prev, const pauli_op* O_cur,
                            double b_prev, const pauli_trunc* t, pauli_op* O_next,
                            double* b_out, pauli_ws* ws, void* stream) {
  if (!O_cur) return PAULI_EINVAL;
  return lanczos_step(H0, O_prev, O_cur, b_prev, t, O_cur->n_qubits, O_next, b_out, ws, stream);
}

int pauli_rk4_step(const pauli_op* H, const pauli_op* O, double dt, const pauli_trunc* t,
                   pauli_op* out, pauli_ws* ws, void* stream) {
  if (!ws || check_op(H, false) || check_op(O, false) || check_op(out, true)) return PAULI_EINVAL;
  if (H->dtype != PAULI_C128 || O->dtype != PAULI_C128 || out->dtype != PAULI_C128)
    return PAULI_EINVAL;
  if (H->n_qubits != O->n_qubits || out->n_qubits != O->n_qubits) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  const int W = words_of(O->n_qubits);
  const double h2 = dt / 2.0, c1 = dt / 6.0, c2 = dt / 3.0;
  const OpV Ov = view(O);
  // k = i [H, S], kept at the top of the workspace.  Every use of k below
  // (the stage inputs and the final sum) is truncated with t's length cap
  // first, and the cap acts on each string alone, so strings of k above it
  // are not emitted at all: every result equals the one from the full k.
  pauli_trunc tl;
  memset(&tl, 0, sizeof(tl));
  if (t) tl.max_len = t->max_len;
  auto comm_i = [&](const OpV& S, OpV* k) -> int {
    Call c;
    c.W = W;
    c.has_comm = true;
    c.H = view(H);
    c.O = S;
    c.n_groups = 1;
    c.groups[0].kind = G_SUM;
    c.groups[0].alpha = make_double2(0.0, 1.0);
    c.trunc = tl.max_len > 0 ? &tl : nullptr;
    c.out.to_arena = true;
    int rc = run_call(ar, ws, stream, c);
    *k = c.out.arena_op;
    return rc;
  };
  // S = trunc(O + h k)
  auto stage = [&](const OpV& k, double h, OpV* S) -> int {
    Call c;
    c.W = W;
    c.n_terms = 2;
    c.T[0] = Ov;
    c.T[1] = k;
    c.tgroup[0] = 0;
    c.tgroup[1] = 1;
    c.n_groups = 2;
    c.groups[1].alpha = make_double2(h, 0.0);
    c.trunc = t;
    c.out.to_arena = true;
    int rc = run_call(ar, ws, stream, c);
    *S = c.out.arena_op;
    return rc;
  };
  OpV k1, k2, k3, k4, S2, S3, S4;
  TRY(comm_i(Ov, &k1));
  TRY(stage(k1, h2, &S2));
  TRY(comm_i(S2, &k2));
  TRY(stage(k2, h2, &S3));
  TRY(comm_i(S3, &k3));
  TRY(stage(k3, dt, &S4));
  TRY(comm_i(S4, &k4));
  Call c;
  c.W = W;
  c.n_terms = 5;
  c.T[0] = Ov;
  c.T[1] = k1;
  c.T[2] = k2;
  c.T[3] = k3;
  c.T[4] = k4;
  const double al[5] = {1.0, c1, c2, c2, c1};
  for (int g = 0; g < 5; g++) {
    c.tgroup[g] = g;
    c.groups[g].alpha = make_double2(al[g], 0.0);
  }
  c.n_groups = 5;
  c.trunc = t;
  c.out.user = out;
  return run_call(ar, ws, stream, c);
}

int pauli_add_noise(pauli_op* A, double lambda, void* stream_) {
  if (check_op(A, false) || !(lambda >= 0.0)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (A->size == 0) return PAULI_OK;
  NoiseTable t;
  for (int w = 0; w < NOISE_TABLE; w++) t.f[w] = std::exp(-lambda * (double)w);
  const int W = words_of(A->n_qubits);
  const int blocks = (int)std::min<int64_t>((A->size + 255) / 256, 8192);
  const int f32 = A->dtype == PAULI_C64K ? 1 : 0;
  if (W == 1)
    LAUNCH("k_add_noise", k_add_noise<1>, blocks, 256, A->x, A->z, A->capacity, A->size,
           A->coef, f32, t);
  else
    LAUNCH("k_add_noise", k_add_noise<2>, blocks, 256, A->x, A->z, A->capacity, A->size,
           A->coef, f32, t);
  return PAULI_OK;
}

int pauli_dagger(pauli_op* A, void* stream_) {
  if (check_op(A, false)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (A->size == 0) return PAULI_OK;
  const int blocks = (int)std::min<int64_t>((A->size + 255) / 256, 8192);
  LAUNCH("k_conj", k_conj, blocks, 256, A->coef, A->size, A->dtype == PAULI_C64K ? 1 : 0);
  return PAULI_OK;
}

int pauli_coefficients(const pauli_op* A, const pauli_op* Q, double* out, pauli_ws* ws,
                       void* stream_) {
  if (!ws || check_op(A, false) || check_op(Q, false) || (Q->size && !out)) return PAULI_EINVAL;
  if (A->n_qubits != Q->n_qubits) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (Q->size == 0) return PAULI_OK;
  const int W = words_of(A->n_qubits);
  Arena ar = make_arena(ws);
  double2* res = (double2*)ar.take((size_t)Q->size * 16);
  if (ar.short_) return ws_short(ar, ws);
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  static_assert(LOOKUP_PINNED <= RED_SUMS * RED_BLOCKS, "results take the partials' room");
  const bool direct = Q->size <= LOOKUP_PINNED;
  if (direct) res = h->part;
  const int64_t bq = (Q->size + 63) / 64;
  const int af32 = A->dtype == PAULI_C64K ? 1 : 0;
  if (W == 1)
    LAUNCH("k_lookup", k_lookup<1>, bq, 64, A->x, A->z, A->capacity, A->coef, af32, A->size, Q->x,
           Q->z, Q->capacity, Q->size, res);
  else
    LAUNCH("k_lookup", k_lookup<2>, bq, 64, A->x, A->z, A->capacity, A->coef, af32, A->size, Q->x,
           Q->z, Q->capacity, Q->size, res);
  if (!direct)
    HIP_TRY(hipMemcpyAsync(out, res, (size_t)Q->size * 16, hipMemcpyDeviceToHost, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  if (direct) memcpy(out, res, (size_t)Q->size * 16);
  return PAULI_OK;
}

int pauli_order_keys(const pauli_op* A, uint64_t* keys, void* stream_) {
  if (!keys || check_op(A, false)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  const int64_t n = A->size;
  if (n == 0) return PAULI_OK;
  const int W = words_of(A->n_qubits);
  const int64_t blocks = (n + 255) / 256;
  if (W == 1)
    LAUNCH("k_order_keys", k_order_keys<1>, blocks, 256, A->x, A->z, A->capacity, n,
           reinterpret_cast<Key<1>*>(keys));
  else
    LAUNCH("k_order_keys", k_order_keys<2>, blocks, 256, A->x, A->z, A->capacity, n,
           reinterpret_cast<Key<2>*>(keys));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

int pauli_strings_from_order_keys(int32_t n_qubits, const uint64_t* keys, int64_t n, uint64_t* x,
                                  uint64_t* z, int64_t cap, void* stream_) {
  if (n_qubits < 1 || n_qubits > 128 || n < 0 || cap < n || (n && (!keys || !x || !z)))
    return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  if (n == 0) return PAULI_OK;
  const int W = words_of(n_qubits);
  const int64_t blocks = (n + 255) / 256;
  if (W == 1)
    LAUNCH("k_from_order_keys", k_from_order_keys<1>, blocks, 256,
           reinterpret_cast<const Key<1>*>(keys), n, x, z, cap);
  else
    LAUNCH("k_from_order_keys", k_from_order_keys<2>, blocks, 256,
           reinterpret_cast<const Key<2>*>(keys), n, x, z, cap);
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

int pauli_workspace_query(int op, const pauli_op* A, const pauli_op* B, const pauli_op* C,
                          const pauli_trunc* t, size_t* ws_bytes, int64_t* out_capacity_upper) {
  return workspace_query(op, A, B, C, t, ws_bytes, out_capacity_upper);
}

int pauli_correlator(const pauli_op* O0, const pauli_op* O, double out[2], pauli_ws* ws,
                     void* stream_) {
  if (!out || check_op(O0, false) || check_op(O, false)) return PAULI_EINVAL;
  if (!ws || O0->n_qubits != O->n_qubits) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  void* bmk = nullptr;
  TRY(red_room(ws, (size_t)O0->size * 16 * words_of(O->n_qubits), &bmk));
  if (O0->size == 0) return PAULI_EINVAL;  // <O0, O0> = 0
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  h->bad = 0;
  TRY(launch_norm(stream, O0, h, 0));
  // <O, O0> looped over O with order-key lookups in O0, then conjugated
  if (O->size) TRY(launch_inner(stream, view(O), O0, bmk, h, 1));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  if (h->bad) return PAULI_EINVAL;
  const double n0 = host_sum(h, 0, red_blocks(O0->size));
  if (!(n0 > 0.0)) return PAULI_EINVAL;
  const double re = O->size ? host_sum(h, 1, red_blocks(O->size)) : 0.0;
  const double im = O->size ? host_sum(h, 2, red_blocks(O->size)) : 0.0;
  out[0] = re / n0;
  out[1] = -im / n0;
  return PAULI_OK;
}

int pauli_norm2(const pauli_op* A, double* out, pauli_ws* ws, void* stream_) {
  if (!ws || !out || check_op(A, false)) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  TRY(red_room(ws, 0));
  if (A->size == 0) {
    *out = 0.0;
    return PAULI_OK;
  }
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  TRY(launch_norm(stream, A, h, 0));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  *out = host_sum(h, 0, red_blocks(A->size));
  return PAULI_OK;
}

int pauli_inner(const pauli_op* A, const pauli_op* B, double out[2], pauli_ws* ws,
                void* stream_) {
  if (!ws || !out || check_op(A, false) || check_op(B, false)) return PAULI_EINVAL;
  if (A->n_qubits != B->n_qubits) return PAULI_EINVAL;
  hipStream_t stream = (hipStream_t)stream_;
  void* bmk = nullptr;
  TRY(red_room(ws, (size_t)B->size * 16 * words_of(A->n_qubits), &bmk));
  out[0] = out[1] = 0.0;
  if (A->size == 0 || B->size == 0) return PAULI_OK;
  HostBlock* h = nullptr;
  TRY(host_block(&h));
  h->bad = 0;
  TRY(launch_inner(stream, view(A), B, bmk, h, 0));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  if (h->bad) return PAULI_EINVAL;
  out[0] = host_sum(h, 0, red_blocks(A->size));
  out[1] = host_sum(h, 1, red_blocks(A->size));
  return PAULI_OK;
}


// ---------------------------------------------------------------------------
// b_n continuation network
// ---------------------------------------------------------------------------
int64_t pauli_mlp_num_params(void) { return mlp::NPARAM; }

static int mlp_check(const pauli_mlp* net) {
  if (!net || net->n_in != mlp::NIN || net->n_hidden != mlp::NHID || net->n_out != mlp::NOUT)
    return PAULI_EINVAL;
  if (!net->params || !net->params_bf16) return PAULI_EINVAL;
  return PAULI_OK;
}

static int gemm_launch(hipStream_t stream, const uint16_t* A, int lda, int transA,
                       const uint16_t* B, int ldb, int transB, float* C, uint16_t* Cb, int ldc,
                       const float* bias, int M, int N, int K, int epilogue) {
  if (M <= 0 || N <= 0 || K <= 0 || M % 16 || N % 16) return PAULI_EINVAL;
  mlp::GemmArgs g;
  g.A = A;
  g.B = B;
  g.C = C;
  g.Cb = Cb;
  g.bias = bias;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  g.transA = transA;
  g.transB = transB;
  g.M = M;
  g.N = N;
  g.K = K;
  g.epilogue = epilogue;
  // both operands read along k in 16-byte words
  const bool nt = !transA && transB && K % 8 == 0 && lda % 8 == 0 && ldb % 8 == 0 &&
                  ((uintptr_t)A | (uintptr_t)B) % 16 == 0;
  if (nt)
    LAUNCH("k_gemm_nt", mlp::k_gemm_nt,
           dim3((N + 16 * mlp::NT_TILES - 1) / (16 * mlp::NT_TILES), (M + 63) / 64), 256, g);
  else
    LAUNCH("k_gemm_bf16", mlp::k_gemm_bf16, dim3((N + 31) / 32, (M + 31) / 32), 256, g);
  return PAULI_OK;
}

int pauli_gemm_bf16(const uint16_t* A, int lda, int transA, const uint16_t* B, int ldb, int transB,
                    float* C, int ldc, int M, int N, int K, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!A || !B || !C) return PAULI_EINVAL;
  TRY(gemm_launch(stream, A, lda, transA, B, ldb, transB, C, nullptr, ldc, nullptr, M, N, K,
                  mlp::EP_STORE));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

int pauli_mlp_sync(const pauli_mlp* net, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  TRY(mlp_check(net));
  LAUNCH("k_to_bf16", mlp::k_to_bf16, (mlp::NPARAM + 255) / 256, 256, net->params,
         net->params_bf16, mlp::NPARAM);
  HIP_TRY(hipStreamSynchronize(stream));
  return PAULI_OK;
}

namespace {
struct MlpBufs {
  uint16_t *xb, *y1b, *y2b, *dyb, *dz2b, *dz1b;
  float *z1, *z2, *yh, *dy, *dy2, *dz2, *dy1, *dz1;
  double *row_err, *row_cnt, *loss;
};
int mlp_bufs(Arena& ar, int64_t B, MlpBufs& m) {
  const size_t b = (size_t)B;
  m.xb = (uint16_t*)ar.take(b * 16 * 2);
  m.y1b = (uint16_t*)ar.take(b * 256 * 2);
  m.y2b = (uint16_t*)ar.take(b * 256 * 2);
  m.dyb = (uint16_t*)ar.take(b * 16 * 2);
  m.dz2b = (uint16_t*)ar.take(b * 256 * 2);
  m.dz1b = (uint16_t*)ar.take(b * 256 * 2);
  m.z1 = (float*)ar.take(b * 256 * 4);
  m.z2 = (float*)ar.take(b * 256 * 4);
  m.yh = (float*)ar.take(b * 16 * 4);
  m.dy = (float*)ar.take(b * 16 * 4);
  m.dy2 = (float*)ar.take(b * 256 * 4);
  m.dz2 = (float*)ar.take(b * 256 * 4);
  m.dy1 = (float*)ar.take(b * 256 * 4);
  m.dz1 = (float*)ar.take(b * 256 * 4);
  m.row_err = (double*)ar.take(b * 8);
  m.row_cnt = (double*)ar.take(b * 8);
  m.loss = (double*)ar.take(16);
  return ar.short_ ? PAULI_EWORKSPACE : PAULI_OK;
}

// forward pass into the buffers
int mlp_forward_bufs(hipStream_t stream, const pauli_mlp* net, const float* x, int64_t B,
                     MlpBufs& m) {
  using namespace mlp;
  const uint16_t* P = net->params_bf16;
  const float* Pf = net->params;
  LAUNCH("k_to_bf16", k_to_bf16, (B * NIN + 255) / 256, 256, x, m.xb, B * NIN);
  // Z1 = X W1^T + b1, Y1 = GELU(Z1)
  TRY(gemm_launch(stream, m.xb, NIN, 0, P + OFF_W1, NIN, 1, m.z1, m.y1b, NHID, Pf + OFF_B1,
                  (int)B, NHID, NIN, EP_BIAS_GELU));
  TRY(gemm_launch(stream, m.y1b, NHID, 0, P + OFF_W2, NHID, 1, m.z2, m.y2b, NHID, Pf + OFF_B2,
                  (int)B, NHID, NHID, EP_BIAS_GELU));
  TRY(gemm_launch(stream, m.y2b, NHID, 0, P + OFF_W3, NHID, 1, m.yh, nullptr, NOUT, Pf + OFF_B3,
                  (int)B, NOUT, NHID, EP_BIAS));
  return PAULI_OK;
}
}  // namespace

int pauli_mlp_forward(const pauli_mlp* net, const float* x, int64_t B, float* y, pauli_ws* ws,
                      void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!ws || !x || !y || B <= 0 || B % 32) return PAULI_EINVAL;
  TRY(mlp_check(net));
  Arena ar = make_arena(ws);
  MlpBufs m;
  if (mlp_bufs(ar, B, m) != PAULI_OK) return ws_short(ar, ws);
  TRY(mlp_forward_bufs(stream, net, x, B, m));
  HIP_TRY(hipMemcpyAsync(y, m.yh, (size_t)B * mlp::NOUT * 4, hipMemcpyDeviceToDevice, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

int pauli_mlp_loss_grad(const pauli_mlp* net, const float* x, const float* t, const float* mask,
                        int64_t B, double* loss, float* acts, pauli_ws* ws, void* stream_) {
  using namespace mlp;
  hipStream_t stream = (hipStream_t)stream_;
  if (!ws || !x || !t || !mask || B <= 0 || B % 32) return PAULI_EINVAL;
  TRY(mlp_check(net));
  if (!net->grads) return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  MlpBufs m;
  if (mlp_bufs(ar, B, m) != PAULI_OK) return ws_short(ar, ws);
  TRY(mlp_forward_bufs(stream, net, x, B, m));
  const uint16_t* P = net->params_bf16;
  float* G = net->grads;
  const int64_t nb = (B + 255) / 256;
  LAUNCH("k_mse_rows", k_mse_rows, nb, 256, m.yh, t, mask, B, m.row_err, m.row_cnt);
  LAUNCH("k_sum_rows", k_sum_rows, 1, 256, m.row_err, m.row_cnt, B, m.loss);
  LAUNCH("k_mse_grad", k_mse_grad, (B * NOUT + 255) / 256, 256, m.yh, t, mask, B * NOUT, m.loss,
         m.dy, m.dyb);
  // layer 3: dW3[16][256] = dY^T Y2, db3 = column sums of dY, dY2 = dY W3
  TRY(gemm_launch(stream, m.dyb, NOUT, 1, m.y2b, NHID, 0, G + OFF_W3, nullptr, NHID, nullptr,
                  NOUT, NHID, (int)B, EP_STORE));
  LAUNCH("k_col_sum", k_col_sum, 1, 256, m.dy, B, NOUT, G + OFF_B3);
  TRY(gemm_launch(stream, m.dyb, NOUT, 0, P + OFF_W3, NHID, 0, m.dy2, nullptr, NHID, nullptr,
                  (int)B, NHID, NOUT, EP_STORE));
  LAUNCH("k_gelu_back", k_gelu_back, (B * NHID + 255) / 256, 256, m.dy2, m.z2, B * NHID, m.dz2,
         m.dz2b);
  // layer 2
  TRY(gemm_launch(stream, m.dz2b, NHID, 1, m.y1b, NHID, 0, G + OFF_W2, nullptr, NHID, nullptr,
                  NHID, NHID, (int)B, EP_STORE));
  LAUNCH("k_col_sum", k_col_sum, 1, 256, m.dz2, B, NHID, G + OFF_B2);
  TRY(gemm_launch(stream, m.dz2b, NHID, 0, P + OFF_W2, NHID, 0, m.dy1, nullptr, NHID, nullptr,
                  (int)B, NHID, NHID, EP_STORE));
  LAUNCH("k_gelu_back", k_gelu_back, (B * NHID + 255) / 256, 256, m.dy1, m.z1, B * NHID, m.dz1,
         m.dz1b);
  // layer 1
  TRY(gemm_launch(stream, m.dz1b, NHID, 1, m.xb, NIN, 0, G + OFF_W1, nullptr, NIN, nullptr, NHID,
                  NIN, (int)B, EP_STORE));
  LAUNCH("k_col_sum", k_col_sum, 1, 256, m.dz1, B, NHID, G + OFF_B1);
  if (acts) {
    float* o = acts;
    auto bf = [&](const uint16_t* src, int64_t n) -> int {
      LAUNCH("k_bf_to_f", k_bf_to_f, (n + 255) / 256, 256, src, o, n);
      o += n;
      return PAULI_OK;
    };
    auto fc = [&](const float* src, int64_t n) -> int {
      HIP_TRY(hipMemcpyAsync(o, src, (size_t)n * 4, hipMemcpyDeviceToDevice, stream));
      o += n;
      return PAULI_OK;
    };
    TRY(bf(m.xb, B * NIN));
    TRY(fc(m.z1, B * NHID));
    TRY(bf(m.y1b, B * NHID));
    TRY(fc(m.z2, B * NHID));
    TRY(bf(m.y2b, B * NHID));
    TRY(fc(m.yh, B * NOUT));
    TRY(bf(m.dyb, B * NOUT));
    TRY(fc(m.dy2, B * NHID));
    TRY(bf(m.dz2b, B * NHID));
    TRY(fc(m.dy1, B * NHID));
    TRY(bf(m.dz1b, B * NHID));
  }
  double h[2];
  HIP_TRY(hipMemcpyAsync(h, m.loss, 16, hipMemcpyDeviceToHost, stream));
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  if (loss) *loss = h[0];
  return PAULI_OK;
}

int pauli_mlp_train(const pauli_mlp* net, const float* x, const float* t, const float* mask,
                    int64_t n, const int32_t* order, int64_t epochs, int32_t batch, double lr,
                    double b1, double b2, double eps, int64_t t0, double* losses, pauli_ws* ws,
                    void* stream_) {
  using namespace mlp;
  hipStream_t stream = (hipStream_t)stream_;
  TRY(mlp_check(net));
  if (!ws || !x || !t || !mask || !order || !losses || n <= 0 || epochs < 0 || batch <= 0 ||
      batch > 4096 || t0 < 0 || !net->grads || !net->adam_m || !net->adam_v)
    return PAULI_EINVAL;
  Arena ar = make_arena(ws);
  // a minibatch's activations, in the room of one gradient share per SR rows
  const int nblk_max = (batch + SR - 1) / SR;
  char* part = (char*)ar.take((size_t)nblk_max * NPARAM * 4);
  ar.take((size_t)nblk_max * 16);
  if (ar.short_) return ws_short(ar, ws);
  static_assert(step_out_bytes(SR) + 16 * 256 <= NPARAM * 4, "the activations fit their room");
  // W2 transposed for the backward product, where the workspace has room for it
  uint16_t* w2t = (uint16_t*)ar.take((size_t)NHID * NHID * 2);
  if (w2t) LAUNCH("k_w2_transpose", k_w2_transpose, NHID * NHID / 256, 256, net->params_bf16, w2t);
  const int64_t spe = (n + batch - 1) / batch;  // minibatches per epoch
  int64_t step = t0;
  for (int64_t e = 0; e < epochs; e++) {
    for (int64_t k = 0; k < spe; k++) {
      const int64_t s0 = k * batch;
      const int rows = (int)std::min<int64_t>(batch, n - s0);
      const int nblk = (rows + SR - 1) / SR;
      StepOut so;
      so.Bp = nblk * SR;
      Arena room;
      room.base = part;
      room.cap = (size_t)nblk_max * NPARAM * 4;
      const size_t Bp = (size_t)so.Bp;
      so.x = (uint16_t*)room.take(Bp * NIN * 2);
      so.y1 = (uint16_t*)room.take(Bp * NHID * 2);
      so.y2 = (uint16_t*)room.take(Bp * NHID * 2);
      so.dz1 = (uint16_t*)room.take(Bp * NHID * 2);
      so.dz2 = (uint16_t*)room.take(Bp * NHID * 2);
      so.dy = (uint16_t*)room.take(Bp * NOUT * 2);
      so.fz1 = (float*)room.take(Bp * NHID * 4);
      so.fz2 = (float*)room.take(Bp * NHID * 4);
      so.fy = (float*)room.take(Bp * NOUT * 4);
      so.err = (double*)room.take(Bp * NOUT * 8);
      so.cnt = (double*)room.take(8);
      StepArgs sa;
      sa.params = net->params;
      sa.pb = net->params_bf16;
      sa.w2t = w2t;
      sa.X = x;
      sa.T = t;
      sa.Mk = mask;
      sa.order = order + e * n + s0;
      sa.rows = rows;
      sa.o = so;
      if ((uintptr_t)net->params_bf16 % 16 == 0)
        LAUNCH("k_mlp_step", k_mlp_step<true>, so.Bp / SB, STEP_THREADS, sa);
      else
        LAUNCH("k_mlp_step", k_mlp_step<false>, so.Bp / SB, STEP_THREADS, sa);
      step++;
      GradArgs ga;
      ga.o = so;
      ga.grads = net->grads;
      ga.p = net->params;
      ga.m = net->adam_m;
      ga.v = net->adam_v;
      ga.pb = net->params_bf16;
      ga.w2t = w2t;
      ga.lr = (float)lr;
      ga.b1 = (float)b1;
      ga.omb1 = (float)(1.0 - b1);
      ga.b2 = (float)b2;
      ga.omb2 = (float)(1.0 - b2);
      ga.eps = (float)eps;
      ga.c1 = (float)(1.0 - std::pow(b1, (double)step));
      ga.c2 = (float)(1.0 - std::pow(b2, (double)step));
      ga.loss = losses + e * spe + k;
      LAUNCH("k_mlp_grad_adam", k_mlp_grad_adam, GRAD_BLOCKS, 64, ga);
    }
  }
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

int pauli_mlp_adam(const pauli_mlp* net, double lr, double b1, double b2, double eps, int64_t t,
                   void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  TRY(mlp_check(net));
  if (!net->grads || !net->adam_m || !net->adam_v || t < 1) return PAULI_EINVAL;
  const float c1 = (float)(1.0 - std::pow(b1, (double)t));
  const float c2 = (float)(1.0 - std::pow(b2, (double)t));
  LAUNCH("k_adam", mlp::k_adam, (mlp::NPARAM + 255) / 256, 256, net->params, net->grads,
         net->adam_m, net->adam_v, net->params_bf16, mlp::NPARAM, (float)lr, (float)b1,
         (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)eps, c1, c2);
  HIP_TRY(hipStreamSynchronize(stream));
  g_prof.resolve();
  return PAULI_OK;
}

}  // extern "C"
