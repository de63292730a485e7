// Host runtime of libtrioseq: validation, 2-bit packing, planning (axis
// choice, longest-first ordering, workspace sizing), launches, hipGraph
// replay, and the synchronous single/batch entry points.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "common.h"

namespace trioseq {

static thread_local std::string g_err;

trioseq_status fail(trioseq_status st, const std::string& msg) {
  g_err = msg;
  return st;
}

trioseq_status fail_hip(hipError_t e, const char* what) {
  if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation)
    return fail(TRIOSEQ_ERR_NOMEM, std::string(what) + ": " + hipGetErrorString(e));
  return fail(TRIOSEQ_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

static const uint8_t* build_code_table() {
  static uint8_t t[256];
  std::memset(t, 255, sizeof t);
  const char* up = "ACGT";
  const char* lo = "acgt";
  for (int c = 0; c < 4; ++c) {
    t[(uint8_t)up[c]] = (uint8_t)c;
    t[(uint8_t)lo[c]] = (uint8_t)c;
  }
  return t;
}
static const uint8_t* g_code = build_code_table();

uint8_t residue_code(char ch) { return g_code[(uint8_t)ch]; }

uint64_t now_ns() {
  return (uint64_t)std::chrono::duration_cast<std::chrono::nanoseconds>(
             std::chrono::steady_clock::now().time_since_epoch())
      .count();
}

trioseq_status validate_scoring(const trioseq_scoring* sc) {
  if (!sc) return fail(TRIOSEQ_ERR_INVALID_ARG, "scoring is NULL");
  if (sc->kind != kGlobal && sc->kind != kSemiGlobal && sc->kind != kLocal)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "scoring kind must be global, semi-global or local");
  // The semi-global and local kernels rely on M' = M - 2*gap*(i+j+k) >= 0
  // for their axis values and floors.
  if (sc->kind != kGlobal && sc->gap > 0)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "semi-global and local scoring need gap <= 0");
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y) {
      if (sc->sub[x][y] != sc->sub[y][x])
        return fail(TRIOSEQ_ERR_INVALID_ARG, "substitution matrix is not symmetric");
      const int64_t term = (int64_t)sc->sub[x][y] - 2 * (int64_t)sc->gap;
      if (term < -127 || term > 127)
        return fail(TRIOSEQ_ERR_INVALID_ARG,
                    "sub[x][y] - 2*gap must lie in [-127, 127] for every pair");
    }
  return TRIOSEQ_OK;
}

trioseq_status check_range(const trioseq_scoring& sc, uint64_t a, uint64_t b, uint64_t c,
                           size_t index) {
  const uint64_t d = a + b + c;
  int64_t maxterm = 0;
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y)
      maxterm = std::max<int64_t>(maxterm, (int64_t)sc.sub[x][y] - 2 * (int64_t)sc.gap);
  // Shifted scores lie in [0, d * maxterm]; the true score adds 2*gap*d.
  // Semi-global axes and local floors put cells at M' = -2*gap*(i+j+k).
  if (sc.kind != kGlobal) maxterm = std::max<int64_t>(maxterm, -2 * (int64_t)sc.gap);
  const long double hi = (long double)d * (long double)maxterm;
  const long double shift = (long double)d * 2.0L * (long double)sc.gap;
  if (hi >= (long double)(1 << 27) || shift >= (long double)(1 << 30) ||
      shift <= -(long double)(1 << 30))
    return fail(TRIOSEQ_ERR_OVERFLOW,
                "triplet " + std::to_string(index) + ": score range exceeds int32 headroom");
  return TRIOSEQ_OK;
}

DevScoring make_dev_scoring(const trioseq_scoring& sc) {
  DevScoring d;
  for (int r = 0; r < 4; ++r) {
    uint32_t w = 0;
    for (int x = 0; x < 4; ++x) {
      const int v = sc.sub[x][r] - 2 * sc.gap;
      w |= (uint32_t)(uint8_t)(int8_t)v << (8 * x);
    }
    d.byte_tab[r] = w;
  }
  d.byte_tab[4] = 0x80808080u;
  for (int r = 0; r < 4; ++r)
    for (int s = 0; s < 4; ++s) d.pair_tab[4 * r + s] = sc.sub[r][s] - 2 * sc.gap;
  d.gap2 = 2 * sc.gap;
  d.kind = sc.kind;
  return d;
}

// When the plan picks engines itself, a triplet is split into panel jobs if
// sweeping it whole on one wavefront would hold the launch up: it is alone,
// it has at least kSplitCells cells (one wave takes ~0.1 s on 2.5e8 cells),
// or more than kSplitFactor times the batch's mean cells per wavefront.
const double kSplitCells = 2.5e8;
const double kSplitFactor = 4.0;

uint64_t panel_steps(const uint32_t l[3], const KernelShape& ks) {
  const uint64_t pj = l[1] / (uint32_t)panel_rows(ks) + 1;
  const uint64_t pk = l[2] / (uint32_t)panel_cols(ks) + 1;
  return pj * pk * (uint64_t)(l[0] + 1 + kSkew);
}

static const uint8_t kPerms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};

AxisChoice choose_axes_batch(const uint32_t len[3], const KernelShape& ks) {
  AxisChoice best{{0, 1, 2}};
  uint64_t best_cost = UINT64_MAX;
  for (const auto& p : kPerms) {
    const uint32_t l[3] = {len[p[0]], len[p[1]], len[p[2]]};
    if (l[0] > (uint32_t)kMaxSweepLen) continue;
    const uint64_t cost = panel_steps(l, ks);
    if (cost < best_cost) {
      best_cost = cost;
      std::memcpy(best.perm, p, 3);
    }
  }
  return best;
}

AxisChoice choose_axes_wide(const uint32_t len[3]) {
  // Sweep the longest sequence that fits the LDS residue buffer: the fill of
  // the panel pipeline is paid once per sweep, so a long sweep amortises it.
  AxisChoice best{{0, 1, 2}};
  int64_t best_len = -1;
  for (const auto& p : kPerms) {
    if (len[p[0]] > (uint32_t)kMaxSweepLen) continue;
    const int64_t key = (int64_t)len[p[0]] * 4 + (len[p[1]] >= len[p[2]] ? 1 : 0);
    if (key > best_len) {
      best_len = key;
      std::memcpy(best.perm, p, 3);
    }
  }
  return best;
}

uint64_t boundary_ints(const KernelShape& ks, uint32_t max_n0) {
  const uint64_t rows = face_rows(max_n0);
  return 3 * (2 * rows * panel_cols(ks) + rows * right_face_row(ks));  // plain + tagged
}

Boundary carve_boundary(const KernelShape& ks, uint32_t max_n0, int* q) {
  const uint64_t rows = face_rows(max_n0);
  const uint64_t top = rows * panel_cols(ks), left = rows * right_face_row(ks);
  Boundary b;
  b.plain[0] = q;
  b.plain[1] = q + top;
  b.plain[2] = q + 2 * top;
  q += 2 * top + left;
  b.tagged[0] = q;
  b.tagged[1] = q + 2 * top;
  b.tagged[2] = q + 4 * top;
  b.rows = (uint32_t)rows;
  return b;
}

SweepArgs make_sweep_args(const uint32_t* words, const TripletDesc* desc, const JobDesc* jobs,
                          uint32_t njobs, uint32_t lds_n0, int32_t* scores, int* counter, int* ctl,
                          int* face, uint64_t face_stride, int* pface, const Boundary& bnd,
                          int* red, const DevScoring& sc) {
  SweepArgs a;
  a.words = words;
  a.desc = desc;
  a.jobs = jobs;
  a.njobs = njobs;
  a.lds_n0 = lds_n0;
  a.scores = scores;
  a.counter = counter;
  a.ctl = ctl;
  a.face = face;
  a.face_stride = face_stride;
  a.pface = pface;
  for (int k = 0; k < 3; ++k) {
    a.bnd_plain[k] = bnd.plain[k];
    a.bnd_tagged[k] = bnd.tagged[k];
  }
  a.red = red;
  a.plane = nullptr;
  a.plane_off = nullptr;
  a.wait_ticks = wait_limit_ticks();
  a.sc = sc;
  return a;
}

// 2 s in ticks of the 100 MHz wall clock the kernels read.
constexpr uint64_t kDefaultWaitTicks = 200000000ull;
static std::atomic<uint64_t> g_wait_ticks{kDefaultWaitTicks};

uint64_t wait_limit_ticks() { return g_wait_ticks.load(std::memory_order_relaxed); }

// A private non-blocking stream per thread and device for the one-off work
// of plan creation (clearing control words and face pools, uploading the job
// tables, writing sentinel faces). Waiting for it stalls nothing else: no
// caller stream and no other thread's work is synchronised. Never destroyed
// (the HIP runtime may be gone at thread exit).
hipError_t init_stream(int device, hipStream_t* out) {
  static thread_local std::vector<hipStream_t>* streams = nullptr;
  if (!streams) streams = new std::vector<hipStream_t>;
  if ((int)streams->size() <= device) streams->resize(device + 1, nullptr);
  hipStream_t& st = (*streams)[device];
  if (!st) {
    hipError_t e = hipStreamCreateWithFlags(&st, hipStreamNonBlocking);
    if (e != hipSuccess) {
      st = nullptr;
      return e;
    }
  }
  *out = st;
  return hipSuccess;
}

trioseq_status device_props(DeviceProps* p) {
  TRIOSEQ_HIP(hipGetDevice(&p->device), "hipGetDevice");
  TRIOSEQ_HIP(hipDeviceGetAttribute(&p->cus, hipDeviceAttributeMultiprocessorCount, p->device),
              "hipDeviceGetAttribute");
  size_t fr = 0, tot = 0;
  TRIOSEQ_HIP(hipMemGetInfo(&fr, &tot), "hipMemGetInfo");
  p->hbm_bytes = tot;
  return TRIOSEQ_OK;
}

}  // namespace trioseq

using namespace trioseq;

struct trioseq_plan {
  int device = 0;
  size_t n = 0;
  int engine = 0;  // 0: all triplets whole, 1: all split into panel jobs, 2: mixed
  int modes = 1;   // kernel variant: bit 0 whole-triplet jobs, bit 1 panel jobs
  KernelShape ks{4, 4, 4};
  int grid = 0, waves_per_cu = 0, panels = 0;
  uint32_t njobs = 0, lds_n0 = 0;
  DevScoring sc{};
  double cells = 0;
  uint64_t workspace_bytes = 0;
  TripletDesc* d_desc = nullptr;
  JobDesc* d_jobs = nullptr;
  int* d_counter = nullptr;  // job queue head
  int* d_ctl = nullptr;      // [0] generation, [1] error flag, [2] meeting counter (0 between runs), [3] highest tag
  int* d_face = nullptr;     // per-wave workspace of whole-triplet jobs
  uint64_t face_stride = 0;
  int* d_pface = nullptr;    // panel-face pool of split triplets
  uint64_t pool_ints = 0;    // its size (a borrowed plan's: the whole region's)
  int* d_bnd = nullptr;      // sentinel faces
  Boundary bnd{};
  int* d_red = nullptr;      // per-triplet reduction pairs (semi-global, local)
  uint32_t red_pairs = 0;
  // Half-split scoring of a lone triplet (see half_split_layout).
  bool half = false;
  uint32_t h_words_n = 0, h_nchunk = 0;
  uint32_t* d_hwords = nullptr;     // the two halves' sequences, gathered every run
  GatherDesc* d_gather = nullptr;   // 6 gather descriptors
  int* d_plane = nullptr;           // the two last-slice planes
  uint64_t* d_plane_off = nullptr;  // {0, plane ints}
  SplitDesc* d_sdesc = nullptr;     // the meeting boxes, the box of every chunk and a
  uint32_t* d_chunk_box = nullptr;  // counter each (null for one box, which uses d_ctl[2])
  int* d_meet = nullptr;
  int* d_partial = nullptr;         // per chunk: its best
  int32_t* d_hscores = nullptr;     // the halves' own scores (unused)
  // graph replay
  bool use_graph = false;
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  const uint32_t* g_words = nullptr;
  int32_t* g_scores = nullptr;
  // Device buffers carved from a caller's region (not owned).
  bool borrowed = false;
  // Packed pairs: sentinel faces (top, left) and the stored value of M' = 0.
  bool packed = false;
  uint32_t pk_base = 0, pk_kc = 0;
  bool pk_self = false;
  bool pk_reuse = false;
  int tag_step = 1;
  int* d_pkbnd = nullptr;
  uint64_t pk_top_words = 0;
};

static void plan_free(trioseq_plan* p) {
  if (!p) return;
  if (p->gexec) (void)hipGraphExecDestroy(p->gexec);
  if (p->graph) (void)hipGraphDestroy(p->graph);
  if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
  if (p->borrowed) {
    // Carved from a caller's region: nothing to free on the device.
    delete p;
    return;
  }
  (void)hipFree(p->d_desc);
  (void)hipFree(p->d_jobs);
  (void)hipFree(p->d_counter);
  (void)hipFree(p->d_ctl);
  (void)hipFree(p->d_face);
  (void)hipFree(p->d_pface);
  (void)hipFree(p->d_bnd);
  (void)hipFree(p->d_red);
  (void)hipFree(p->d_pkbnd);
  for (void* q : {(void*)p->d_hwords, (void*)p->d_gather, (void*)p->d_plane, (void*)p->d_plane_off,
                  (void*)p->d_sdesc, (void*)p->d_partial, (void*)p->d_hscores, (void*)p->d_chunk_box, (void*)p->d_meet})
    (void)hipFree(q);
  delete p;
}

extern "C" {

void trioseq_scoring_simple(trioseq_scoring* s, int32_t match, int32_t mismatch, int32_t gap) {
  if (!s) return;
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y) s->sub[x][y] = x == y ? match : mismatch;
  s->gap = gap;
  s->kind = TRIOSEQ_GLOBAL;
}

const char* trioseq_last_error(void) { return g_err.c_str(); }

const char* trioseq_version(void) { return "trioseq-mi355x 0.2 (gfx950)"; }

void trioseq_set_wait_limit(uint64_t ns) {
  g_wait_ticks.store(ns ? ns / 10 : kDefaultWaitTicks, std::memory_order_relaxed);
}

trioseq_status trioseq_pack(const char* seq, uint32_t len, uint32_t* words) {
  if (len && (!seq || !words)) return fail(TRIOSEQ_ERR_INVALID_ARG, "pack: NULL pointer");
  const uint8_t* in = (const uint8_t*)seq;
  // Validate first (codes of A, C, G, T are 0..3, anything else has a
  // higher bit set), so an error leaves the words untouched.
  uint32_t bad = 0;
  for (uint32_t p = 0; p < len; ++p) bad |= g_code[in[p]];
  if (bad > 3) {
    uint32_t p = 0;
    while (g_code[in[p]] <= 3) ++p;
    return fail(TRIOSEQ_ERR_BAD_RESIDUE, "pack: character at position " + std::to_string(p) + " is not ACGT");
  }
  const uint32_t full = len / 16;
  for (uint32_t w = 0; w < full; ++w) {
    const uint8_t* r = in + 16 * (size_t)w;
    uint32_t v = 0;
    for (int q = 0; q < 16; ++q) v |= (uint32_t)g_code[r[q]] << (2 * q);
    words[w] = v;
  }
  if (len % 16) {
    uint32_t v = 0;
    for (uint32_t q = 0; q < len % 16; ++q) v |= (uint32_t)g_code[in[16 * (size_t)full + q]] << (2 * q);
    words[full] = v;
  }
  return TRIOSEQ_OK;
}

trioseq_status trioseq_packed_layout(const uint32_t* lens, size_t n, uint64_t* word_off,
                                     uint64_t* total_words) {
  if ((n && (!lens || !word_off)) || !total_words)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "packed_layout: NULL pointer");
  uint64_t acc = 0;
  for (size_t q = 0; q < 3 * n; ++q) {
    word_off[q] = acc;
    acc += (lens[q] + 15u) / 16u;
  }
  *total_words = acc;
  return TRIOSEQ_OK;
}

}  // extern "C"

namespace trioseq {

// 0 .. n - 1 in ascending order of their keys (equal keys in index order): by
// comparison for a few, else byte by byte from the last, leaving out the bytes
// that all keys share (20000 triplets of 8-31 residues: a plan's three sorts 0.6
// ms, 11 ms when they compared descriptors through the indices).
struct SortKey {
  uint64_t w[3];
};
template <class F>
static std::vector<uint32_t> sorted_by(size_t n, F key) {
  std::vector<SortKey> k(n);
  std::vector<uint32_t> idx(n), to(n);
  for (size_t t = 0; t < n; ++t) k[t] = key(t);
  std::iota(idx.begin(), idx.end(), 0u);
  if (n < 256) {
    std::stable_sort(idx.begin(), idx.end(), [&](uint32_t x, uint32_t y) {
      return std::lexicographical_compare(k[x].w, k[x].w + 3, k[y].w, k[y].w + 3);
    });
    return idx;
  }
  for (int w = 2; w >= 0; --w) {
    uint64_t differ = 0;
    for (const SortKey& x : k) differ |= x.w[w] ^ k[0].w[w];
    for (int shift = 0; shift < 64; shift += 8) {
      if (!((differ >> shift) & 255u)) continue;
      size_t at[257] = {0};
      for (const SortKey& x : k) ++at[1 + ((x.w[w] >> shift) & 255u)];
      for (int v = 0; v < 255; ++v) at[v + 1] += at[v];
      for (uint32_t t : idx) to[at[(k[t].w[w] >> shift) & 255u]++] = t;
      idx.swap(to);
    }
  }
  return idx;
}

// Packed pairs (two triplets per lane, one 16-bit half each): the batch's
// whole triplets, sorted by their axis lengths, are paired neighbour with
// neighbour (a lone last one with itself) and each pair is one job over the
// common panel grid. Qualifies when the scoring is global, every
// substitution term sub - 2*gap is >= 0, and every value a lane can hold
// stays within [kPackedSentinel, kPackedMax]: values outside the tensor
// start at kPackedSentinel and grow by at most maxA per residue along the
// fill region (kSkew slices plus the padded panel box), M' = 0 is stored as
// base above all of them, and base + maxA * (the longest path of the padded
// box, drain included) must not pass kPackedMax.
static bool pair_up(Layout* L, const trioseq_scoring& sc, const KernelShape& ks) {
  const size_t n = L->desc.size();
  if (L->modes != 1 || L->planes || n < 2) return false;
  int mina = INT32_MAX, maxa = INT32_MIN;
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y) {
      mina = std::min(mina, sc.sub[x][y] - 2 * sc.gap);
      maxa = std::max(maxa, sc.sub[x][y] - 2 * sc.gap);
    }
  if (mina < 0 || maxa > 255 || !pk_shape_supported(ks, sc.kind)) return false;
  const int H = panel_rows(ks), W = panel_cols(ks), RR = (int)right_face_row(ks);
  const size_t np = (n + 1) / 2;
  // A pair costs the panels of its common grid times its steps. Neighbours
  // in two sort orders are paired, and the cheaper pairing is kept: by the
  // lengths (similar sweep lengths), or by the panel counts of the other two
  // axes first (no pair crosses a panel boundary the two do not share).
  auto pair_cost = [&](const TripletDesc& a, const TripletDesc& b) {
    const uint64_t n0 = std::max(a.len[0], b.len[0]);
    const uint64_t PJ = std::max(a.len[1], b.len[1]) / H + 1, PK = std::max(a.len[2], b.len[2]) / W + 1;
    return PJ * PK * (n0 + 1 + kSkew);
  };
  auto total_cost = [&](const std::vector<uint32_t>& v) {
    uint64_t c = 0;
    for (size_t q = 0; q < np; ++q) c += pair_cost(L->desc[v[2 * q]], L->desc[v[std::min(2 * q + 1, n - 1)]]);
    return c;
  };
  const std::vector<TripletDesc>& in = L->desc;
  const std::vector<uint32_t> by_len = sorted_by(n, [&](size_t t) {
    return SortKey{{in[t].len[0], in[t].len[1], in[t].len[2]}};
  });
  const std::vector<uint32_t> by_panels = sorted_by(n, [&](size_t t) {
    return SortKey{{(uint64_t)(in[t].len[1] / H) << 32 | in[t].len[2] / W, in[t].len[0],
                    (uint64_t)in[t].len[1] << 32 | in[t].len[2]}};
  });
  const std::vector<uint32_t>& idx = total_cost(by_panels) < total_cost(by_len) ? by_panels : by_len;
  uint64_t box_jk = 0, n0max = 0, stride = 0;
  std::vector<uint64_t> cost(np);
  for (size_t q = 0; q < np; ++q) {
    const TripletDesc& a = L->desc[idx[2 * q]];
    const TripletDesc& b = L->desc[idx[std::min(2 * q + 1, n - 1)]];
    const uint32_t n0 = std::max(a.len[0], b.len[0]), n1 = std::max(a.len[1], b.len[1]),
                   n2 = std::max(a.len[2], b.len[2]);
    const uint64_t PJ = n1 / H + 1, PK = n2 / W + 1, rows = face_rows(n0);
    box_jk = std::max(box_jk, PJ * H + PK * W);
    n0max = std::max<uint64_t>(n0max, n0);
    stride = std::max(stride, rows * (PK * W + RR));
    cost[q] = pair_cost(a, b);
  }
  // Real values: base + M' with M' <= mx per unit of index sum (a move adds
  // at most one term per residue it consumes; the local floor and the
  // semi-global axes add g = -2*gap per unit), over the padded box and the
  // drain steps. Semi-global candidates M + kc need kc above g times every
  // index sum and must stay within 16 bits (see sweep.hip).
  const uint64_t g = sc.kind == kGlobal ? 0 : (uint64_t)(-2 * sc.gap);  // gap <= 0 for the others
  const uint64_t mx = sc.kind == kGlobal ? (uint64_t)maxa : std::max<uint64_t>(maxa, g);
  const uint64_t base = kPackedSentinel + 512 + (uint64_t)maxa * (kSkew + box_jk);
  if (base + mx * (n0max + kSkew + kChunk + box_jk) > kPackedMax) return false;
  uint64_t kc = 0;
  if (sc.kind == kSemiGlobal) {
    kc = g * (n0max + box_jk) + 1;
    if (kPackedMax - base + kc > 0xFFFF) return false;
  }
  std::vector<TripletDesc> desc(2 * np);
  for (size_t q = 0; q < np; ++q) {
    desc[2 * q] = L->desc[idx[2 * q]];
    desc[2 * q + 1] = L->desc[idx[std::min(2 * q + 1, n - 1)]];
  }
  const std::vector<uint32_t> order = sorted_by(np, [&](size_t q) { return SortKey{{~cost[q], 0, 0}}; });
  L->jobs.clear();
  for (size_t q : order) L->jobs.push_back(JobDesc{(uint32_t)(2 * q), kWholeTriplet});
  L->desc.swap(desc);
  L->ks = ks;
  L->packed = true;
  L->pk_base = (uint32_t)base;
  L->pk_kc = (uint32_t)kc;
  L->face_stride = (stride + 63) / 64 * 64;
  L->lds_n0 = (uint32_t)n0max;
  return true;
}

// Estimated times of the panel jobs of packed pairs (see panel_jobs).
struct PkTime {
  double steps = 0, chain = 0;
  void add(uint32_t n0, uint32_t n1, uint32_t n2) {
    const double slices = n0 + 1 + kSkew, PJ = n1 / kPkPanel + 1, PK = n2 / kPkPanel + 1;
    steps += PJ * PK * (slices + 12);  // (a panel's start costs about 12 steps)
    chain = std::max(chain, slices + 21 * (PJ + PK));
  }
  // 256 compute units: 2048 single waves, 1024 wave pairs.
  double single_us() const {
    const double s = steps / 2048 * 0.66, c = chain * 24 / 21 * 0.4;
    return std::max(s, c) + 0.4 * std::min(s, c);
  }
  double wave_pair_us() const {
    const double s = steps / 1024 * 0.385, c = chain * 0.4;
    return std::max(s, c) + 0.25 * std::min(s, c);
  }
};
static PkTime pk_panel_time(const std::vector<TripletDesc>& desc) {
  PkTime t;
  for (size_t p = 0; p + 1 < desc.size(); p += 2) {
    const TripletDesc &a = desc[p], &b = desc[p + 1];
    t.add(std::max(a.len[0], b.len[0]), std::max(a.len[1], b.len[1]), std::max(a.len[2], b.len[2]));
  }
  return t;
}

// What a pair must keep to for its panels to run packed (the reasons are in
// packed_panel.hip). With every term >= 0, M' grows by at most `step` per unit
// of an index, so a panel's window is step * (slices + rows + columns); off
// puts the panel's base above every value from outside the tensor. A cell's M'
// itself is recovered from 16 bits where it leaves the panel (score, plane), so
// it must stay below 2^16: at most maxA per residue pair that two sequences can
// form, or per residue with the semi-global axes and local floors.
struct PanelValues {
  uint64_t off, kc;  // stored value of a panel's base, offset of semi-global candidates
};
static bool panel_values(const std::vector<TripletDesc>& desc, const trioseq_scoring& sc, bool planes, PanelValues* v) {
  int mina = INT32_MAX, maxa = 0, maxs = 0;
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y) {
      mina = std::min(mina, sc.sub[x][y] - 2 * sc.gap);
      maxa = std::max(maxa, sc.sub[x][y] - 2 * sc.gap);
      maxs = std::max(maxs, sc.sub[x][y]);
    }
  if (desc.empty() || desc.size() % 2 || mina < 0) return false;
  const uint64_t A = (uint64_t)maxa, g = sc.kind == kGlobal ? 0 : (uint64_t)(-2 * sc.gap);
  const uint64_t step = std::max(2 * A, g);
  // Outside values: kPackedSentinel plus the terms of a path over the fill
  // region (kSkew slices) and the panel, and of one move more.
  const uint64_t off = kPackedSentinel + A * (kSkew + 2 * kPkPanel + 3) + step + 64;
  uint64_t kc = 0;
  for (const TripletDesc& d : desc) {
    const uint64_t a = d.len[0], b = d.len[1], c = d.len[2];
    const uint64_t pairs = std::min(a, b) + std::min(a, c) + std::min(b, c);
    // (Where every term is 0 nothing but the kernels' own limit bounds the sweep.)
    if (a > (uint64_t)kMaxSweepLen) return false;
    if (off + step * (a + 2 * kPkPanel + 2) > kPackedMax) return false;
    const uint64_t most = sc.kind == kGlobal ? A * pairs : std::max(A, g) * (a + b + c);
    const uint64_t score = (uint64_t)maxs * pairs;  // no score is larger
    // (Floors are told from live values by their distance, below 2^15.)
    const bool floors = sc.kind == kLocal || (sc.kind == kSemiGlobal && planes);
    if (most > 0xFFFF || (floors && score > 30000)) return false;
  }
  // Semi-global candidates M + kc must be positive on every cell of a pair's
  // common panel grid: a triplet's last slice is taken with its padding.
  if (sc.kind == kSemiGlobal)
    for (size_t p = 0; p + 1 < desc.size(); p += 2) {
      const TripletDesc &a = desc[p], &b = desc[p + 1];
      uint64_t sum = std::max(a.len[0], b.len[0]);
      for (int k = 1; k < 3; ++k) sum += (uint64_t)(std::max(a.len[k], b.len[k]) / kPkPanel + 1) * kPkPanel;
      kc = std::max(kc, g * sum + 1);
    }
  for (const TripletDesc& d : desc)
    if (sc.kind == kSemiGlobal &&
        kc + (uint64_t)maxs * (std::min(d.len[0], d.len[1]) + std::min(d.len[0], d.len[2]) + std::min(d.len[1], d.len[2])) >
            0xFFFF)
      return false;
  *v = PanelValues{off, kc};
  return true;
}

// Panels that a diagonal of a group of pairs has at least, on average.
constexpr double kPkWidth = 2048;

// The job queue and buffers of pairs whose values fit (panel_values).
static bool panel_jobs(std::vector<TripletDesc> desc, const trioseq_scoring& sc, bool planes, const PanelValues& v,
                       Layout* L) {
  const size_t np = desc.size() / 2;
  L->desc = std::move(desc);
  L->jobs.clear();
  std::vector<uint32_t> PJ(np), PK(np);
  std::vector<uint64_t> cost(np);
  uint64_t jobs = 0;
  uint32_t n0max = 0;
  double cells = 0;
  for (size_t p = 0; p < np; ++p) {
    TripletDesc &a = L->desc[2 * p], &b = L->desc[2 * p + 1];
    const uint32_t n0 = std::max(a.len[0], b.len[0]);
    PJ[p] = std::max(a.len[1], b.len[1]) / kPkPanel + 1;
    PK[p] = std::max(a.len[2], b.len[2]) / kPkPanel + 1;
    jobs += (uint64_t)PJ[p] * PK[p];
    cost[p] = (uint64_t)PJ[p] * PK[p] * (n0 + 1 + kSkew);
    n0max = std::max(n0max, n0);
    cells += (double)a.len[0] * a.len[1] * a.len[2] + (double)b.len[0] * b.len[1] * b.len[2];
  }
  if (jobs > (uint64_t)INT32_MAX / 2) return false;
  // In groups of pairs, by anti-diagonal across a group's pairs (the costlier
  // first): every panel comes after those it reads from, and a diagonal of a
  // group has about as many panels as single waves fit the device, so that the
  // panels of the next one rarely wait for them. (8192 triplets of 100-400
  // residues: 27.8 ms with 512 panels a diagonal, 26.7 with 2048 and with all
  // pairs in one group.) Two sets of face buffers serve the groups in turn: a
  // group's panels start when all jobs of the group two before are finished,
  // which is long before they are popped.
  const std::vector<uint32_t> idx = sorted_by(np, [&](size_t p) { return SortKey{{~cost[p], 0, 0}}; });
  L->jobs.reserve(jobs);
  uint64_t region[2] = {0, 0}, done[2] = {0, 0};  // per set: ints of buffers, jobs of its groups so far
  uint64_t tags = 0;
  uint32_t group = 0;
  std::vector<std::pair<size_t, size_t>> groups;
  for (size_t g0 = 0; g0 < np; ++group) {
    const size_t before = L->jobs.size();
    double width = 0;
    size_t g1 = g0;
    uint32_t gd = 0, longest = 0;
    uint64_t at = 0;
    while (g1 < np && width < kPkWidth) {
      const size_t p = idx[g1++];
      width += (double)PJ[p] * PK[p] / (PJ[p] + PK[p] - 1);
      gd = std::max(gd, PJ[p] + PK[p] - 1);
      longest = std::max({longest, PJ[p], PK[p]});
      TripletDesc &a = L->desc[2 * p], &b = L->desc[2 * p + 1];
      a.face_off = at;
      a.set = group & 1;
      a.after = (uint32_t)done[group & 1];
      a.tag0 = (uint32_t)tags;
      at += pk_pair_ints(std::max(a.len[0], b.len[0]), PJ[p], PK[p]);
    }
    for (uint32_t d = 0; d < gd; ++d)
      for (size_t q = g0; q < g1; ++q) {
        const size_t p = idx[q];
        if (d + 1 >= PJ[p] + PK[p]) continue;
        for (uint32_t pj = (d >= PK[p] ? d - PK[p] + 1 : 0); pj <= std::min(d, PJ[p] - 1); ++pj)
          L->jobs.push_back(JobDesc{(uint32_t)(2 * p), pj * PK[p] + (d - pj)});
      }
    region[group & 1] = std::max(region[group & 1], at);
    done[group & 1] += L->jobs.size() - before;
    tags += longest + 1;
    groups.emplace_back(g0, g1);
    g0 = g1;
  }
  for (size_t g = 1; g < groups.size(); g += 2)
    for (size_t q = groups[g].first; q < groups[g].second; ++q) L->desc[2 * idx[q]].face_off += region[0];
  if (tags + 2 > (1u << 24)) return false;
  const uint64_t pool = region[0] + region[1];
  L->pk_reuse = groups.size() > 2 && pool != 0;
  L->tag_step = (int)tags + 2;
  L->ks = KernelShape{4, 4, 2};
  L->kind = sc.kind;
  L->planes = planes;
  L->modes = kModePkPanel;
  L->engine = 1;
  L->panels = (int)(2 * jobs);
  L->lds_n0 = n0max;
  L->cells = cells;
  L->face_stride = 0;
  L->pool_ints = pool;
  L->packed = true;
  L->pk_base = (uint32_t)v.off;
  L->pk_kc = (uint32_t)v.kc;
  // Single-wave workgroups (two computing waves on a SIMD) or a computing and a
  // memory wave each (shorter hops from panel to panel): whichever the batch's
  // total work and its longest chain of panels make faster, at the steps both
  // were measured to take: 0.66 us a step of a single wave (two share a SIMD),
  // 0.385 us of a computing wave; a panel starts 24 or 21 steps after its
  // neighbour. Lone 1024 x 1000 x 1048: 0.82 ms single, 0.62 ms in pairs; 2560 x
  // 2500 x 2600: 3.49 and 3.48; 3072 x 3000 x 3120: 5.13 and 5.74; 4096 x 4000 x
  // 4150: 10.9 and 12.9.
  // Pairs of one panel each have no faces to move: single waves (halves of 1000
  // x 31 x 31: 191 us, 198 in wave pairs, 192 in int32 lanes; local 241, 253,
  // 248; 250 x 31 x 31: 75.5, 77.4, 75.0).
  const PkTime t = pk_panel_time(L->desc);
  L->pk_self = t.single_us() < t.wave_pair_us() || jobs == np;
  return true;
}

bool pair_panel_layout(const std::vector<TripletDesc>& desc, const trioseq_scoring& sc, bool planes, Layout* L) {
  PanelValues v;
  return panel_values(desc, sc, planes, &v) && panel_jobs(desc, sc, planes, v, L);
}

// The halved axis of a triplet (its longest) and the other two.
static void half_order(const uint32_t* l, int order[3]) {
  int ax = 0;
  for (int q = 1; q < 3; ++q)
    if (l[q] > l[ax]) ax = q;
  order[0] = ax;
  order[1] = ax == 0 ? 1 : 0;
  order[2] = ax == 2 ? 1 : 2;
}

// The halves of a triplet as two descriptors (the longest sequence cut in two,
// the second half read backwards), and the size of their last slices.
static void half_descs(const uint32_t* l, const uint64_t* off, TripletDesc d[2], SplitDesc* box) {
  int order[3];
  half_order(l, order);
  const int ax = order[0];
  const uint32_t mid = l[ax] / 2;
  for (int h = 0; h < 2; ++h) {
    d[h] = TripletDesc{};
    for (int k = 0; k < 3; ++k) {
      d[h].off[k] = off[order[k]];
      d[h].len[k] = l[order[k]];
      d[h].start[k] = 0;
    }
    d[h].len[0] = h ? l[ax] - mid : mid;
    d[h].start[0] = h ? mid : 0;
    d[h].rev = (uint32_t)h;
  }
  *box = SplitDesc{0, 0, l[order[1]] + 1, l[order[2]] + 1, 0, 0, 0};
}

// At least nine panels across the two shorter axes.
static bool nine_panels(const uint32_t* l) {
  const uint32_t lo = std::min({l[0], l[1], l[2]}), hi = std::max({l[0], l[1], l[2]});
  const uint32_t mid = (uint32_t)((uint64_t)l[0] + l[1] + l[2] - lo - hi);
  return (uint64_t)(lo / kPkPanel + 1) * (mid / kPkPanel + 1) >= 9;
}

// Semi-global halves (packed only): at least nine panels across the two shorter
// axes. Halves / the triplet as a pair with itself: 128 x 125 x 131 142 / 152
// us, 300 x 290 x 305 271 / 319, 723 x 651 x 698 595 / 737, 2048 x 2000 x 2080
// 2.79 / 4.74 ms, 4096 x 4000 x 4150 12.7 / 35.2 ms (int32). Thin triplets would
// gain as well, but their plans have always reported the panels of one sweep.
// Beyond the longest sweep the pair with itself takes a shorter axis: 17000 x 64
// x 64 3.65 ms (halves 5.73, int32 4.80), 30000 x 1000 x 1000 14.2 ms (19.9,
// 16.4); 16000 x 64 x 64 by halves 5.3 ms, 8.9 as a pair with itself.
bool semi_global_halves(const uint32_t* l) {
  return nine_panels(l) && std::max({l[0], l[1], l[2]}) <= (uint32_t)kMaxSweepLen;
}

// Lone triplets that run as a pair with themselves unless they have halves:
// short ones of every kind, and semi-global ones of nine panels or of a length
// no sweep takes. Long thin semi-global ones keep int32 lanes (pair with itself
// / int32: 64 x 40 x 40 81 / 84 us, 250 x 40 x 40 190 / 188, 2000 x 40 x 40 1191 /
// 1145; 20000 x 40 x 40 4.2 / 5.5 ms).
bool self_pair(int kind, const uint32_t* l) {
  const uint32_t longest = std::max({l[0], l[1], l[2]});
  if (longest < kHalfSplitMin) return true;
  return kind == kSemiGlobal && (longest > (uint32_t)kMaxSweepLen || nine_panels(l));
}

bool packed_halves_layout(const uint32_t* lens, const uint64_t* off, const trioseq_scoring& sc, Layout* L) {
  TripletDesc h[2];
  SplitDesc box;
  half_descs(lens, off, h, &box);
  const uint64_t cells = (uint64_t)box.rows * box.cols;
  Layout P;
  if (!pair_panel_layout({h[0], h[1]}, sc, true, &P)) return false;
  box.bwd = cells;
  box.nchunk = (uint32_t)((cells + kSplitChunk - 1) / kSplitChunk);
  P.halves = true;
  P.boxes = {box};
  P.chunk_box.assign(box.nchunk, 0u);
  P.plane_off = {0, cells};
  P.plane_ints = 2 * cells;
  *L = std::move(P);
  return true;
}

bool packed_self_layout(const uint32_t* lens, const uint64_t* off, const trioseq_scoring& sc, Layout* L) {
  const AxisChoice w = choose_axes_wide(lens);
  TripletDesc d{};
  for (int k = 0; k < 3; ++k) {
    d.off[k] = off[w.perm[k]];
    d.len[k] = lens[w.perm[k]];
  }
  Layout P;
  if (!pair_panel_layout({d, d}, sc, false, &P)) return false;
  P.panels /= 2;
  *L = std::move(P);
  return true;
}

// The axes of a triplet among others: the fewest panel steps (whole chunks of
// them, and about 12 for a panel's start). 8192 triplets of 100-400 residues:
// 0.862 of the executed cells are theirs, 0.846 with the longest axis swept.
static AxisChoice choose_axes_panels(const uint32_t len[3]) {
  AxisChoice best{{0, 1, 2}};
  uint64_t best_cost = UINT64_MAX;
  for (const auto& p : kPerms) {
    if (len[p[0]] > (uint32_t)kMaxSweepLen) continue;
    const uint64_t cost = (uint64_t)(len[p[1]] / kPkPanel + 1) * (len[p[2]] / kPkPanel + 1) *
                          ((len[p[0]] + 1 + kSkew + kChunk - 1) / kChunk * kChunk + 12);
    if (cost < best_cost) {
      best_cost = cost;
      std::memcpy(best.perm, p, 3);
    }
  }
  return best;
}

// Whether a batch runs better as whole pairs (one wavefront a pair) than as the
// panel jobs chosen for it (P in pairs, or by halves), or in pairs after all.
// Panel jobs use the device where whole pairs leave it waiting for their
// longest; where the pairs are many and alike, or too short to be worth
// splitting, the jobs' own costs decide: a panel takes one pop of the queue (16
// ns, whatever its size), its faces pass through memory, and halves add their
// planes' meeting. Microseconds, whole pairs / panel jobs in pairs / by halves,
// at the lines drawn here:
//   one panel a pair: 20000 of 20 residues 256 / 308 / -, 2048 of 128 x 31 x 31
//     90 / 98 / 172, 512 of them 73 / 74 / 77, 128 of them 70 / 71 / 61, 1024 of
//     500 x 31 x 31 207 / 229 / 171, 1300 of them 208 / 235 / 281;
//   two by two panels: 2000 of 32 114 / 127, 2300 of them 153 / 137, 3800 168 /
//     185, 30000 908 / 1320; 1700 of 40-60 151 / 145; 8192 of 5-60 on every
//     axis 179 / 190, 4096 of them 166 / 129; semi-global, 8000 of 63: 685 /
//     623, 6000 of them 421 / 473, 15000 of 20-60 616 / 702;
//   more: 20000 of 64 1979 / 2337, 8192 of 100 2252 / 2188, 20000 of 30-100
//     1721 / 2018, 8192 of 30-150 2121 / 1891.
// *W: the batch as whole pairs, made from the triplets of `unsplit` when kWhole is
// in question.
enum BatchForm { kChosen, kPairs, kWhole };
static BatchForm batch_form(const std::vector<TripletDesc>& P, bool halves, const Layout& unsplit,
                            const trioseq_scoring& sc, int waves, Layout* W) {
  const double np = (double)(P.size() / 2);
  double steps = 0, panels = 0, sweeps = 0, most = 0;  // of the panel pairs
  for (size_t p = 0; p + 1 < P.size(); p += 2) {
    const TripletDesc &a = P[p], &b = P[p + 1];
    const double n0 = std::max(a.len[0], b.len[0]);
    const double k = (std::max(a.len[1], b.len[1]) / kPkPanel + 1.0) * (std::max(a.len[2], b.len[2]) / kPkPanel + 1);
    steps += k * (n0 + 1 + kSkew);
    panels += k;
    sweeps += k * n0;
    most = std::max(most, k);
  }
  const bool one_panel = panels <= 1.1 * np && (most <= 1 || np > waves / 2), long_pairs = steps > 400 * np;
  // One panel a pair: halves are worth their meeting while there is room for
  // them and the sweep is long.
  if (one_panel && halves && np <= waves / 4 && steps / np >= 64 + 0.4 * np) return kChosen;
  if (!one_panel && !halves && long_pairs && !(sweeps <= 115 * panels && np > 5.4 * waves)) return kChosen;
  *W = unsplit;
  if (!pair_up(W, sc, KernelShape{4, 4, 2})) return kChosen;
  // Whole pairs: steps, and with about 12 for a panel's start and 27 for a
  // pair's, what the longest-first queue makes of them.
  const int H = panel_rows(W->ks), C = panel_cols(W->ks);
  double wsteps = 0, wpanels = 0, longest = 0;
  std::vector<double> cost;
  cost.reserve(P.size() / 2);
  for (size_t p = 0; p + 1 < W->desc.size(); p += 2) {
    const TripletDesc &a = W->desc[p], &b = W->desc[p + 1];
    const double n0 = std::max(a.len[0], b.len[0]) + 1 + kSkew;
    const double k = (std::max(a.len[1], b.len[1]) / H + 1.0) * (std::max(a.len[2], b.len[2]) / C + 1);
    wsteps += k * n0;
    wpanels += k;
    longest = std::max(longest, k * n0);
    cost.push_back(k * (n0 + 12) + 27);
  }
  const bool global = sc.kind == kGlobal, semi = sc.kind == kSemiGlobal;
  if (one_panel) {
    // (Whole pairs may take other axes, of more panels: 20000 of 64 x 10 x 10 354
    // / 350 us, of 64 x 5 x 5 294 / 344, of 1000 x 10 x 10 3078 / 2577.)
    const bool dearer = 1.08 * (steps + 40 * panels) < wsteps + 12 * wpanels + 27 * np;
    return dearer && !semi && (np > 0.93 * waves || (global && np <= waves / 2)) ? kPairs : kWhole;
  }
  const double fill = wsteps / waves / longest;  // rounds of the longest pair's
  if (halves) return fill > 1. / 3 ? kWhole : kChosen;
  if (fill <= 1. / 3) return kChosen;
  // Where the two are close: few rounds of unlike panel counts; about two of
  // semi-global pairs that are alike.
  if ((most > 4 && fill < 1.2) || (semi && fill > 1.55 && fill < 3 && wsteps >= 0.8 * longest * np)) return kChosen;
  if (long_pairs && wpanels > 12.5 * np) return kChosen;
  std::sort(cost.begin(), cost.end(), std::greater<double>());
  std::vector<double> busy(waves, 0.);  // a min-heap of the waves' ends
  double total = 0, end = 0;
  for (double c : cost) {
    std::pop_heap(busy.begin(), busy.end(), std::greater<double>());
    busy.back() += c;
    total += c;
    end = std::max(end, busy.back());
    std::push_heap(busy.begin(), busy.end(), std::greater<double>());
  }
  const double use = total / waves / end;
  return use > (long_pairs ? 0.75 : np <= waves / 2 ? 0.4 : fill < 1.2 ? 0.75 : 0.7) ? kWhole : kChosen;
}

bool packed_batch_layout(const uint32_t* lens, const uint64_t* off, size_t n, const trioseq_scoring& sc, Layout* L,
                         PackedPanels allow, const Layout* unsplit, int waves) {
  // Panel pairs: neighbours by size (the panels of the common grid, then the
  // slices; the largest first), or each triplet's own two halves, whichever the
  // times above make shorter.
  std::vector<AxisChoice> ax(n);
  for (size_t t = 0; t < n; ++t) ax[t] = choose_axes_panels(lens + 3 * t);
  const std::vector<uint32_t> order = sorted_by(n, [&](size_t t) {
    const uint32_t* l = lens + 3 * t;
    const uint32_t pj = l[ax[t].perm[1]] / kPkPanel + 1, pk = l[ax[t].perm[2]] / kPkPanel + 1;
    return SortKey{{~((uint64_t)pj * pk), ~((uint64_t)pj << 32 | l[ax[t].perm[0]]), 0}};
  });
  std::vector<TripletDesc> P;
  P.reserve(n + 1);
  for (size_t q = 0; q < n + n % 2; ++q) {
    const size_t t = order[std::min(q, n - 1)];
    TripletDesc e{};
    for (int k = 0; k < 3; ++k) {
      e.off[k] = off[3 * t + ax[t].perm[k]];
      e.len[k] = lens[3 * t + ax[t].perm[k]];
    }
    e.out = (uint32_t)t;
    P.push_back(e);
  }
  PkTime ht;
  for (size_t t = 0; t < n; ++t) {
    const uint32_t* l = lens + 3 * t;
    int o[3];
    half_order(l, o);
    ht.add(l[o[0]] - l[o[0]] / 2, l[o[1]], l[o[2]]);
  }
  // (The halves' estimate leaves out their second start per panel and their
  // meeting: measured, they had to be ahead by 3 % on single waves, 25 % on wave
  // pairs. 16 triplets of 800-1200 residues: 2.84 ms by halves, 3.10 in pairs;
  // four of 1000: 1.27 and 1.11; 2000 of 100-400: 8.5 and 6.6.)
  const PkTime pt = pk_panel_time(P);
  PanelValues vp, vh;
  const bool have_p = panel_values(P, sc, false, &vp);
  bool use_h = allow == PackedPanels::kAny &&
               (!have_p || std::min(ht.single_us() * 1.03, ht.wave_pair_us() * 1.25) <
                               std::min(pt.single_us(), pt.wave_pair_us()));
  if (!use_h && !have_p) return false;
  Layout Q;
  std::vector<TripletDesc> H;
  if (use_h) {
    uint64_t chunks = 0;
    H.reserve(2 * n);
    Q.boxes.reserve(n);
    for (size_t t : order) {
      TripletDesc h[2];
      SplitDesc box;
      half_descs(lens + 3 * t, off + 3 * t, h, &box);
      h[0].out = h[1].out = box.out = (uint32_t)t;
      const uint64_t cells = (uint64_t)box.rows * box.cols;
      box.fwd = Q.plane_ints;
      box.bwd = Q.plane_ints + cells;
      box.chunk0 = (uint32_t)chunks;
      box.nchunk = (uint32_t)((cells + kSplitChunk - 1) / kSplitChunk);
      Q.boxes.push_back(box);
      Q.plane_ints += 2 * cells;
      chunks += box.nchunk;
      H.insert(H.end(), h, h + 2);
    }
    use_h = chunks <= INT32_MAX && Q.plane_ints * 4 <= kHalvesBytes && panel_values(H, sc, true, &vh);
    if (!use_h && !have_p) return false;
  }
  if (unsplit && have_p) {
    Layout W;
    const BatchForm form = batch_form(P, use_h, *unsplit, sc, waves, &W);
    if (form == kWhole) {
      *L = std::move(W);
      return true;
    }
    if (form == kPairs) use_h = false;
  }
  if (use_h) {
    Q.halves = true;
    for (const SplitDesc& box : Q.boxes) {
      Q.plane_off.push_back(box.fwd);
      Q.plane_off.push_back(box.bwd);
      Q.chunk_box.insert(Q.chunk_box.end(), box.nchunk, (uint32_t)(&box - Q.boxes.data()));
    }
  } else {
    Q.boxes.clear();
    Q.plane_ints = 0;
  }
  if (!panel_jobs(std::move(use_h ? H : P), sc, use_h, use_h ? vh : vp, &Q)) return false;
  Q.cells = L->cells;
  Q.engine = L->engine;  // (reported: which triplets the split rule of the options calls split)
  *L = std::move(Q);
  return true;
}

trioseq_status build_layout(const uint32_t* lens, const uint64_t* off, size_t n,
                            const trioseq_scoring& sc, const trioseq_plan_options& o, int waves_hint,
                            Layout* L, bool planes, PackedPanels panels_allowed) {
  if (n && !lens) return fail(TRIOSEQ_ERR_INVALID_ARG, "lens is NULL");
  if (n > (size_t)INT32_MAX) return fail(TRIOSEQ_ERR_TOO_LARGE, "too many triplets");
  trioseq_status st = validate_scoring(&sc);
  if (st != TRIOSEQ_OK) return st;
  if (o.engine < -1 || o.engine > 1) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: bad engine");
  if (o.grid < 0) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: negative grid");
  if (o.split_factor < 0) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: negative split_factor");
  if (o.half_split_min < -1) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: bad half_split_min");
  if (o.packed < 0 || o.packed > 2) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: packed must be 0, 1 or 2");
  if (o.staging < 0 || o.staging > 2) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: staging must be 0, 1 or 2");
  if (o.panel_group != 0 && o.panel_group != 1 && o.panel_group != 4)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: panel_group must be 0, 1 or 4");
  static_assert(kStripPanels == 4, "panel_group option values");
  KernelShape ks{o.tile_rows ? o.tile_rows : 4, o.tile_cols ? o.tile_cols : 4,
                 o.waves_per_simd ? o.waves_per_simd : 2};
  ks.group = o.panel_group ? o.panel_group : kDefaultPanelGroup;
  if (o.lane_exchange < 0 || o.lane_exchange > 2)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: lane_exchange must be 0, 1 or 2");
  ks.xch = o.lane_exchange ? o.lane_exchange - 1 : kDefaultLaneExchange;
  // A shape only the packed kernels have is accepted when packing is asked
  // for; the batch must then qualify for it (checked at the end).
  const bool int32_shape = shape_supported(ks, sc.kind);
  KernelShape pks = ks;
  pks.dma = o.staging == 2 ? 1 : 0;
  if (!int32_shape && !(o.packed == 2 && pk_shape_supported(pks, sc.kind)))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "plan: unsupported tile shape for this scoring kind");
  std::vector<uint64_t> offs;
  if (!off) {
    offs.resize(3 * n);
    uint64_t tw = 0;
    trioseq_packed_layout(lens, n, offs.data(), &tw);
    off = offs.data();
  }
  double cells = 0;
  for (size_t t = 0; t < n; ++t) {
    const uint32_t* l = lens + 3 * t;
    if (std::min({l[0], l[1], l[2]}) > (uint32_t)kMaxSweepLen)
      return fail(TRIOSEQ_ERR_TOO_LARGE, "triplet " + std::to_string(t) +
                                             ": every sequence exceeds " +
                                             std::to_string(kMaxSweepLen) + " residues");
    if (planes && l[0] > (uint32_t)kMaxSweepLen)
      return fail(TRIOSEQ_ERR_TOO_LARGE, "triplet " + std::to_string(t) + ": sweep sequence exceeds " +
                                             std::to_string(kMaxSweepLen) + " residues");
    st = check_range(sc, l[0], l[1], l[2], t);
    if (st != TRIOSEQ_OK) return st;
    cells += (double)l[0] * (double)l[1] * (double)l[2];
  }
  const int H = panel_rows(ks), W = panel_cols(ks), RR = (int)right_face_row(ks);

  // Which triplets are split into panel jobs: forced by the engine option,
  // else by the rule at kSplitCells.
  const double per_wave = cells / std::max(1, waves_hint);
  L->desc.assign(n, TripletDesc{});
  std::vector<char> split(n, 0);
  std::vector<uint64_t> cost(n, 0);
  uint64_t stride = 0, pool = 0;
  uint32_t max_n0 = 0;
  int n_split = 0, panels = 0;
  for (size_t t = 0; t < n; ++t) {
    const uint32_t* l = lens + 3 * t;
    const double c = (double)l[0] * l[1] * l[2];
    const double factor = o.split_factor > 0 ? (double)o.split_factor : kSplitFactor;
    const bool sp = o.engine == 1 ||
                    (o.engine == -1 && (n == 1 || c >= kSplitCells || c > factor * per_wave));
    // Plane runs keep the caller's axes: the plane is the last slice of S0.
    AxisChoice ax = planes ? AxisChoice{{0, 1, 2}} : sp ? choose_axes_wide(l) : choose_axes_batch(l, ks);
    TripletDesc& d = L->desc[t];
    for (int a = 0; a < 3; ++a) {
      d.off[a] = off[3 * t + ax.perm[a]];
      d.len[a] = l[ax.perm[a]];
    }
    d.out = (uint32_t)t;
    d.face_off = 0;
    const uint64_t rows = face_rows(d.len[0]);
    const uint64_t PJ = d.len[1] / H + 1, PK = d.len[2] / W + 1;
    if (sp && PJ * PK > 1) {
      split[t] = 1;
      ++n_split;
      d.face_off = pool;
      pool += PJ * PK * rows * (uint64_t)(W + RR) * 2;
      panels += (int)(PJ * PK);
    } else {
      stride = std::max(stride, rows * (PK * W + RR));
    }
    cost[t] = panel_steps(d.len, ks);
    max_n0 = std::max(max_n0, d.len[0]);
  }
  L->engine = n_split == 0 ? 0 : (n_split == (int)n ? 1 : 2);
  L->modes = n_split == 0 ? 1 : (n_split == (int)n ? 2 : 3);
  // Strip workgroups serve plans of panel jobs only.
  if (L->modes != 2) ks.group = 1;
  // Whole-triplet-only plans fit four waves per SIMD without much spilling
  // on 4x4 tiles; panel jobs carry tag registers and use the two-wave budget.
  if (!planes && !o.waves_per_simd && L->modes == 1 && ks.rj * ks.rk <= 16) {
    KernelShape k4 = ks;
    k4.wpe = 4;
    if (shape_supported(k4, sc.kind)) ks = k4;
  }
  L->ks = ks;
  L->kind = sc.kind;
  L->planes = planes;
  L->panels = panels;
  L->lds_n0 = max_n0;
  L->cells = cells;
  L->face_stride = (stride + 63) / 64 * 64;
  L->pool_ints = pool;
  L->packed = false;

  // A batch of packed panel jobs needs nothing of the int32 job queue. (Whole
  // pairs are looked at where the split rule splits none of the batch.)
  const bool default_shape = (o.tile_rows == 0 || o.tile_rows == 4) && (o.tile_cols == 0 || o.tile_cols == 4) &&
                             (o.waves_per_simd == 0 || o.waves_per_simd == 2) && o.lane_exchange != 2 && o.staging != 2;
  const bool any_shape = o.tile_rows || o.tile_cols || o.waves_per_simd || o.lane_exchange || o.staging;
  if (panels_allowed != PackedPanels::kNone && !planes && n > 1 && o.engine == -1 && !o.grid && ks.group == 1 &&
      (o.packed == 2 ? default_shape : o.packed == 0 && !any_shape) &&
      packed_batch_layout(lens, off, n, sc, L, panels_allowed, L->modes == 1 ? L : nullptr, std::max(4, waves_hint)))
    return TRIOSEQ_OK;

  // Job order: split triplets' panels first, by anti-diagonal d = pj + pk
  // across all split triplets (largest first within a diagonal), so every
  // panel comes after the panels it reads from and several split triplets
  // fill their pipelines together; then whole triplets longest first so the
  // queue drains with short ones.
  const std::vector<uint32_t> idx = sorted_by(n, [&](size_t t) { return SortKey{{~cost[t], 0, 0}}; });
  L->jobs.clear();
  L->jobs.reserve(n + panels);
  uint32_t diagonals = 0;
  for (size_t t : idx)
    if (split[t]) diagonals = std::max(diagonals, L->desc[t].len[1] / H + L->desc[t].len[2] / W + 1);
  // With strip workgroups a job is a strip of kStripPanels panels of one
  // panel row (panel = its first panel), ordered by the diagonal of (panel
  // row, strip index): its top faces come from the strip above, its left face
  // from the strip before it in the row.
  const uint32_t sw = ks.group > 1 ? (uint32_t)kStripPanels : 1u;
  for (uint32_t d = 0; d < diagonals; ++d)
    for (size_t t : idx) {
      if (!split[t]) continue;
      const uint32_t PJ = L->desc[t].len[1] / H + 1, PK = L->desc[t].len[2] / W + 1;
      const uint32_t NS = (PK + sw - 1) / sw;  // strips (or panels) per panel row
      if (d + 1 >= PJ + NS) continue;
      for (uint32_t pj = (d >= NS ? d - NS + 1 : 0); pj <= std::min(d, PJ - 1); ++pj)
        L->jobs.push_back(JobDesc{(uint32_t)t, pj * PK + (d - pj) * sw});
    }
  for (size_t t : idx)
    if (!split[t]) L->jobs.push_back(JobDesc{(uint32_t)t, kWholeTriplet});
  // Packed pairs when asked for (any lane tile a packed kernel exists for),
  // or by default when the tile is left to the library (4 x 4, two waves per
  // SIMD); the batch keeps int32 lanes when it does not qualify (pair_up).
  if (o.packed == 2) {
    KernelShape pks{o.tile_rows ? o.tile_rows : 4, o.tile_cols ? o.tile_cols : 4,
                    o.waves_per_simd ? o.waves_per_simd : 2};
    pks.xch = o.lane_exchange == 2 ? 1 : 0;
    pks.dma = o.staging == 2 ? 1 : 0;
    pair_up(L, sc, pks);
  } else if (o.packed == 0 && !any_shape) {
    pair_up(L, sc, KernelShape{4, 4, 2});
  }
  if (!L->packed && !int32_shape)
    return fail(TRIOSEQ_ERR_INVALID_ARG,
                "plan: this tile shape exists for packed pairs only, and the batch does not qualify");
  return TRIOSEQ_OK;
}

// Autotuning cache: the best options per batch length profile.
static std::mutex g_tune_mu;
static std::vector<std::pair<std::string, trioseq_plan_options>> g_tuned;
// Bumped whenever a tuned choice is remembered: cached plans made before it
// are rebuilt so they take the choice.
std::atomic<uint64_t> g_tune_epoch{0};

static int log2_bucket(double v) {
  int b = 0;
  while (v >= 2.0 && b < 80) {
    v /= 2.0;
    ++b;
  }
  return b;
}

std::string length_profile(const uint32_t* lens, size_t n, int kind) {
  uint32_t mx = 0;
  double cells = 0;
  for (size_t t = 0; t < n; ++t) {
    const uint32_t* l = lens + 3 * t;
    mx = std::max({mx, l[0], l[1], l[2]});
    cells += (double)l[0] * l[1] * l[2];
  }
  return std::to_string(kind) + "/" + std::to_string(log2_bucket((double)n)) + "/" +
         std::to_string(log2_bucket(mx)) + "/" + std::to_string(log2_bucket(cells));
}

void apply_tuned(const uint32_t* lens, size_t n, int kind, trioseq_plan_options* o) {
  const std::string key = length_profile(lens, n, kind);
  std::lock_guard<std::mutex> lk(g_tune_mu);
  for (const auto& kv : g_tuned)
    if (kv.first == key) {
      o->tile_rows = kv.second.tile_rows;
      o->tile_cols = kv.second.tile_cols;
      o->waves_per_simd = kv.second.waves_per_simd;
      if (!o->panel_group) o->panel_group = kv.second.panel_group;
      if (!o->lane_exchange) o->lane_exchange = kv.second.lane_exchange;
      if (!o->split_factor) o->split_factor = kv.second.split_factor;
      if (!o->half_split_min) o->half_split_min = kv.second.half_split_min;
      if (!o->packed) o->packed = kv.second.packed;
      if (!o->staging) o->staging = kv.second.staging;
    }
}

static void remember_tuned(const std::string& key, const trioseq_plan_options& o) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  g_tune_epoch.fetch_add(1, std::memory_order_relaxed);
  for (auto& kv : g_tuned)
    if (kv.first == key) {
      kv.second = o;
      return;
    }
  g_tuned.emplace_back(key, o);
}

// Occupancy per (device, kernel variant, dynamic LDS bytes): the runtime
// query costs about 0.2 ms, and plans of one process ask the same few.
static std::mutex g_occ_mu;
static std::vector<std::pair<std::string, int>> g_occ;

static hipError_t cached_occupancy(const Layout& L, int device, int* w) {
  const std::string key = std::to_string(device) + "/" + std::to_string(L.ks.rj) + "x" +
                          std::to_string(L.ks.rk) + "/" + std::to_string(L.ks.wpe) + "/" +
                          std::to_string(L.ks.group) + "/" + std::to_string(L.ks.xch) + "/" +
                          std::to_string((int)L.packed + 2 * (int)L.pk_self) + "/" +
                          std::to_string(L.modes) + "/" + std::to_string(L.kind) + "/" +
                          std::to_string((int)L.planes) + "/" + std::to_string(shift_lds_bytes(L.lds_n0)) + "/" +
                          std::to_string(pk_waves_per_simd(L.kind, L.planes, L.pk_self, L.lds_n0, L.jobs.size()));
  {
    std::lock_guard<std::mutex> lk(g_occ_mu);
    for (const auto& kv : g_occ)
      if (kv.first == key) {
        *w = kv.second;
        return hipSuccess;
      }
  }
  hipError_t e = L.modes == kModePkPanel ? panel_pk_occupancy(L.kind, L.planes, L.pk_self, L.lds_n0, L.jobs.size(), w)
                 : L.packed ? sweep_pk_occupancy(L.ks, L.kind, L.lds_n0, w)
                         : sweep_occupancy(L.ks, L.modes, L.kind, L.planes, L.lds_n0, w);
  if (e == hipSuccess && L.modes == 2 && L.ks.group > 1) {
    // A strip workgroup's 2 * kStripPanels waves fill 4 SIMDs x (waves per
    // SIMD) slots of a compute unit; the runtime's figure for these
    // workgroups was measured above that (launches beyond it only queue).
    *w = std::max(1, std::min(*w, 4 * L.ks.wpe / (2 * kStripPanels)));
  }
  if (e == hipSuccess) {
    std::lock_guard<std::mutex> lk(g_occ_mu);
    g_occ.emplace_back(key, *w);
  }
  return e;
}

trioseq_status layout_grid(const Layout& L, const DeviceProps& dp, int requested, int* grid,
                           int* waves_per_cu) {
  int w = 0;
  TRIOSEQ_HIP(cached_occupancy(L, dp.device, &w), "occupancy");
  int g = requested ? requested : dp.cus * std::max(1, w);
  g = (int)std::min<size_t>((size_t)g, std::max<size_t>(L.jobs.size(), 1));
  *grid = g;
  // Waves per compute unit: workgroups of 1 (whole triplets), 2 (panel jobs)
  // or 2 * kStripPanels (strip jobs) waves.
  *waves_per_cu = w * (L.modes == 1 || L.modes == 3 || L.pk_self ? 1 : L.ks.group > 1 ? 2 * kStripPanels : 2);
  return TRIOSEQ_OK;
}

}  // namespace trioseq

namespace trioseq {

bool half_split_layout(const uint32_t* lens, const uint64_t* word_off, int32_t min_len, HalfSplit* h) {
  int ax = 0;
  for (int q = 1; q < 3; ++q)
    if (lens[q] > lens[ax]) ax = q;
  const uint32_t na = lens[ax];
  if (min_len < 0) return false;
  const uint32_t lo = min_len ? (uint32_t)std::max(min_len, 2) : kHalfSplitMin;
  if (na < lo || (na + 1) / 2 > (uint32_t)kMaxSweepLen) return false;
  const int r = ax == 0 ? 1 : 0, c = ax == 2 ? 1 : 2;
  const uint32_t mid = na / 2;
  uint64_t src[3];
  if (word_off) {
    for (int q = 0; q < 3; ++q) src[q] = word_off[q];
  } else {
    uint64_t tw = 0;
    trioseq_packed_layout(lens, 1, src, &tw);
  }
  const int order[3] = {ax, r, c};
  uint64_t w = 0;
  for (int half = 0; half < 2; ++half)
    for (int k = 0; k < 3; ++k) {
      const int q = order[k];
      const uint32_t start = (k == 0 && half == 1) ? mid : 0;
      const uint32_t len = k == 0 ? (half == 0 ? mid : na - mid) : lens[q];
      const int i = 3 * half + k;
      h->lens[i] = len;
      h->offs[i] = w;
      h->gather[i] = GatherDesc{src[q], w, start, len, (uint32_t)half};
      w += (len + 15) / 16;
    }
  h->words = (uint32_t)w;
  h->rows = lens[r] + 1;
  h->cols = lens[c] + 1;
  return true;
}

bool half_split_choice(const uint32_t* lens, const uint64_t* word_off, size_t n, int kind,
                       const trioseq_plan_options& o, HalfSplit* h) {
  if (n != 1 || o.lane_exchange == 2) return false;
  if (kind == kLocal) {
    if (o.half_split_min == 0 && std::max({lens[0], lens[1], lens[2]}) >= kHalfSplitMaxLocal) return false;
  } else if (kind != kGlobal) {
    return false;
  }
  return half_split_layout(lens, word_off, o.half_split_min, h);
}

}  // namespace trioseq

// panels: the packed panel jobs a batch may use; left at those it does use.
static trioseq_status plan_create_with(const uint32_t* lens, const uint64_t* word_off, size_t n,
                                       const trioseq_scoring* scp, const trioseq_plan_options* opts,
                                       trioseq_plan** out, const PlanMemory* mem, PackedPanels* panels) {
  if (!out) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan_create: plan output is NULL");
  if (!scp) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan_create: scoring is NULL");
  trioseq_plan_options o{-1, 0, 0, 0, 0, 0};
  if (opts) o = *opts;
  // A lone global triplet is scored by halves under the automatic engine and
  // grid when the options leave the tile at (or set it to) the plane
  // kernels' 4 x 4 at two waves per SIMD.
  const bool defaults = o.engine == -1 && !o.grid && (o.tile_rows == 0 || o.tile_rows == 4) &&
                        (o.tile_cols == 0 || o.tile_cols == 4) &&
                        (o.waves_per_simd == 0 || o.waves_per_simd == 2);
  if (!o.tile_rows && !o.tile_cols && !o.waves_per_simd && lens) apply_tuned(lens, n, scp->kind, &o);
  // Inputs are validated (by the layout) before the device is touched; the
  // layout is redone if the device's size changes the split rule's hint.
  Layout L;
  int hint = 256 * kWavesPerCuHint;
  trioseq_status st = build_layout(lens, word_off, n, *scp, o, hint, &L, false, *panels);
  if (st != TRIOSEQ_OK) return st;
  // A lone global or local triplet under the automatic options is scored by
  // halves (local: the best of the two halves' own bests and of the paths
  // that cross the middle plane).
  HalfSplit hs;
  bool half = defaults && half_split_choice(lens, word_off, n, scp->kind, o, &hs);
  const trioseq_plan_options ho{-1, 4, 4, 0, 0, 2, o.panel_group, o.lane_exchange};  // the plane kernels' shape
  DeviceProps dp;
  st = device_props(&dp);
  if (st != TRIOSEQ_OK) return st;
  if (half || dp.cus * kWavesPerCuHint != hint) {
    hint = dp.cus * kWavesPerCuHint;
    st = half ? build_layout(hs.lens, hs.offs, 2, *scp, ho, hint, &L, true)
              : build_layout(lens, word_off, n, *scp, o, hint, &L, false, *panels);
    if (st != TRIOSEQ_OK) return st;
  }
  if (n < 2 || L.modes != kModePkPanel) *panels = PackedPanels::kNone;
  else if (!L.halves) *panels = PackedPanels::kPairs;
  // A batch carved from a region whose pool cannot hold its split triplets'
  // faces sweeps every triplet whole instead (same scores, no face pool).
  if (mem && !half && n > 1 && o.engine == -1 && L.pool_ints * sizeof(int) > mem->pool_bytes) {
    o.engine = 0;
    st = build_layout(lens, word_off, n, *scp, o, hint, &L);
    if (st != TRIOSEQ_OK) return st;
  }
  // The halves run as one packed pair where their values fit 16 bits: one
  // sweep of 3.5 instructions per cell over both, against 7 in int32 (the
  // 1024 x 1000 x 1048 triplet 975 -> 620 us, 4096 x 4000 x 4150 31.3 -> 10.9 ms).
  // Packed, they also beat the classic split on long local triplets, which
  // stay on it in int32 (2048 x 2000 x 2080: 5.62 -> 2.58 ms, 4096 x 4000 x
  // 4150: 38.8 -> 14.6 ms).
  const bool may_pack = o.packed != 1 && o.panel_group <= 1;
  // Semi-global halves exist in packed form only.
  const bool packed_half =
      defaults && !half && n == 1 && !mem && may_pack && o.lane_exchange != 2 &&
      ((scp->kind == kSemiGlobal && semi_global_halves(lens)) || (scp->kind == kLocal && o.half_split_min == 0 && L.cells >= kSplitCells)) &&
      half_split_layout(lens, word_off, o.half_split_min, &hs);
  if ((half && may_pack) || packed_half) {
    const uint64_t int32_pool = L.pool_ints * sizeof(int);
    const double cells = L.cells;
    std::vector<uint64_t> def(3);
    uint64_t tw = 0;
    if (!word_off) trioseq_packed_layout(lens, 1, def.data(), &tw);
    Layout P;
    if (packed_halves_layout(lens, word_off ? word_off : def.data(), *scp, &P)) {
      if (mem && int32_pool > mem->pool_bytes)
        return fail(TRIOSEQ_ERR_TOO_LARGE,
                    "allocation-free scoring: panel faces of split triplets exceed the scratch array's face pool");
      L = std::move(P);
      L.cells = cells;
      half = true;
    }
  }
  // A lone triplet that takes no halves may run as a pair with itself: per cell
  // as many instructions as int32 lanes take, but the packed kernel's shorter
  // hops and polls (semi-global 723 x 651 x 698: 824 -> 721 us; global 48 x 45 x
  // 51: 68 -> 58 us, 100 x 97 x 104: 119 -> 95 us).
  if (n == 1 && defaults && may_pack && !mem && !half && o.lane_exchange != 2 && L.modes == 2 &&
      (scp->kind == kSemiGlobal || o.half_split_min == 0) && self_pair(scp->kind, lens)) {
    std::vector<uint64_t> def(3);
    uint64_t tw = 0;
    if (!word_off) trioseq_packed_layout(lens, 1, def.data(), &tw);
    const double cells = L.cells;
    if (packed_self_layout(lens, word_off ? word_off : def.data(), *scp, &L)) L.cells = cells;
  }
  const size_t nd = L.desc.size();  // triplets the kernels see

  trioseq_plan* p = new (std::nothrow) trioseq_plan;
  if (!p) return fail(TRIOSEQ_ERR_NOMEM, "plan: host allocation");
  p->device = dp.device;
  p->n = n;
  p->ks = L.ks;
  p->modes = L.modes;
  p->engine = L.engine;
  p->panels = L.panels;
  p->lds_n0 = L.lds_n0;
  p->njobs = (uint32_t)L.jobs.size();
  p->sc = make_dev_scoring(*scp);
  p->cells = L.cells;
  p->use_graph = o.use_graph != 0 && !mem;
  p->face_stride = L.face_stride;
  auto hip_bail = [&](hipError_t e, const char* what) {
    fail_hip(e, what);
    trioseq_status s2 = (e == hipErrorOutOfMemory) ? TRIOSEQ_ERR_NOMEM : TRIOSEQ_ERR_DEVICE;
    plan_free(p);
    return s2;
  };
  st = layout_grid(L, dp, o.grid, &p->grid, &p->waves_per_cu);
  if (st != TRIOSEQ_OK) {
    plan_free(p);
    return st;
  }
  hipError_t e;
  // One-off initialisation runs on this thread's private stream, which is
  // waited for alone before the plan is returned (or, for a plan carved from
  // a caller's region, on the caller's stream).
  hipStream_t is = nullptr;
  if (mem) {
    is = mem->stream;
  } else if ((e = init_stream(dp.device, &is)) != hipSuccess) {
    return hip_bail(e, "hipStreamCreate");
  }
  // Device buffers: hipMalloc'd and owned by the plan, or carved in order
  // from the region's plain part (256-byte aligned); what is carved is never
  // freed.
  p->borrowed = mem != nullptr;
  uint64_t carved = 0;
  auto dalloc = [&](void** dst, uint64_t bytes) -> hipError_t {
    if (!mem) return hipMalloc(dst, bytes);
    const uint64_t at = (carved + 255) & ~255ull;
    if (at + bytes > mem->plain_bytes) return hipErrorOutOfMemory;
    *dst = mem->plain + at;
    carved = at + bytes;
    return hipSuccess;
  };
  auto too_large = [&](const std::string& what) {
    plan_free(p);
    return fail(TRIOSEQ_ERR_TOO_LARGE, "allocation-free scoring: " + what);
  };
  auto region_fail = [&](hipError_t e2, const char* what) {
    if (mem && e2 == hipErrorOutOfMemory) return too_large(std::string(what) + " exceeds the scratch region");
    return hip_bail(e2, what);
  };
  const uint64_t pool_bytes = L.pool_ints * sizeof(int);
  if (mem) {
    // The generation word, error flag and queue head persist in the region
    // (the generation only grows, so no stale tag ever looks current).
    p->d_ctl = mem->ctl;
    p->d_counter = mem->counter;
  } else {
    if ((e = hipMalloc((void**)&p->d_counter, kCounterBytes)) != hipSuccess) return hip_bail(e, "hipMalloc");
    if ((e = hipMalloc((void**)&p->d_ctl, 256)) != hipSuccess) return hip_bail(e, "hipMalloc");
    if ((e = hipMemsetAsync(p->d_ctl, 0, 256, is)) != hipSuccess) return hip_bail(e, "hipMemset");
  }
  if (nd) {
    if ((e = dalloc((void**)&p->d_desc, nd * sizeof(TripletDesc))) != hipSuccess)
      return region_fail(e, "triplet table");
    if ((e = hipMemcpyAsync(p->d_desc, L.desc.data(), nd * sizeof(TripletDesc), hipMemcpyHostToDevice,
                            is)) != hipSuccess)
      return hip_bail(e, "hipMemcpy desc");
    if ((e = dalloc((void**)&p->d_jobs, L.jobs.size() * sizeof(JobDesc))) != hipSuccess)
      return region_fail(e, "job table");
    if ((e = hipMemcpyAsync(p->d_jobs, L.jobs.data(), L.jobs.size() * sizeof(JobDesc),
                            hipMemcpyHostToDevice, is)) != hipSuccess)
      return hip_bail(e, "hipMemcpy jobs");
  }
  if (mem) {
    p->d_pface = mem->pool;
    p->pool_ints = mem->pool_bytes / 4;
  }
  if (pool_bytes) {
    if (mem) {
      // The region's pool part only ever holds (value, tag) pairs at even
      // offsets from its fixed base, or the zeros it started with.
      if (pool_bytes > mem->pool_bytes)
        return too_large("panel faces of split triplets exceed the scratch array's face pool");
    } else {
      p->pool_ints = L.pool_ints;
      // Tagged faces start at tag 0, which no run uses, so nothing stale matches.
      if ((e = hipMalloc((void**)&p->d_pface, pool_bytes)) != hipSuccess)
        return hip_bail(e, "hipMalloc panel faces");
      if ((e = hipMemsetAsync(p->d_pface, 0, pool_bytes, is)) != hipSuccess) return hip_bail(e, "hipMemset");
    }
  }
  p->red_pairs = L.red_pairs();
  if (p->red_pairs &&
      (e = dalloc((void**)&p->d_red, (uint64_t)p->red_pairs * 2 * sizeof(int))) != hipSuccess)
    return region_fail(e, "reduction pairs");
  const bool pk_panel = L.modes == kModePkPanel;
  p->packed = L.packed;
  p->pk_base = L.pk_base;
  p->pk_kc = L.pk_kc;
  p->pk_self = L.pk_self;
  p->pk_reuse = L.pk_reuse;
  p->tag_step = L.tag_step;
  // (Packed panel jobs make their own edge values.)
  const uint64_t bnd_ints = pk_panel ? 0 : boundary_ints(L.ks, L.lds_n0);
  if (bnd_ints && (e = dalloc((void**)&p->d_bnd, bnd_ints * sizeof(int))) != hipSuccess)
    return region_fail(e, "sentinel faces");
  if (bnd_ints) {
    p->bnd = carve_boundary(L.ks, L.lds_n0, p->d_bnd);
    if ((e = launch_init_boundary(L.ks, p->bnd, is)) != hipSuccess) return hip_bail(e, "boundary init");
  }
  if (L.packed && !pk_panel) {
    const uint64_t rows = face_rows(L.lds_n0);
    p->pk_top_words = rows * panel_cols(L.ks);
    const uint64_t words = p->pk_top_words + rows * right_face_row(L.ks);
    if ((e = dalloc((void**)&p->d_pkbnd, words * 4)) != hipSuccess) return region_fail(e, "packed sentinel faces");
    if ((e = launch_fill_packed_sentinel((uint32_t*)p->d_pkbnd, words, is)) != hipSuccess)
      return hip_bail(e, "packed sentinel faces");
  }
  p->workspace_bytes = pool_bytes + (L.packed && !pk_panel ? (p->pk_top_words + face_rows(L.lds_n0) * right_face_row(L.ks)) * 4 : 0) + bnd_ints * sizeof(int) +
                       (uint64_t)p->red_pairs * 2 * sizeof(int) +
                       nd * sizeof(TripletDesc) + L.jobs.size() * sizeof(JobDesc) + 512;
  if (half || L.halves) {
    p->half = true;
    if (!L.halves) {
      // (int32 halves of a lone triplet, gathered in every run.)
      const uint64_t cells = (uint64_t)hs.rows * hs.cols;
      L.boxes = {SplitDesc{0, cells, hs.rows, hs.cols, 0, (uint32_t)((cells + kSplitChunk - 1) / kSplitChunk), 0}};
      L.plane_off = {0, cells};
      L.plane_ints = 2 * cells;
      p->h_words_n = hs.words;
      if ((e = dalloc((void**)&p->d_hwords, std::max<uint64_t>(hs.words, 1) * 4)) != hipSuccess ||
          (e = dalloc((void**)&p->d_gather, sizeof hs.gather)) != hipSuccess ||
          (e = dalloc((void**)&p->d_hscores, 8)) != hipSuccess)
        return region_fail(e, "half-split buffers");
      if ((e = hipMemcpyAsync(p->d_gather, hs.gather, sizeof hs.gather, hipMemcpyHostToDevice, is)) != hipSuccess)
        return hip_bail(e, "half-split buffers");
    }
    const size_t nb = L.boxes.size();
    p->h_nchunk = L.boxes.back().chunk0 + L.boxes.back().nchunk;
    if ((e = dalloc((void**)&p->d_plane, L.plane_ints * 4)) != hipSuccess ||
        (e = dalloc((void**)&p->d_plane_off, L.plane_off.size() * 8)) != hipSuccess ||
        (e = dalloc((void**)&p->d_sdesc, nb * sizeof(SplitDesc))) != hipSuccess ||
        (e = dalloc((void**)&p->d_partial, (uint64_t)p->h_nchunk * 4)) != hipSuccess ||
        (nb > 1 && ((e = dalloc((void**)&p->d_chunk_box, (uint64_t)p->h_nchunk * 4)) != hipSuccess ||
                    (e = dalloc((void**)&p->d_meet, nb * 4)) != hipSuccess)))
      return region_fail(e, "half-split buffers");
    if ((e = hipMemcpyAsync(p->d_plane_off, L.plane_off.data(), L.plane_off.size() * 8, hipMemcpyHostToDevice, is)) !=
            hipSuccess ||
        (e = hipMemcpyAsync(p->d_sdesc, L.boxes.data(), nb * sizeof(SplitDesc), hipMemcpyHostToDevice, is)) !=
            hipSuccess ||
        (nb > 1 && ((e = hipMemcpyAsync(p->d_chunk_box, L.chunk_box.data(), (uint64_t)p->h_nchunk * 4,
                                        hipMemcpyHostToDevice, is)) != hipSuccess ||
                    (e = hipMemsetAsync(p->d_meet, 0, nb * 4, is)) != hipSuccess)))
      return hip_bail(e, "half-split buffers");
    p->workspace_bytes += L.plane_ints * 4 + (uint64_t)p->h_words_n * 4 + (uint64_t)p->h_nchunk * 8 +
                          nb * (sizeof(SplitDesc) + 20);
  }
  // The whole-triplet workspace comes last: a carved plan launches no more
  // waves than the rest of the region holds workspaces for.
  if (L.face_stride) {
    const uint64_t per_wave = L.face_stride * sizeof(int);
    if (mem) {
      const uint64_t at = (carved + 255) & ~255ull;
      const uint64_t fit = at < mem->plain_bytes ? (mem->plain_bytes - at) / per_wave : 0;
      if (fit == 0) return too_large("the largest whole triplet's face workspace exceeds the scratch region");
      p->grid = (int)std::min<uint64_t>((uint64_t)p->grid, fit);
    }
    const uint64_t face_bytes = (uint64_t)p->grid * per_wave;
    if ((e = dalloc((void**)&p->d_face, face_bytes)) != hipSuccess)
      return region_fail(e, "hipMalloc face workspace");
    p->workspace_bytes += face_bytes;
  }
  if ((e = hipStreamSynchronize(is)) != hipSuccess) return hip_bail(e, "plan init");
  if (p->use_graph) {
    if ((e = hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking)) != hipSuccess)
      return hip_bail(e, "hipStreamCreate");
  }
  *out = p;
  return TRIOSEQ_OK;
}

// A batch whose packed panel jobs do not fit the device's free memory takes the
// next smaller form: pairs instead of halves (whose planes are all held at
// once), then whole triplets.
static trioseq_status plan_create_impl(const uint32_t* lens, const uint64_t* word_off, size_t n,
                                       const trioseq_scoring* scp, const trioseq_plan_options* opts,
                                       trioseq_plan** out, const PlanMemory* mem = nullptr) {
  // (A carved plan keeps to the int32 layout's memory limits.)
  PackedPanels panels = mem ? PackedPanels::kNone : PackedPanels::kAny;
  for (;;) {
    PackedPanels used = panels;
    const trioseq_status st = plan_create_with(lens, word_off, n, scp, opts, out, mem, &used);
    if (st != TRIOSEQ_ERR_NOMEM || used == PackedPanels::kNone) return st;
    (void)hipGetLastError();  // the failed allocation's
    panels = used == PackedPanels::kAny ? PackedPanels::kPairs : PackedPanels::kNone;
  }
}

namespace trioseq {

PlaneWorkspace::~PlaneWorkspace() {
  for (Buf* b : {&ctl, &desc, &jobs, &face, &pool, &bnd, &red, &plane, &plane_off, &words, &scores, &sd,
                 &split_out, &chunk_box, &partial, &lwords, &leaves, &cols, &ncols, &lscore, &tables})
    (void)hipFree(b->p);
  (void)hipHostFree(h_stage);
  (void)hipHostFree(h_out);
}

uint64_t ws_bytes(const PlaneWorkspace& ws) {
  uint64_t t = ws.h_stage_bytes + ws.h_out_ints * 4;
  for (const PlaneWorkspace::Buf* b :
       {&ws.ctl, &ws.desc, &ws.jobs, &ws.face, &ws.pool, &ws.bnd, &ws.red, &ws.plane, &ws.plane_off,
        &ws.words, &ws.scores, &ws.sd, &ws.split_out, &ws.chunk_box, &ws.partial, &ws.lwords, &ws.leaves,
        &ws.cols, &ws.ncols, &ws.lscore, &ws.tables})
    t += b->bytes;
  return t;
}

hipError_t ws_grow(PlaneWorkspace::Buf& b, uint64_t bytes, bool zero, hipStream_t s) {
  bytes = std::max<uint64_t>(bytes, 256);
  if (b.bytes >= bytes) return hipSuccess;
  hipError_t e = hipStreamSynchronize(s);  // the old buffer may still be in use
  if (e != hipSuccess) return e;
  (void)hipFree(b.p);
  b.p = nullptr;
  b.bytes = 0;
  const uint64_t cap = bytes + bytes / 4;  // room for the next, similar run
  if ((e = hipMalloc(&b.p, cap)) != hipSuccess) return e;
  b.bytes = cap;
  if (zero) e = hipMemsetAsync(b.p, 0, cap, s);
  return e;
}

trioseq_status run_planes(PlaneWorkspace& ws, const uint32_t* lens, const uint64_t* offs, size_t n,
                          const uint32_t* words, size_t nwords, const trioseq_scoring& sc,
                          const uint64_t* plane_off, uint64_t plane_ints, hipStream_t s) {
  if (n == 0) return TRIOSEQ_OK;
  if (!ws.have_props) {
    trioseq_status st = device_props(&ws.dp);
    if (st != TRIOSEQ_OK) return st;
    ws.have_props = true;
  }
  const trioseq_plan_options o{-1, 4, 4, 0, 0, 2};  // the plane kernels' shape
  Layout L;
  trioseq_status st = build_layout(lens, offs, n, sc, o, ws.dp.cus * kWavesPerCuHint, &L, true);
  if (st != TRIOSEQ_OK) return st;
  int grid = 0, wpc = 0;
  st = layout_grid(L, ws.dp, 0, &grid, &wpc);
  if (st != TRIOSEQ_OK) return st;
  hipError_t e;
#define WS(call, what)                                  \
  do {                                                  \
    if ((e = (call)) != hipSuccess) return fail_hip(e, what); \
  } while (0)
  if (!ws.ctl.p) {
    // [0] generation, [1] error flag, [64] queue head and counters; the generation
    // keeps growing across runs, so a zeroed pool's tags (0) are never current.
    WS(ws_grow(ws.ctl, 256 + kCounterBytes, true, s), "align: workspace");
  }
  WS(ws_grow(ws.desc, n * sizeof(TripletDesc), false, s), "align: workspace");
  WS(ws_grow(ws.jobs, L.jobs.size() * sizeof(JobDesc), false, s), "align: workspace");
  WS(ws_grow(ws.face, (uint64_t)grid * L.face_stride * 4, false, s), "align: workspace");
  WS(ws_grow(ws.pool, L.pool_ints * 4, true, s), "align: workspace");
  WS(ws_grow(ws.plane, plane_ints * 4, false, s), "align: workspace");
  WS(ws_grow(ws.plane_off, n * 8, false, s), "align: workspace");
  WS(ws_grow(ws.words, nwords * 4, false, s), "align: workspace");
  WS(ws_grow(ws.scores, n * 4, false, s), "align: workspace");
  if (!ws.bnd.p || L.lds_n0 > ws.bnd_n0) {
    WS(hipStreamSynchronize(s), "align: workspace");
    (void)hipFree(ws.bnd.p);
    ws.bnd = PlaneWorkspace::Buf{};
    WS(ws_grow(ws.bnd, boundary_ints(L.ks, L.lds_n0) * 4, false, s), "align: workspace");
    ws.boundary = carve_boundary(L.ks, L.lds_n0, (int*)ws.bnd.p);
    ws.bnd_n0 = L.lds_n0;
    WS(launch_init_boundary(L.ks, ws.boundary, s), "align: boundary");
  }
  WS(hipStreamSynchronize(s), "align: workspace");  // the previous run's host copies
  ws.h_desc.swap(L.desc);
  ws.h_jobs.swap(L.jobs);
  WS(hipMemcpyAsync(ws.desc.p, ws.h_desc.data(), n * sizeof(TripletDesc), hipMemcpyHostToDevice, s),
     "align: upload");
  WS(hipMemcpyAsync(ws.jobs.p, ws.h_jobs.data(), ws.h_jobs.size() * sizeof(JobDesc),
                    hipMemcpyHostToDevice, s),
     "align: upload");
  WS(hipMemcpyAsync(ws.plane_off.p, plane_off, n * 8, hipMemcpyHostToDevice, s), "align: upload");
  if (nwords) WS(hipMemcpyAsync(ws.words.p, words, nwords * 4, hipMemcpyHostToDevice, s), "align: upload");
  int* ctl = (int*)ws.ctl.p;
  WS(launch_prepare(ctl, ctl + 64, nullptr, 0, (int*)ws.pool.p, ws.pool.bytes / 4, L.tag_step, s), "align: prepare");
  SweepArgs a = make_sweep_args((const uint32_t*)ws.words.p, (const TripletDesc*)ws.desc.p,
                                (const JobDesc*)ws.jobs.p, (uint32_t)ws.h_jobs.size(), L.lds_n0,
                                (int32_t*)ws.scores.p, ctl + 64, ctl, (int*)ws.face.p, L.face_stride,
                                (int*)ws.pool.p, ws.boundary, nullptr, make_dev_scoring(sc));
  a.plane = (int*)ws.plane.p;
  a.plane_off = (const uint64_t*)ws.plane_off.p;
  WS(launch_sweep(L.ks, L.modes, a, grid, s), "align: sweep");
#undef WS
  return TRIOSEQ_OK;
}

}  // namespace trioseq

extern "C" {

static trioseq_status trioseq_plan_create_body(const uint32_t* lens, const uint64_t* word_off, size_t n,
                                   const trioseq_scoring* scp, const trioseq_plan_options* opts,
                                   trioseq_plan** out) {
  return plan_create_impl(lens, word_off, n, scp, opts, out);
}

static hipError_t plan_enqueue(trioseq_plan* p, const uint32_t* d_words, int32_t* d_scores,
                               hipStream_t s) {
  if (p->n == 0) return hipSuccess;
  hipError_t e;
  const bool pk_panel = p->modes == kModePkPanel;
  // The int32 halves are gathered in every run (the gather kernel also prepares
  // the run when there are no reduction pairs to reset); packed jobs read them
  // from the caller's words in place.
  const bool gather = p->half && !pk_panel;
  if ((!gather || p->red_pairs) &&
      (e = launch_prepare(p->d_ctl, p->d_counter, p->d_red, p->red_pairs, p->d_pface, p->pool_ints, p->tag_step, s)) != hipSuccess)
    return e;
  if (gather &&
      (e = launch_gather(d_words, p->d_gather, 6, p->h_words_n, p->d_hwords, p->red_pairs ? nullptr : p->d_ctl,
                         p->d_counter, p->d_pface, p->pool_ints, s)) != hipSuccess)
    return e;
  SweepArgs a = make_sweep_args(gather ? p->d_hwords : d_words, p->d_desc, p->d_jobs, p->njobs, p->lds_n0,
                                gather ? p->d_hscores : d_scores, p->d_counter, p->d_ctl, p->d_face,
                                p->face_stride, p->d_pface, p->bnd, p->d_red, p->sc);
  const int* pk_left = p->d_pkbnd + p->pk_top_words;
  if (p->half) {
    a.plane = p->d_plane;
    a.plane_off = p->d_plane_off;
  }
  if (pk_panel) {
    e = launch_panel_pk(p->sc.kind, p->pk_self, a, p->pk_base, p->pk_kc, p->pk_reuse, p->grid, s);
  } else if (p->packed) {
    e = launch_sweep_pk(p->ks, p->sc.kind, a, p->d_pkbnd, pk_left, p->pk_base, p->pk_kc, p->grid, s);
  } else {
    e = launch_sweep(p->ks, p->modes, a, p->grid, s);
  }
  if (e != hipSuccess || !p->half) return e;
  // The planes of the halves meet. Under local scoring the score is the best
  // of the crossing paths and the halves' own bests.
  const int* own = p->sc.kind == kGlobal ? nullptr : pk_panel ? p->d_red : p->d_hscores;
  return launch_meet(p->d_sdesc, p->d_chunk_box, p->h_nchunk, p->d_plane, p->d_partial, p->d_ctl + 1, own,
                     pk_panel ? 2 : 1, pk_panel ? (int)p->pk_kc : 0, p->d_meet ? p->d_meet : p->d_ctl + 2, d_scores, s);
}

trioseq_status trioseq_plan_run(trioseq_plan* p, const uint32_t* d_words, int32_t* d_scores,
                                void* hip_stream) {
  if (!p) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan_run: plan is NULL");
  if (p->n && (!d_words || !d_scores))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "plan_run: NULL device buffer");
  hipStream_t s = (hipStream_t)hip_stream;
  if (!p->use_graph) {
    TRIOSEQ_HIP(plan_enqueue(p, d_words, d_scores, s), "kernel launch");
    return TRIOSEQ_OK;
  }
  if (!p->gexec || p->g_words != d_words || p->g_scores != d_scores) {
    if (p->gexec) {
      (void)hipGraphExecDestroy(p->gexec);
      p->gexec = nullptr;
    }
    if (p->graph) {
      (void)hipGraphDestroy(p->graph);
      p->graph = nullptr;
    }
    TRIOSEQ_HIP(hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal),
                "hipStreamBeginCapture");
    hipError_t le = plan_enqueue(p, d_words, d_scores, p->cap_stream);
    hipError_t ce = hipStreamEndCapture(p->cap_stream, &p->graph);
    if (le != hipSuccess) return fail_hip(le, "kernel launch during capture");
    if (ce != hipSuccess) return fail_hip(ce, "hipStreamEndCapture");
    TRIOSEQ_HIP(hipGraphInstantiate(&p->gexec, p->graph, nullptr, nullptr, 0), "hipGraphInstantiate");
    p->g_words = d_words;
    p->g_scores = d_scores;
  }
  TRIOSEQ_HIP(hipGraphLaunch(p->gexec, s), "hipGraphLaunch");
  return TRIOSEQ_OK;
}

trioseq_status trioseq_plan_get_info(const trioseq_plan* p, trioseq_plan_info* info) {
  if (!p || !info) return fail(TRIOSEQ_ERR_INVALID_ARG, "plan_get_info: NULL pointer");
  info->engine = p->engine;
  info->tile_rows = p->ks.rj;
  info->tile_cols = p->ks.rk;
  info->grid = p->grid;
  info->waves_per_cu = p->waves_per_cu;
  info->panels = p->panels;
  info->packed = p->packed ? 1 : 0;
  info->workspace_bytes = p->workspace_bytes;
  info->cells = p->cells;
  return TRIOSEQ_OK;
}

trioseq_status trioseq_plan_destroy(trioseq_plan* p) {
  plan_free(p);
  return TRIOSEQ_OK;
}

// Host packing threads: batches of at least kPackParallelMin residues are
// split over up to kPackThreadsMax threads (the calling one included).
constexpr uint64_t kPackParallelMin = 1u << 20;
constexpr size_t kPackThreadsMax = 16;

// Validates and packs host ASCII triplets into one word array.
static trioseq_status pack_triplets(const trioseq_triplet* t, size_t n, std::vector<uint32_t>* lens,
                                    std::vector<uint64_t>* offs, std::vector<uint32_t>* words) {
  if (n && !t) return fail(TRIOSEQ_ERR_INVALID_ARG, "triplet array is NULL");
  lens->resize(3 * n);
  offs->resize(3 * n);
  for (size_t q = 0; q < n; ++q)
    for (int s = 0; s < 3; ++s) {
      (*lens)[3 * q + s] = t[q].len[s];
      if (t[q].len[s] && !t[q].seq[s])
        return fail(TRIOSEQ_ERR_INVALID_ARG,
                    "triplet " + std::to_string(q) + ": sequence " + std::to_string(s) + " is NULL");
    }
  uint64_t total = 0;
  trioseq_packed_layout(lens->data(), n, offs->data(), &total);
  words->assign(std::max<uint64_t>(total, 1), 0u);
  // Large batches are packed by several host threads, each over a run of
  // whole triplets of about equal residue count. Each records its first bad
  // sequence; the first over all is packed again here for its message
  // (messages are per thread).
  const uint64_t residues = 16 * total;
  const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
  const size_t nthreads = residues < kPackParallelMin ? 1 : std::min<size_t>({hw, kPackThreadsMax, n});
  std::vector<size_t> first_bad(nthreads, SIZE_MAX);
  auto pack_range = [&](size_t th, size_t q0, size_t q1) {
    for (size_t q = q0; q < q1; ++q)
      for (int s = 0; s < 3; ++s) {
        bool ok = false;
        try {  // nothing may leave a worker thread
          ok = trioseq_pack(t[q].seq[s], t[q].len[s], words->data() + (*offs)[3 * q + s]) == TRIOSEQ_OK;
        } catch (...) {
        }
        if (!ok) {
          first_bad[th] = 3 * q + s;
          return;
        }
      }
  };
  std::vector<std::thread> pool;
  size_t q0 = 0;
  for (size_t th = 0; th < nthreads; ++th) {
    // Triplets that start before the (th+1)-th share of the words; the last
    // range runs on this thread, and so does any range whose thread could
    // not be started.
    const uint64_t goal = total * (th + 1) / nthreads;
    size_t q1 = q0;
    while (q1 < n && (th + 1 == nthreads || (*offs)[3 * q1] < goal)) ++q1;
    bool started = false;
    if (th + 1 < nthreads) {
      try {
        pool.emplace_back(pack_range, th, q0, q1);
        started = true;
      } catch (...) {
      }
    }
    if (!started) pack_range(th, q0, q1);
    q0 = q1;
  }
  for (std::thread& th : pool) th.join();
  const size_t bad = *std::min_element(first_bad.begin(), first_bad.end());
  if (bad != SIZE_MAX) {
    const size_t q = bad / 3;
    const int s = (int)(bad % 3);
    const trioseq_status st = trioseq_pack(t[q].seq[s], t[q].len[s], words->data() + (*offs)[bad]);
    return fail(st, "triplet " + std::to_string(q) + ", sequence " + std::to_string(s) + ": " + g_err);
  }
  return TRIOSEQ_OK;
}

// trioseq_score_batch_packed: this thread's last plan, reused while the
// batch (lengths, word offsets, scoring, device) stays the same. It is never
// freed at thread exit (the HIP runtime may already be gone then).
struct PackedCache {
  std::vector<uint32_t> lens;
  std::vector<uint64_t> offs;
  trioseq_scoring sc{};
  int device = -1;
  trioseq_plan* plan = nullptr;
  hipStream_t stream = nullptr;  // where the plan last ran
};
static thread_local PackedCache* g_packed = nullptr;

static trioseq_status score_batch_packed_body(const uint32_t* d_words, const uint64_t* d_word_off,
                                              const uint32_t* d_len, size_t n, const trioseq_scoring* sc,
                                              int32_t* d_scores, void* hip_stream) {
  if (!sc) return fail(TRIOSEQ_ERR_INVALID_ARG, "score_batch_packed: scoring is NULL");
  if (n && (!d_words || !d_word_off || !d_len || !d_scores))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "score_batch_packed: NULL device buffer");
  trioseq_status st = validate_scoring(sc);
  if (st != TRIOSEQ_OK) return st;
  if (n == 0) return TRIOSEQ_OK;
  hipStream_t s = (hipStream_t)hip_stream;
  std::vector<uint32_t> lens(3 * n);
  std::vector<uint64_t> offs(3 * n);
  hipError_t e;
  if ((e = hipMemcpyAsync(lens.data(), d_len, 3 * n * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(offs.data(), d_word_off, 3 * n * 8, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return fail_hip(e, "score_batch_packed: reading lengths");
  int device = 0;
  TRIOSEQ_HIP(hipGetDevice(&device), "hipGetDevice");
  if (!g_packed) g_packed = new PackedCache;
  PackedCache& c = *g_packed;
  const bool same = c.plan && c.device == device && c.lens == lens && c.offs == offs &&
                    std::memcmp(&c.sc, sc, sizeof *sc) == 0;
  if (!same) {
    trioseq_plan* plan = nullptr;
    st = trioseq_plan_create(lens.data(), offs.data(), n, sc, nullptr, &plan);
    if (st != TRIOSEQ_OK) return st;
    if (c.plan) {
      // The old plan's workspace may still be in use on the stream it ran on.
      (void)hipStreamSynchronize(c.stream);
      trioseq_plan_destroy(c.plan);
    }
    c.plan = plan;
    c.lens.swap(lens);
    c.offs.swap(offs);
    c.sc = *sc;
    c.device = device;
  }
  // Runs of one plan share its workspace: a run on another stream waits for
  // the previous one.
  if (c.stream != s) (void)hipStreamSynchronize(c.stream);
  c.stream = s;
  return trioseq_plan_run(c.plan, d_words, d_scores, hip_stream);
}

}  // extern "C"

namespace trioseq {

trioseq_status score_packed_in_region(const uint32_t* d_words, const uint64_t* d_word_off,
                                      const uint32_t* d_len, size_t n, const trioseq_scoring* sc,
                                      int32_t* d_scores, const PlanMemory& mem) {
  if (!sc) return fail(TRIOSEQ_ERR_INVALID_ARG, "score_batch_packed_noalloc: scoring is NULL");
  if (n && (!d_words || !d_word_off || !d_len || !d_scores))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "score_batch_packed_noalloc: NULL device buffer");
  trioseq_status st = validate_scoring(sc);
  if (st != TRIOSEQ_OK) return st;
  if (n == 0) return TRIOSEQ_OK;
  // Host copies of the lengths and offsets, in buffers of this thread that
  // only grow.
  static thread_local std::vector<uint32_t>* lens = nullptr;
  static thread_local std::vector<uint64_t>* offs = nullptr;
  if (!lens) lens = new std::vector<uint32_t>;
  if (!offs) offs = new std::vector<uint64_t>;
  lens->resize(3 * n);
  offs->resize(3 * n);
  hipError_t e;
  if ((e = hipMemcpyAsync(lens->data(), d_len, 3 * n * 4, hipMemcpyDeviceToHost, mem.stream)) != hipSuccess ||
      (e = hipMemcpyAsync(offs->data(), d_word_off, 3 * n * 8, hipMemcpyDeviceToHost, mem.stream)) !=
          hipSuccess ||
      (e = hipStreamSynchronize(mem.stream)) != hipSuccess)
    return fail_hip(e, "score_batch_packed_noalloc: reading lengths");
  trioseq_plan* plan = nullptr;
  st = plan_create_impl(lens->data(), offs->data(), n, sc, nullptr, &plan, &mem);
  if (st != TRIOSEQ_OK) return st;
  const hipError_t le = plan_enqueue(plan, d_words, d_scores, mem.stream);
  plan_free(plan);  // host bookkeeping only: the device buffers are the region's
  if (le != hipSuccess) return fail_hip(le, "score_batch_packed_noalloc: kernel launch");
  return TRIOSEQ_OK;
}

}  // namespace trioseq

extern "C" {

// trioseq_score / trioseq_score_batch: the plans (with their device inputs
// and outputs) of this thread's last few batch shapes, reused when the same
// lengths, scoring and device come again, so a repeated call only uploads,
// launches and downloads. Plans whose workspace exceeds kHostCacheBytes are
// freed after their call. Never freed at thread exit (the HIP runtime may
// already be gone then).
constexpr size_t kHostCacheEntries = 4;
constexpr uint64_t kHostCacheBytes = 4ull << 30;
struct HostBatchEntry {
  int device = -1;
  int engine = 0;
  uint64_t epoch = 0;
  std::vector<uint32_t> lens;
  trioseq_scoring sc{};
  trioseq_plan* plan = nullptr;
  uint32_t* d_words = nullptr;
  int32_t* d_scores = nullptr;
  uint64_t last_use = 0;
};
static thread_local std::vector<HostBatchEntry>* g_host_cache = nullptr;
static thread_local uint64_t g_host_clock = 0;

static void host_entry_free(HostBatchEntry& c) {
  (void)hipFree(c.d_words);
  (void)hipFree(c.d_scores);
  trioseq_plan_destroy(c.plan);
  c = HostBatchEntry{};
}

static trioseq_status run_host_batch(const trioseq_triplet* t, size_t n, const trioseq_scoring* sc,
                                     int32_t* scores, hipStream_t s, int engine) {
  if (n && !scores) return fail(TRIOSEQ_ERR_INVALID_ARG, "scores is NULL");
  trioseq_status st = validate_scoring(sc);
  if (st != TRIOSEQ_OK) return st;
  std::vector<uint32_t> lens, words;
  std::vector<uint64_t> offs;
  st = pack_triplets(t, n, &lens, &offs, &words);
  if (st != TRIOSEQ_OK) return st;
  if (n == 0) return TRIOSEQ_OK;
  // A cached plan is only looked for on a working device; otherwise
  // plan_create below validates the batch (before any device work) and
  // reports the problem.
  int device = -1;
  if (hipGetDevice(&device) != hipSuccess) device = -1;
  if (!g_host_cache) g_host_cache = new std::vector<HostBatchEntry>;
  std::vector<HostBatchEntry>& cache = *g_host_cache;
  const uint64_t epoch = g_tune_epoch.load(std::memory_order_relaxed);
  HostBatchEntry* hit = nullptr;
  for (HostBatchEntry& c : cache)
    if (device >= 0 && c.plan && c.device == device && c.engine == engine && c.epoch == epoch && c.lens == lens &&
        std::memcmp(&c.sc, sc, sizeof *sc) == 0)
      hit = &c;
  HostBatchEntry fresh;
  if (!hit) {
    trioseq_plan_options o{engine, 0, 0, 0, 0, 0};
    st = trioseq_plan_create(lens.data(), offs.data(), n, sc, &o, &fresh.plan);
    if (st != TRIOSEQ_OK) return st;
    hipError_t e = hipMalloc((void**)&fresh.d_words, words.size() * 4);
    if (e == hipSuccess) e = hipMalloc((void**)&fresh.d_scores, n * 4);
    if (e != hipSuccess) {
      host_entry_free(fresh);
      return fail_hip(e, "batch: device buffers");
    }
    fresh.device = device;
    fresh.engine = engine;
    fresh.epoch = epoch;
    fresh.lens = lens;
    fresh.sc = *sc;
    hit = &fresh;
  }
  hit->last_use = ++g_host_clock;
  hipError_t e = hipMemcpyAsync(hit->d_words, words.data(), words.size() * 4, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) {
    st = trioseq_plan_run(hit->plan, hit->d_words, hit->d_scores, s);
    if (st == TRIOSEQ_OK) {
      e = hipMemcpyAsync(scores, hit->d_scores, n * 4, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
    }
  }
  if (hit == &fresh) {
    // Keep it when it is small enough, in place of the least recently used.
    if (st == TRIOSEQ_OK && e == hipSuccess && fresh.plan->workspace_bytes <= kHostCacheBytes) {
      if (cache.size() < kHostCacheEntries) {
        cache.push_back(std::move(fresh));
      } else {
        HostBatchEntry* lru = &cache[0];
        for (HostBatchEntry& c : cache)
          if (c.last_use < lru->last_use) lru = &c;
        host_entry_free(*lru);
        *lru = std::move(fresh);
      }
    } else {
      host_entry_free(fresh);
    }
  }
  if (st != TRIOSEQ_OK) return st;
  if (e != hipSuccess) return fail_hip(e, "batch");
  return TRIOSEQ_OK;
}

static trioseq_status trioseq_autotune_body(const uint32_t* lens, const uint64_t* word_off, size_t n,
                                const trioseq_scoring* sc, const uint32_t* d_words, int32_t reps,
                                void* hip_stream, trioseq_tune_result* out) {
  if (!out || !sc || (n && (!lens || !d_words)))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "autotune: NULL pointer");
  if (n == 0) return fail(TRIOSEQ_ERR_INVALID_ARG, "autotune: empty batch");
  if (reps < 1) reps = 1;
  hipStream_t s = (hipStream_t)hip_stream;
  // Candidates: the reference in int32 lanes first, then every lane tile (the
  // panel a wave owns is 8 x 8 tiles) and register budget, the register lane
  // exchange, other split factors (which triplets of a batch become panel
  // jobs), strip workgroups, and for a lone triplet other half-split
  // thresholds. Options a layout ignores are not tried. A lone triplet's
  // defaults are packed lanes: a candidate of their own, as 16-bit values are
  // held against 32-bit ones and not the other way round.
  std::vector<trioseq_plan_options> cands;
  cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2, 0, 0, 0, 0, n == 1 ? 1 : 0});
  const size_t defaults = n == 1 ? 1 : 0;  // the candidate that plans without options run as
  if (n == 1) cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2});
  const int shapes[][3] = {{4, 4, 4}, {8, 4, 2}, {4, 8, 2}};
  for (const auto& sh : shapes) cands.push_back(trioseq_plan_options{-1, sh[0], sh[1], 0, 0, sh[2]});
  if (sc->kind == kGlobal) {
    cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2, 0, 2});
    cands.push_back(trioseq_plan_options{-1, 8, 4, 0, 0, 2, 0, 2});
  }
  if (n > 1) {
    for (int f : {2, 8, 16}) cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2, 0, 0, f});
    // Packed shapes: tile, waves per SIMD, lane exchange, staging (the
    // other kinds have the plain forms only).
    const int pks[][5] = {{4, 4, 2, 0, 0}, {4, 4, 3, 0, 0}, {8, 4, 2, 0, 0}, {4, 8, 2, 0, 0},
                          {4, 4, 2, 2, 0}, {4, 4, 2, 0, 2}, {4, 4, 3, 0, 2}, {8, 4, 2, 0, 2},
                          {4, 8, 2, 0, 2}};
    for (const auto& sh : pks)
      if (sc->kind == kGlobal || (sh[3] == 0 && sh[4] == 0))
        cands.push_back(trioseq_plan_options{-1, sh[0], sh[1], 0, 0, sh[2], 0, sh[3], 0, 0, 2, sh[4]});
  } else {
    cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2, 4});
    if (sc->kind == kGlobal)
      for (int h : {-1, 128, 512}) cands.push_back(trioseq_plan_options{-1, 4, 4, 0, 0, 2, 0, 0, 0, h});
  }
  int32_t* d_ref = nullptr;
  int32_t* d_out = nullptr;
  TRIOSEQ_HIP(hipMalloc((void**)&d_ref, n * 4), "hipMalloc");
  hipError_t e = hipMalloc((void**)&d_out, n * 4);
  if (e != hipSuccess) {
    (void)hipFree(d_ref);
    return fail_hip(e, "hipMalloc");
  }
  std::vector<int32_t> ref(n), got(n);
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  (void)hipEventCreate(&ev0);
  (void)hipEventCreate(&ev1);
  trioseq_tune_result r{};
  r.best_ms = 1e300;
  trioseq_status st = TRIOSEQ_OK;
  for (size_t c = 0; c < cands.size() && st == TRIOSEQ_OK; ++c) {
    trioseq_plan_options o = cands[c];
    trioseq_plan* plan = nullptr;
    // Shapes that need more registers than a budget allows are skipped.
    if (trioseq_plan_create(lens, word_off, n, sc, &o, &plan) != TRIOSEQ_OK) continue;
    trioseq_plan_info info;
    trioseq_plan_get_info(plan, &info);
    int32_t* dst = c == 0 ? d_ref : d_out;
    st = trioseq_plan_run(plan, d_words, dst, s);  // warm-up, and the scores to compare
    if (st == TRIOSEQ_OK && (e = hipStreamSynchronize(s)) != hipSuccess) st = fail_hip(e, "autotune");
    float ms = 0;
    if (st == TRIOSEQ_OK) {
      (void)hipEventRecord(ev0, s);
      for (int k = 0; k < reps && st == TRIOSEQ_OK; ++k) st = trioseq_plan_run(plan, d_words, d_out, s);
      (void)hipEventRecord(ev1, s);
      if (st == TRIOSEQ_OK && (e = hipEventSynchronize(ev1)) != hipSuccess) st = fail_hip(e, "autotune");
      (void)hipEventElapsedTime(&ms, ev0, ev1);
      ms /= (float)reps;
    }
    trioseq_plan_destroy(plan);
    if (st != TRIOSEQ_OK) break;
    ++r.tried;
    if (c == 0) {
      if ((e = hipMemcpy(ref.data(), d_ref, n * 4, hipMemcpyDeviceToHost)) != hipSuccess) {
        st = fail_hip(e, "autotune");
        break;
      }
      r.reference_ms = ms;  // (of a lone triplet until its defaults agree)
    } else {
      if ((e = hipMemcpy(got.data(), d_out, n * 4, hipMemcpyDeviceToHost)) != hipSuccess) {
        st = fail_hip(e, "autotune");
        break;
      }
      if (got != ref) {  // parity gate: never pick a configuration that disagrees
        ++r.rejected;
        continue;
      }
      if (c == defaults) r.reference_ms = ms;
    }
    if (ms < r.best_ms) {
      r.best_ms = ms;
      r.best = cands[c];
      r.best.tile_rows = info.tile_rows;
      r.best.tile_cols = info.tile_cols;
      r.best.waves_per_simd = c == defaults ? 0 : cands[c].waves_per_simd;
    }
    if (std::getenv("TRIOSEQ_TUNE_LOG"))
      std::fprintf(stderr, "autotune: %dx%d wpe %d xch %d group %d split %d half %d packed %d staging %d: %.4f ms\n",
                   info.tile_rows, info.tile_cols, cands[c].waves_per_simd, cands[c].lane_exchange,
                   cands[c].panel_group, cands[c].split_factor, cands[c].half_split_min, info.packed,
                   cands[c].staging, ms);
  }
  (void)hipEventDestroy(ev0);
  (void)hipEventDestroy(ev1);
  (void)hipFree(d_ref);
  (void)hipFree(d_out);
  if (st != TRIOSEQ_OK) return st;
  if (r.tried == 0) return fail(TRIOSEQ_ERR_DEVICE, "autotune: no configuration could be planned");
  if (r.best.waves_per_simd) remember_tuned(length_profile(lens, n, sc->kind), r.best);
  *out = r;
  return TRIOSEQ_OK;
}

static trioseq_status trioseq_score_body(const trioseq_triplet* t, const trioseq_scoring* sc, int32_t* score) {
  if (!t || !score) return fail(TRIOSEQ_ERR_INVALID_ARG, "score: NULL pointer");
  return run_host_batch(t, 1, sc, score, nullptr, -1);
}

static trioseq_status trioseq_score_batch_body(const trioseq_triplet* t, size_t n, const trioseq_scoring* sc,
                                   int32_t* scores, void* hip_stream) {
  return run_host_batch(t, n, sc, scores, (hipStream_t)hip_stream, -1);
}

}  // extern "C"

// Entry points: every body runs guarded (no exception crosses the ABI).
extern "C" {

trioseq_status trioseq_plan_create(const uint32_t* lens, const uint64_t* word_off, size_t n, const trioseq_scoring* scp, const trioseq_plan_options* opts, trioseq_plan** out) {
  return guarded([&] { return trioseq_plan_create_body(lens, word_off, n, scp, opts, out); });
}

trioseq_status trioseq_autotune(const uint32_t* lens, const uint64_t* word_off, size_t n, const trioseq_scoring* sc, const uint32_t* d_words, int32_t reps, void* hip_stream, trioseq_tune_result* out) {
  return guarded([&] { return trioseq_autotune_body(lens, word_off, n, sc, d_words, reps, hip_stream, out); });
}

trioseq_status trioseq_score(const trioseq_triplet* t, const trioseq_scoring* sc, int32_t* score) {
  return guarded([&] { return trioseq_score_body(t, sc, score); });
}

trioseq_status trioseq_score_batch_packed(const uint32_t* d_words, const uint64_t* d_word_off,
                                          const uint32_t* d_len, size_t n, const trioseq_scoring* sc,
                                          int32_t* d_scores, void* hip_stream) {
  return guarded([&] {
    return score_batch_packed_body(d_words, d_word_off, d_len, n, sc, d_scores, hip_stream);
  });
}

trioseq_status trioseq_score_batch(const trioseq_triplet* t, size_t n, const trioseq_scoring* sc, int32_t* scores, void* hip_stream) {
  return guarded([&] { return trioseq_score_batch_body(t, n, sc, scores, hip_stream); });
}

}  // extern "C"
