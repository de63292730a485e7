// Traceback: optimal global alignments of triplets (paper, Section II, Eq. 1;
// the paper returns alignments by Hirschberg's linear-space divide and
// conquer), computed level by level on the GPU for a whole batch at once:
//  * every box (sub-problem) larger than kLeafCells table cells is halved on
//    its longest axis; one batched plane run per level sweeps, for every such
//    box, the first half forward and the second half reversed, and k_split
//    picks where an optimal alignment of the box crosses the middle slice;
//  * the remaining small boxes are solved whole by k_leaf (table and walk
//    back), and their columns, in path order, are the alignment.
// The host only lays out the boxes, moves data and formats the rows.
// A level sweeps packed panel jobs, the two halves of a box in one register,
// where the values fit 16 bits (split_level_packed), int32 jobs otherwise.
#include <algorithm>
#include <array>
#include <cstring>
#include <numeric>
#include <string>
#include <vector>

#include "common.h"

namespace trioseq {
namespace {

struct Box {
  uint32_t trip;
  uint32_t lo[3], hi[3];
  uint64_t cells() const {
    return (uint64_t)(hi[0] - lo[0] + 1) * (hi[1] - lo[1] + 1) * (hi[2] - lo[2] + 1);
  }
  uint64_t corner() const { return (uint64_t)lo[0] + lo[1] + lo[2]; }
};

template <class T>
T* as(const PlaneWorkspace::Buf& b) {
  return (T*)b.p;
}

// Appends codes[from, to) (reversed if asked), packed 16 per word from a
// fresh word; returns its word offset.
uint64_t pack_range(const std::vector<uint8_t>& codes, uint32_t from, uint32_t to, bool reverse,
                    std::vector<uint32_t>& words) {
  const uint64_t off = words.size();
  const uint32_t n = to - from;
  words.resize(off + (n + 15) / 16, 0u);
  for (uint32_t p = 0; p < n; ++p) {
    const uint8_t c = reverse ? codes[to - 1 - p] : codes[from + p];
    words[off + p / 16] |= (uint32_t)c << (2 * (p % 16));
  }
  return off;
}

trioseq_status hip_err(hipError_t e, const char* what) { return fail_hip(e, what); }

// Leaves solved per k_leaf launch (bounds the column buffers of a launch).
constexpr size_t kLeavesPerLaunch = 1 << 18;

// Traceback workspace of this thread (see align_batch_impl).
constexpr uint64_t kKeepBytes = 2ull << 30;
thread_local PlaneWorkspace* g_ws = nullptr;
thread_local int g_ws_device = -1;

// The axes of a box's split: the halved (longest) one, then the plane's rows and
// columns; mid = where it is halved.
struct Split {
  int ax, r, c;
  uint32_t mid;
};
Split split_of(const Box& b) {
  Split q;
  q.ax = 0;
  for (int a = 1; a < 3; ++a)
    if (b.hi[a] - b.lo[a] > b.hi[q.ax] - b.lo[q.ax]) q.ax = a;
  q.r = q.ax == 0 ? 1 : 0;
  q.c = q.ax == 2 ? 1 : 2;
  q.mid = b.lo[q.ax] + (b.hi[q.ax] - b.lo[q.ax]) / 2;
  return q;
}

// Takes a level's split points (out[3q] = score, out[3q + 1], out[3q + 2] = the
// cell of box q's middle slice, negative if the level's sweep gave up): the boxes' halves go to `next`.
// root_score[t] is set when the box is triplet t's root (its first split).
trioseq_status take_splits(const std::vector<Box>& boxes, const int* out, std::vector<char>& split_seen,
                           std::vector<int32_t>& root_score, std::vector<Box>& next) {
  for (size_t q = 0; q < boxes.size(); ++q) {
    const Box& b = boxes[q];
    const Split sp = split_of(b);
    if (out[3 * q + 1] < 0) return fail(TRIOSEQ_ERR_DEVICE, "align: a wait of the sweep gave up");
    const uint32_t p = (uint32_t)out[3 * q + 1], pc = (uint32_t)out[3 * q + 2];
    if (p > b.hi[sp.r] - b.lo[sp.r] || pc > b.hi[sp.c] - b.lo[sp.c])
      return fail(TRIOSEQ_ERR_DEVICE, "align: split point outside its box");
    if (!split_seen[b.trip]) {  // a triplet's first split is of its root box
      split_seen[b.trip] = 1;
      root_score[b.trip] = out[3 * q];
    }
    Box left = b, right = b;
    left.hi[sp.ax] = sp.mid;
    right.lo[sp.ax] = sp.mid;
    left.hi[sp.r] = right.lo[sp.r] = b.lo[sp.r] + p;
    left.hi[sp.c] = right.lo[sp.c] = b.lo[sp.c] + pc;
    next.push_back(left);
    next.push_back(right);
  }
  return TRIOSEQ_OK;
}

// One level on packed panel jobs: the two halves of a box are a pair, read in
// place from the sequences uploaded once (words at ws.lwords, soff). All
// tables of the level go up in one copy and the split points come back in mapped
// host memory. *done = false, with nothing launched, if a box's values do not
// fit 16 bits. (The alignment of 1024 x 1000 x
// 1048: 2.69 -> 1.60 ms, with the leaves' kernel.)
trioseq_status split_level_packed(PlaneWorkspace& ws, const std::vector<Box>& boxes,
                                  const std::vector<uint64_t>& soff, const trioseq_scoring& sc,
                                  std::vector<char>& split_seen, std::vector<int32_t>& root_score,
                                  std::vector<Box>& next, hipStream_t s, bool* done) {
  *done = false;
  const size_t nb = boxes.size();
  std::vector<TripletDesc> desc(2 * nb);
  std::vector<uint64_t> poff(2 * nb);
  std::vector<SplitDesc> sd(nb);
  std::vector<uint32_t> chunk_box;
  uint64_t pints = 0;
  for (size_t q = 0; q < nb; ++q) {
    const Box& b = boxes[q];
    const Split sp = split_of(b);
    const int order[3] = {sp.ax, sp.r, sp.c};
    for (int h = 0; h < 2; ++h) {
      TripletDesc& d = desc[2 * q + h];
      d = TripletDesc{};
      for (int k = 0; k < 3; ++k) {
        const int a = order[k];
        const uint32_t lo = k == 0 && h ? sp.mid : b.lo[a], hi = k == 0 && !h ? sp.mid : b.hi[a];
        d.off[k] = soff[3 * b.trip + a];
        d.start[k] = lo;
        d.len[k] = hi - lo;
      }
      d.rev = (uint32_t)h;
    }
    const uint32_t rows = b.hi[sp.r] - b.lo[sp.r] + 1, cols = b.hi[sp.c] - b.lo[sp.c] + 1;
    const uint64_t cells = (uint64_t)rows * cols;
    poff[2 * q] = pints;
    poff[2 * q + 1] = pints + cells;
    const uint32_t nchunk = (uint32_t)((cells + kSplitChunk - 1) / kSplitChunk);
    sd[q] = SplitDesc{pints, pints + cells, rows, cols, (uint32_t)chunk_box.size(), nchunk, 0};
    chunk_box.insert(chunk_box.end(), nchunk, (uint32_t)q);
    pints += 2 * cells;
  }
  Layout L;
  if (!pair_panel_layout(desc, sc, true, &L)) return TRIOSEQ_OK;
  hipError_t e;
#define AL(call)                                                      \
  do {                                                                \
    if ((e = (call)) != hipSuccess) return hip_err(e, "align: level"); \
  } while (0)
  if (!ws.have_props) {
    trioseq_status st = device_props(&ws.dp);
    if (st != TRIOSEQ_OK) return st;
    ws.have_props = true;
  }
  int grid = 0, wpc = 0;
  trioseq_status st = layout_grid(L, ws.dp, 0, &grid, &wpc);
  if (st != TRIOSEQ_OK) return st;
  const size_t nc = chunk_box.size();
  uint64_t at[6] = {0};
  const uint64_t part[5] = {2 * nb * sizeof(TripletDesc), L.jobs.size() * sizeof(JobDesc), 2 * nb * 8,
                            nb * sizeof(SplitDesc), nc * 4};
  for (int k = 0; k < 5; ++k) at[k + 1] = (at[k] + part[k] + 15) & ~15ull;
  const void* src[5] = {L.desc.data(), L.jobs.data(), poff.data(), sd.data(), chunk_box.data()};
  if (ws.h_stage_bytes < at[5]) {
    (void)hipHostFree(ws.h_stage);
    ws.h_stage = nullptr;
    ws.h_stage_bytes = 0;
    const uint64_t cap = at[5] + at[5] / 4 + 4096;
    AL(hipHostMalloc((void**)&ws.h_stage, cap, 0));
    ws.h_stage_bytes = cap;
  }
  if (ws.h_out_ints < 3 * nb) {
    (void)hipHostFree(ws.h_out);
    ws.h_out = nullptr;
    ws.h_out_ints = 0;
    const uint64_t cap = 3 * nb + 3 * nb / 4 + 256;
    AL(hipHostMalloc((void**)&ws.h_out, cap * 4, hipHostMallocMapped));
    AL(hipHostGetDevicePointer((void**)&ws.d_out, ws.h_out, 0));
    ws.h_out_ints = cap;
  }
  for (int k = 0; k < 5; ++k)
    if (part[k]) std::memcpy(ws.h_stage + at[k], src[k], part[k]);
  if (!ws.ctl.p) AL(ws_grow(ws.ctl, 256 + kCounterBytes, true, s));
  AL(ws_grow(ws.tables, at[5], false, s));
  AL(ws_grow(ws.pool, L.pool_ints * 4, true, s));
  AL(ws_grow(ws.plane, pints * 4, false, s));
  AL(ws_grow(ws.scores, 256, false, s));
  AL(ws_grow(ws.partial, nc * 8, false, s));
  char* t = (char*)ws.tables.p;
  AL(hipMemcpyAsync(t, ws.h_stage, at[5], hipMemcpyHostToDevice, s));
  int* ctl = as<int>(ws.ctl);
  AL(launch_prepare(ctl, ctl + 64, nullptr, 0, as<int>(ws.pool), ws.pool.bytes / 4, L.tag_step, s));
  SweepArgs a = make_sweep_args(as<uint32_t>(ws.lwords), (const TripletDesc*)(t + at[0]), (const JobDesc*)(t + at[1]),
                                (uint32_t)L.jobs.size(), L.lds_n0, as<int32_t>(ws.scores), ctl + 64, ctl, nullptr, 0,
                                as<int>(ws.pool), Boundary{}, nullptr, make_dev_scoring(sc));
  a.plane = as<int>(ws.plane);
  a.plane_off = (const uint64_t*)(t + at[2]);
  AL(launch_panel_pk(kGlobal, L.pk_self, a, L.pk_base, L.pk_kc, L.pk_reuse, grid, s));
  AL(launch_split(as<int>(ws.plane), (const SplitDesc*)(t + at[3]), (uint32_t)nb, (const uint32_t*)(t + at[4]),
                  (uint32_t)nc, as<int>(ws.partial), ctl + 1, ws.d_out, s));
  // The level's only wait: its split points are needed to lay out the next.
  AL(hipStreamSynchronize(s));
#undef AL
  *done = true;
  return take_splits(boxes, ws.h_out, split_seen, root_score, next);
}

// One level in int32 lanes: every box in `boxes` is split.
trioseq_status split_level(PlaneWorkspace& ws, const std::vector<Box>& boxes,
                           const std::vector<std::vector<uint8_t>>& codes, const trioseq_scoring& sc,
                           std::vector<char>& split_seen, std::vector<int32_t>& root_score,
                           std::vector<Box>& next, hipStream_t s) {
  const size_t nb = boxes.size();
  // Triplet 2q = first half of box q forward, 2q + 1 = second half reversed;
  // the halved axis is swept, the other two stay in index order.
  std::vector<uint32_t> lens(6 * nb), words;
  std::vector<uint64_t> offs(6 * nb), poff(2 * nb);
  std::vector<SplitDesc> sd(nb);
  std::vector<uint32_t> chunk_box;
  uint64_t pints = 0;
  for (size_t q = 0; q < nb; ++q) {
    const Box& b = boxes[q];
    const Split sp = split_of(b);
    const int ax = sp.ax, r = sp.r, c = sp.c;
    const uint32_t mid = sp.mid;
    const int order[3] = {ax, r, c};
    for (int half = 0; half < 2; ++half) {
      const size_t tr = 2 * q + half;
      for (int sidx = 0; sidx < 3; ++sidx) {
        const int a = order[sidx];
        uint32_t from = b.lo[a], to = b.hi[a];
        if (sidx == 0) (half == 0 ? to : from) = mid;
        lens[3 * tr + sidx] = to - from;
        offs[3 * tr + sidx] = pack_range(codes[3 * b.trip + a], from, to, half == 1, words);
      }
    }
    const uint32_t prow = b.hi[r] - b.lo[r] + 1, pcol = b.hi[c] - b.lo[c] + 1;
    poff[2 * q] = pints;
    pints += (uint64_t)prow * pcol;
    poff[2 * q + 1] = pints;
    pints += (uint64_t)prow * pcol;
    const uint32_t nchunk = (uint32_t)(((uint64_t)prow * pcol + kSplitChunk - 1) / kSplitChunk);
    sd[q] = SplitDesc{poff[2 * q], poff[2 * q + 1], prow, pcol, (uint32_t)chunk_box.size(), nchunk, 0};
    chunk_box.insert(chunk_box.end(), nchunk, (uint32_t)q);
  }
  trioseq_status st = run_planes(ws, lens.data(), offs.data(), 2 * nb, words.data(), words.size(), sc,
                                 poff.data(), pints, s);
  if (st != TRIOSEQ_OK) return st;
  std::vector<int> out(3 * nb);
  const size_t nchunks = chunk_box.size();
  hipError_t e;
  // The level's only wait: its split points are needed to lay out the next.
  if ((e = ws_grow(ws.sd, nb * sizeof(SplitDesc), false, s)) != hipSuccess ||
      (e = ws_grow(ws.split_out, 3 * nb * 4, false, s)) != hipSuccess ||
      (e = ws_grow(ws.chunk_box, nchunks * 4, false, s)) != hipSuccess ||
      (e = ws_grow(ws.partial, nchunks * 8, false, s)) != hipSuccess ||
      (e = hipMemcpyAsync(ws.sd.p, sd.data(), nb * sizeof(SplitDesc), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = hipMemcpyAsync(ws.chunk_box.p, chunk_box.data(), nchunks * 4, hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = launch_split((const int*)ws.plane.p, as<SplitDesc>(ws.sd), (uint32_t)nb, as<uint32_t>(ws.chunk_box),
                        (uint32_t)nchunks, as<int>(ws.partial), as<int>(ws.ctl) + 1, as<int>(ws.split_out),
                        s)) != hipSuccess ||
      (e = hipMemcpyAsync(out.data(), ws.split_out.p, 3 * nb * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return hip_err(e, "align: split");
  return take_splits(boxes, out.data(), split_seen, root_score, next);
}

// Solves leaves[first, first + n) with k_leaf; columns and scores to host.
trioseq_status solve_leaves(PlaneWorkspace& ws, const std::vector<Box>& leaves, size_t first, size_t n,
                            const std::vector<uint64_t>& soff, const trioseq_scoring& sc, std::vector<LeafDesc>& ld,
                            std::vector<uint8_t>& cols, std::vector<uint32_t>& ncols,
                            std::vector<int32_t>& lscore, hipStream_t s) {
  ld.assign(n, LeafDesc{});
  uint64_t col_bytes = 0;
  for (size_t q = 0; q < n; ++q) {
    const Box& b = leaves[first + q];
    if (b.cells() > kLeafCells) return fail(TRIOSEQ_ERR_DEVICE, "align: leaf larger than its table");
    for (int a = 0; a < 3; ++a) {
      ld[q].off[a] = soff[3 * b.trip + a];
      ld[q].lo[a] = b.lo[a];
      ld[q].len[a] = b.hi[a] - b.lo[a];
    }
    ld[q].out = col_bytes;
    col_bytes += 3ull * (ld[q].len[0] + ld[q].len[1] + ld[q].len[2]);
  }
  cols.assign(col_bytes, 0);
  ncols.assign(n, 0);
  lscore.assign(n, 0);
  hipError_t e;
  if ((e = ws_grow(ws.leaves, n * sizeof(LeafDesc), false, s)) != hipSuccess ||
      (e = ws_grow(ws.cols, col_bytes, false, s)) != hipSuccess ||
      (e = ws_grow(ws.ncols, n * 4, false, s)) != hipSuccess ||
      (e = ws_grow(ws.lscore, n * 4, false, s)) != hipSuccess)
    return hip_err(e, "align: leaf buffers");
  LeafArgs la;
  la.words = as<uint32_t>(ws.lwords);
  la.leaves = as<LeafDesc>(ws.leaves);
  la.n = (uint32_t)n;
  la.cols = as<uint8_t>(ws.cols);
  la.ncols = as<uint32_t>(ws.ncols);
  la.score = as<int32_t>(ws.lscore);
  for (int x = 0; x < 4; ++x)
    for (int y = 0; y < 4; ++y) la.sub[4 * x + y] = sc.sub[x][y];
  la.gap = sc.gap;
  if ((e = hipMemcpyAsync(ws.leaves.p, ld.data(), n * sizeof(LeafDesc), hipMemcpyHostToDevice, s)) !=
          hipSuccess ||
      (e = launch_leaf(la, s)) != hipSuccess ||
      (e = hipMemcpyAsync(cols.data(), ws.cols.p, col_bytes, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(ncols.data(), ws.ncols.p, n * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipMemcpyAsync(lscore.data(), ws.lscore.p, n * 4, hipMemcpyDeviceToHost, s)) != hipSuccess ||
      (e = hipStreamSynchronize(s)) != hipSuccess)
    return hip_err(e, "align: leaves");
  return TRIOSEQ_OK;
}

// rows: triplet u's row a at rows + 3 * cap_before[u] + a * cap[u].
trioseq_status align_batch_impl(const trioseq_triplet* t, size_t n, const trioseq_scoring& sc,
                                char* rows, uint32_t* ncols_out, int32_t* scores_out, hipStream_t s) {
  // The sequences, packed; uploaded once for all levels and the leaves.
  std::vector<uint32_t> words;
  std::vector<uint64_t> soff(3 * n);
  std::vector<uint64_t> cap(n), cap_before(n);
  uint64_t total_cap = 0;
  for (size_t u = 0; u < n; ++u) {
    for (int q = 0; q < 3; ++q) {
      if (t[u].len[q] && !t[u].seq[q]) return fail(TRIOSEQ_ERR_INVALID_ARG, "align: NULL sequence");
      if (t[u].len[q] > (uint32_t)kMaxSweepLen)
        return fail(TRIOSEQ_ERR_TOO_LARGE, "align: triplet " + std::to_string(u) +
                                               ": every length must be at most " +
                                               std::to_string(kMaxSweepLen));
      const uint64_t at = words.size();
      soff[3 * u + q] = at;
      words.resize(at + (t[u].len[q] + 15) / 16);
      if (trioseq_pack(t[u].seq[q], t[u].len[q], words.data() + at) != TRIOSEQ_OK)
        return fail(TRIOSEQ_ERR_BAD_RESIDUE, "align: residue outside ACGT");
    }
    trioseq_status st = check_range(sc, t[u].len[0], t[u].len[1], t[u].len[2], u);
    if (st != TRIOSEQ_OK) return st;
    cap[u] = (uint64_t)t[u].len[0] + t[u].len[1] + t[u].len[2];
    cap_before[u] = total_cap;
    total_cap += cap[u];
  }
  if (n == 0) return TRIOSEQ_OK;

  std::vector<Box> work, leaves;
  for (size_t u = 0; u < n; ++u) work.push_back(Box{(uint32_t)u, {0, 0, 0}, {t[u].len[0], t[u].len[1], t[u].len[2]}});
  std::vector<char> split_seen(n, 0);
  std::vector<int32_t> root_score(n, 0);
  // This thread's traceback workspace, kept from call to call (and from
  // level to level) so that a repeated alignment allocates nothing; one
  // grown past kKeepBytes is released when the call ends.
  int device = 0;
  TRIOSEQ_HIP(hipGetDevice(&device), "hipGetDevice");
  if (!g_ws || g_ws_device != device) {
    delete g_ws;  // the previous device's buffers (synchronous calls: idle)
    g_ws = new PlaneWorkspace;
    g_ws_device = device;
  }
  PlaneWorkspace& ws = *g_ws;
  struct Release {
    hipStream_t s;
    bool done = false;
    ~Release() {
      // (After an error work may still read the staged tables.)
      if (!done) (void)hipStreamSynchronize(s);
      if (g_ws && ws_bytes(*g_ws) > kKeepBytes) {
        delete g_ws;
        g_ws = nullptr;
      }
    }
  } release{s};
  hipError_t e = ws_grow(ws.lwords, words.size() * 4, false, s);
  if (e == hipSuccess && !words.empty())
    e = hipMemcpyAsync(ws.lwords.p, words.data(), words.size() * 4, hipMemcpyHostToDevice, s);
  if (e != hipSuccess) return hip_err(e, "align: sequences");
  std::vector<std::vector<uint8_t>> codes;  // of every sequence, for int32 levels
  while (!work.empty()) {
    std::vector<Box> boxes, next;
    for (const Box& b : work) (b.cells() <= kLeafCells ? leaves : boxes).push_back(b);
    if (boxes.empty()) break;
    bool done = false;
    trioseq_status st = split_level_packed(ws, boxes, soff, sc, split_seen, root_score, next, s, &done);
    if (st == TRIOSEQ_OK && !done && codes.empty()) {
      codes.resize(3 * n);
      for (size_t q = 0; q < 3 * n; ++q) {
        const trioseq_triplet& tr = t[q / 3];
        codes[q].resize(tr.len[q % 3]);
        for (uint32_t p = 0; p < tr.len[q % 3]; ++p) codes[q][p] = residue_code(tr.seq[q % 3][p]);
      }
    }
    if (st == TRIOSEQ_OK && !done) st = split_level(ws, boxes, codes, sc, split_seen, root_score, next, s);
    if (st != TRIOSEQ_OK) return st;
    work.swap(next);
  }

  // Leaves in path order per triplet: along an alignment every coordinate
  // grows, and a leaf holds at least one residue, so the sum of a leaf's
  // lower corner strictly increases from leaf to leaf.
  std::sort(leaves.begin(), leaves.end(), [](const Box& x, const Box& y) {
    return x.trip != y.trip ? x.trip < y.trip : x.corner() < y.corner();
  });
  std::vector<char> out(3 * total_cap);  // laid out like rows
  std::vector<uint32_t> len(n, 0);       // columns so far
  std::vector<std::array<uint32_t, 3>> used(n, {0, 0, 0});  // residues in each row
  std::vector<int64_t> sum(n, 0);
  static const char kLetter[8] = {'A', 'C', 'G', 'T', '-', '?', '?', '?'};
  std::vector<LeafDesc> ld;
  std::vector<uint8_t> cols;
  std::vector<uint32_t> ncols;
  std::vector<int32_t> lscore;
  for (size_t first = 0; first < leaves.size(); first += kLeavesPerLaunch) {
    const size_t cnt = std::min(kLeavesPerLaunch, leaves.size() - first);
    trioseq_status st = solve_leaves(ws, leaves, first, cnt, soff, sc, ld, cols, ncols, lscore, s);
    if (st != TRIOSEQ_OK) return st;
    for (size_t q = 0; q < cnt; ++q) {
      const uint32_t u = leaves[first + q].trip;
      const uint64_t most = (uint64_t)ld[q].len[0] + ld[q].len[1] + ld[q].len[2];
      if (ncols[q] > most) return fail(TRIOSEQ_ERR_DEVICE, "align: leaf wrote too many columns");
      sum[u] += lscore[q];
      const uint8_t* c = cols.data() + ld[q].out;
      if (len[u] + (uint64_t)ncols[q] > cap[u]) return fail(TRIOSEQ_ERR_DEVICE, "align: too many columns");
      uint8_t top = 0;
      for (int a = 0; a < 3; ++a) {
        char* r = out.data() + 3 * cap_before[u] + a * cap[u] + len[u];
        uint32_t res = 0;
        for (uint32_t k = 0; k < ncols[q]; ++k) {  // written last column first
          const uint8_t v = c[3 * (uint64_t)(ncols[q] - 1 - k) + a];
          top = std::max(top, v);
          r[k] = kLetter[v & 7];
          res += v < 4;
        }
        used[u][a] += res;
      }
      if (top > 4) return fail(TRIOSEQ_ERR_DEVICE, "align: bad column code");
      len[u] += ncols[q];
    }
  }
  // Checks before any output is written: the leaves' scores add up to the
  // alignment's score (the sum-of-pairs score is a sum over columns), which
  // must be the root box's optimum, and every row holds its whole sequence.
  for (size_t u = 0; u < n; ++u) {
    const int64_t total = split_seen[u] ? root_score[u] : sum[u];
    if (sum[u] != total) return fail(TRIOSEQ_ERR_DEVICE, "align: leaf scores do not add up to the optimum");
    for (int a = 0; a < 3; ++a)
      if (used[u][a] != t[u].len[a]) return fail(TRIOSEQ_ERR_DEVICE, "align: a row does not hold its whole sequence");
  }
  for (size_t u = 0; u < n; ++u) {
    for (int a = 0; a < 3; ++a) {
      const uint64_t at = 3 * cap_before[u] + a * cap[u];
      std::memcpy(rows + at, out.data() + at, len[u]);
    }
    ncols_out[u] = len[u];
    scores_out[u] = (int32_t)sum[u];
  }
  release.done = true;
  return TRIOSEQ_OK;
}

}  // namespace
}  // namespace trioseq

using namespace trioseq;

static trioseq_status trioseq_align_batch_body(const trioseq_triplet* t, size_t n,
                                              const trioseq_scoring* sc, char* rows, uint32_t* ncols,
                                              int32_t* scores, void* hip_stream) {
  if (!sc || (n && (!t || !rows || !ncols || !scores)))
    return fail(TRIOSEQ_ERR_INVALID_ARG, "align_batch: NULL pointer");
  trioseq_status st = validate_scoring(sc);
  if (st != TRIOSEQ_OK) return st;
  if (sc->kind != kGlobal) return fail(TRIOSEQ_ERR_INVALID_ARG, "align: only global alignments");
  return align_batch_impl(t, n, *sc, rows, ncols, scores, (hipStream_t)hip_stream);
}

static trioseq_status trioseq_align_body(const trioseq_triplet* t, const trioseq_scoring* sc,
                                        char* row0, char* row1, char* row2, uint32_t cap,
                                        uint32_t* ncols, int32_t* score, void* hip_stream) {
  if (!t || !sc || !row0 || !row1 || !row2 || !ncols || !score)
    return fail(TRIOSEQ_ERR_INVALID_ARG, "align: NULL pointer");
  trioseq_status st = validate_scoring(sc);
  if (st != TRIOSEQ_OK) return st;
  if (sc->kind != kGlobal) return fail(TRIOSEQ_ERR_INVALID_ARG, "align: only global alignments");
  const uint64_t need = (uint64_t)t->len[0] + t->len[1] + t->len[2];
  if (cap < need) return fail(TRIOSEQ_ERR_INVALID_ARG, "align: row capacity below the sum of the lengths");
  std::vector<char> buf(3 * need + 1);
  uint32_t nc = 0;
  int32_t sco = 0;
  st = align_batch_impl(t, 1, *sc, buf.data(), &nc, &sco, (hipStream_t)hip_stream);
  if (st != TRIOSEQ_OK) return st;
  std::memcpy(row0, buf.data(), nc);
  std::memcpy(row1, buf.data() + need, nc);
  std::memcpy(row2, buf.data() + 2 * need, nc);
  *ncols = nc;
  *score = sco;
  return TRIOSEQ_OK;
}

// Entry points: every body runs guarded (no exception crosses the ABI).
extern "C" {

trioseq_status trioseq_align_batch(const trioseq_triplet* t, size_t n, const trioseq_scoring* sc, char* rows, uint32_t* ncols, int32_t* scores, void* hip_stream) {
  return guarded([&] { return trioseq_align_batch_body(t, n, sc, rows, ncols, scores, hip_stream); });
}

trioseq_status trioseq_align(const trioseq_triplet* t, const trioseq_scoring* sc, char* row0, char* row1, char* row2, uint32_t cap, uint32_t* ncols, int32_t* score, void* hip_stream) {
  return guarded([&] { return trioseq_align_body(t, sc, row0, row1, row2, cap, ncols, score, hip_stream); });
}

}  // extern "C"
