// gfx950 kernel for panel jobs of packed pairs: two triplets (or the two
// halves of one) swept together, two 16-bit values per register, panel by
// panel over many workgroups.
//
// Values. A panel stores M' - B + off in every half, B being the panel's own
// base: its first real halo value at slice 0 (M'(0, j0 - 1, k0), or M'(0, 0,
// k0 - 1) in the first panel row, 0 in the first panel). M' grows by at most
// 2 * maxA (maxA = the largest term sub - 2*gap; g = -2*gap for local scoring
// if that is more) per unit of any index when every term is >= 0: dropping the
// last residue from an alignment turns its column into a move that scores at
// most two terms less. So a panel's real values stay within a window of that
// times (slices + panel rows + panel columns) above B, whatever the lengths of
// the other two sequences, and the host admits pairs whose window keeps every
// value within the range the half-precision maximum needs (packed.hip).
// Faces carry M' modulo 2^16 per half; a consumer subtracts its own base,
// which is exact modulo 2^16 because its true window is below 2^15.
// Outside the tensor (slices before 0, virtual faces) values start at
// kSentP and grow inside the panel only, to below off minus one step.
//
// Work split, as in k_panel: a workgroup of two waves, one computing (it
// touches only LDS), one moving faces between LDS rings and (value, tag)
// entries in memory. An entry holds both triplets, so a pair moves the bytes
// that one triplet of the int32 kernel moves; a poll takes five loads (16
// lanes cover a row with two entries each) and three ballots.
//
// What bounds it. Batches and long triplets run on single-wave workgroups, two
// or three to a SIMD, bound by VALU issue (about 139 instructions a step
// against the recurrence's 112; 93 % of the issue slots of the batch): 8192
// triplets of lengths 100-400 24.9 ms (whole pairs, one wavefront each: 31.3
// ms, their unequal sizes leave the device half empty at the end; int32: 46.5
// ms), 1999 of them under local scoring 8.5 ms (34.8 ms), 4096 x 4000 x 4150 by
// halves 10.8 ms (int32 halves: 31.3 ms). Short lone triplets are a chain of
// panel hops: 1024 x 1000 x 1048 by halves on wave pairs 613 us (int32: 976 us),
// 0.39 us a step and 21 steps a hop.
#include <type_traits>

#include "packed.h"

namespace trioseq {
namespace {

constexpr int kSideLanes = kPkPanel / 2;   // lanes covering one face row, two entries each
constexpr int kSideRows = 64 / kSideLanes; // rows per load
constexpr int kSideLoads = kChunk / kSideRows;

// R: halo and out rows kept (kRing with a memory wave, kChunk without).
template <int R>
struct PkPanelLds {
  static constexpr int kRows = R, kRowsC = 2 * R;         // corner rows are staged one step ahead
  __attribute__((aligned(16))) int sR[64][4];             // right column of each lane
  __attribute__((aligned(16))) int sB[64][4];             // bottom row of each lane
  __attribute__((aligned(16))) int T[R][kPkPanel];        // halo rings: row t mod R serves step t
  __attribute__((aligned(16))) int Lf[R][kPkPanel];
  // Corners of the top lanes; entry 8 is the corner that the panel to the
  // right takes for the step before the row's.
  int C[kRowsC][kGK + 1];
  __attribute__((aligned(16))) int ob[R][kPkPanel];       // out rows
  __attribute__((aligned(16))) int orr[R][kPkPanel];
  int sX[64];                                             // bottom of each lane's left halo
  int cap[2][16];                                         // score tiles of both triplets
  int in_ready, out_done, out_flushed, job;
  uint32_t base;
};

// A panel's faces. A pair has two bottom-face buffers per panel column and two
// right-face buffers (corner face behind them) per panel row (fewer where a
// column or row has fewer panels that write), written in turn:
// a panel reads the one its neighbour wrote and overwrites the one written two
// panels before. 260 buffers instead of two for each of 4225 panels of a
// 2048-residue triplet (1024 x 1000 x 1048: 711 us against 734 with faces of its
// own for every panel; with a single buffer, read and written in the same
// lines, 764). Every face byte still leaves the L2, as the device-coherent stores
// write through: the smaller buffers are for the memory-side cache. Nothing that is needed is
// overwritten: a panel's row t depends, through its neighbour's row t + 7, on
// the neighbour having read row t + 14 of the buffer in question. The tag of
// an entry is gen + 1 + the panel row (bottom faces) or column (right faces)
// that wrote it; a consumer takes exactly its neighbour's.
struct PkPanelIO {
  int *col_in, *col_out;  // bottom faces of this panel column: read if has_top, written if bot
  int *row_in, *row_out;  // right faces of this panel row: read if has_left, written if right
  bool has_top, has_left, bot, right;
  int top_tag, left_tag;  // the neighbours' tags; this panel's are one more
  int* err;
  uint64_t wait_ticks;
};

// One wave's view of a panel's faces. For steps u .. u + 7 a load fetches rows
// u + 7 .. u + 14 of the top, left and corner faces, five instructions: lane l
// holds entries 2(l mod 16), +1 of row l / 16 (+ 4 in the second load), so the
// first row with a stale entry is the lowest set bit of a ballot.
template <class Lds>
struct PkFaces {
  static constexpr uint32_t RB = kPkPanel * 8u;  // bytes of a face row
  Lds& S;
  const PkPanelIO& io;
  int n0, lane, rr0, pr, grp;
  uint32_t side, vside, off2, delta;  // delta: off - base, per half modulo 2^16
  Rsrc r_top, r_left, r_bot, r_right;
  bool have_base;
  v4i tv[kSideLoads], lv[kSideLoads];
  v2i cv;

  // A face that does not exist (tensor edge) or has no consumer is an empty
  // resource: its loads give 0 and its stores are dropped. It is never waited
  // for (its tag is 0 as well), and every slice counts as before the tensor.
  int top_tag, left_tag, top_from, left_from;

  __device__ __forceinline__ PkFaces(Lds& S_, const PkPanelIO& io_, int n0_, uint32_t off2_)
      : S(S_), io(io_), n0(n0_), off2(off2_), delta(off2_) {
    lane = threadIdx.x & 63;
    rr0 = lane / kSideLanes;
    pr = lane % kSideLanes;
    grp = pr >> 1;
    vside = (uint32_t)(rr0 * RB + pr * 16);
    const uint64_t rows = pk_face_rows((uint32_t)n0);
    side = (uint32_t)(rows * RB);
    const uint32_t both = side + (uint32_t)rows * 8u;  // right faces, then corners
    r_top = make_rsrc(io.col_in, io.has_top ? side : 0);
    r_left = make_rsrc(io.row_in, io.has_left ? both : 0);
    r_bot = make_rsrc(io.col_out, io.bot ? side : 0);
    r_right = make_rsrc(io.row_out, io.right ? both : 0);
    top_tag = io.has_top ? io.top_tag : 0;
    left_tag = io.has_left ? io.left_tag : 0;
    top_from = io.has_top ? 0 : INT32_MAX;
    left_from = io.has_left ? 0 : INT32_MAX;
    have_base = !io.has_top && !io.has_left;
  }

  // Before the first put, by the wave that stages: the corners of step 0 lie
  // before slice 0 (lane 0's comes with the corner face, or lies outside).
  __device__ __forceinline__ void begin() {
    if (lane < kGK) S.C[0][lane] = (int)(kSentP * 0x10001u);
  }

  __device__ __forceinline__ void load(int u) {
    const uint32_t z = opaque_zero();
    const uint32_t vo = vside + (uint32_t)(u + kGJ - 1) * RB;
#pragma unroll
    for (int q = 0; q < kSideLoads; ++q) {
      tv[q] = __builtin_amdgcn_raw_buffer_load_b128(r_top, vo + q * kSideRows * RB, z, kCohDevice);
      lv[q] = __builtin_amdgcn_raw_buffer_load_b128(r_left, vo + q * kSideRows * RB, z, kCohDevice);
    }
    cv = __builtin_amdgcn_raw_buffer_load_b64(
        r_left, lane < kChunk ? side + (uint32_t)(u + kGJ - 1 + lane) * 8u : kOob, z, kCohDevice);
  }

  // How many of the steps u .. u + 7 have every entry they need (entries of
  // slices past n0 are never needed, those before 0 are not read).
  __device__ __forceinline__ int ready(int u) const {
    int k = kChunk;
#pragma unroll
    for (int q = kSideLoads - 1; q >= 0; --q) {
      const int slice = u + rr0 + q * kSideRows - grp;
      const int stale =
          (tv[q].y ^ top_tag) | (tv[q].w ^ top_tag) | (lv[q].y ^ left_tag) | (lv[q].w ^ left_tag);
      const uint64_t m = __builtin_amdgcn_ballot_w64((uint32_t)slice <= (uint32_t)n0 && stale != 0);
      if (m) k = q * kSideRows + __builtin_ctzll(m) / kSideLanes;
    }
    // (In the first panel row nobody writes or needs corners.)
    const uint64_t m =
        __builtin_amdgcn_ballot_w64(io.has_top && lane < kChunk && u + lane <= n0 && cv.y != left_tag);
    if (m) k = min(k, __builtin_ctzll(m));
    return k;
  }

  // Writes the halo rows of steps u .. u + k - 1 to the rings, relative to the
  // panel's base (taken from the first entry of slice 0). ALL: k = kChunk.
  template <bool ALL>
  __device__ __forceinline__ void put(int u, int k) {
    const uint32_t sent2 = kSentP * 0x10001u;
    if (!have_base) {
      // Lane 0 holds entry 0 of row 7, slice 0.
      const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(io.has_top ? tv[0].x : lv[0].x);
      delta = psub(off2, b);
      if (lane == 0) S.base = b;
      have_base = true;
    }
#pragma unroll
    for (int q = 0; q < kSideLoads; ++q) {
      const int rr = rr0 + q * kSideRows, st = u + rr;
      if (ALL || rr < k) {
        // Slices before 0 lie outside the tensor.
        const bool no_top = st - grp < top_from, no_left = st - grp < left_from;
        const uint32_t t0 = no_top ? sent2 : paddw((uint32_t)tv[q].x, delta);
        const uint32_t t1 = no_top ? sent2 : paddw((uint32_t)tv[q].z, delta);
        const uint32_t l0 = no_left ? sent2 : paddw((uint32_t)lv[q].x, delta);
        const uint32_t l1 = no_left ? sent2 : paddw((uint32_t)lv[q].z, delta);
        *reinterpret_cast<v2i*>(&S.T[st & (Lds::kRows - 1)][2 * pr]) = (v2i){(int)t0, (int)t1};
        *reinterpret_cast<v2i*>(&S.Lf[st & (Lds::kRows - 1)][2 * pr]) = (v2i){(int)l0, (int)l1};
        // Entry 4x + 3 is the corner of lane x + 1 at the next step (x = 7:
        // of the panel to the right, at this step).
        if (pr & 1) S.C[(st + 1) & (Lds::kRowsC - 1)][grp + 1] = (int)t1;
      }
    }
    if (lane < (ALL ? kChunk : k))
      S.C[(u + lane) & (Lds::kRowsC - 1)][0] =
          (int)(io.has_top && io.has_left ? paddw((uint32_t)cv.x, delta) : sent2);
  }

  // Stores out rows t0 .. t0 + nf - 1, back to M' modulo 2^16.
  template <bool ALL>
  __device__ __forceinline__ void flush(int t0, int nf) const {
    const int bot_tag = io.top_tag + 1, right_tag = io.left_tag + 1;
    v2i bv[kSideLoads], rv[kSideLoads];
#pragma unroll
    for (int q = 0; q < kSideLoads; ++q) {
      const int ro = (t0 + rr0 + q * kSideRows) & (Lds::kRows - 1);
      bv[q] = *reinterpret_cast<const v2i*>(&S.ob[ro][2 * pr]);
      rv[q] = *reinterpret_cast<const v2i*>(&S.orr[ro][2 * pr]);
    }
    const int c = S.C[(t0 + (lane & (kChunk - 1)) + 1) & (Lds::kRowsC - 1)][kGK];
    const uint32_t vo = vside + (uint32_t)t0 * RB;
#pragma unroll
    for (int q = 0; q < kSideLoads; ++q) {
      const uint32_t o = ALL || rr0 + q * kSideRows < nf ? vo + q * kSideRows * RB : kOob;
      __builtin_amdgcn_raw_buffer_store_b128(
          (v4i){(int)psub((uint32_t)bv[q].x, delta), bot_tag, (int)psub((uint32_t)bv[q].y, delta), bot_tag}, r_bot,
          o, 0, kCohDevice);
      __builtin_amdgcn_raw_buffer_store_b128(
          (v4i){(int)psub((uint32_t)rv[q].x, delta), right_tag, (int)psub((uint32_t)rv[q].y, delta), right_tag},
          r_right, o, 0, kCohDevice);
    }
    __builtin_amdgcn_raw_buffer_store_b64((v2i){(int)psub((uint32_t)c, delta), right_tag}, r_right,
                                          lane < (ALL ? kChunk : nf) ? side + (uint32_t)(t0 + lane) * 8u : kOob, 0,
                                          kCohDevice);
  }
};

__device__ __forceinline__ void lds_put4(int* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  *reinterpret_cast<v4i*>(__builtin_assume_aligned(p, 16)) = (v4i){(int)a, (int)b, (int)c, (int)d};
}

// b where the mask is set, else a.
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t b, uint32_t a) { return (b & mask) | (a & ~mask); }

// The compute wave. Folds local and semi-global bests into `best`, as the
// whole-triplet kernel does (local: M; semi-global: M + kc). SELF: the wave
// moves its faces itself, a chunk of steps at a time (loads of the next chunk
// issued at step kSelfStageAt of this one).
constexpr int kSelfStageAt = 5;
template <int KIND, bool PLANE, bool SELF, int WPS, class Lds>
__device__ void pk_panel_compute(Lds& S, const uint32_t* sel, const DevScoring& sc,
                                 const uint32_t* __restrict__ words, const TripletDesc& ta, const TripletDesc& tb,
                                 int n0, int pj, int pk, const PkPanelIO& io, uint16_t* capt, uint32_t off2,
                                 uint32_t& best, uint32_t kc) {
  constexpr int RJ = 4, RK = 4;
  constexpr int H = kPkPanel, W = kPkPanel;
  constexpr bool PAD = KIND != kGlobal;
  // Semi-global halves. An alignment ends on any last face, so the reversed
  // half starts with 0 on all three of its faces (M' = g * index sum there),
  // and what it finds of its own are the alignments that start on the cut axis
  // past the middle: those through its row n1, column n2. The first half starts
  // on the axes as ever, and its own best takes the last row and column only:
  // its last slice is the cut, not a face.
  constexpr bool kFaces = KIND == kSemiGlobal && PLANE;
  const int lane = threadIdx.x & 63;
  const int y = lane >> 3, x = lane & 7;
  const int j0 = pj * H + y * RJ, k0 = pk * W + x * RK;
  PkTables<RJ, RK> tabs;
  pk_tables<PAD>(tabs, sc, words, ta, tb, j0, k0);

  const uint32_t sent2 = kSentP * 0x10001u;
  uint32_t P[RJ][RK], D[RJ][RK], Lp[RJ], Tp[RK];
#pragma unroll
  for (int r = 0; r < RJ; ++r) {
    Lp[r] = sent2;
#pragma unroll
    for (int c = 0; c < RK; ++c) P[r][c] = D[r][c] = sent2;
  }
#pragma unroll
  for (int c = 0; c < RK; ++c) Tp[c] = sent2;

  const int nchunks = (n0 + 1 + kSkew + kChunk - 1) / kChunk;
  const int n0a = (int)ta.len[0], n0b = (int)tb.len[0];
  const int rsa = (int)ta.len[1] - j0, csa = (int)ta.len[2] - k0;
  const int rsb = (int)tb.len[1] - j0, csb = (int)tb.len[2] - k0;
  const bool own_a = rsa >= 0 && rsa < RJ && csa >= 0 && csa < RK;
  const bool own_b = rsb >= 0 && rsb < RJ && csb >= 0 && csb < RK;

  constexpr int ND = RJ + RK - 1;
  const int g = -sc.gap2;
  const uint32_t g2 = (uint32_t)g * 0x10001u;
  int fi = g * (j0 + k0 - y - x);  // g * (i + j0 + k0) for the lane's slice i
  uint32_t RM[RJ], CM[RK], rcany = 0;
#pragma unroll
  for (int r = 0; r < RJ; ++r) {
    RM[r] = (r == rsa ? 0xFFFFu : 0u) | (r == rsb ? 0xFFFF0000u : 0u);
    rcany |= RM[r];
  }
#pragma unroll
  for (int c = 0; c < RK; ++c) {
    CM[c] = (c == csa ? 0xFFFFu : 0u) | (c == csb ? 0xFFFF0000u : 0u);
    rcany |= CM[c];
  }
  const bool axis_panel = pj == 0 || pk == 0;
  const bool seed_lane = pj == 0 && pk == 0 && lane == 0;

#pragma unroll
  for (int r = 0; r < RJ; ++r) S.sR[lane][r] = (int)sent2;
#pragma unroll
  for (int c = 0; c < RK; ++c) S.sB[lane][c] = (int)sent2;
  S.sX[lane] = (int)sent2;

  // Halo sources: ring rows for edge lanes, neighbours' slots otherwise. As
  // byte offsets that advance by their stride every step: with pointers plus
  // step times stride the compiler kept the addresses of all eight steps (wave
  // pairs 192 VGPRs, now 170; 8192 triplets 26.2 ms, now 26.0).
  const bool y0 = y == 0, x0 = x == 0;
  char* const lds = reinterpret_cast<char*>(&S);
  const auto at = [lds](const int* p) { return (int)(reinterpret_cast<const char*>(p) - lds); };
  const int t_off = y0 ? at(&S.T[0][x * RK]) : at(&S.sB[y0 ? 0 : lane - 8][0]);
  const int c_off = y0 ? at(&S.C[0][x]) : at(&S.sX[y0 ? 0 : lane - 8]);
  const int l_off = x0 ? at(&S.Lf[0][y * RJ]) : at(&S.sR[x0 ? 0 : lane - 1][0]);
  const int t_str = y0 ? W * 4 : 0, c_str = y0 ? (kGK + 1) * 4 : 0, l_str = x0 ? H * 4 : 0;
  // Where the tile's bottom row and right column go: the lane's slots, or the
  // out rows for the panel's last lanes (whose slots nobody reads).
  const bool y7 = y == kGJ - 1, x7 = x == kGK - 1;
  const int b_off = y7 ? at(&S.ob[0][x * RK]) : at(&S.sB[lane][0]);
  const int r_off = x7 ? at(&S.orr[0][y * RJ]) : at(&S.sR[lane][0]);
  const int b_str = y7 ? W * 4 : 0, r_str = x7 ? H * 4 : 0;
  const uint32_t* sl = sel + kShiftPre - y - x;

  int fin = 0, ffl = 0;
  bool gave_up = false;
  PkFaces<Lds> f(S, io, n0, off2);  // (unused, and dropped, without SELF)
  if (SELF) {
    f.begin();
    f.load(0);
  }
  uint32_t zero2 = off2;  // stored value of M' = 0 (set at step 0, once the base is known)
  auto run_chunk = [&](int c, auto capture) __attribute__((always_inline)) {
    constexpr bool CAP = decltype(capture)::value;
    const int cb0 = c * kChunk;
    constexpr int kPh = Lds::kRows / kChunk - 1, kPhC = Lds::kRowsC / kChunk - 1;
    int to = t_off + (c & kPh) * kChunk * t_str, co = c_off + (c & kPhC) * kChunk * c_str;
    int lo = l_off + (c & kPh) * kChunk * l_str;
    int bo = b_off + (c & kPh) * kChunk * b_str, ro = r_off + (c & kPh) * kChunk * r_str;
    if (SELF) {
      if (!gave_up && f.ready(cb0) < kChunk) {
        const uint64_t t_start = wall_clock64();
        do {
          if (wall_clock64() - t_start > io.wait_ticks) {
            raise_error(io.err);
            gave_up = true;
            break;
          }
          __builtin_amdgcn_s_sleep(2);
          f.load(cb0);
        } while (f.ready(cb0) < kChunk);
      }
      f.template put<true>(cb0, kChunk);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
    }
    uint32_t selv[kChunk];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) selv[s] = sl[cb0 + s];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) {
      const int t = cb0 + s;
      if (SELF && s == kSelfStageAt && c + 1 < nchunks) f.load(cb0 + kChunk);
      // Step t needs its halo rows staged and out row t mod kRing read back;
      // the counters read during the previous step usually already say so.
      if (!SELF && !gave_up && !(fin > t && ffl > t - kRing)) {
        const uint64_t t_start = wall_clock64();
        for (;;) {
          fin = lds_get(&S.in_ready);
          ffl = lds_get(&S.out_flushed);
          if (fin > t && ffl > t - kRing) break;
          if (wall_clock64() - t_start > io.wait_ticks) {
            raise_error(io.err);
            gave_up = true;
            break;
          }
          __builtin_amdgcn_s_sleep(1);
        }
      }
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      int fin_next = 0, ffl_next = 0;
      if (!SELF) {
        fin_next = lds_get(&S.in_ready);
        ffl_next = lds_get(&S.out_flushed);
      }
      if (PAD && s == 0 && c == 0) zero2 = psub(off2, S.base);

      const uint32_t sv = selv[s];
      uint32_t A[RJ], B[RK], T[RK], Lh[RJ];
#pragma unroll
      for (int r = 0; r < RJ; ++r) A[r] = __builtin_amdgcn_perm(tabs.TBb[r], tabs.TBa[r], sv);
#pragma unroll
      for (int cc = 0; cc < RK; ++cc) B[cc] = __builtin_amdgcn_perm(tabs.TCb[cc], tabs.TCa[cc], sv);
      {
        const v4i v = lds_v4(reinterpret_cast<const int*>(lds + to));
        T[0] = (uint32_t)v.x, T[1] = (uint32_t)v.y, T[2] = (uint32_t)v.z, T[3] = (uint32_t)v.w;
        const v4i w = lds_v4(reinterpret_cast<const int*>(lds + lo));
        Lh[0] = (uint32_t)w.x, Lh[1] = (uint32_t)w.y, Lh[2] = (uint32_t)w.z, Lh[3] = (uint32_t)w.w;
      }
      const uint32_t corner = (uint32_t)*reinterpret_cast<const int*>(lds + co);
      const int i = t - y - x;  // this lane's slice
      if (KIND == kSemiGlobal && axis_panel) {
        // The axes hold 0 (M' = g * index): see the whole-triplet kernel. With
        // planes the second half of the pair starts on its whole faces instead
        // (see kFaces).
        const uint32_t keep = kFaces ? 0xFFFFu : 0xFFFFFFFFu;
        const uint32_t faces = kFaces && i >= 0 ? 0xFFFF0000u : 0u;
        if (kFaces && j0 == 0) {
#pragma unroll
          for (int cc = 0; cc < RK; ++cc)
            T[cc] = bfi(faces, paddw(zero2, ((uint32_t)(g * (i + k0 + cc)) & 0xFFFFu) * 0x10001u), T[cc]);
        }
        if (kFaces && k0 == 0) {
#pragma unroll
          for (int r = 0; r < RJ; ++r)
            Lh[r] = bfi(faces, paddw(zero2, ((uint32_t)(g * (i + j0 + r)) & 0xFFFFu) * 0x10001u), Lh[r]);
        }
        if (j0 == 0) {
#pragma unroll
          for (int cc = 0; cc < RK; ++cc) T[cc] = bfi(i == 0 ? keep : 0u, paddw(zero2, (uint32_t)(g * (k0 + cc)) * 0x10001u), T[cc]);
          if (k0 == 0) T[0] = bfi(i >= 0 ? keep : 0u, paddw(zero2, (uint32_t)(g * i) * 0x10001u), T[0]);
        }
        if (k0 == 0) {
#pragma unroll
          for (int r = 0; r < RJ; ++r) Lh[r] = bfi(i == 0 ? keep : 0u, paddw(zero2, (uint32_t)(g * (j0 + r)) * 0x10001u), Lh[r]);
        }
      }
      // Local floors per anti-diagonal class, F_d = F_0 + g*d. A floor below
      // the panel's window (the base has outgrown it) is as good as none: its
      // F_0 is taken as 0, and F_0 + g*d then lies below every live value.
      uint32_t F0 = 0, F[ND];
      if (KIND == kLocal) {
        asm volatile("" : "+v"(fi));  // one step's floors live at a time
        F0 = paddw(zero2, ((uint32_t)fi & 0xFFFFu) * 0x10001u);
        const uint32_t f0 = i >= 0 ? smax2(F0, 0u) : 0u;
#pragma unroll
        for (int d = 0; d < ND; ++d) F[d] = f0 + (uint32_t)d * g2;
      }
      uint32_t Q[RJ][RK], X7[RJ][RK], N[RJ][RK];
#pragma unroll
      for (int r = 0; r < RJ; ++r)
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) {
          const uint32_t up_prev = r ? P[r - 1][cc] : Tp[cc];
          const uint32_t left_prev = cc ? P[r][cc - 1] : Lp[r];
          Q[r][cc] = pmax3(P[r][cc], padd(up_prev, A[r]), padd(left_prev, B[cc]));
          X7[r][cc] = D[r][cc] + A[r] + B[cc];
          if (KIND == kLocal) Q[r][cc] = pmax3(Q[r][cc], X7[r][cc], F[r + cc]);
        }
      if (kFaces && c < 2 && i == 0) {
        // Slice 0 of the second half is a face (lanes reach it in steps 0 .. 14).
        // A value below the window counts as none, as the local floors do.
        const uint32_t f0 = smax2(paddw(zero2, ((uint32_t)(g * (j0 + k0)) & 0xFFFFu) * 0x10001u), 0u) & 0xFFFF0000u;
#pragma unroll
        for (int r = 0; r < RJ; ++r)
#pragma unroll
          for (int cc = 0; cc < RK; ++cc)
            Q[r][cc] = pmax2(Q[r][cc], f0 + ((uint32_t)((r + cc) * g) << 16));
      }
#pragma unroll
      for (int r = 0; r < RJ; ++r)
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) {
          const uint32_t up_cur = r ? N[r - 1][cc] : T[cc];
          const uint32_t left_cur = cc ? N[r][cc - 1] : Lh[r];
          const uint32_t diag_cur = r ? (cc ? N[r - 1][cc - 1] : Lh[r - 1]) : (cc ? T[cc - 1] : corner);
          const uint32_t x6 = padd(diag_cur, tabs.C2[r][cc]);
          if (KIND == kLocal)
            N[r][cc] = pmax3(pmax2(Q[r][cc], x6), up_cur, left_cur);
          else
            N[r][cc] = pmax3(pmax3(Q[r][cc], X7[r][cc], x6), up_cur, left_cur);
          // Global M'(0,0,0) = 0, the one real start.
          if (KIND == kGlobal && s == 0 && r == 0 && cc == 0) N[0][0] = (c == 0 && seed_lane) ? off2 : N[0][0];
          D[r][cc] = x6;
        }

      if (KIND != kGlobal) {
        const uint32_t vm =
            ((uint32_t)i <= (uint32_t)n0a ? 0xFFFFu : 0u) | ((uint32_t)i <= (uint32_t)n0b ? 0xFFFF0000u : 0u);
        if (KIND == kLocal) {
          // Best class maximum less g*d, then less F_0 (modulo 2^16: M itself).
          uint32_t sb = 0;
#pragma unroll
          for (int d = 0; d < ND; ++d) {
            uint32_t m = 0, hold = 0;
            int cnt = 0;
#pragma unroll
            for (int r = 0; r < RJ; ++r) {
              if (d - r < 0 || d - r >= RK) continue;
              const uint32_t v = N[r][d - r];
              if (cnt == 0) m = v;
              else if (cnt & 1) hold = v;
              else m = pmax3(m, hold, v);
              ++cnt;
            }
            if (!(cnt & 1)) m = pmax2(m, hold);
            sb = umax2(sb, psub(m, (uint32_t)d * g2));
          }
          best = umax2(best, psub(sb, F0) & vm);
          // Formed here: sunk to where `best` is used, the end of the chunk,
          // it would keep the tiles of all its steps in registers.
          asm volatile("" : "+v"(best));
        } else {
          const uint32_t sm = kFaces ? 0u : (i == n0a ? 0xFFFFu : 0u) | (i == n0b ? 0xFFFF0000u : 0u);
          if (((rcany | sm) & vm) != 0u) {
            // M + kc = stored - zero2 - g*(i + j + k) + kc.
            const uint32_t off0 = psub(((kc - (uint32_t)fi) & 0xFFFFu) * 0x10001u, zero2);
            uint32_t sb = 0;
#pragma unroll
            for (int r = 0; r < RJ; ++r)
#pragma unroll
              for (int cc = 0; cc < RK; ++cc)
                sb = umax2(sb, paddw(N[r][cc], psub(off0, (uint32_t)(r + cc) * g2)) &
                                   (kFaces ? bfi(0xFFFFu, RM[r] | CM[cc], RM[r] & CM[cc]) : RM[r] | CM[cc] | sm));
            best = umax2(best, sb & vm);
            asm volatile("" : "+v"(best));
          }
        }
        fi += g;
      }

      lds_put4(reinterpret_cast<int*>(lds + bo), N[RJ - 1][0], N[RJ - 1][1], N[RJ - 1][2], N[RJ - 1][3]);
      lds_put4(reinterpret_cast<int*>(lds + ro), N[0][RK - 1], N[1][RK - 1], N[2][RK - 1], N[3][RK - 1]);
      S.sX[lane] = (int)Lh[RJ - 1];
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (!SELF && lane == 0) lds_put(&S.out_done, t + 1);
      fin = fin_next;
      ffl = ffl_next;

      if (CAP) {
        if (PLANE) {
          // (Halves interleaved: 16-bit stores straight from the registers.)
          if (i == n0a) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q) capt[(lane * (RJ * RK) + q) * 2] = (uint16_t)N[q / RK][q % RK];
          }
          if (i == n0b) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q)
              capt[(lane * (RJ * RK) + q) * 2 + 1] = (uint16_t)(N[q / RK][q % RK] >> 16);
          }
        } else if (KIND == kGlobal) {
          if (own_a && i == n0a) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q) S.cap[0][q] = (int)N[q / RK][q % RK];
          }
          if (own_b && i == n0b) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q) S.cap[1][q] = (int)N[q / RK][q % RK];
          }
        }
      }
#pragma unroll
      for (int r = 0; r < RJ; ++r) {
        Lp[r] = Lh[r];
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) P[r][cc] = N[r][cc];
      }
#pragma unroll
      for (int cc = 0; cc < RK; ++cc) Tp[cc] = T[cc];
      to += t_str, co += c_str, lo += l_str, bo += b_str, ro += r_str;
      // (Formed step by step: all steps' addresses at once do not fit.)
      if (WPS == 3) asm volatile("" : "+v"(to), "+v"(co), "+v"(lo), "+v"(bo), "+v"(ro));
    }
    if (SELF) {
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      f.template flush<true>(cb0, kChunk);
    }
  };
  // A triplet's last slice n0 is captured in the chunks from n0 / kChunk on: a
  // copy of the body of their own keeps the tests out of all others.
  constexpr bool kCaptures = PLANE || KIND == kGlobal;
  const int ccap = kCaptures ? min(n0a, n0b) / kChunk : nchunks;
  for (int c = 0; c < ccap; ++c) run_chunk(c, std::false_type{});
  if constexpr (kCaptures)
    for (int c = ccap; c < nchunks; ++c) run_chunk(c, std::true_type{});
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
}

// Last slices of a panel, unshifted, from the captured tiles (half h of the pair).
__device__ __forceinline__ void pk_write_plane(const uint16_t* capt, int* plane, const TripletDesc& td, int pj, int pk,
                                               uint32_t zero, int gap2) {
  const int lane = threadIdx.x & 63;
  const int j0 = pj * kPkPanel + (lane >> 3) * 4, k0 = pk * kPkPanel + (lane & 7) * 4;
  const int n0 = (int)td.len[0], n1 = (int)td.len[1], n2 = (int)td.len[2];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int j = j0 + q / 4, k = k0 + q % 4;
    if (j <= n1 && k <= n2)
      plane[(uint64_t)j * (uint64_t)(n2 + 1) + (uint64_t)k] =
          (int)((capt[(lane * 16 + q) * 2] - zero) & 0xFFFFu) + gap2 * (n0 + j + k);
  }
}

// The memory wave: keeps the compute wave's halo rings filled and stores its
// out rows. Every wait is bounded (past the limit the error flag is raised and
// the rows are staged as they are).
__device__ void pk_panel_memory(PkPanelLds<kRing>& S, int n0, const PkPanelIO& io, uint32_t off2) {
  const int lane = threadIdx.x & 63;
  const int stepsp = (n0 + 1 + kSkew + kChunk - 1) / kChunk * kChunk;
  PkFaces<PkPanelLds<kRing>> f(S, io, n0, off2);
  f.begin();
  int staged = 0, flushed = 0;
  uint64_t stall_since = 0;
  bool gave_up = false;
  while (staged < stepsp || flushed < stepsp) {
    const int done = lds_get(&S.out_done);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    bool progress = false;
    const int nb = min(min(kChunk, stepsp - staged), done + kRing - staged);
    if (nb > 0) {
      f.load(staged);
      int k = min(f.ready(staged), nb);
      if (gave_up) k = nb;
      if (k <= 0 && stall_since && wall_clock64() - stall_since > io.wait_ticks) {
        raise_error(io.err);
        gave_up = true;
        k = nb;
      }
      if (k > 0) {
        f.template put<false>(staged, k);
        staged += k;
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0) lds_put(&S.in_ready, staged);
        progress = true;
      }
    }
    const int nf = min(kChunk, lds_get(&S.out_done) - flushed);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (nf > 0) {
      f.template flush<false>(flushed, nf);
      flushed += nf;
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (lane == 0) lds_put(&S.out_flushed, flushed);
      progress = true;
    }
    if (progress) {
      stall_since = 0;
    } else {
      if (!stall_since) stall_since = wall_clock64();
      __builtin_amdgcn_s_sleep(1);
    }
  }
}

// Workgroups pop panel jobs (jd.trip = the pair's first descriptor) in the
// host's dependency order, so every producer was popped earlier by a running
// workgroup and every wait ends. Pairs that reuse the face buffers of earlier
// ones (see pair_panel_layout) also wait until those are over; all their jobs
// were popped before.
template <int KIND, bool PLANE, bool SELF, int WPS>
__global__ void __launch_bounds__(SELF ? 64 : 128) __attribute__((amdgpu_waves_per_eu(WPS)))
k_panel_pk(SweepArgs a, uint32_t off, uint32_t kc, uint32_t count) {
  constexpr int H = kPkPanel, W = kPkPanel;
  typedef PkPanelLds<SELF ? kChunk : kRing> Lds;
  __shared__ Lds S;
  __shared__ __attribute__((aligned(16))) uint16_t capt[PLANE ? 2 * 64 * 16 : 1];
  extern __shared__ uint32_t selw[];
  const int wave = threadIdx.x >> 6;
  const uint32_t off2 = off * 0x10001u;
  const int gen = __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t staged = 0xFFFFFFFFu, seen[2] = {0, 0};
  for (;;) {
    if (threadIdx.x == 0) S.job = atomicAdd(a.counter, 1);
    __syncthreads();
    const int idx = S.job;
    if (idx >= (int)a.njobs) break;
    const JobDesc jd = a.jobs[idx];
    const TripletDesc ta = a.desc[jd.trip], tb = a.desc[jd.trip + 1];
    const int n0 = (int)max(ta.len[0], tb.len[0]);
    const int n1 = (int)max(ta.len[1], tb.len[1]), n2 = (int)max(ta.len[2], tb.len[2]);
    // (Counts only grow, so a group's first wait serves its other panels.)
    if (count && ta.after > seen[ta.set]) {
      if (threadIdx.x == 0) {
        const uint64_t t_start = wall_clock64();
        while (__hip_atomic_load(a.counter + kFinished * (1 + ta.set), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
               (int)ta.after) {
          if (wall_clock64() - t_start > a.wait_ticks) {
            raise_error(a.ctl + 1);
            break;
          }
          __builtin_amdgcn_s_sleep(8);
        }
      }
      seen[ta.set] = ta.after;
    }
    if (jd.trip != staged) {
      stage_selectors(selw, a.words, ta, tb, n0, (int)threadIdx.x, SELF ? 64 : 128);
      staged = jd.trip;
    }
    if (threadIdx.x == 0) {
      S.in_ready = 0;
      S.out_done = 0;
      S.out_flushed = 0;
      S.base = 0;
    }
    __syncthreads();
    const int PJ = n1 / H + 1, PK = n2 / W + 1;
    const uint64_t rows = pk_face_rows((uint32_t)n0);
    const uint32_t p = jd.panel;
    const int pj = (int)(p / (uint32_t)PK), pk = (int)(p % (uint32_t)PK);
    int* pool = a.pface + ta.face_off;
    PkPanelIO io;
    // (The buffer a panel at the edge would read or write may not exist: it is
    // an empty resource then.)
    const uint64_t cs = rows * (2 * kPkPanel), rs = rows * (2 * kPkPanel + 2);
    int* rpool = pool + pk_face_buffers((uint64_t)PJ) * (uint64_t)PK * cs;
    io.col_in = pool + (uint64_t)(((pj & 1) ^ 1) * PK + pk) * cs;
    io.col_out = pool + (uint64_t)((pj & 1) * PK + pk) * cs;
    io.row_in = rpool + (uint64_t)(((pk & 1) ^ 1) * PJ + pj) * rs;
    io.row_out = rpool + (uint64_t)((pk & 1) * PJ + pj) * rs;
    io.has_top = pj > 0;
    io.has_left = pk > 0;
    io.bot = pj + 1 < PJ;
    io.right = pk + 1 < PK;
    io.top_tag = gen + (int)ta.tag0 + pj;
    io.left_tag = gen + (int)ta.tag0 + pk;
    io.err = a.ctl + 1;
    io.wait_ticks = a.wait_ticks;
    uint32_t best = 0;
    if constexpr (SELF) {
      pk_panel_compute<KIND, PLANE, true, WPS>(S, selw, a.sc, a.words, ta, tb, n0, pj, pk, io, capt, off2, best, kc);
    } else {
      if (wave == 0)
        pk_panel_compute<KIND, PLANE, false, WPS>(S, selw, a.sc, a.words, ta, tb, n0, pj, pk, io, capt, off2, best, kc);
      else
        pk_panel_memory(S, n0, io, off2);
    }
    if (count) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's face stores
    __syncthreads();
    // Both waves are done: a wait of this job that gave up has raised the flag
    // by now, and upstream panels raised theirs before writing the faces this
    // job read.
    if (count && threadIdx.x == 0) {
      // (Every wave's face stores have reached memory: a later pair may
      // overwrite them.)
      __hip_atomic_fetch_add(a.counter + kFinished * (1 + ta.set), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint32_t zero2 = psub(off2, S.base);
    if (PLANE) {
      // One half's plane by each wave.
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (SELF || wave == h)
          pk_write_plane(capt + h, a.plane + a.plane_off[jd.trip + h], h ? tb : ta, pj, pk,
                         h ? zero2 >> 16 : zero2 & 0xFFFFu, a.sc.gap2);
    }
    if (KIND == kGlobal && !PLANE && threadIdx.x < 2) {
      const int h = (int)threadIdx.x;
      const TripletDesc& td = h ? tb : ta;
      const int r = (int)td.len[1] - pj * H, c = (int)td.len[2] - pk * W;
      if (r >= 0 && r < H && c >= 0 && c < W) {
        const uint32_t v = psub((uint32_t)S.cap[h][(r & 3) * 4 + (c & 3)], zero2);
        const int m = (int)(h ? v >> 16 : v & 0xFFFFu);
        // (The faces this panel read had arrived before the barrier above, so
        // this load of the flag comes after them.)
        const bool bad = __hip_atomic_load(io.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
        // System scope: the score may live in mapped host memory (serving).
        __hip_atomic_store(a.scores + td.out,
                           bad ? INT32_MIN : m + a.sc.gap2 * (int)(td.len[0] + td.len[1] + td.len[2]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
    if (KIND != kGlobal && wave == 0) {
      // Fold the panel's best into both triplets' accumulators; the panel
      // that finishes last writes the scores (see finish_panel of sweep.hip).
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) best = umax2(best, (uint32_t)__shfl_xor((int)best, o));
      if (threadIdx.x == 0) {
        int* acc = a.red + 2 * (uint64_t)jd.trip;
        __hip_atomic_fetch_max(acc, (int)(best & 0xFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_fetch_max(acc + 2, (int)(best >> 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // (Halves: the meeting of their planes reads both bests.) The folds have
        // reached memory before this panel counts itself finished: waiting for
        // them is enough, as every access here is device-coherent; a release
        // would write back the whole L2 for every panel.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const int prev = PLANE ? 0 : __hip_atomic_fetch_add(acc + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!PLANE && prev == PJ * PK - 1) {
          const int sub = KIND == kSemiGlobal ? (int)kc : 0;
          const bool bad = __hip_atomic_load(io.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int v = __hip_atomic_load(acc + 2 * h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - sub;
            __hip_atomic_store(a.scores + (h ? tb.out : ta.out), bad ? INT32_MIN : v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_SYSTEM);
          }
        }
      }
    }
  }
}

// Kind, planes, single waves, waves per SIMD (see pk_waves_per_simd).
#define TRIOSEQ_PKP(X)                                                                           \
  X(0, true, false, 2) X(0, true, true, 2) X(0, false, false, 2) X(0, false, true, 2)            \
  X(0, false, true, 3)                                                                           \
  X(1, true, false, 2) X(1, true, true, 2) X(1, false, false, 2) X(1, false, true, 2)            \
  X(2, true, false, 2) X(2, true, true, 2) X(2, false, false, 2) X(2, false, true, 2)

}  // namespace

hipError_t launch_panel_pk(int kind, bool self, const SweepArgs& a, uint32_t off, uint32_t kc, bool count, int grid,
                           hipStream_t s) {
  const size_t lds = (size_t)(a.lds_n0 + 64) * 4;
  const bool plane = a.plane != nullptr;
  const int wps = pk_waves_per_simd(kind, plane, self, a.lds_n0, a.njobs);
#define X(k, p, f, w)                                                                                \
  if (kind == k && plane == p && self == f && wps == w) {                                            \
    hipLaunchKernelGGL((k_panel_pk<k, p, f, w>), dim3(grid), dim3(f ? 64 : 128), lds, s, a, off, kc, \
                       count ? 1u : 0u);                                                             \
    return hipGetLastError();                                                                        \
  }
  TRIOSEQ_PKP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t panel_pk_occupancy(int kind, bool plane, bool self, uint32_t lds_n0, uint64_t njobs, int* blocks_per_cu) {
  const int wps = pk_waves_per_simd(kind, plane, self, lds_n0, njobs);
#define X(k, p, f, w)                                                                                        \
  if (kind == k && plane == p && self == f && wps == w)                                                      \
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_panel_pk<k, p, f, w>, f ? 64 : 128, \
                                                        (size_t)(lds_n0 + 64) * 4);
  TRIOSEQ_PKP(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace trioseq
