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
// What bounds it: long triplets (4096 x 4000 x 4150 by halves, 31.3 -> 15.5 ms
// against the int32 halves) the issue of the lone computing wave on each SIMD;
// shorter ones (1024 x 1000 x 1048, 975 -> 727 us) the chain of panel hops.
#include "packed.h"

namespace trioseq {
namespace {

constexpr int kRingC = 2 * kRing;  // corner rows: staged one step ahead of the other rings
constexpr int kSideLanes = kPkPanel / 2;   // lanes covering one face row, two entries each
constexpr int kSideRows = 64 / kSideLanes; // rows per load
constexpr int kSideLoads = kChunk / kSideRows;

struct PkPanelLds {
  __attribute__((aligned(16))) int sR[64][4];             // right column of each lane
  __attribute__((aligned(16))) int sB[64][4];             // bottom row of each lane
  int sX[64];                                             // bottom of each lane's left halo
  __attribute__((aligned(16))) int T[kRing][kPkPanel];    // halo rings: ring row t mod kRing serves step t
  __attribute__((aligned(16))) int Lf[kRing][kPkPanel];
  __attribute__((aligned(16))) int C[kRingC][kGK];
  __attribute__((aligned(16))) int ob[kRing][kPkPanel];   // out rows of the compute wave
  __attribute__((aligned(16))) int orr[kRing][kPkPanel];
  int oc[kRing];
  int cap[2][16];                                         // score tiles of both triplets
  int in_ready, out_done, out_flushed, job;
  uint32_t base;
};

// One panel's faces. Null: tensor edge (inputs) or not needed (outputs).
struct PkPanelIO {
  const int* top;     // bottom face of the panel above
  const int* left;    // right face of the panel to the left, its corner face behind it
  int* out;           // this panel's faces: bottom, right, corner
  bool bot, right;    // whether they have a consumer
  int gen;
  int* err;
  uint64_t wait_ticks;
};

// Half-wise a - b and a + b modulo 2^16 are psub and paddw.

// The compute wave. Folds local and semi-global bests into `best`, as the
// whole-triplet kernel does (local: M; semi-global: M + kc).
template <int KIND, bool PLANE>
__device__ void pk_panel_compute(PkPanelLds& S, const uint32_t* sel, const DevScoring& sc,
                                 const uint32_t* __restrict__ words, const TripletDesc& ta, const TripletDesc& tb,
                                 int n0, int pj, int pk, const PkPanelIO& io, uint16_t* capt, uint32_t off2,
                                 uint32_t& best, uint32_t kc) {
  constexpr int RJ = 4, RK = 4;
  constexpr int H = kPkPanel, W = kPkPanel;
  constexpr bool PAD = KIND != kGlobal;
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

  // Halo sources: ring rows for edge lanes, neighbours' slots otherwise.
  const bool y0 = y == 0, x0 = x == 0;
  const int* t_base = y0 ? &S.T[0][x * RK] : &S.sB[y0 ? 0 : lane - 8][0];
  const int* c_base = y0 ? &S.C[0][x] : &S.sX[y0 ? 0 : lane - 8];
  const int* l_base = x0 ? &S.Lf[0][y * RJ] : &S.sR[x0 ? 0 : lane - 1][0];
  const int t_str = y0 ? W : 0, c_str = y0 ? kGK : 0, l_str = x0 ? H : 0;
  const uint32_t* sl = sel + kShiftPre - y - x;

  int fin = 0, ffl = 0;
  bool gave_up = false;
  uint32_t zero2 = off2;  // stored value of M' = 0 (set at step 0, once the base is known)
  for (int c = 0; c < nchunks; ++c) {
    const int cb0 = c * kChunk;
    const bool cap_chunk = (n0a >= cb0 - kSkew && n0a <= cb0 + kChunk - 1) ||
                           (n0b >= cb0 - kSkew && n0b <= cb0 + kChunk - 1);
    const int* tb_ = t_base + (c & 1) * kChunk * t_str;
    const int* cb_ = c_base + (c & 3) * kChunk * c_str;
    const int* lb_ = l_base + (c & 1) * kChunk * l_str;
    uint32_t selv[kChunk];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) selv[s] = sl[cb0 + s];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) {
      const int t = cb0 + s;
      // Step t needs its halo rows staged and out row t mod kRing read back;
      // the counters read during the previous step usually already say so.
      if (!gave_up && !(fin > t && ffl > t - kRing)) {
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
      const int fin_next = lds_get(&S.in_ready);
      const int ffl_next = lds_get(&S.out_flushed);
      if (PAD && s == 0 && c == 0) zero2 = psub(off2, S.base);

      const uint32_t sv = selv[s];
      uint32_t A[RJ], B[RK], T[RK], Lh[RJ];
#pragma unroll
      for (int r = 0; r < RJ; ++r) A[r] = __builtin_amdgcn_perm(tabs.TBb[r], tabs.TBa[r], sv);
#pragma unroll
      for (int cc = 0; cc < RK; ++cc) B[cc] = __builtin_amdgcn_perm(tabs.TCb[cc], tabs.TCa[cc], sv);
      {
        const v4i v = lds_v4(tb_ + s * t_str);
        T[0] = (uint32_t)v.x, T[1] = (uint32_t)v.y, T[2] = (uint32_t)v.z, T[3] = (uint32_t)v.w;
        const v4i w = lds_v4(lb_ + s * l_str);
        Lh[0] = (uint32_t)w.x, Lh[1] = (uint32_t)w.y, Lh[2] = (uint32_t)w.z, Lh[3] = (uint32_t)w.w;
      }
      const uint32_t corner = (uint32_t)cb_[s * c_str];
      const int i = t - y - x;  // this lane's slice
      if (KIND == kSemiGlobal && axis_panel) {
        // The axes hold 0 (M' = g * index): see the whole-triplet kernel.
        if (j0 == 0) {
#pragma unroll
          for (int cc = 0; cc < RK; ++cc) T[cc] = i == 0 ? paddw(zero2, (uint32_t)(g * (k0 + cc)) * 0x10001u) : T[cc];
          if (k0 == 0) T[0] = i >= 0 ? paddw(zero2, (uint32_t)(g * i) * 0x10001u) : T[0];
        }
        if (k0 == 0) {
#pragma unroll
          for (int r = 0; r < RJ; ++r) Lh[r] = i == 0 ? paddw(zero2, (uint32_t)(g * (j0 + r)) * 0x10001u) : Lh[r];
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
        } else {
          const uint32_t sm = (i == n0a ? 0xFFFFu : 0u) | (i == n0b ? 0xFFFF0000u : 0u);
          if (((rcany | sm) & vm) != 0u) {
            // M + kc = stored - zero2 - g*(i + j + k) + kc.
            const uint32_t off0 = psub(((kc - (uint32_t)fi) & 0xFFFFu) * 0x10001u, zero2);
            uint32_t sb = 0;
#pragma unroll
            for (int r = 0; r < RJ; ++r)
#pragma unroll
              for (int cc = 0; cc < RK; ++cc)
                sb = umax2(sb, paddw(N[r][cc], psub(off0, (uint32_t)(r + cc) * g2)) & (RM[r] | CM[cc] | sm));
            best = umax2(best, sb & vm);
          }
        }
        fi += g;
      }

#pragma unroll
      for (int r = 0; r < RJ; ++r) S.sR[lane][r] = (int)N[r][RK - 1];
#pragma unroll
      for (int cc = 0; cc < RK; ++cc) S.sB[lane][cc] = (int)N[RJ - 1][cc];
      S.sX[lane] = (int)Lh[RJ - 1];

      // Out rows (row t mod kRing).
      const int ro = (c & 1) * kChunk + s;
      if (y == kGJ - 1) {
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) S.ob[ro][x * RK + cc] = (int)N[RJ - 1][cc];
      }
      if (x == kGK - 1) {
#pragma unroll
        for (int r = 0; r < RJ; ++r) S.orr[ro][y * RJ + r] = (int)N[r][RK - 1];
        if (y == 0) S.oc[ro] = (int)T[RK - 1];
      }
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (lane == 0) lds_put(&S.out_done, t + 1);
      fin = fin_next;
      ffl = ffl_next;

      if (cap_chunk) {
        if (PLANE) {
          if (i == n0a) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q) capt[lane * (RJ * RK) + q] = (uint16_t)(N[q / RK][q % RK] & 0xFFFFu);
          }
          if (i == n0b) {
#pragma unroll
            for (int q = 0; q < RJ * RK; ++q)
              capt[64 * RJ * RK + lane * (RJ * RK) + q] = (uint16_t)(N[q / RK][q % RK] >> 16);
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
    }
  }
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
          (int)((capt[lane * 16 + q] - zero) & 0xFFFFu) + gap2 * (n0 + j + k);
  }
}

// The memory wave: keeps the compute wave's halo rings filled from the
// neighbours' tagged faces and writes its out rows. For steps u .. u + 7 one
// poll loads rows u + 7 .. u + 14 of the top, right and corner faces; lane l of
// a load holds entries 2(l mod 16), +1 of row l / 16 (+ 4 in the second load),
// so the first row with a stale entry is the lowest set bit of a ballot. Every
// wait is bounded (past the limit the error flag is raised and the rows are
// staged as they are).
__device__ void pk_panel_memory(PkPanelLds& S, int n0, const PkPanelIO& io, uint32_t off2) {
  constexpr uint32_t RB = kPkPanel * 8u;  // bytes of a face row
  const int lane = threadIdx.x & 63;
  const int stepsp = (n0 + 1 + kSkew + kChunk - 1) / kChunk * kChunk;
  const uint64_t rows = pk_face_rows((uint32_t)n0);
  const bool has_top = io.top != nullptr, has_left = io.left != nullptr;
  const uint32_t side = (uint32_t)(rows * RB), all = side * 2 + (uint32_t)rows * 8u;
  const int* any = has_top ? io.top : io.left;
  const Rsrc r_top = make_rsrc(any, has_top ? side : 0);
  // Left neighbour: right face, then the corner face.
  const Rsrc r_left = make_rsrc(has_left ? io.left : any, has_left ? side + (uint32_t)rows * 8u : 0);
  const Rsrc r_out = make_rsrc(io.out, all);
  const int gen = io.gen;
  const int rr0 = lane / kSideLanes, pr = lane % kSideLanes, grp = pr >> 1;
  const uint32_t sent2 = kSentP * 0x10001u;
  const uint32_t vside = (uint32_t)(rr0 * RB + pr * 16);
  const bool has_corner = has_top && has_left;

  // Rings that nothing fills hold the outside value; so does the corner row of
  // step 0 (its slices lie before 0, lane 0's comes with the corner face).
  for (int q = lane; q < kRing * kPkPanel; q += 64) {
    if (!has_top) (&S.T[0][0])[q] = (int)sent2;
    if (!has_left) (&S.Lf[0][0])[q] = (int)sent2;
  }
  for (int q = lane; q < kRingC * kGK; q += 64) (&S.C[0][0])[q] = (int)sent2;
  bool have_base = !has_top && !has_left;
  uint32_t delta = off2;  // off - base, per half modulo 2^16

  int staged = 0, flushed = 0;
  uint64_t stall_since = 0;
  bool gave_up = false;
  while (staged < stepsp || flushed < stepsp) {
    const int done = lds_get(&S.out_done);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    bool progress = false;
    const int u = staged;
    // (The corner rows run one step ahead.)
    const int nb = min(min(kChunk, stepsp - u), done + kRing - u);
    if (nb > 0) {
      v4i tv[kSideLoads], lv[kSideLoads];
      v2i cv = {0, 0};
      const uint32_t z = opaque_zero();
      const uint32_t vo = vside + (uint32_t)(u + kGJ - 1) * RB;
      uint64_t m[kSideLoads], mc = 0;
#pragma unroll
      for (int q = 0; q < kSideLoads; ++q) {
        if (has_top) tv[q] = __builtin_amdgcn_raw_buffer_load_b128(r_top, vo + q * kSideRows * RB, z, kCohDevice);
        if (has_left) lv[q] = __builtin_amdgcn_raw_buffer_load_b128(r_left, vo + q * kSideRows * RB, z, kCohDevice);
      }
      if (has_corner)
        cv = __builtin_amdgcn_raw_buffer_load_b64(
            r_left, lane < kChunk ? side + (uint32_t)(u + kGJ - 1 + lane) * 8u : kOob, z, kCohDevice);
#pragma unroll
      for (int q = 0; q < kSideLoads; ++q) {
        const int slice = u + rr0 + q * kSideRows - grp;
        int tag = kTagAlways;
        if (has_top) tag = min(tv[q].y, tv[q].w);
        if (has_left) tag = min(tag, min(lv[q].y, lv[q].w));
        m[q] = __builtin_amdgcn_ballot_w64((uint32_t)slice <= (uint32_t)n0 && tag < gen);
      }
      if (has_corner) mc = __builtin_amdgcn_ballot_w64(lane < kChunk && u + lane <= n0 && cv.y < gen);
      int k = nb;
#pragma unroll
      for (int q = kSideLoads - 1; q >= 0; --q)
        if (m[q]) k = min(k, q * kSideRows + __builtin_ctzll(m[q]) / kSideLanes);
      if (mc) k = min(k, __builtin_ctzll(mc));
      if (gave_up) k = nb;
      if (k <= 0 && stall_since && wall_clock64() - stall_since > io.wait_ticks) {
        raise_error(io.err);
        gave_up = true;
        k = nb;
      }
      if (k > 0) {
        if (!have_base) {
          // Lane 0 holds entry 0 of row 7, slice 0.
          const uint32_t b = (uint32_t)__builtin_amdgcn_readfirstlane(has_top ? tv[0].x : lv[0].x);
          delta = psub(off2, b);
          if (lane == 0) S.base = b;
          have_base = true;
        }
#pragma unroll
        for (int q = 0; q < kSideLoads; ++q) {
          const int rr = rr0 + q * kSideRows, st = u + rr;
          const bool before = st - grp < 0;  // slices before 0 lie outside the tensor
          if (rr < k) {
            if (has_top) {
              const uint32_t v0 = before ? sent2 : paddw((uint32_t)tv[q].x, delta);
              const uint32_t v1 = before ? sent2 : paddw((uint32_t)tv[q].z, delta);
              *reinterpret_cast<v2i*>(&S.T[st & (kRing - 1)][2 * pr]) = (v2i){(int)v0, (int)v1};
              // Entry 4x + 3 is the corner of lane x + 1 at the next step.
              if ((pr & 1) && grp + 1 < kGK) S.C[(st + 1) & (kRingC - 1)][grp + 1] = (int)v1;
            }
            if (has_left) {
              const uint32_t v0 = before ? sent2 : paddw((uint32_t)lv[q].x, delta);
              const uint32_t v1 = before ? sent2 : paddw((uint32_t)lv[q].z, delta);
              *reinterpret_cast<v2i*>(&S.Lf[st & (kRing - 1)][2 * pr]) = (v2i){(int)v0, (int)v1};
            }
          }
        }
        if (has_corner && lane < k) S.C[(u + lane) & (kRingC - 1)][0] = (int)paddw((uint32_t)cv.x, delta);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        if (lane == 0) lds_put(&S.in_ready, u + k);
        staged = u + k;
        progress = true;
      }
    }
    // Flush finished out rows, back to M' modulo 2^16.
    const int nf = min(kChunk, lds_get(&S.out_done) - flushed);
    if (nf > 0) {
      v2i bv[kSideLoads], rv[kSideLoads];
#pragma unroll
      for (int q = 0; q < kSideLoads; ++q) {
        const int ro = (flushed + rr0 + q * kSideRows) & (kRing - 1);
        bv[q] = *reinterpret_cast<const v2i*>(&S.ob[ro][2 * pr]);
        rv[q] = *reinterpret_cast<const v2i*>(&S.orr[ro][2 * pr]);
      }
      const int cv = S.oc[(flushed + lane) & (kRing - 1)];
      const uint32_t vo = vside + (uint32_t)flushed * RB;
#pragma unroll
      for (int q = 0; q < kSideLoads; ++q) {
        const bool live = rr0 + q * kSideRows < nf;
        const uint32_t o = live ? vo + q * kSideRows * RB : kOob;
        if (io.bot)
          __builtin_amdgcn_raw_buffer_store_b128((v4i){(int)psub((uint32_t)bv[q].x, delta), gen,
                                                       (int)psub((uint32_t)bv[q].y, delta), gen},
                                                 r_out, o, 0, kCohDevice);
        if (io.right)
          __builtin_amdgcn_raw_buffer_store_b128((v4i){(int)psub((uint32_t)rv[q].x, delta), gen,
                                                       (int)psub((uint32_t)rv[q].y, delta), gen},
                                                 r_out, live ? o + side : kOob, 0, kCohDevice);
      }
      if (io.right)
        __builtin_amdgcn_raw_buffer_store_b64((v2i){(int)psub((uint32_t)cv, delta), gen}, r_out,
                                              lane < nf ? 2 * side + (uint32_t)(flushed + lane) * 8u : kOob, 0,
                                              kCohDevice);
      __atomic_signal_fence(__ATOMIC_SEQ_CST);
      if (lane == 0) lds_put(&S.out_flushed, flushed + nf);
      flushed += nf;
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
// workgroup and every wait ends.
template <int KIND, bool PLANE>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2)))
k_panel_pk(SweepArgs a, uint32_t off, uint32_t kc) {
  constexpr int H = kPkPanel, W = kPkPanel;
  __shared__ PkPanelLds S;
  __shared__ __attribute__((aligned(16))) uint16_t capt[PLANE ? 2 * 64 * 16 : 1];
  extern __shared__ uint32_t selw[];
  const int wave = threadIdx.x >> 6;
  const uint32_t off2 = off * 0x10001u;
  const int gen = __hip_atomic_load(a.ctl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t staged = 0xFFFFFFFFu;
  for (;;) {
    if (threadIdx.x == 0) S.job = atomicAdd(a.counter, 1);
    __syncthreads();
    const int idx = S.job;
    if (idx >= (int)a.njobs) break;
    const JobDesc jd = a.jobs[idx];
    const TripletDesc ta = a.desc[jd.trip], tb = a.desc[jd.trip + 1];
    const int n0 = (int)max(ta.len[0], tb.len[0]);
    const int n1 = (int)max(ta.len[1], tb.len[1]), n2 = (int)max(ta.len[2], tb.len[2]);
    if (jd.trip != staged) {
      stage_selectors(selw, a.words, ta, tb, n0, (int)threadIdx.x, 128);
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
    const uint64_t per_panel = pk_panel_ints((uint32_t)n0), side = pk_face_rows((uint32_t)n0) * (2 * kPkPanel);
    const uint32_t p = jd.panel;
    const int pj = (int)(p / (uint32_t)PK), pk = (int)(p % (uint32_t)PK);
    int* pool = a.pface + ta.face_off;
    PkPanelIO io;
    io.top = pj ? pool + (uint64_t)(p - PK) * per_panel : nullptr;
    io.left = pk ? pool + (uint64_t)(p - 1) * per_panel + side : nullptr;
    io.out = pool + (uint64_t)p * per_panel;
    io.bot = pj + 1 < PJ;
    io.right = pk + 1 < PK;
    io.gen = gen;
    io.err = a.ctl + 1;
    io.wait_ticks = a.wait_ticks;
    uint32_t best = 0;
    if (wave == 0)
      pk_panel_compute<KIND, PLANE>(S, selw, a.sc, a.words, ta, tb, n0, pj, pk, io, capt, off2, best, kc);
    else
      pk_panel_memory(S, n0, io, off2);
    __syncthreads();
    // Both waves are done: a wait of this job that gave up has raised the flag
    // by now, and upstream panels raised theirs before writing the faces this
    // job read.
    const uint32_t zero2 = psub(off2, S.base);
    if (PLANE) {
      // One half's plane by each wave.
      const TripletDesc& td = wave ? tb : ta;
      pk_write_plane(capt + wave * 64 * 16, a.plane + a.plane_off[jd.trip + wave], td, pj, pk,
                     wave ? zero2 >> 16 : zero2 & 0xFFFFu, a.sc.gap2);
    }
    if (KIND == kGlobal && !PLANE && threadIdx.x < 2) {
      const int h = (int)threadIdx.x;
      const TripletDesc& td = h ? tb : ta;
      const int r = (int)td.len[1] - pj * H, c = (int)td.len[2] - pk * W;
      if (r >= 0 && r < H && c >= 0 && c < W) {
        const uint32_t v = psub((uint32_t)S.cap[h][(r & 3) * 4 + (c & 3)], zero2);
        const int m = (int)(h ? v >> 16 : v & 0xFFFFu);
        publish_score(a.scores + td.out, m + a.sc.gap2 * (int)(td.len[0] + td.len[1] + td.len[2]), io.err);
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
        const int prev = __hip_atomic_fetch_add(acc + 1, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == PJ * PK - 1) {
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

#define TRIOSEQ_PKP(X) X(0, false) X(0, true) X(1, false) X(2, false) X(2, true)

}  // namespace

hipError_t launch_panel_pk(int kind, const SweepArgs& a, uint32_t off, uint32_t kc, int grid, hipStream_t s) {
  const size_t lds = (size_t)(a.lds_n0 + 64) * 4;
  const bool plane = a.plane != nullptr;
#define X(k, p)                                                                                   \
  if (kind == k && plane == p) {                                                                  \
    hipLaunchKernelGGL((k_panel_pk<k, p>), dim3(grid), dim3(128), lds, s, a, off, kc);            \
    return hipGetLastError();                                                                     \
  }
  TRIOSEQ_PKP(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t panel_pk_occupancy(int kind, bool plane, uint32_t lds_n0, int* blocks_per_cu) {
#define X(k, p)           \
  if (kind == k && plane == p) \
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, k_panel_pk<k, p>, 128, (size_t)(lds_n0 + 64) * 4);
  TRIOSEQ_PKP(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace trioseq
