// One wavefront sweeping a pair of whole triplets (packed.hip has the idea).
#pragma once
#include "packed.h"

namespace trioseq {
namespace {

// LDS of a packed wavefront: the lanes' edge slots and the capture tile
// (one object), and the halo rings, one object per chunk half. Staging of
// chunk c + 1 goes to the half that chunk c does not read. Kept as two
// objects, each a fixed object in its copy of the chunk body, the halves
// take static addresses. (The compiler still makes a chunk's first halo
// read wait for the loads in flight, since a lane's read picks between a
// ring row and a slot; the other wave on the SIMD covers that wait.)
template <int RJ, int RK>
struct PkLds {
  __attribute__((aligned(16))) int sR[64][RJ];  // right column of each lane
  __attribute__((aligned(16))) int sB[64][RK];  // bottom row of each lane
  int sX[64];                                   // bottom of each lane's left halo
  int cap[RJ * RK];                             // tile of triplet a's score cell
  int wsync;
};
template <int RJ, int RK>
struct PkRing {
  static constexpr int H = kGJ * RJ, W = kGK * RK;
  __attribute__((aligned(16))) int T[kChunk][W];    // top face rows of the chunk
  __attribute__((aligned(16))) int C[kChunk][kGK];  // corners of the top-edge lanes
  __attribute__((aligned(16))) int L[kChunk][H];    // left face rows of the chunk
};

// One panel of a pair (plain faces in the wave's workspace, one 32-bit word
// per entry holding both halves). Global scoring captures each triplet's
// cell (n0, n1, n2) when the panel holds it: triplet a's tile into L.cap,
// b's into capb. Semi-global and local scoring fold the panel's cells into
// the lane's running best (both halves; see k_sweep_pk for its meaning).
template <int RJ, int RK, int KIND, bool FUSED, int XCH, bool DMA>
__device__ void sweep_panel_pk(PkLds<RJ, RK>& L, PkRing<RJ, RK>& R0, PkRing<RJ, RK>& R1, int* capb,
                               const uint32_t* sel, const DevScoring& sc,
                               const uint32_t* __restrict__ words, const TripletDesc& ta,
                               const TripletDesc& tb, int n0, int pj, int pk, const int* top, const int* left,
                               int* bot, int* right, uint32_t base2, uint32_t& best, uint32_t kc) {
  constexpr int H = kGJ * RJ, W = kGK * RK, RR = H + 4;
  constexpr bool PAD = KIND != kGlobal;
  const int lane = threadIdx.x & 63;
  const int y = lane >> 3, x = lane & 7;
  const int j0 = pj * H + y * RJ, k0 = pk * W + x * RK;
  const int n1a = (int)ta.len[1], n1b = (int)tb.len[1], n2a = (int)ta.len[2], n2b = (int)tb.len[2];
  PkTables<RJ, RK> tabs;
  pk_tables<PAD>(tabs, sc, words, ta, tb, j0, k0);
  const auto& TBa = tabs.TBa;
  const auto& TBb = tabs.TBb;
  const auto& TCa = tabs.TCa;
  const auto& TCb = tabs.TCb;
  const auto& C2 = tabs.C2;

  uint32_t P[RJ][RK], D[RJ][RK], Lp[RJ], Tp[RK];
#pragma unroll
  for (int r = 0; r < RJ; ++r) {
    Lp[r] = kSentP * 0x10001u;
#pragma unroll
    for (int c = 0; c < RK; ++c) P[r][c] = D[r][c] = kSentP * 0x10001u;
  }
#pragma unroll
  for (int c = 0; c < RK; ++c) Tp[c] = kSentP * 0x10001u;

  const int nsteps = n0 + 1 + kSkew;
  const int nchunks = (nsteps + kChunk - 1) / kChunk;
  // Capture: the lane holding cell (n1, n2) of a triplet in this panel keeps
  // its tile at that triplet's slice n0.
  const int rsa = n1a - j0, csa = n2a - k0;
  const int rsb = n1b - j0, csb = n2b - k0;
  const bool own_a = rsa >= 0 && rsa < RJ && csa >= 0 && csa < RK;
  const bool own_b = rsb >= 0 && rsb < RJ && csb >= 0 && csb < RK;
  const int n0a = (int)ta.len[0], n0b = (int)tb.len[0];

  // Semi-global and local scoring (g = -2*gap >= 0). fi = g*(i + j0 + k0)
  // for the lane's slice i of the current step; a cell of anti-diagonal
  // class d = r + c of the tile lies at index sum i + j0 + k0 + d.
  constexpr int ND = RJ + RK - 1;
  const int g = -sc.gap2;
  const uint32_t g2 = (uint32_t)g * 0x10001u;
  int fi = g * (j0 + k0 - y - x);
  // Semi-global: the halves of the rows and columns that are a triplet's
  // last row n1 or last column n2 (masks of both halves).
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

  const uint32_t frows = face_rows((uint32_t)n0);
  constexpr uint32_t ts = W * 4u, RRB = RR * 4u;
  const Rsrc r_top = make_rsrc(top, (uint64_t)frows * ts);
  const Rsrc r_left = make_rsrc(left, (uint64_t)frows * RRB);
  const Rsrc r_bot = make_rsrc(bot ? bot : top, bot ? (uint64_t)frows * ts : 0);
  const Rsrc r_right = make_rsrc(right ? right : left, right ? (uint64_t)frows * RRB : 0);

  // Staging, as in sweep_panel (plain faces): value q of a chunk is entry
  // lane + 64 q of the top, corner or left ring.
  constexpr int QT = kChunk * W / 64, QC = kChunk * kGK / 64, QL = kChunk * H / 64;
  constexpr int NPF = QT + QC + QL;
  constexpr int RT = 64 / W, RL = 64 / H;
  static_assert(64 % W == 0 && 64 % H == 0 && QC == 1, "ring widths must divide 64");
  const int eT = lane % W;
  const uint32_t offT = (uint32_t)((kGJ - 1 + lane / W) * (int)ts + eT * 4);
  const int eC = lane % kGK;
  const bool corner_from_left = eC == 0;
  const uint32_t offC = corner_from_left ? (uint32_t)((kGK - 1 + lane / kGK) * (int)RRB)
                                         : (uint32_t)((kGJ - 2 + lane / kGK) * (int)ts + (eC * RK - 1) * 4);
  const int eL = lane % H;
  const uint32_t offL = (uint32_t)((kGK - 1 + lane / H) * (int)RRB + (4 + eL) * 4);
  int pf[DMA ? 1 : NPF];
  auto stage_load = [&](int c, PkRing<RJ, RK>& dst) {
    const uint32_t cb0 = (uint32_t)(c * kChunk);
    if (DMA) {
      // Straight into the ring half of chunk c (lane l's word of each load
      // lands at the destination + 4 l, which is where it belongs); the
      // corner loads go to the same slots from the top or the left face,
      // so each lane takes only one of them.
      typedef __attribute__((address_space(3))) void* LdsPtr;
#pragma unroll
      for (int q = 0; q < QT; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_top, (LdsPtr)(&dst.T[0][0] + 64 * q), 4, offT,
                                                 (cb0 + q * RT) * ts, 0, 0);
      if (corner_from_left)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_left, (LdsPtr)&dst.C[0][0], 4, offC, cb0 * RRB, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_top, (LdsPtr)&dst.C[0][0], 4, offC, cb0 * ts, 0, 0);
#pragma unroll
      for (int q = 0; q < QL; ++q)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r_left, (LdsPtr)(&dst.L[0][0] + 64 * q), 4, offL,
                                                 (cb0 + q * RL) * RRB, 0, 0);
      return;
    }
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      if (q < QT) {
        pf[q] = (int)__builtin_amdgcn_raw_buffer_load_b32(r_top, offT, (cb0 + q * RT) * ts, 0);
      } else if (q < QT + QC) {
        const uint32_t ot = corner_from_left ? kOob : offC, ol = corner_from_left ? offC : kOob;
        pf[q] = (int)(__builtin_amdgcn_raw_buffer_load_b32(r_top, ot, cb0 * ts, 0) |
                      __builtin_amdgcn_raw_buffer_load_b32(r_left, ol, cb0 * RRB, 0));
      } else {
        pf[q] = (int)__builtin_amdgcn_raw_buffer_load_b32(r_left, offL, (cb0 + (q - QT - QC) * RL) * RRB, 0);
      }
    }
  };
  auto stage_finish = [&](int c, PkRing<RJ, RK>& dst) {
    if (DMA) {
      // The loads of chunk c were issued at the first step of chunk c - 1,
      // ahead of that chunk's face stores (kStores per step); vector memory
      // operations complete in issue order, so once no more than those
      // stores are outstanding the loads are done, and the stores need not
      // be waited for. Chunk 0's loads were issued just before, with no
      // store after them.
      constexpr int kStores = RK / 4 + RJ / 4 + 1;
      constexpr int kAfter = kStores * kChunk;
      static_assert(kAfter < 64, "vmcnt holds at most 63");
      constexpr int kWaitAfter = (kAfter & 15) | ((kAfter >> 4) << 14) | (0x7 << 4) | (0xF << 8);
      if (c == 0)
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      else
        __builtin_amdgcn_s_waitcnt(kWaitAfter);  // vmcnt(kAfter)
      return;
    }
#pragma unroll
    for (int q = 0; q < NPF; ++q) {
      if (q < QT)
        (&dst.T[0][0])[lane + 64 * q] = pf[q];
      else if (q < QT + QC)
        dst.C[0][lane] = pf[q];
      else
        (&dst.L[0][0])[lane + 64 * (q - QT - QC)] = pf[q];
    }
  };
  stage_load(0, R0);
#pragma unroll
  for (int r = 0; r < RJ; ++r) L.sR[lane][r] = (int)(kSentP * 0x10001u);
#pragma unroll
  for (int c = 0; c < RK; ++c) L.sB[lane][c] = (int)(kSentP * 0x10001u);
  L.sX[lane] = (int)(kSentP * 0x10001u);

  const bool y0 = y == 0, x0 = x == 0;
  const bool tring = XCH || y0, lring = XCH || x0;
  // Halo rows: edge lanes read the chunk's ring half, inner lanes their
  // neighbour's slot (the same every step).
  const int* t_slot = &L.sB[y0 ? 0 : lane - 8][0];
  const int t_str = tring ? W : 0;
  const int* c_slot = &L.sX[y0 ? 0 : lane - 8];
  const int c_str = tring ? kGK : 0;
  const int* l_slot = &L.sR[x0 ? 0 : lane - 1][0];
  const int l_str = lring ? H : 0;
  const int up_addr = ((lane + 64 - kGK) & 63) << 2;
  const uint32_t vo_bot = (y == kGJ - 1) ? (uint32_t)(x * RK * 4) : kOob;
  const uint32_t vo_right = (x == kGK - 1) ? (uint32_t)((4 + y * RJ) * 4) : kOob;
  const uint32_t vo_corner = (x == kGK - 1 && y == 0) ? 0u : kOob;
  const int sl_base = kShiftPre - y - x;
  const bool seed_lane = pj == 0 && pk == 0 && lane == 0;

  // Chunk c reads ring half cur and stages chunk c + 1 into nxt. With loads
  // straight to LDS the loop below takes two chunks per turn, so that both
  // halves are fixed objects in each copy of the body.
  auto run_chunk = [&](int c, PkRing<RJ, RK>& cur, PkRing<RJ, RK>& nxt) __attribute__((always_inline)) {
    stage_finish(c, cur);
    const bool more = c + 1 < nchunks;
    const int cb0 = c * kChunk;
    const bool cap_chunk = (n0a >= cb0 - kSkew && n0a <= cb0 + kChunk - 1) ||
                           (n0b >= cb0 - kSkew && n0b <= cb0 + kChunk - 1);
    const uint32_t vb = vo_bot + (uint32_t)cb0 * ts, vr = vo_right + (uint32_t)cb0 * RRB,
                   vc = vo_corner + (uint32_t)cb0 * RRB;
    const int* tb = tring ? &cur.T[0][x * RK] : t_slot;
    const int* cbp = tring ? &cur.C[0][x] : c_slot;
    const int* lb = lring ? &cur.L[0][y * RJ] : l_slot;
    const uint32_t* sp = sel + sl_base + cb0;
    uint32_t selv[kChunk];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) selv[s] = sp[s];
#pragma unroll
    for (int s = 0; s < kChunk; ++s) {
      if (s == 0 && more) stage_load(c + 1, nxt);
      const int t = cb0 + s;
      const uint32_t sv = selv[s];
      uint32_t A[RJ], B[RK];
#pragma unroll
      for (int r = 0; r < RJ; ++r) A[r] = __builtin_amdgcn_perm(TBb[r], TBa[r], sv);
#pragma unroll
      for (int cc = 0; cc < RK; ++cc) B[cc] = __builtin_amdgcn_perm(TCb[cc], TCa[cc], sv);
      uint32_t T[RK], Lh[RJ];
#pragma unroll
      for (int cc = 0; cc < RK; cc += 4) {
        const v4i v = lds_v4(tb + s * t_str + cc);
        T[cc] = (uint32_t)v.x, T[cc + 1] = (uint32_t)v.y, T[cc + 2] = (uint32_t)v.z, T[cc + 3] = (uint32_t)v.w;
      }
#pragma unroll
      for (int r = 0; r < RJ; r += 4) {
        const v4i v = lds_v4(lb + s * l_str + r);
        Lh[r] = (uint32_t)v.x, Lh[r + 1] = (uint32_t)v.y, Lh[r + 2] = (uint32_t)v.z, Lh[r + 3] = (uint32_t)v.w;
      }
      uint32_t corner = (uint32_t)cbp[s * c_str];
      if (XCH) {
        // As in sweep_panel: inner lanes take their upper neighbour's row
        // and corner through ds_bpermute and their left neighbour's column
        // through a DPP row shift, from its previous-step registers.
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) {
          const uint32_t nb = (uint32_t)__builtin_amdgcn_ds_bpermute(up_addr, (int)P[RJ - 1][cc]);
          T[cc] = y0 ? T[cc] : nb;
        }
        {
          const uint32_t nb = (uint32_t)__builtin_amdgcn_ds_bpermute(up_addr, (int)Lp[RJ - 1]);
          corner = y0 ? corner : nb;
        }
#pragma unroll
        for (int r = 0; r < RJ; ++r) {
          const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)P[r][RK - 1], 0x111, 0xF, 0xF, true);
          Lh[r] = x0 ? Lh[r] : nb;
        }
      }
      const int i = t - y - x;  // this lane's slice
      if (KIND == kSemiGlobal && axis_panel) {
        // The axes hold 0 (stored base + g*index, both halves): at slice 0
        // the virtual row above the first panel row holds base + g*k and the
        // virtual column left of the first panel column base + g*j, and at
        // k = 0 the virtual row holds base + g*i; the single move (+0)
        // copies them in. Other moves from there take the zero row/column-0
        // tables and give values the single moves already reach.
        if (j0 == 0) {
#pragma unroll
          for (int cc = 0; cc < RK; ++cc) T[cc] = i == 0 ? base2 + (uint32_t)(g * (k0 + cc)) * 0x10001u : T[cc];
          if (k0 == 0) T[0] = i >= 0 ? base2 + (uint32_t)(g * i) * 0x10001u : T[0];
        }
        if (k0 == 0) {
#pragma unroll
          for (int r = 0; r < RJ; ++r) Lh[r] = i == 0 ? base2 + (uint32_t)(g * (j0 + r)) * 0x10001u : Lh[r];
        }
      }
      // Local floors per anti-diagonal class, F_d = base + fi + g*d in both
      // halves (M >= 0); none before slice 0 (0 there, below every value).
      uint32_t F[ND];
      if (KIND == kLocal) {
        asm volatile("" : "+v"(fi));  // one step's floors live at a time
        const uint32_t f0 = i >= 0 ? base2 + (uint32_t)fi * 0x10001u : 0u;
#pragma unroll
        for (int d = 0; d < ND; ++d) F[d] = f0 + (uint32_t)d * g2;
      }
      // Terms of the previous slice first (formed while the halo reads are
      // in flight): Q = best of the single move along S0 and its two double
      // moves, X7 the triple move. The fused form computes them cell by cell
      // instead (no registers held for them across the tile). Local scoring
      // folds X7 and the floor into Q.
      uint32_t Q[RJ][RK], X7[RJ][RK], N[RJ][RK];
      auto prev_terms = [&](int r, int cc) {
        const uint32_t up_prev = r ? P[r - 1][cc] : Tp[cc];
        const uint32_t left_prev = cc ? P[r][cc - 1] : Lp[r];
        Q[r][cc] = pmax3(P[r][cc], padd(up_prev, A[r]), padd(left_prev, B[cc]));
        X7[r][cc] = D[r][cc] + A[r] + B[cc];
        if (KIND == kLocal) Q[r][cc] = pmax3(Q[r][cc], X7[r][cc], F[r + cc]);
      };
      if (!FUSED) {
#pragma unroll
        for (int r = 0; r < RJ; ++r)
#pragma unroll
          for (int cc = 0; cc < RK; ++cc) prev_terms(r, cc);
      }
#pragma unroll
      for (int r = 0; r < RJ; ++r)
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) {
          if (FUSED) prev_terms(r, cc);
          const uint32_t up_cur = r ? N[r - 1][cc] : T[cc];
          const uint32_t left_cur = cc ? N[r][cc - 1] : Lh[r];
          const uint32_t diag_cur = r ? (cc ? N[r - 1][cc - 1] : Lh[r - 1]) : (cc ? T[cc - 1] : corner);
          const uint32_t x6 = padd(diag_cur, C2[r][cc]);
          if (KIND == kLocal)
            N[r][cc] = pmax3(pmax2(Q[r][cc], x6), up_cur, left_cur);
          else
            N[r][cc] = pmax3(pmax3(Q[r][cc], X7[r][cc], x6), up_cur, left_cur);
          // Global M'(0,0,0) = 0: the one real start, cell (0,0) of lane 0
          // of the first panel at step 0, set before any other cell reads it.
          if (KIND == kGlobal && r == 0 && cc == 0) N[0][0] = (t == 0 && seed_lane) ? base2 : N[0][0];
          D[r][cc] = x6;
        }

      // Masks of the halves whose triplet has this slice (0 <= i <= its n0)
      // and of those whose last slice it is.
      const uint32_t vm = ((uint32_t)i <= (uint32_t)n0a ? 0xFFFFu : 0u) | ((uint32_t)i <= (uint32_t)n0b ? 0xFFFF0000u : 0u);
      if (KIND == kLocal) {
        // M = stored value - F_d, never negative on slices from 0 (every
        // cell is floored); the best class maximum minus its floor.
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
          sb = umax2(sb, psub(m, F[d]));
        }
        best = umax2(best, sb & vm);
      } else if (KIND == kSemiGlobal) {
        // Cells of a triplet's last slice, row or column (on its slices 0
        // .. n0), as M + kc = stored - base - g*(i + j + k) + kc, which the
        // host keeps within [1, 0xFFFF]; masked cells give 0.
        const uint32_t sm = (i == n0a ? 0xFFFFu : 0u) | (i == n0b ? 0xFFFF0000u : 0u);
        if (((rcany | sm) & vm) != 0u) {
          const uint32_t off0 = ((uint32_t)(kc - (base2 & 0xFFFFu) - (uint32_t)fi) & 0xFFFFu) * 0x10001u;
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

      if (!XCH) {
#pragma unroll
        for (int r = 0; r < RJ; ++r) L.sR[lane][r] = (int)N[r][RK - 1];
#pragma unroll
        for (int cc = 0; cc < RK; ++cc) L.sB[lane][cc] = (int)N[RJ - 1][cc];
        L.sX[lane] = (int)Lh[RJ - 1];
      }
#pragma unroll
      for (int cc = 0; cc < RK; cc += 4)
        __builtin_amdgcn_raw_buffer_store_b128(
            (v4i){(int)N[RJ - 1][cc], (int)N[RJ - 1][cc + 1], (int)N[RJ - 1][cc + 2], (int)N[RJ - 1][cc + 3]},
            r_bot, vb + (s * ts + cc * 4), 0, 0);
#pragma unroll
      for (int r = 0; r < RJ; r += 4)
        __builtin_amdgcn_raw_buffer_store_b128(
            (v4i){(int)N[r][RK - 1], (int)N[r + 1][RK - 1], (int)N[r + 2][RK - 1], (int)N[r + 3][RK - 1]},
            r_right, vr + (s * RRB + r * 4), 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32((int)T[RK - 1], r_right, vc + s * RRB, 0, 0);
      if (KIND == kGlobal && cap_chunk) {
        if (own_a && i == n0a) {
#pragma unroll
          for (int r = 0; r < RJ; ++r)
#pragma unroll
            for (int cc = 0; cc < RK; ++cc) L.cap[r * RK + cc] = (int)N[r][cc];
        }
        if (own_b && i == n0b) {
#pragma unroll
          for (int r = 0; r < RJ; ++r)
#pragma unroll
            for (int cc = 0; cc < RK; ++cc) capb[r * RK + cc] = (int)N[r][cc];
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
  };
  if constexpr (DMA) {
    for (int c = 0; c < nchunks; c += 2) {
      run_chunk(c, R0, R1);
      if (c + 1 < nchunks) run_chunk(c + 1, R1, R0);
    }
  } else {
    // Staged through registers, the rings are written by LDS stores, which
    // need no such care; one copy of the body keeps register pressure down.
    for (int c = 0; c < nchunks; ++c) run_chunk(c, (c & 1) ? R1 : R0, (c & 1) ? R0 : R1);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
}

// A pair of whole triplets (descriptors jd.trip and the next) swept by one
// wavefront over all panels of the common grid, row by row, in the wave's own
// face workspace. pk_top / pk_left: plain sentinel faces holding kSentP in
// both halves. base: the stored value of M' = 0. Local scoring keeps each
// lane's best M per half, semi-global its best M + kc (kc > 0 keeps every
// candidate positive); the wave's maxima are the scores.
template <int RJ, int RK, int KIND, bool FUSED, int XCH, bool DMA>
__device__ void pk_whole_pair(PkLds<RJ, RK>& L, PkRing<RJ, RK>& R0, PkRing<RJ, RK>& R1, int* capb, uint32_t* selw,
                              const SweepArgs& a, const JobDesc& jd, int* face, const int* pk_top,
                              const int* pk_left, uint32_t base, uint32_t kc) {
  constexpr int H = kGJ * RJ, W = kGK * RK;
  const uint32_t base2 = base * 0x10001u;
  const TripletDesc ta = a.desc[jd.trip], tb = a.desc[jd.trip + 1];
  const int n0 = (int)max(ta.len[0], tb.len[0]);
  const int n1 = (int)max(ta.len[1], tb.len[1]), n2 = (int)max(ta.len[2], tb.len[2]);
  stage_selectors(selw, a.words, ta, tb, n0, threadIdx.x & 63, 64);
  const int PJ = n1 / H + 1, PK = n2 / W + 1;
  const uint64_t rows = face_rows((uint32_t)n0);
  int* fb = face;
  int* fr = face + rows * (uint64_t)(PK * W);
  const int pja = (int)ta.len[1] / H, pka = (int)ta.len[2] / W;
  const int pjb = (int)tb.len[1] / H, pkb = (int)tb.len[2] / W;
  uint32_t best = 0;
  for (int pj = 0; pj < PJ; ++pj) {
    for (int pk = 0; pk < PK; ++pk) {
      int* col = fb + (uint64_t)pk * rows * W;
      sweep_panel_pk<RJ, RK, KIND, FUSED, XCH, DMA>(L, R0, R1, capb, selw, a.sc, a.words, ta, tb, n0, pj, pk,
                                                    pj ? col : pk_top, pk ? fr : pk_left,
                                                    pj + 1 < PJ ? col : nullptr, pk + 1 < PK ? fr : nullptr,
                                                    base2, best, kc);
      // Scores of the triplets whose last cell this panel held (the owner
      // lane's tile is in LDS; lane 0 reads the cell and stores the score).
      if (KIND == kGlobal && (threadIdx.x & 63) == 0) {
        if (pj == pja && pk == pka) {
          const int r = (int)ta.len[1] - pja * H, cc = (int)ta.len[2] - pka * W;
          const int v = L.cap[(r % RJ) * RK + (cc % RK)] & 0xFFFF;
          __hip_atomic_store(a.scores + ta.out,
                             v - (int)base + a.sc.gap2 * (int)(ta.len[0] + ta.len[1] + ta.len[2]),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        if (pj == pjb && pk == pkb) {
          const int r = (int)tb.len[1] - pjb * H, cc = (int)tb.len[2] - pkb * W;
          const int v = (int)((uint32_t)capb[(r % RJ) * RK + (cc % RK)] >> 16);
          __hip_atomic_store(a.scores + tb.out,
                             v - (int)base + a.sc.gap2 * (int)(tb.len[0] + tb.len[1] + tb.len[2]),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    }
  }
  if (KIND != kGlobal) {
    // The wave's best per half; lane 0 stores both scores.
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) best = umax2(best, (uint32_t)__shfl_xor((int)best, o));
    if ((threadIdx.x & 63) == 0) {
      const int off = KIND == kSemiGlobal ? (int)kc : 0;
      __hip_atomic_store(a.scores + ta.out, (int)(best & 0xFFFFu) - off, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(a.scores + tb.out, (int)(best >> 16) - off, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

}  // namespace
}  // namespace trioseq
