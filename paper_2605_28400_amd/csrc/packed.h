// Device pieces shared by the packed-pair kernels: whole triplets (packed.hip)
// and panel jobs (packed_panel.hip). A register holds one cell of two
// triplets, one 16-bit half each (see packed.hip for why this is exact).
#pragma once
#include "device.h"

namespace trioseq {
namespace {

typedef _Float16 h2v __attribute__((ext_vector_type(2)));
typedef unsigned short u2v __attribute__((ext_vector_type(2)));
constexpr uint32_t kSentP = 0x0400u;  // 1024 in both halves (see above)

// Sum of both halves as one 32-bit addition: no half of a live lane ever
// passes 31743, so nothing carries from the low half into the high one (lanes
// past their pair's last slice may overflow, both halves of them dead). Unlike
// v_pk_add_u16 it also takes three terms at once (v_add3_u32), and plain
// 32-bit additions of two waves on a SIMD can issue together (a chain of them
// runs at 2.5 cycles an instruction against 4.5 for the packed form). The
// kernel is bound by VALU issue: the 8192-triplet batch of lengths 100-400
// took 34.8 ms with v_pk_add_u16 and takes 31.3 ms with these.
__device__ __forceinline__ uint32_t padd(uint32_t a, uint32_t b) { return a + b; }
// Sum of each half modulo 2^16.
__device__ __forceinline__ uint32_t paddw(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u2v, a) + __builtin_bit_cast(u2v, b));
}
__device__ __forceinline__ uint32_t pmax3(uint32_t a, uint32_t b, uint32_t c) {
  const h2v x = __builtin_bit_cast(h2v, a), y = __builtin_bit_cast(h2v, b), z = __builtin_bit_cast(h2v, c);
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z));
}
__device__ __forceinline__ uint32_t pmax2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_maximum(__builtin_bit_cast(h2v, a), __builtin_bit_cast(h2v, b)));
}
// Integer forms, for differences that need not be normal half patterns.
__device__ __forceinline__ uint32_t psub(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u2v, a) - __builtin_bit_cast(u2v, b));
}
__device__ __forceinline__ uint32_t umax2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u2v, a), __builtin_bit_cast(u2v, b)));
}

// Larger of each half as signed 16-bit integers.
typedef short s2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t smax2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s2v, a), __builtin_bit_cast(s2v, b)));
}

// Residue p of sequence `axis` of a descriptor (a sub-range, possibly read
// backwards, of the packed sequence).
__device__ __forceinline__ uint32_t residue_of(const uint32_t* __restrict__ words, const TripletDesc& td, int axis,
                                               uint32_t p) {
  return residue_at(words, td.off[axis], td.start[axis] + (td.rev ? td.len[axis] - 1 - p : p));
}

// Per-slice byte selectors of a pair, for v_perm_b32: slice i of the common
// sweep picks byte code_a(i) of triplet a's table into the low half and byte
// code_b(i) of b's table into the high half (codes of S0[i-1] for 1 <= i <=
// n0 of that triplet, 0 elsewhere); covers slices -kShiftPre .. n0 + 47.
__device__ __forceinline__ void stage_selectors(uint32_t* sel, const uint32_t* __restrict__ words,
                                                const TripletDesc& ta, const TripletDesc& tb, int n0, int tid,
                                                int nthreads) {
  const int total = n0 + 64;
  for (int q = tid; q < total; q += nthreads) {
    const int i = q - kShiftPre;
    const uint32_t ca = (i >= 1 && i <= (int)ta.len[0]) ? residue_of(words, ta, 0, (uint32_t)(i - 1)) : 0u;
    const uint32_t cb = (i >= 1 && i <= (int)tb.len[0]) ? residue_of(words, tb, 0, (uint32_t)(i - 1)) : 0u;
    sel[q] = ca | 0x0C00u | ((cb + 4u) << 16) | 0x0C000000u;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
}

// Row and column tables of a lane's tile for both triplets of a pair (code 0
// outside a sequence), and C2, the term of the move along rows and columns.
// PAD (semi-global and local scoring): all-zero tables, per triplet, on row
// 0, column 0 and past the triplet's own last row and column: a move that
// consumes a residue which is not there then scores no better than the gaps
// it replaces, so those cells never beat a cell of the triplet itself (the
// padding argument of the int32 kernels, with 0 for -128, as no term may be
// negative here).
template <int RJ, int RK>
struct PkTables {
  uint32_t TBa[RJ], TBb[RJ], TCa[RK], TCb[RK], C2[RJ][RK];
};
template <bool PAD, int RJ, int RK>
__device__ __forceinline__ void pk_tables(PkTables<RJ, RK>& t, const DevScoring& sc,
                                          const uint32_t* __restrict__ words, const TripletDesc& ta,
                                          const TripletDesc& tb, int j0, int k0) {
  const int n1a = (int)ta.len[1], n1b = (int)tb.len[1], n2a = (int)ta.len[2], n2b = (int)tb.len[2];
  const uint32_t* bt = sc.byte_tab;
  uint32_t cca[RK], ccb[RK];
  bool za[RK], zb[RK];
#pragma unroll
  for (int r = 0; r < RJ; ++r) {
    const int j = j0 + r;
    const uint32_t ba = (j >= 1 && j <= n1a) ? residue_of(words, ta, 1, (uint32_t)(j - 1)) : 0u;
    const uint32_t bb = (j >= 1 && j <= n1b) ? residue_of(words, tb, 1, (uint32_t)(j - 1)) : 0u;
    t.TBa[r] = (PAD && (j == 0 || j > n1a)) ? 0u : pick4(ba, bt[0], bt[1], bt[2], bt[3]);
    t.TBb[r] = (PAD && (j == 0 || j > n1b)) ? 0u : pick4(bb, bt[0], bt[1], bt[2], bt[3]);
  }
#pragma unroll
  for (int c = 0; c < RK; ++c) {
    const int k = k0 + c;
    cca[c] = (k >= 1 && k <= n2a) ? residue_of(words, ta, 2, (uint32_t)(k - 1)) : 0u;
    ccb[c] = (k >= 1 && k <= n2b) ? residue_of(words, tb, 2, (uint32_t)(k - 1)) : 0u;
    za[c] = PAD && (k == 0 || k > n2a);
    zb[c] = PAD && (k == 0 || k > n2b);
    t.TCa[c] = za[c] ? 0u : pick4(cca[c], bt[0], bt[1], bt[2], bt[3]);
    t.TCb[c] = zb[c] ? 0u : pick4(ccb[c], bt[0], bt[1], bt[2], bt[3]);
  }
#pragma unroll
  for (int r = 0; r < RJ; ++r)
#pragma unroll
    for (int c = 0; c < RK; ++c)
      t.C2[r][c] = (za[c] ? 0u : ((t.TBa[r] >> (cca[c] << 3)) & 0xFFu)) |
                   ((zb[c] ? 0u : ((t.TBb[r] >> (ccb[c] << 3)) & 0xFFu)) << 16);
}

}  // namespace
}  // namespace trioseq
