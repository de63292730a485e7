// gfx950 kernels for packed pairs: two triplets per lane, one 16-bit half
// each (batches of whole triplets, and panel jobs of split ones).
#include "packed_whole.h"

namespace trioseq {
namespace {

// ---- Packed pairs: two triplets per lane, one 16-bit half each. ----------
//
// Two triplets of a batch are swept together by one wavefront over a common
// panel grid (each axis padded to the longer of the two), every register
// holding the pair's two values of one cell, one per 16-bit half. A cell
// takes 4 additions (one of three terms) and 3 packed three-input maxima
// (v_pk_maximum3_f16), 3.5 instructions per cell update against 7 in int32.
//
// The maximum is a half-precision instruction used on integers, exactly:
// every value a lane ever holds is an integer in [1024, 31743], whose bit
// patterns are positive normal half-precision numbers (0x0400 .. 0x7BFF:
// no zero, no subnormal, no infinity, no NaN), and for those the float
// order of the bit patterns is the integer order; a maximum returns one of
// its inputs unchanged. The additions are plain 32-bit integer additions of
// both halves at once, exact as no half passes 65535 and nothing is carried
// from the low half into the high one.
// What keeps every value in range (checked on the host per batch, otherwise
// the batch takes the int32 kernels):
//  * every substitution term s - 2*gap is >= 0, so no addition lowers a
//    value and the lookups need no sign extension;
//  * predecessors outside the tensor (the virtual faces, and the slices
//    before 0 that skewed lanes compute while filling) start at kSentP =
//    1024 and grow only along their own paths, by at most maxA per residue
//    of the path (maxA = the largest term), to below base - 512;
//  * a real cell holds base + M', with base above every such value and
//    M' >= 0, so a move from outside the tensor never wins (this also
//    replaces the -128 row and column tables of the int32 kernels); the one
//    real start, M'(0,0,0) = 0, is set explicitly;
//  * base + maxA * (the longest path in the padded box, drain included)
//    stays at or below 31743.
// Persistent kernel of a packed plan: every job is a pair of whole triplets
// (a lone last triplet is paired with itself).
template <int RJ, int RK, int WPE, int KIND, bool FUSED, int XCH, bool DMA>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
k_sweep_pk(SweepArgs a, const int* pk_top, const int* pk_left, uint32_t base, uint32_t kc) {
  __shared__ PkLds<RJ, RK> L;
  __shared__ PkRing<RJ, RK> R0, R1;
  __shared__ int capb[RJ * RK];
  extern __shared__ uint32_t selw[];
  int* face = a.face + (uint64_t)blockIdx.x * a.face_stride;
  for (;;) {
    if (threadIdx.x == 0) L.wsync = atomicAdd(a.counter, 1);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    const int idx = __builtin_amdgcn_readfirstlane(L.wsync);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    if (idx >= (int)a.njobs) break;
    pk_whole_pair<RJ, RK, KIND, FUSED, XCH, DMA>(L, R0, R1, capb, selw, a, a.jobs[idx], face, pk_top, pk_left, base,
                                                 kc);
  }
}

// Plain sentinel faces of the packed kernels: kSentP in both halves.
__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

}  // namespace

// Packed kernels: lane tile and register budget; the 4 x 4 two-wave form
// holds the previous slice's terms for the whole tile, the others form them
// cell by cell.
// (rows, columns, waves per SIMD, kind, fused, lane exchange, LDS-direct
// staging); semi-global and local scoring exist in the four plain forms.
#define TRIOSEQ_PK_PLAIN(X, k)                                                                    \
  X(4, 4, 2, k, false, 0, false) X(4, 4, 3, k, true, 0, false) X(8, 4, 2, k, true, 0, false)      \
  X(4, 8, 2, k, true, 0, false)
#define TRIOSEQ_PK_SHAPES(X)                                                                      \
  TRIOSEQ_PK_PLAIN(X, 0) TRIOSEQ_PK_PLAIN(X, 1) TRIOSEQ_PK_PLAIN(X, 2)                            \
  X(4, 4, 2, 0, false, 1, false) X(4, 4, 2, 0, false, 0, true) X(4, 4, 3, 0, true, 0, true)       \
  X(8, 4, 2, 0, true, 0, true) X(4, 8, 2, 0, true, 0, true)
#define TRIOSEQ_PK_MATCH(r, c, w, k, x, d) \
  (ks.rj == r && ks.rk == c && ks.wpe == w && kind == k && ks.xch == x && ks.dma == d)

bool pk_shape_supported(const KernelShape& ks, int kind) {
#define X(r, c, w, k, f, x, d) \
  if (TRIOSEQ_PK_MATCH(r, c, w, k, x, d)) return true;
  TRIOSEQ_PK_SHAPES(X)
#undef X
  return false;
}

hipError_t launch_sweep_pk(const KernelShape& ks, int kind, const SweepArgs& a, const int* pk_top,
                           const int* pk_left, uint32_t base, uint32_t kc, int grid, hipStream_t s) {
  const size_t lds = (size_t)(a.lds_n0 + 64) * 4;
#define X(r, c, w, k, f, x, d)                                                                     \
  if (TRIOSEQ_PK_MATCH(r, c, w, k, x, d)) {                                                        \
    hipLaunchKernelGGL((k_sweep_pk<r, c, w, k, f, x, d>), dim3(grid), dim3(64), lds, s, a, pk_top, \
                       pk_left, base, kc);                                                         \
    return hipGetLastError();                                                                      \
  }
  TRIOSEQ_PK_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t sweep_pk_occupancy(const KernelShape& ks, int kind, uint32_t lds_n0, int* blocks_per_cu) {
#define X(r, c, w, k, f, x, d)                                                                     \
  if (TRIOSEQ_PK_MATCH(r, c, w, k, x, d))                                                          \
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(                                           \
        blocks_per_cu, k_sweep_pk<r, c, w, k, f, x, d>, 64, (size_t)(lds_n0 + 64) * 4);
  TRIOSEQ_PK_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}
#undef TRIOSEQ_PK_MATCH

hipError_t launch_fill_packed_sentinel(uint32_t* p, uint64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(256), dim3(256), 0, s, p, n, kSentP * 0x10001u);
  return hipGetLastError();
}


}  // namespace trioseq
