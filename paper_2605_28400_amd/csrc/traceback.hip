// gfx950 kernels of the traceback (Hirschberg's linear-space divide and
// conquer, applied to the 3-way recurrence of the paper, Section II, Eq. 1).
//
// A box is a sub-problem: the global alignment of S0[lo0, hi0), S1[lo1, hi1)
// and S2[lo2, hi2). The host halves a box's longest axis at mid; the sweep
// kernels (plane variant) give the last slice of the forward tensor of the
// first half, F[p][q], and of the tensor of the reversed second half,
// R[p'][q'], over the two other axes. Every optimal alignment of the box
// crosses the slice mid at some (p, q) with F[p][q] + R[P-p][Q-q] equal to
// the box's score, so the split kernels pick such a cell and the box becomes
// two. Boxes of at most kLeafCells cells are solved by k_leaf: the full
// table of the box in LDS and a walk back from its far corner.
#include "device.h"

namespace trioseq {
namespace {

__device__ __forceinline__ uint32_t leaf_residue(const uint32_t* __restrict__ words, uint64_t off,
                                                 uint32_t p) {
  return (words[off + (p >> 4)] >> ((p & 15u) << 1)) & 3u;
}

constexpr int kSplitBatch = 32;

// Split, stage 1: one workgroup per chunk of kSplitChunk cells of one box's
// plane; its best F[p][q] + R[P-p][Q-q] and the smallest linear index
// p * cols + q reaching it.
__global__ void __launch_bounds__(256) k_split_part(const int* __restrict__ planes,
                                                    const SplitDesc* __restrict__ boxes,
                                                    const uint32_t* __restrict__ chunk_box,
                                                    uint32_t nchunks, int* __restrict__ partial) {
  __shared__ int s_val[256];
  __shared__ uint32_t s_idx[256];
  const uint32_t ch = blockIdx.x;
  if (ch >= nchunks) return;
  const SplitDesc d = boxes[chunk_box[ch]];
  const int* F = planes + d.fwd;
  const int* R = planes + d.bwd;
  const uint32_t cells = d.rows * d.cols;
  const uint32_t lo = (ch - d.chunk0) * kSplitChunk;
  const uint32_t hi = min(cells, lo + kSplitChunk);
  int best = INT32_MIN;
  uint32_t bidx = 0xFFFFFFFFu;
  // kSplitBatch cells per thread per pass, their loads issued together: one
  // workgroup covers a whole chunk, so a pass at a time would wait out a full
  // memory latency per cell.
  for (uint32_t q0 = lo + threadIdx.x; q0 < hi; q0 += kSplitBatch * blockDim.x) {
    int v[kSplitBatch];
#pragma unroll
    for (int u = 0; u < kSplitBatch; ++u) {
      // Cells past the chunk load its last cell (no branch between the
      // loads) and are then discarded.
      const uint32_t q = q0 + u * blockDim.x, qc = min(q, hi - 1);
      const uint32_t p = qc / d.cols, c = qc - p * d.cols;
      const int s = F[qc] + R[(d.rows - 1 - p) * d.cols + (d.cols - 1 - c)];
      v[u] = q < hi ? s : INT32_MIN;
    }
#pragma unroll
    for (int u = 0; u < kSplitBatch; ++u) {
      if (v[u] > best) {  // q grows with u, so the first maximum of this thread is kept
        best = v[u];
        bidx = q0 + u * blockDim.x;
      }
    }
  }
  s_val[threadIdx.x] = best;
  s_idx[threadIdx.x] = bidx;
  __syncthreads();
  for (uint32_t w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      const int v2 = s_val[threadIdx.x + w];
      const uint32_t i2 = s_idx[threadIdx.x + w];
      if (v2 > s_val[threadIdx.x] || (v2 == s_val[threadIdx.x] && i2 < s_idx[threadIdx.x])) {
        s_val[threadIdx.x] = v2;
        s_idx[threadIdx.x] = i2;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * ch] = s_val[0];
    partial[2 * ch + 1] = (int)s_idx[0];
  }
}

// Split, stage 2: one wave per box folds its chunks' results (same order:
// larger value, then smaller index) into out[3b] = best, (p, q); (-1, -1) if a
// wait of the run gave up, as the planes are then not to be trusted.
__global__ void __launch_bounds__(64) k_split_final(const SplitDesc* __restrict__ boxes, uint32_t n,
                                                    const int* __restrict__ partial, const int* __restrict__ err,
                                                    int* __restrict__ out) {
  const uint32_t b = blockIdx.x;
  if (b >= n) return;
  const SplitDesc d = boxes[b];
  int best = INT32_MIN;
  uint32_t bidx = 0xFFFFFFFFu;
  for (uint32_t c = threadIdx.x; c < d.nchunk; c += 64) {
    const int v = partial[2 * (d.chunk0 + c)];
    const uint32_t i = (uint32_t)partial[2 * (d.chunk0 + c) + 1];
    if (v > best || (v == best && i < bidx)) {
      best = v;
      bidx = i;
    }
  }
  for (int m = 32; m >= 1; m >>= 1) {
    const int v2 = __shfl_xor(best, m, 64);
    const uint32_t i2 = (uint32_t)__shfl_xor((int)bidx, m, 64);
    if (v2 > best || (v2 == best && i2 < bidx)) {
      best = v2;
      bidx = i2;
    }
  }
  if (threadIdx.x == 0) {
    const bool bad = *err != 0;
    out[3 * b] = best;
    out[3 * b + 1] = bad ? -1 : (int)(bidx / d.cols);
    out[3 * b + 2] = bad ? -1 : (int)(bidx % d.cols);
  }
}

// One workgroup per leaf box: the table of Eq. 1 over the box (global
// initialisation: the box's corner is 0, moves leaving the box do not exist)
// in LDS, filled one anti-diagonal plane i + j + k = const at a time (every
// predecessor lies on one of the three previous planes), then the first wave
// walks back from the far corner, taking at every cell the first move, in a
// fixed order, whose predecessor plus column score gives the cell's value.
// Columns are written last first, one byte per sequence (0..3 a residue, 4 a
// gap). Both parts are chains of LDS latencies, not work: four waves share a
// plane, the substitution scores are in LDS (read from the kernel arguments,
// they were a memory access per lane), and the walk tests a cell's seven moves
// on seven lanes. With one wave
// a box the boxes of a 1024 x 1000 x 1048 alignment took 107 us, now 29; 1000
// alignments of 8-64 residues 240, now 71.
constexpr int kLeafThreads = 256;
__global__ void __launch_bounds__(kLeafThreads) k_leaf(LeafArgs a) {
  __shared__ int T[kLeafCells];
  __shared__ uint8_t res[kLeafCells + 4];  // the three sequences, one behind the other
  __shared__ int sub[16];
  const uint32_t leaf = blockIdx.x;
  if (leaf >= a.n) return;
  const LeafDesc d = a.leaves[leaf];
  const int A = (int)d.len[0], B = (int)d.len[1], C = (int)d.len[2];
  const int tid = threadIdx.x;
  // (Residue p of a sequence sits at index p of its part; index -1 is read for
  // cells on a face and not used.)
  uint8_t *rx = res + 1, *ry = rx + A, *rz = ry + B;
  for (int q = tid; q < A; q += kLeafThreads) rx[q] = (uint8_t)leaf_residue(a.words, d.off[0], d.lo[0] + q);
  for (int q = tid; q < B; q += kLeafThreads) ry[q] = (uint8_t)leaf_residue(a.words, d.off[1], d.lo[1] + q);
  for (int q = tid; q < C; q += kLeafThreads) rz[q] = (uint8_t)leaf_residue(a.words, d.off[2], d.lo[2] + q);
  if (tid == 0) {
#pragma unroll
    for (int q = 0; q < 16; ++q) sub[q] = a.sub[q];
    res[0] = 0;
    T[0] = 0;
  }
  __syncthreads();
  const int sB = (B + 1) * (C + 1), sC = C + 1;
  const int g2 = 2 * a.gap;
  constexpr int kNone = INT32_MIN / 2;
  const int pairs = (A + 1) * (B + 1);
  // q / (B + 1) for q < 4096 (exact: the quotient's distance to an integer is
  // far above the rounding).
  const float inv = 1.0f / (float)(B + 1);
  for (int dd = 1; dd <= A + B + C; ++dd) {
    for (int q = tid; q < pairs; q += kLeafThreads) {
      const int i = (int)(((float)q + 0.5f) * inv), j = q - i * (B + 1), k = dd - i - j;
      if (k < 0 || k > C) continue;
      const int at = i * sB + j * sC + k;
      const int x = 4 * rx[i - 1], y = ry[j - 1], z = rz[k - 1];
      const int sxy = sub[x + y], sxz = sub[x + z], syz = sub[4 * y + z];
      // Predecessors outside the box are read from the corner and dropped.
      const bool ij = i && j, ik = i && k, jk = j && k, ijk = ij && k;
      const int t7 = T[ijk ? at - sB - sC - 1 : 0], t6 = T[ij ? at - sB - sC : 0], t5 = T[ik ? at - sB - 1 : 0],
                t4 = T[jk ? at - sC - 1 : 0], t3 = T[i ? at - sB : 0], t2 = T[j ? at - sC : 0], t1 = T[k ? at - 1 : 0];
      int m = kNone;
      m = max(m, ijk ? t7 + sxy + sxz + syz : kNone);
      m = max(m, ij ? t6 + sxy + g2 : kNone);
      m = max(m, ik ? t5 + sxz + g2 : kNone);
      m = max(m, jk ? t4 + syz + g2 : kNone);
      m = max(m, i ? t3 + g2 : kNone);
      m = max(m, j ? t2 + g2 : kNone);
      m = max(m, k ? t1 + g2 : kNone);
      T[at] = m;
    }
    __syncthreads();
  }
  if (tid >= 64) return;
  if (tid == 0) a.score[leaf] = T[A * sB + B * sC + C];
  // Lane m < 7 tests move m: which sequences it consumes (bits 0, 1, 2).
  const int move = tid < 7 ? (0x4216537 >> (4 * tid)) & 7 : 0;  // ijk, ij, ik, jk, i, j, k
  const int ui = move & 1, uj = (move >> 1) & 1, uk = (move >> 2) & 1;
  const int back = ui * sB + uj * sC + uk;
  uint8_t* out = a.cols + d.out;
  int i = A, j = B, k = C, n = 0;
  while (i || j || k) {
    const int at = i * sB + j * sC + k;
    const int x = rx[i - 1], y = ry[j - 1], z = rz[k - 1];
    const bool legal = move && (!ui || i) && (!uj || j) && (!uk || k);
    const int v = T[at], p = T[legal ? at - back : 0];
    // A pair of residues scores its substitution, a residue and a gap the gap.
    const int s = (ui && uj ? sub[4 * x + y] : 0) + (ui && uk ? sub[4 * x + z] : 0) + (uj && uk ? sub[4 * y + z] : 0) +
                  (ui + uj + uk == 3 ? 0 : g2);
    const uint64_t hits = __builtin_amdgcn_ballot_w64(legal && p + s == v);
    // (The last move is taken when no earlier one fits, as the only one left.)
    const int which = hits ? __builtin_ctzll(hits) : 6;
    const int w = (0x4216537 >> (4 * which)) & 7;
    if (which == 6 && !k) break;  // an inconsistent table
    const int di = w & 1, dj = (w >> 1) & 1, dk = (w >> 2) & 1;
    if (tid < 3) out[3 * n + tid] = (uint8_t)(tid == 0 ? (di ? x : 4) : tid == 1 ? (dj ? y : 4) : (dk ? z : 4));
    ++n;
    i -= di;
    j -= dj;
    k -= dk;
  }
  if (tid == 0) a.ncols[leaf] = (uint32_t)n;
}

// Gather: one thread per output word packs 16 residues of one output
// sequence (forward or reversed) from the caller's packed sequences.
__global__ void __launch_bounds__(256) k_gather(const uint32_t* __restrict__ in,
                                                const GatherDesc* __restrict__ d, uint32_t n,
                                                uint32_t words_out, uint32_t* __restrict__ out,
                                                int* __restrict__ ctl, int* __restrict__ counter,
                                                int* __restrict__ pool, uint64_t pool_ints) {
  const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
  // With ctl given, also the per-run preparation of the sweep that follows,
  // saving its launch: nothing here reads these words.
  if (ctl && blockIdx.x == 0) next_run(ctl, counter, pool, pool_ints, 1);
  if (w >= words_out) return;
  // The output sequence holding word w (sequences start on fresh words).
  uint32_t q = 0;
  while (q + 1 < n && d[q + 1].dst_off <= w) ++q;
  const GatherDesc g = d[q];
  const uint32_t first = (uint32_t)(w - g.dst_off) * 16;
  uint32_t v = 0;
  for (uint32_t b = 0; b < 16; ++b) {
    const uint32_t p = first + b;
    if (p >= g.len) break;
    const uint32_t src = g.reverse ? g.start + g.len - 1 - p : g.start + p;
    v |= leaf_residue(in, g.src_off, src) << (2 * b);
  }
  out[w] = v;
}

// Meet, in one launch: a workgroup reduces one chunk of kSplitChunk plane cells
// of a box to its best F + R; the workgroup that finishes its box last folds
// the chunks' bests, and the halves' own bests when given, into the box's score
// (INT32_MIN if a wait of the run gave up) and clears the box's counter for
// the next run.
__global__ void __launch_bounds__(256) k_meet(const int* __restrict__ planes, const SplitDesc* __restrict__ boxes,
                                              const uint32_t* __restrict__ chunk_box, int* partial,
                                              const int* __restrict__ err, const int* __restrict__ own, int own_step,
                                              int own_base, int* counters, int32_t* out) {
  __shared__ int s_val[256];
  __shared__ int s_last;
  const uint32_t box = chunk_box ? chunk_box[blockIdx.x] : 0u;
  const SplitDesc d = boxes[box];
  const int* F = planes + d.fwd;
  const int* R = planes + d.bwd;
  const uint32_t cells = d.rows * d.cols;
  const uint32_t lo = (blockIdx.x - d.chunk0) * kSplitChunk;
  const uint32_t hi = min(cells, lo + kSplitChunk);
  int best = INT32_MIN;
  // kSplitBatch cells per thread per pass, their loads issued together.
  for (uint32_t q0 = lo + threadIdx.x; q0 < hi; q0 += kSplitBatch * blockDim.x) {
    int v[kSplitBatch];
#pragma unroll
    for (int u = 0; u < kSplitBatch; ++u) {
      const uint32_t q = q0 + u * blockDim.x, qc = min(q, hi - 1);
      const uint32_t p = qc / d.cols, c = qc - p * d.cols;
      const int sv = F[qc] + R[(d.rows - 1 - p) * d.cols + (d.cols - 1 - c)];
      v[u] = q < hi ? sv : INT32_MIN;
    }
#pragma unroll
    for (int u = 0; u < kSplitBatch; ++u) best = max(best, v[u]);
  }
  s_val[threadIdx.x] = best;
  __syncthreads();
  for (uint32_t w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) s_val[threadIdx.x] = max(s_val[threadIdx.x], s_val[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    __hip_atomic_store(&partial[blockIdx.x], s_val[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int done = __hip_atomic_fetch_add(counters + box, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    s_last = done == (int)d.nchunk - 1;
  }
  __syncthreads();
  if (!s_last) return;
  int b = (own && threadIdx.x < 2) ? own[4 * (uint64_t)box + threadIdx.x * own_step] - own_base : INT32_MIN;
  for (uint32_t c = threadIdx.x; c < d.nchunk; c += blockDim.x)
    b = max(b, __hip_atomic_load(&partial[d.chunk0 + c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  __syncthreads();
  s_val[threadIdx.x] = b;
  __syncthreads();
  for (uint32_t w = blockDim.x / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) s_val[threadIdx.x] = max(s_val[threadIdx.x], s_val[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const bool bad = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    __hip_atomic_store(out + d.out, bad ? INT32_MIN : s_val[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(counters + box, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

}  // namespace

hipError_t launch_gather(const uint32_t* in, const GatherDesc* d, uint32_t n, uint32_t words_out,
                         uint32_t* out, int* ctl, int* counter, int* pool, uint64_t pool_ints, hipStream_t s) {
  if (words_out == 0 && !ctl) return hipSuccess;
  const uint32_t blocks = words_out == 0 ? 1 : (words_out + 255) / 256;
  hipLaunchKernelGGL(k_gather, dim3(blocks), dim3(256), 0, s, in, d, n, words_out, out, ctl, counter,
                     pool, pool_ints);
  return hipGetLastError();
}

hipError_t launch_meet(const SplitDesc* boxes, const uint32_t* chunk_box, uint32_t nchunks, const int* planes,
                       int* partial, const int* err, const int* own, int own_step, int own_base, int* counters,
                       int32_t* out, hipStream_t s) {
  if (nchunks == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_meet, dim3(nchunks), dim3(256), 0, s, planes, boxes, chunk_box, partial, err, own, own_step,
                     own_base, counters, out);
  return hipGetLastError();
}

hipError_t launch_split(const int* planes, const SplitDesc* boxes, uint32_t n, const uint32_t* chunk_box,
                        uint32_t nchunks, int* partial, const int* err, int* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_split_part, dim3(nchunks), dim3(256), 0, s, planes, boxes, chunk_box, nchunks,
                     partial);
  hipLaunchKernelGGL(k_split_final, dim3(n), dim3(64), 0, s, boxes, n, partial, err, out);
  return hipGetLastError();
}

hipError_t launch_leaf(const LeafArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_leaf, dim3(a.n), dim3(kLeafThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace trioseq
