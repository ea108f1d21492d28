// Tall-skinny FP64 subspace kernels of the Rayleigh-Ritz step (DFT-FE 1.0,
// Section 4.4 and Algorithm 2): the overlap / projected-Hamiltonian Gram
// products A = X^H Y (lower triangle only, split over rows with a
// deterministic two-phase reduction, the single-GPU counterpart of the
// blocked, all-reduced N x B_v slabs), the subspace rotation X' = X Z, and
// residual column norms.  Complex data is handled through its real view
// (interleaved re, im): X^H Y and X Z become real products of twice the width
// whose entries are recombined, which costs exactly the complex flop count.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.h"

namespace chfsi {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator register i holds D[4 i + l / 16][l % 16].
__device__ __forceinline__ d4 mma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int acc_row(int lane, int i) { return 4 * i + lane / 16; }

// The same products for FP64 and FP32 data.  v_mfma_f32_16x16x4f32 takes its
// operands in the same lanes as the f64 instruction; its accumulator
// register i holds D[4 (l / 16) + i][l % 16].
template <typename T> struct Mfma;
template <> struct Mfma<double> {
  using Acc = d4;
  static __device__ __forceinline__ Acc mma(double a, double b, Acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int i) { return 4 * i + lane / 16; }
};
template <> struct Mfma<float> {
  using Acc = f4;
  static __device__ __forceinline__ Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int i) { return 4 * (lane / 16) + i; }
};

// ---- Gram: lower blocks of X^T Y ------------------------------------------
// One wave computes a 64 x 64 block (I, J), I >= J, over the rows of one
// chunk.  In a 4-row k step, lanes 16 q .. 16 q + 15 read 16 consecutive
// columns of row 4 s + q, which is both the A operand (X^T) and the B operand
// (Y) layout of the f64 MFMA, so the fragments go straight from memory into
// registers: buffer loads from the chunk's first row, the row offset in the
// lane's voffset, the 16-column groups in the instruction offset.  Loads run
// two k steps ahead of the MFMAs; no LDS, no barriers.
// Bound by the matrix cores, so no product is made for padding: the last block
// row takes only its groups of 16 columns and diagonal blocks only their lower
// 16 x 16 tiles.  The blocks then differ in work; as single-wave workgroups,
// in two rounds over the device, they level out.  On 2,985,984 x 256 FP64
// (136 of the 192 tiles that 128 x 128 workgroups multiplied):
// 5.9 -> 4.3 ms, 77 % of the cycles multiplying; on 216,000 x 160, 0.384 ->
// 0.166 ms.  (2048 waves: 0.177 ms there; 8192: 0.170 ms and a longer sum.)
constexpr int kGB = kGramBlock;  // columns of a block
constexpr int kGramStages = 3;   // register stages (loads GS - 1 steps ahead)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
template <typename T, int OFF>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, int voff);
template <int OFF>
__device__ __forceinline__ double bload64(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, voff + OFF, 0, 0));
}
template <int OFF>
__device__ __forceinline__ float bload32(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff + OFF, 0, 0));
}
template <typename T, int G>   // 16-column group G of the lane's row
__device__ __forceinline__ T bload_group(__amdgpu_buffer_rsrc_t r, int voff) {
  if constexpr (sizeof(T) == 8) return bload64<G * 128>(r, voff);
  else return bload32<G * 64>(r, voff);
}

template <typename T> struct GramArgs {
  const T* X; const T* Y;
  int64_t ldx, ldy, M;
  int n, nblk;                     // columns; blocks
  int64_t rows;                    // per chunk
  double* part;                    // [chunk][block][64][64]
  int64_t offx, offy;              // first columns' positions in their rows
};

// RA groups of 16 rows of the block, CA of its columns.
template <typename T, int GS, int RA, int CA, bool DIAG>
__device__ __forceinline__ void gram_block(const GramArgs<T>& a, const int I, const int J, const int64_t m0,
                                           const int nrows, double* __restrict__ out) {
  const int lane = threadIdx.x % 64;
  using Acc = typename Mfma<T>::Acc;
  Acc acc[RA][CA];
#pragma unroll
  for (int i = 0; i < RA; ++i)
#pragma unroll
    for (int j = 0; j < CA; ++j) acc[i][j] = Acc{0, 0, 0, 0};
  // X and Y may start offx / offy columns into their rows (a column slice):
  // the ranges then end offx / offy elements before the last row's end, so
  // the padding columns of the last chunk never reach past the allocation.
  // What columns beyond n hold (the rest of the row, the next row, or zero
  // past the range) goes to entries that are never read.
  const int64_t ex = min(nrows * a.ldx, (a.M - m0) * a.ldx - a.offx);
  const int64_t ey = min(nrows * a.ldy, (a.M - m0) * a.ldy - a.offy);
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X + m0 * a.ldx, static_cast<uint32_t>(ex * sizeof(T)));
  const __amdgpu_buffer_rsrc_t ry = rsrc(a.Y + m0 * a.ldy, static_cast<uint32_t>(ey * sizeof(T)));
  const int ldx = static_cast<int>(a.ldx), ldy = static_cast<int>(a.ldy);
  auto load = [&](T (&xv)[RA], T (&yv)[CA], int s) {
    const int row = min(4 * s + lane / 16, nrows - 1);
    const int vx = (row * ldx + I * kGB + lane % 16) * static_cast<int>(sizeof(T));
    const int vy = (row * ldy + J * kGB + lane % 16) * static_cast<int>(sizeof(T));
    xv[0] = bload_group<T, 0>(rx, vx);
    if constexpr (RA > 1) xv[1] = bload_group<T, 1>(rx, vx);
    if constexpr (RA > 2) xv[2] = bload_group<T, 2>(rx, vx);
    if constexpr (RA > 3) xv[3] = bload_group<T, 3>(rx, vx);
    yv[0] = bload_group<T, 0>(ry, vy);
    if constexpr (CA > 1) yv[1] = bload_group<T, 1>(ry, vy);
    if constexpr (CA > 2) yv[2] = bload_group<T, 2>(ry, vy);
    if constexpr (CA > 3) yv[3] = bload_group<T, 3>(ry, vy);
  };
  auto compute = [&](const T (&x)[RA], const T (&y)[CA]) {
#pragma unroll
    for (int i = 0; i < RA; ++i)
#pragma unroll
      for (int j = 0; j < CA; ++j)
        if (!DIAG || j <= i) acc[i][j] = Mfma<T>::mma(x[i], y[j], acc[i][j]);
  };
  // GS register stages with fixed roles (the loop is unrolled by GS; three:
  // four or five measured no faster): the rows of step s + GS - 1 are in
  // flight while step s multiplies.  A copy between stages would make the
  // compiler wait for the loads in flight into the source.  Loads past the
  // chunk read its last row; steps past it are left out, and the rows of the
  // last step that lie past it count as zero.
  const int KS = (nrows + 3) / 4;
  T xq[GS][RA], yq[GS][CA];
#pragma unroll
  for (int j = 0; j < GS - 1; ++j) load(xq[j], yq[j], j);
  int s = 0;
  for (; s + GS < KS; s += GS) {
#pragma unroll
    for (int j = 0; j < GS; ++j) {
      load(xq[(j + GS - 1) % GS], yq[(j + GS - 1) % GS], s + j + GS - 1);
      compute(xq[j], yq[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < GS; ++j) {
    load(xq[(j + GS - 1) % GS], yq[(j + GS - 1) % GS], s + j + GS - 1);
    const bool ok = 4 * (s + j) + lane / 16 < nrows;
#pragma unroll
    for (int i = 0; i < RA; ++i) xq[j][i] = ok ? xq[j][i] : T(0);
#pragma unroll
    for (int i = 0; i < CA; ++i) yq[j][i] = ok ? yq[j][i] : T(0);
    compute(xq[j], yq[j]);
  }
#pragma unroll
  for (int i = 0; i < RA; ++i)
#pragma unroll
    for (int j = 0; j < CA; ++j)
      if (!DIAG || j <= i) {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          out[(i * 16 + Mfma<T>::row(lane, k)) * kGB + j * 16 + lane % 16] = static_cast<double>(acc[i][j][k]);
      }
}

// lower-triangular block index -> (I, J)
__device__ __forceinline__ int tri_row(int t) {
  int I = static_cast<int>((sqrt(8.0 * t + 1.0) - 1.0) / 2.0);
  while ((I + 1) * (I + 2) / 2 <= t) ++I;
  while (I * (I + 1) / 2 > t) --I;
  return I;
}

template <typename T, int GS>
__global__ void __attribute__((amdgpu_flat_work_group_size(64, 64), amdgpu_waves_per_eu(2, 2)))
gram_kernel(const GramArgs<T> a) {
  // workgroups go round-robin over the 8 XCDs: the blocks of a chunk, which
  // read the same rows, are given to one of them
  const int nwg = gridDim.x, full = nwg / 8, rest = nwg % 8;
  const int xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const int w = xcd < rest ? xcd * (full + 1) + slot : rest * (full + 1) + (xcd - rest) * full + slot;
  const int chunk = w / a.nblk, t = w % a.nblk;
  const int I = __builtin_amdgcn_readfirstlane(tri_row(t));
  const int J = t - I * (I + 1) / 2;
  const int64_t m0 = chunk * a.rows;
  const int nrows = static_cast<int>(min(a.rows, a.M - m0));
  double* out = a.part + static_cast<int64_t>(w) * kGB * kGB;
  const int ra = min((a.n - I * kGB + 15) / 16, 4);
  if (I == J) {
    if (ra == 4) gram_block<T, GS, 4, 4, true>(a, I, J, m0, nrows, out);
    else if (ra == 3) gram_block<T, GS, 3, 3, true>(a, I, J, m0, nrows, out);
    else if (ra == 2) gram_block<T, GS, 2, 2, true>(a, I, J, m0, nrows, out);
    else gram_block<T, GS, 1, 1, true>(a, I, J, m0, nrows, out);
  } else {
    if (ra == 4) gram_block<T, GS, 4, 4, false>(a, I, J, m0, nrows, out);
    else if (ra == 3) gram_block<T, GS, 3, 4, false>(a, I, J, m0, nrows, out);
    else if (ra == 2) gram_block<T, GS, 2, 4, false>(a, I, J, m0, nrows, out);
    else gram_block<T, GS, 1, 4, false>(a, I, J, m0, nrows, out);
  }
}

// G = sums of the chunks' blocks, 64 entries per workgroup (one row of a
// block): 4 waves take every 4th chunk, their sums are added in a fixed order.
// Entries above the 16 x 16 tiles of the diagonal are left as they are.  A grid
// holds 65535 in y: the blocks beyond (from 23,105 columns on) are taken by the
// same workgroups in turn.
__global__ void __launch_bounds__(256)
gram_reduce_kernel(const double* __restrict__ part, int nchunks, int nblk, int n, double* __restrict__ G, int64_t ldg) {
  __shared__ double red[4][64];
  const int r = blockIdx.x, c = threadIdx.x % 64, wave = threadIdx.x / 64;
  for (int t = blockIdx.y; t < nblk; t += gridDim.y) {
    const int I = tri_row(t), J = t - I * (I + 1) / 2;
    const int i = I * kGB + r, j = J * kGB + c;
    double s = 0.0;
    if (i < n && j / 16 <= i / 16) {
      const double* p = part + (static_cast<int64_t>(t) * kGB + r) * kGB + c;
      const int64_t step = static_cast<int64_t>(nblk) * kGB * kGB;
#pragma unroll 8
      for (int q = wave; q < nchunks; q += 4) s += p[q * step];
    }
    red[wave][c] = s;
    __syncthreads();
    if (wave == 0 && i < n && j < n && j / 16 <= i / 16)
      G[static_cast<int64_t>(i) * ldg + j] = ((s + red[1][c]) + red[2][c]) + red[3][c];
    __syncthreads();
  }
}

// Real symmetric result from the lower entries: S[i][j] = G[max][min].
__global__ void sym_from_lower_kernel(const double* __restrict__ G, int64_t ldg, double* __restrict__ S,
                                      int n) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int i = static_cast<int>(idx / n), j = static_cast<int>(idx % n);
  const int a = i > j ? i : j, b = i > j ? j : i;
  S[idx] = G[static_cast<int64_t>(a) * ldg + b];
}

// Complex Hermitian S (n x n, column-major interleaved) from the real-view
// Gram G2 (2n x 2n) of interleaved X, Y:
// S_ij = (G[2i][2j] + G[2i+1][2j+1]) + i (G[2i][2j+1] - G[2i+1][2j]) for
// i >= j, S_ji = conj(S_ij).
__global__ void gram_combine_complex_kernel(const double* __restrict__ G, int64_t ldg,
                                            double* __restrict__ S, int n) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int i = static_cast<int>(idx / n), j = static_cast<int>(idx % n);
  const int a = i > j ? i : j, b = i > j ? j : i;
  const double g00 = G[static_cast<int64_t>(2 * a) * ldg + 2 * b];
  const double g11 = G[static_cast<int64_t>(2 * a + 1) * ldg + 2 * b + 1];
  const double g01 = G[static_cast<int64_t>(2 * a) * ldg + 2 * b + 1];
  const double g10 = G[static_cast<int64_t>(2 * a + 1) * ldg + 2 * b];
  const double re = g00 + g11;
  double im = g01 - g10;
  if (i < j) im = -im;   // conjugate for the upper triangle
  if (i == j) im = 0.0;
  // column-major: element (i, j) at i + j n
  const int64_t o = (static_cast<int64_t>(i) + static_cast<int64_t>(j) * n) * 2;
  S[o] = re;
  S[o + 1] = im;
}

// ---- rotation C = X Z by tiles -------------------------------------------------
// Workgroup tile 128 x 128, 4 waves of 64 x 64 (4 x 4 MFMA tiles: each A and
// B fragment read from LDS serves four MFMAs).  X rows are staged through
// LDS (the A operand needs 16 rows per fragment), Z through LDS as well; both
// double buffered, with the next 16-deep k chunk loaded into registers from
// global memory while the current one multiplies, so there is one barrier
// per chunk (64 MFMAs per wave) and the global latency overlaps the MFMAs.
// The two stages take 70 KB of LDS at FP64: two workgroups per CU.
// For a full Z whose columns fill the tiles (see rotate_t): the values of Z that
// a workgroup stages serve 128 rows, those that the row kernel below reads
// serve 32.
constexpr int kTM = 128;  // rows per workgroup
constexpr int kTN = 128;  // columns per workgroup
constexpr int kTK = 16;   // k per stage
constexpr int kZP = kTN + 8;  // padded LDS row of the Z stage

template <typename T>
__global__ void __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
rotate_tile_kernel(const T* __restrict__ X, int64_t ldx, const T* __restrict__ Z, int64_t ldz,
                   T* __restrict__ C, int64_t ldc, int64_t M, int K, int N2) {
  __shared__ T xs[2][kTM][kTK + 1];
  __shared__ T zs[2][kTK][kZP];
  const int64_t r0 = blockIdx.x * static_cast<int64_t>(kTM);
  const int c0 = blockIdx.y * kTN;
  const int tid = threadIdx.x, wave = tid / 64, lane = tid % 64;
  const int wr = (wave / 2) * 64, wc = (wave % 2) * 64;
  using Acc = typename Mfma<T>::Acc;
  Acc acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = Acc{0, 0, 0, 0};
  // loaders: X 128 rows x 16 k (8 per thread, 16 threads per row), Z 16 k x
  // 128 columns (8 per thread, one row per 128 threads); addresses clamped,
  // out-of-range values zeroed when stored to LDS
  const int xk = tid % kTK, xr = tid / kTK;
  const int zc = tid % kTN, zr = tid / kTN;
  T gx[8], gz[8];
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      int64_t row = r0 + xr + 16 * i;
      row = row < M ? row : M - 1;
      int k = k0 + xk;
      k = k < K ? k : K - 1;
      gx[i] = X[row * ldx + k];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      int k = k0 + zr + 2 * i;
      k = k < K ? k : K - 1;
      int c = c0 + zc;
      c = c < N2 ? c : N2 - 1;
      gz[i] = Z[static_cast<int64_t>(k) * ldz + c];
    }
  };
  auto sstore = [&](int buf, int k0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool ok = r0 + xr + 16 * i < M && k0 + xk < K;
      xs[buf][xr + 16 * i][xk] = ok ? gx[i] : T(0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool ok = k0 + zr + 2 * i < K && c0 + zc < N2;
      zs[buf][zr + 2 * i][zc] = ok ? gz[i] : T(0);
    }
  };
  if (K > 0) {
    gload(0);
    sstore(0, 0);
  }
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < K; k0 += kTK) {
    const bool more = k0 + kTK < K;
    if (more) gload(k0 + kTK);
#pragma unroll
    for (int ks = 0; ks < kTK / 4; ++ks) {
      const int kr = ks * 4 + lane / 16;
      T av[4], bv[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) av[a] = xs[buf][wr + a * 16 + lane % 16][kr];
#pragma unroll
      for (int b = 0; b < 4; ++b) bv[b] = zs[buf][kr][wc + b * 16 + lane % 16];
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = Mfma<T>::mma(av[a], bv[b], acc[a][b]);
    }
    if (more) sstore(buf ^ 1, k0 + kTK);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = r0 + wr + a * 16 + Mfma<T>::row(lane, i);
        const int col = c0 + wc + b * 16 + lane % 16;
        if (row < M && col < N2) C[row * ldc + col] = acc[a][b][i];
      }
}

// ---- rotation C = X Z by rows ------------------------------------------------
// For triangular and narrow Z.  A workgroup owns 32 rows and makes their columns in slabs of 256, from the
// last to the first: the slab's X values go through LDS in panels of 256
// columns, and 4 waves multiply them with groups of 16 columns of Z, which all
// workgroups read from their L2 straight into B operands, 32 k ahead of their
// use.  66 KB of LDS: two workgroups per CU, one loads while the other
// multiplies.
// upper: Z is upper triangular (in its 16 x 16 tiles: the real view of a
// complex triangle counts too).  A group then takes the k up to its own last
// column, the waves share the groups from the longest to the shortest in
// alternating order so that their sums agree, and C may be X: a slab is
// stored after all X columns that it or a slab to its left needs were read.
// Bound by the matrix cores (56 % of the cycles multiply) and by Z's way from
// the L2; reading X and writing C take half the time.  On 2,985,984 x 256 FP64,
// upper, the products of whole 128 x 128 tiles into a second block took 6.45 ms
// and the copy back 2.7 ms; this takes 5.45 ms.  216,000 x 160: 0.281 -> 0.182
// ms.  (4 or 8 units in flight: 5.47 and 5.90 ms; the next panel fetched during
// the multiplications by workgroups that stay for 8 row blocks: 5.6 ms; 64 rows
// by 8 waves: 5.9 ms.)
constexpr int kRM = 32;    // rows per workgroup
constexpr int kRK = 256;   // columns per slab and panel
constexpr int kRing = 2;   // units of 16 k in flight

template <typename T>
__global__ void __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2, 2)))
rotate_kernel(const T* X, int64_t ldx, const T* __restrict__ Z, int64_t ldz, T* C, int64_t ldc, int64_t M, int K,
              int N2, int upper) {
  // rows end 4 banks apart: the 16 rows of an operand are read without conflicts
  constexpr int S = kRK + 16 / static_cast<int>(sizeof(T));
  __shared__ T xs[kRM][S];
  using Acc = typename Mfma<T>::Acc;
  constexpr uint32_t kBeyond = 0xfffffff0u;   // past any range: loads 0
  const int64_t r0 = blockIdx.x * static_cast<int64_t>(kRM);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lane = threadIdx.x % 64, q = lane / 16, cl = lane % 16;
  for (int c0 = (N2 - 1) / kRK * kRK; c0 >= 0; c0 -= kRK) {
    const int G = min(kRK / 16, (N2 - c0 + 15) / 16);
    const int g[4] = {G - 1 - wave, G - 8 + wave, G - 9 - wave, G - 16 + wave};   // negative: none
    Acc acc[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[r][i] = Acc{0, 0, 0, 0};
    const int kend = upper ? min(K, c0 + kRK) : K;
    for (int kb = 0; kb < kend; kb += kRK) {
      const int nk = min(kRK, kend - kb);
      __syncthreads();
      // the panel: 8 rows per wave, 4 columns per lane 64 apart
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        T v[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int64_t row = min(r0 + wave * 8 + h * 4 + r, M - 1);
            v[r][c] = X[row * ldx + kb + min(lane + 64 * c, nk - 1)];
          }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < 4; ++c) xs[wave * 8 + h * 4 + r][lane + 64 * c] = lane + 64 * c < nk ? v[r][c] : T(0);
      }
      __syncthreads();
      const bool diag = upper && kb == c0;
      const int rows = min(K - kb, kRK);
      const __amdgpu_buffer_rsrc_t rz =
          rsrc(Z + static_cast<int64_t>(kb) * ldz, static_cast<uint32_t>((static_cast<int64_t>(rows - 1) * ldz + N2) * sizeof(T)));
      const uint32_t zstep = static_cast<uint32_t>(ldz * 4 * sizeof(T));   // 4 rows of Z
      const uint32_t zlane = static_cast<uint32_t>((q * ldz + c0 + cl) * sizeof(T));
      // units of 16 k of one group, group after group; the list of loads runs
      // kRing units ahead of the multiplications
      const int nkc = (nk + 15) / 16;
      int len[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) len[i] = g[i] < 0 ? 0 : (diag ? min(g[i] + 1, nkc) : nkc);
      int lg = 0, lk = 0;                     // group and unit of the next load
      T b[kRing][4];
      auto load = [&](T (&u)[4]) {
        const int n = lg == 0 ? len[0] : lg == 1 ? len[1] : lg == 2 ? len[2] : lg == 3 ? len[3] : 0;
        const int gi = lg == 0 ? g[0] : lg == 1 ? g[1] : lg == 2 ? g[2] : g[3];
        const uint32_t o = zlane + lk * 4 * zstep + static_cast<uint32_t>(gi * 16 * static_cast<int>(sizeof(T)));
#pragma unroll
        for (int s = 0; s < 4; ++s) u[s] = bload_group<T, 0>(rz, lk < n ? o + s * zstep : kBeyond);
        ++lk;
        if (lk % kRing == 0 && lk >= n) {
          lk = 0;
          ++lg;
          if (lg == 1 && len[1] == 0) ++lg;
          if (lg == 2 && len[2] == 0) ++lg;
          if (lg == 3 && len[3] == 0) ++lg;
        }
      };
      if (len[0] == 0) continue;
#pragma unroll
      for (int u = 0; u < kRing; ++u) load(b[u]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll 1
        for (int kc = 0; kc < len[i]; kc += kRing) {
#pragma unroll
          for (int u = 0; u < kRing; ++u) {
            if (kc + u < len[i]) {
              T a[4][2];
#pragma unroll
              for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int r = 0; r < 2; ++r) a[s][r] = xs[r * 16 + cl][(kc + u) * 16 + s * 4 + q];
#pragma unroll
              for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int r = 0; r < 2; ++r) acc[r][i] = Mfma<T>::mma(a[s][r], b[u][s], acc[r][i]);
            }
            load(b[u]);
          }
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int col = c0 + g[i] * 16 + cl;
      if (g[i] < 0 || col >= N2) continue;
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int64_t row = r0 + r * 16 + Mfma<T>::row(lane, k);
          if (row < M) C[row * ldc + col] = acc[r][i][k];
        }
    }
  }
}

// ---- residual column sums ------------------------------------------------
__global__ void __launch_bounds__(256)
resid_kernel(const double* __restrict__ HX, int64_t ldh, const double* __restrict__ X, int64_t ldx,
             const double* __restrict__ th, int64_t M, int ncols, int cplx, int64_t rows_per_chunk,
             double* __restrict__ part) {
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j >= ncols) return;
  const int64_t m0 = blockIdx.x * rows_per_chunk;
  int64_t m1 = m0 + rows_per_chunk;
  if (m1 > M) m1 = M;
  const double t = th[j];
  double s = 0.0;
  if (cplx) {
    for (int64_t r = m0; r < m1; ++r) {
      const double dr = HX[(r * ldh + j) * 2] - t * X[(r * ldx + j) * 2];
      const double di = HX[(r * ldh + j) * 2 + 1] - t * X[(r * ldx + j) * 2 + 1];
      s += dr * dr + di * di;
    }
  } else {
    for (int64_t r = m0; r < m1; ++r) {
      const double d = HX[r * ldh + j] - t * X[r * ldx + j];
      s += d * d;
    }
  }
  part[static_cast<int64_t>(blockIdx.x) * ncols + j] = s;
}

// ---- vector helpers --------------------------------------------------------
constexpr int kDotBlocks = 1024;

__global__ void __launch_bounds__(256)
dot_kernel(const double* __restrict__ x, const double* __restrict__ y, int64_t n, double* part) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += static_cast<int64_t>(gridDim.x) * 256)
    s += x[i] * y[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// sum of the kDotBlocks partial sums, by every workgroup in the same order
__device__ __forceinline__ double sum_parts(const double* __restrict__ part, double* red) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kDotBlocks / 256; ++i) s += part[threadIdx.x + 256 * i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  return red[0];
}
__device__ __forceinline__ void store_part(double s, double* red, double* part) {
  __syncthreads();
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// The vector work of a Lanczos step, kDotBlocks workgroups.  With the scalars
// read by the host a step waited for two reductions to reach it; these are
// launched back to back.
__global__ void __launch_bounds__(256)
lanczos_scale_kernel(const double* __restrict__ part1, double* bb, const double* __restrict__ f,
                     double* __restrict__ v, int64_t n) {
  __shared__ double red[256];
  const double b = sum_parts(part1, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) *bb = b;
  const double inv = b > 0.0 ? 1.0 / sqrt(b) : 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += kDotBlocks * 256) v[i] = inv * f[i];
}
__global__ void __launch_bounds__(256)
lanczos_orth_kernel(const double* __restrict__ bb, const double* __restrict__ vprev, const double* __restrict__ v,
                    double* __restrict__ f, int64_t n, double* __restrict__ part2) {
  __shared__ double red[256];
  const double beta = vprev ? sqrt(*bb) : 0.0;
  double s = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += kDotBlocks * 256) {
    double x = f[i];
    if (vprev) f[i] = x -= beta * vprev[i];
    s += v[i] * x;
  }
  store_part(s, red, part2);
}
__global__ void __launch_bounds__(256)
lanczos_close_kernel(const double* __restrict__ part2, double* alpha, const double* __restrict__ v,
                     double* __restrict__ f, int64_t n, double* __restrict__ part1) {
  __shared__ double red[256];
  const double a = sum_parts(part2, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = a;
  double s = 0.0;
  for (int64_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += kDotBlocks * 256) {
    const double x = f[i] - a * v[i];
    f[i] = x;
    s += x * x;
  }
  store_part(s, red, part1);
}

__global__ void axpby_kernel(double a, const double* __restrict__ x, double b, double* __restrict__ y,
                             int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    y[i] = a * x[i] + b * y[i];
}

__global__ void transpose_kernel(const double* __restrict__ in, double* __restrict__ out, int n) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int i = static_cast<int>(idx / n), j = static_cast<int>(idx % n);
  out[static_cast<int64_t>(j) * n + i] = in[idx];
}

// out (cols x rows, ldo) = in^T, in rows x cols (ldi), row-major
__global__ void transpose_rect_kernel(const double* __restrict__ in, int64_t ldi, int rows, int cols,
                                      double* __restrict__ out, int64_t ldo) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(rows) * cols) return;
  const int i = static_cast<int>(idx / cols), j = static_cast<int>(idx % cols);
  out[static_cast<int64_t>(j) * ldo + i] = in[static_cast<int64_t>(i) * ldi + j];
}

// Splits the upper-triangular n x n Z (row-major, ldz): Zo = FP32 copy with
// the diagonal removed, d = the diagonal in FP64.
__global__ void split_diag_kernel(const double* __restrict__ Z, int64_t ldz, int n, float* __restrict__ Zo,
                                  double* __restrict__ d) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int i = static_cast<int>(idx / n), j = static_cast<int>(idx % n);
  const double z = Z[static_cast<int64_t>(i) * ldz + j];
  Zo[idx] = i == j ? 0.0f : static_cast<float>(z);
  if (i == j) d[i] = z;
}

// X[r][j] <- C[r][j] + d[j] X[r][j]   (C in FP32, X and d in FP64)
__global__ void add_scaled_cols_kernel(const float* __restrict__ C, int64_t ldc, const double* __restrict__ d,
                                       double* __restrict__ X, int64_t ldx, int64_t M, int n) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= M * n) return;
  const int64_t r = idx / n;
  const int j = static_cast<int>(idx % n);
  double* x = X + r * ldx + j;
  *x = static_cast<double>(C[r * ldc + j]) + d[j] * *x;
}

__global__ void zero_strict_lower_kernel(double* A, int n, int64_t lda) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int i = static_cast<int>(idx / n), j = static_cast<int>(idx % n);
  if (i > j) A[static_cast<int64_t>(i) * lda + j] = 0.0;
}

// Real 2n1 x 2n2 expansion of a complex matrix Z (row-major interleaved,
// Z[k][j] at (k n2 + j)), or of the conjugate of a column-major upper
// Cholesky-inverse read as row-major, so that [re im] rows times it give the
// complex product.  mode 0: Z given row-major.  mode 1: src is column-major
// L^-1 (n1 = n2); Z = L^-H, i.e. Z[k][j] = conj(src[k n + j]) for k <= j,
// 0 below the diagonal.  mode 2: src is column-major Q (eigenvectors); Z = Q,
// Z[k][j] = src[k + j n].
__global__ void expand_complex_kernel(const double* __restrict__ src, int n1, int n2, int mode,
                                      double* __restrict__ Z2) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n1) * n2) return;
  const int k = static_cast<int>(idx / n2), j = static_cast<int>(idx % n2);
  double zr, zi;
  if (mode == 0) {
    zr = src[idx * 2];
    zi = src[idx * 2 + 1];
  } else if (mode == 1) {
    if (k > j) {
      zr = 0.0;
      zi = 0.0;
    } else {
      zr = src[idx * 2];
      zi = -src[idx * 2 + 1];
    }
  } else {
    const int64_t o = (static_cast<int64_t>(k) + static_cast<int64_t>(j) * n1) * 2;
    zr = src[o];
    zi = src[o + 1];
  }
  const int64_t ld = 2 * static_cast<int64_t>(n2);
  Z2[(2 * static_cast<int64_t>(k)) * ld + 2 * j] = zr;
  Z2[(2 * static_cast<int64_t>(k)) * ld + 2 * j + 1] = zi;
  Z2[(2 * static_cast<int64_t>(k) + 1) * ld + 2 * j] = -zi;
  Z2[(2 * static_cast<int64_t>(k) + 1) * ld + 2 * j + 1] = zr;
}

unsigned blocks_for(int64_t total, int per = 256) {
  return static_cast<unsigned>((total + per - 1) / per);
}

}  // namespace

size_t gram_partial_bytes(int64_t M, int n, int64_t ld) {
  // what the widest of all products of up to n columns takes, in either
  // precision (single precision has the more chunks)
  int64_t blocks = 0;
  for (int w = kGB; w < n + kGB; w += kGB)
    blocks = std::max(blocks, static_cast<int64_t>(gram_chunks(M, w, ld, true)) * gram_blocks(w));
  return static_cast<size_t>(blocks) * kGB * kGB * sizeof(double);
}

template <typename T>
hipError_t gram_t(const T* X, int64_t ldx, const T* Y, int64_t ldy, int64_t M, int n, double* partial,
                  double* G, int64_t ldg, hipStream_t s, int64_t offx, int64_t offy) {
  if (offx < 0 || offy < 0 || offx + n > ldx || offy + n > ldy) return hipErrorInvalidValue;
  if (n <= 0) return hipSuccess;
  int nch = gram_chunks(M, n, ldx > ldy ? ldx : ldy, sizeof(T) == 4);
  GramArgs<T> a;
  a.X = X;
  a.Y = Y;
  a.ldx = ldx;
  a.ldy = ldy;
  a.M = M;
  a.n = n;
  a.nblk = gram_blocks(n);
  a.rows = ((M + nch - 1) / nch + 15) / 16 * 16;
  a.part = partial;
  a.offx = offx;
  a.offy = offy;
  nch = static_cast<int>((M + a.rows - 1) / a.rows);   // rounding up can leave trailing chunks empty
  const int64_t nwg = static_cast<int64_t>(nch) * a.nblk;
  if (nwg > 0x7fffffff) return hipErrorInvalidValue;
  if (nwg > 0)
    hipLaunchKernelGGL((gram_kernel<T, kGramStages>), dim3(static_cast<unsigned>(nwg)), dim3(64), 0, s, a);
  hipLaunchKernelGGL(gram_reduce_kernel, dim3(kGB, std::min(a.nblk, 65535)), dim3(256), 0, s, partial, nch, a.nblk, n,
                     G, ldg);
  return hipGetLastError();
}

hipError_t launch_gram(const double* X, int64_t ldx, const double* Y, int64_t ldy, int64_t M, int n,
                       double* partial, double* G, int64_t ldg, hipStream_t s, int64_t offx, int64_t offy) {
  return gram_t(X, ldx, Y, ldy, M, n, partial, G, ldg, s, offx, offy);
}

hipError_t launch_gram(const float* X, int64_t ldx, const float* Y, int64_t ldy, int64_t M, int n,
                       double* partial, double* G, int64_t ldg, hipStream_t s, int64_t offx, int64_t offy) {
  return gram_t(X, ldx, Y, ldy, M, n, partial, G, ldg, s, offx, offy);
}

hipError_t launch_sym_from_lower(const double* G, int64_t ldg, double* S, int n, hipStream_t s) {
  hipLaunchKernelGGL(sym_from_lower_kernel, dim3(blocks_for(static_cast<int64_t>(n) * n)), dim3(256), 0, s,
                     G, ldg, S, n);
  return hipGetLastError();
}

hipError_t launch_gram_combine_complex(const double* G2, int64_t ldg2, double* S, int n, hipStream_t s) {
  hipLaunchKernelGGL(gram_combine_complex_kernel, dim3(blocks_for(static_cast<int64_t>(n) * n)), dim3(256), 0,
                     s, G2, ldg2, S, n);
  return hipGetLastError();
}

template <typename T>
hipError_t rotate_t(const T* X, int64_t ldx, const T* Z, int64_t ldz, T* C, int64_t ldc, int64_t M, int K, int N2,
                    bool upper, hipStream_t s) {
  if (M <= 0 || N2 <= 0) return hipSuccess;
  // By rows: triangular Z, and a full Z of an odd number of 64-column units up
  // to 512 columns, where the tiles' last one would be half empty or worse.
  // Full Z, 373,248 rows, FP64, tiles against rows: 128 columns 0.30 and 0.37 ms,
  // 256: 1.03 and 1.15, 512: 4.2 and 4.5, 1024: 15.6 and 16.5; 216,000 x 160 by
  // 32 columns and 4096 x 32 by 32 the rows take half the time.  Triangular: 128
  // columns 0.30 and 0.28, 256: 0.82 and 0.68, 512: 2.59 and 2.49, 1024: 8.9 and
  // 8.7 ms.  Full Z of 65, 96 and 127 columns, tiles against rows: 193 and 242,
  // 223 and 285, 313 and 368 us on 373,248 rows; 20 and 13, 23 and 16, 29 and 20 us
  // on 13,824, where 108 tiles leave half of the device idle.
  const bool rows = upper || ((N2 + 63) / 64 % 2 == 1 && N2 <= 512);
  if (!rows) {
    const int64_t gt = (M + kTM - 1) / kTM;
    if (gt > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rotate_tile_kernel<T>, dim3(static_cast<unsigned>(gt), (N2 + kTN - 1) / kTN), dim3(256), 0, s, X,
                       ldx, Z, ldz, C, ldc, M, K, N2);
    return hipGetLastError();
  }
  const int64_t gx = (M + kRM - 1) / kRM;
  if (gx > 0x7fffffff) return hipErrorInvalidValue;
  if (ldz > (int64_t{1} << 19)) return hipErrorInvalidValue;   // 32-bit offsets in 256 rows of Z
  hipLaunchKernelGGL(rotate_kernel<T>, dim3(static_cast<unsigned>(gx)), dim3(256), 0, s, X, ldx, Z, ldz, C, ldc, M, K,
                     N2, upper ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_rotate(const double* X, int64_t ldx, const double* Z, int64_t ldz, double* C, int64_t ldc,
                         int64_t M, int K, int N2, bool upper, hipStream_t s) {
  return rotate_t(X, ldx, Z, ldz, C, ldc, M, K, N2, upper, s);
}

hipError_t launch_rotate(const float* X, int64_t ldx, const float* Z, int64_t ldz, float* C, int64_t ldc,
                         int64_t M, int K, int N2, bool upper, hipStream_t s) {
  return rotate_t(X, ldx, Z, ldz, C, ldc, M, K, N2, upper, s);
}

size_t resid_partial_count(int64_t M, int ncols) {
  (void)M;
  const int ny = (ncols + 255) / 256;
  int nch = 1024 / ny;
  if (nch < 1) nch = 1;
  return static_cast<size_t>(nch) * ncols;
}

hipError_t launch_resid(const double* HX, int64_t ldh, const double* X, int64_t ldx, const double* theta,
                        int64_t M, int ncols, bool cplx, double* partial, int* nchunks_out, hipStream_t s) {
  const int ny = (ncols + 255) / 256;
  int nch = 1024 / ny;
  if (nch < 1) nch = 1;
  const int64_t rpc = (M + nch - 1) / nch;
  *nchunks_out = nch;
  hipLaunchKernelGGL(resid_kernel, dim3(nch, ny), dim3(256), 0, s, HX, ldh, X, ldx, theta, M, ncols,
                     cplx ? 1 : 0, rpc, partial);
  return hipGetLastError();
}

int dot_blocks() { return kDotBlocks; }

hipError_t launch_dot(const double* x, const double* y, int64_t n, double* partial, hipStream_t s) {
  hipLaunchKernelGGL(dot_kernel, dim3(kDotBlocks), dim3(256), 0, s, x, y, n, partial);
  return hipGetLastError();
}

hipError_t launch_lanczos_scale(const double* part1, double* bb, const double* f, double* v, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(lanczos_scale_kernel, dim3(kDotBlocks), dim3(256), 0, s, part1, bb, f, v, n);
  return hipGetLastError();
}

hipError_t launch_lanczos_orth(const double* bb, const double* vprev, const double* v, double* f, int64_t n,
                               double* part2, hipStream_t s) {
  hipLaunchKernelGGL(lanczos_orth_kernel, dim3(kDotBlocks), dim3(256), 0, s, bb, vprev, v, f, n, part2);
  return hipGetLastError();
}

hipError_t launch_lanczos_close(const double* part2, double* alpha, const double* v, double* f, int64_t n,
                                double* part1, hipStream_t s) {
  hipLaunchKernelGGL(lanczos_close_kernel, dim3(kDotBlocks), dim3(256), 0, s, part2, alpha, v, f, n, part1);
  return hipGetLastError();
}

hipError_t launch_axpby(double a, const double* x, double b, double* y, int64_t n, hipStream_t s) {
  int64_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  hipLaunchKernelGGL(axpby_kernel, dim3(static_cast<unsigned>(g)), dim3(256), 0, s, a, x, b, y, n);
  return hipGetLastError();
}

hipError_t launch_transpose_rect(const double* in, int64_t ldi, int rows, int cols, double* out, int64_t ldo,
                                 hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  hipLaunchKernelGGL(transpose_rect_kernel, dim3(blocks_for(static_cast<int64_t>(rows) * cols)), dim3(256), 0, s,
                     in, ldi, rows, cols, out, ldo);
  return hipGetLastError();
}

hipError_t launch_split_diag(const double* Z, int64_t ldz, int n, float* Zo, double* d, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(split_diag_kernel, dim3(blocks_for(static_cast<int64_t>(n) * n)), dim3(256), 0, s, Z, ldz, n,
                     Zo, d);
  return hipGetLastError();
}

hipError_t launch_add_scaled_cols(const float* C, int64_t ldc, const double* d, double* X, int64_t ldx, int64_t M,
                                  int n, hipStream_t s) {
  if (M <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(add_scaled_cols_kernel, dim3(blocks_for(M * n)), dim3(256), 0, s, C, ldc, d, X, ldx, M, n);
  return hipGetLastError();
}

hipError_t launch_transpose(const double* in, double* out, int n, hipStream_t s) {
  hipLaunchKernelGGL(transpose_kernel, dim3(blocks_for(static_cast<int64_t>(n) * n)), dim3(256), 0, s, in, out,
                     n);
  return hipGetLastError();
}

hipError_t launch_zero_strict_lower(double* A, int n, int64_t lda, hipStream_t s) {
  hipLaunchKernelGGL(zero_strict_lower_kernel, dim3(blocks_for(static_cast<int64_t>(n) * n)), dim3(256), 0, s,
                     A, n, lda);
  return hipGetLastError();
}

hipError_t launch_expand_complex(const double* Z, int n1, int n2, int mode, double* Z2, hipStream_t s) {
  hipLaunchKernelGGL(expand_complex_kernel, dim3(blocks_for(static_cast<int64_t>(n1) * n2)), dim3(256), 0, s,
                     Z, n1, n2, mode, Z2);
  return hipGetLastError();
}

}  // namespace chfsi
