// Node-level projector contraction of the nonlocal Hamiltonian (DFT-FE 1.0,
// Eq. nonlocalHamDiscrete and Algorithm 4, the steps that form the
// projections P_a = h_a sum_j conj(c~_{a,j}) X_j), and the elementwise
// helpers of the filter (zero fill, precision conversion of a block).
#include <hip/hip_runtime.h>

#include "device_util.h"
#include "internal.h"

namespace chfsi {
namespace {

// ---- node-level projector contraction (Algorithm 4 steps 1-4) -------------
// P_a = h_a * sum_j conj(c~_{a,j}) X[j, :], computed from atom-major node
// lists (each node row read once per atom), in two deterministic phases:
// fixed-size chunks of an atom's list give partial sums, then the chunks of
// each atom are summed in order and scaled by the couplings.
constexpr int kNlChunk = 512;

// One workgroup: one chunk of an atom's node list and 64 columns; wave w
// takes the entries w, w + 4, ...  Entries go in groups of 8 per wave: their
// node ids and projector values are wave-uniform (scalar loads), the 8 row
// loads of X are issued before any is used, so their latencies overlap.
template <typename T, bool CPLX>
__device__ __forceinline__ void nl_partial_item(const int chunk, const int ctile, gptr<const int32_t> chunk_atom,
                                                gptr<const int64_t> chunk_begin, gptr<const int64_t> atom_ptr,
                                                gptr<const int32_t> atom_node, gptr<const double> atom_val,
                                                gptr<const T> X, int64_t ldx, int ncols, gptr<T> partial,
                                                int64_t ldhp) {
  __shared__ T red[4][CPLX ? 8 : 4][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lane = threadIdx.x % 64;
  const int col = ctile * 64 + lane;  // logical column
  const int colc = col < ncols ? col : ncols - 1;
  const int at = chunk_atom[chunk];
  const int64_t e0 = chunk_begin[chunk];
  int64_t e1 = e0 + kNlChunk;
  if (e1 > atom_ptr[at + 1]) e1 = atom_ptr[at + 1];
  constexpr int NV = CPLX ? 8 : 4;
  constexpr int G = 8;
  T acc[NV];
#pragma unroll
  for (int m = 0; m < NV; ++m) acc[m] = T(0);
  auto add = [&](int64_t e, T xr, T xi) {
    const gptr<const double> v = atom_val + e * NV;
    if constexpr (CPLX) {
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const T cr = static_cast<T>(v[2 * m]), ci = static_cast<T>(v[2 * m + 1]);
        acc[2 * m] += cr * xr + ci * xi;       // conj(c) x, real part
        acc[2 * m + 1] += cr * xi - ci * xr;   // imaginary part
      }
    } else {
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] += static_cast<T>(v[m]) * xr;
    }
  };
  int64_t e = e0 + wave;
  for (; e + 4 * (G - 1) < e1; e += 4 * G) {
    T xr[G], xi[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int64_t j = atom_node[e + 4 * g];
      if constexpr (CPLX) {
        xr[g] = X[(j * ldx + colc) * 2];
        xi[g] = X[(j * ldx + colc) * 2 + 1];
      } else {
        xr[g] = X[j * ldx + colc];
        xi[g] = T(0);
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) add(e + 4 * g, xr[g], xi[g]);
  }
  for (; e < e1; e += 4) {
    const int64_t j = atom_node[e];
    if constexpr (CPLX)
      add(e, X[(j * ldx + colc) * 2], X[(j * ldx + colc) * 2 + 1]);
    else
      add(e, X[j * ldx + colc], T(0));
  }
#pragma unroll
  for (int m = 0; m < NV; ++m) red[wave][m][lane] = acc[m];
  __syncthreads();
  if (wave == 0 && col < ncols) {
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const T s = ((red[0][m][lane] + red[1][m][lane]) + red[2][m][lane]) + red[3][m][lane];
      if constexpr (CPLX) {
        partial[(static_cast<int64_t>(chunk) * 4 + m / 2) * ldhp + 2 * col + (m & 1)] = s;
      } else {
        partial[(static_cast<int64_t>(chunk) * 4 + m) * ldhp + col] = s;
      }
    }
  }
}

template <typename T, bool CPLX>
__global__ void __launch_bounds__(256)
nl_partial_kernel(const int32_t* chunk_atom, const int64_t* chunk_begin, const int64_t* atom_ptr,
                  const int32_t* atom_node, const double* atom_val, const T* X, int64_t ldx,
                  int ncols, T* partial, int64_t ldhp) {
  nl_partial_item<T, CPLX>(blockIdx.x, blockIdx.y, to_global(chunk_atom), to_global(chunk_begin),
                           to_global(atom_ptr), to_global(atom_node), to_global(atom_val), to_global(X), ldx, ncols,
                           to_global(partial), ldhp);
}

template <typename T>
__device__ __forceinline__ void nl_reduce_item(const int am, const int jblk, gptr<const int32_t> atom_chunk_ptr,
                                               gptr<const double> hcoef, gptr<const T> partial, gptr<T> hP,
                                               int64_t ldhp, int nreal) {
  const int at = am / 4, m = am % 4;   // am = atom * 4 + component
  const int j = jblk * 256 + threadIdx.x;
  if (j >= ldhp) return;
  T s = T(0);
  if (j < nreal) {
    for (int ch = atom_chunk_ptr[at]; ch < atom_chunk_ptr[at + 1]; ++ch)
      s += partial[(static_cast<int64_t>(ch) * 4 + m) * ldhp + j];
    s *= static_cast<T>(hcoef[am]);
  }
  hP[static_cast<int64_t>(am) * ldhp + j] = s;
}

template <typename T>
__global__ void __launch_bounds__(256)
nl_reduce_kernel(const int32_t* atom_chunk_ptr, const double* hcoef, const T* partial, T* hP,
                 int64_t ldhp, int nreal) {
  nl_reduce_item<T>(blockIdx.x, blockIdx.y, to_global(atom_chunk_ptr), to_global(hcoef), to_global(partial),
                    to_global(hP), ldhp, nreal);
}

// The projection of many operators' blocks in two launches: work units are
// the concatenated chunks (partial sums) and (atom, component) rows (the
// reduction) of every problem; per-problem tables and pointers come from the
// device descriptors d[q].
template <typename T, bool CPLX>
__global__ void __launch_bounds__(256)
nl_partial_batched_kernel(const NlLaunch* __restrict__ d, const int64_t* __restrict__ chunk_off, const int nprob) {
  const int q = problem_of(chunk_off, nprob, blockIdx.x);
  const NlLaunch& L = d[q];
  if (static_cast<int>(blockIdx.y) * 64 >= L.ncols) return;
  nl_partial_item<T, CPLX>(static_cast<int>(blockIdx.x - chunk_off[q]), blockIdx.y, to_global(L.chunk_atom),
                           to_global(L.chunk_begin), to_global(L.atom_ptr), to_global(L.atom_node),
                           to_global(L.atom_val), to_global(static_cast<const T*>(L.X)), L.ldx, L.ncols,
                           to_global(static_cast<T*>(L.partial)), L.ldhp);
}

template <typename T, bool CPLX>
__global__ void __launch_bounds__(256)
nl_reduce_batched_kernel(const NlLaunch* __restrict__ d, const int64_t* __restrict__ am_off, const int nprob) {
  const int q = problem_of(am_off, nprob, blockIdx.x);
  const NlLaunch& L = d[q];
  nl_reduce_item<T>(static_cast<int>(blockIdx.x - am_off[q]), blockIdx.y, to_global(L.atom_chunk_ptr),
                    to_global(L.hcoef), to_global(static_cast<const T*>(L.partial)),
                    to_global(static_cast<T*>(L.hP)), L.ldhp, CPLX ? 2 * L.ncols : L.ncols);
}

template <typename T, bool CPLX>
hipError_t nl_launch(const NlLaunch& L, hipStream_t s) {
  if (L.nchunks <= 0) return hipSuccess;
  const int nct = (L.ncols + 63) / 64;
  hipLaunchKernelGGL((nl_partial_kernel<T, CPLX>), dim3(L.nchunks, nct), dim3(256), 0, s,
                     L.chunk_atom, L.chunk_begin, L.atom_ptr, L.atom_node, L.atom_val,
                     static_cast<const T*>(L.X), L.ldx, L.ncols, static_cast<T*>(L.partial), L.ldhp);
  const int nreal = CPLX ? 2 * L.ncols : L.ncols;
  hipLaunchKernelGGL((nl_reduce_kernel<T>), dim3(L.natoms * 4, (L.ldhp + 255) / 256), dim3(256), 0, s,
                     L.atom_chunk_ptr, L.hcoef, static_cast<const T*>(L.partial), static_cast<T*>(L.hP),
                     L.ldhp, nreal);
  return hipGetLastError();
}

// ---- nonlocal update fused with the next projection -----------------------------
// Y += alpha C (h P) on the nodes that the projectors touch, and, from the
// updated values while they are in registers, the partial projections
// C^H Y of the next step (Algorithm 4 steps 1-6 around one Chebyshev step).
// The tensor-product kernel leaves the nonlocal term out: its waves have no
// registers left for it (in it, with the projector values as A operands of
// one MFMA per (cell, atom) pair, the term cost 0.6-0.9 ms of a 128-column
// FP64 step on the 24^3-cell p = 6 operator; reading and writing the touched
// rows here costs about what reading them for the projection alone did).
// One workgroup of 8 waves per (cell that owns touched nodes, 64 columns).  A
// wave holds its share of the cell's p^3 owned rows in registers (all loads
// in flight together); the projector values are uniform over a wave (scalar
// loads).  Partial projections of a (cell, atom) pair are summed over the
// waves in a fixed order and stored; nl_pair_reduce_kernel sums them per atom.
template <typename T> using cptr = const __attribute__((address_space(4))) T*;

template <int P, typename T, bool CPLX>
__device__ __forceinline__ void nl_update_item(const NlUpdate& a, const int item, const int ctile) {
  constexpr int P3 = P * P * P, NW = 8, NPW = (P3 + NW - 1) / NW, CF = CPLX ? 2 : 1;
  __shared__ T red[NW][4 * CF][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lane = threadIdx.x % 64;
  const int col = ctile * 64 + lane;   // logical column
  const bool ok = col < a.ncols;
  const int colc = ok ? col : a.ncols - 1;
  const int cell = a.cells[item];
  const int p0 = a.pair_ptr[item], p1 = a.pair_ptr[item + 1];
  const int nc = a.nc, n = nc * P;
  const int64_t base = static_cast<int64_t>(cell % nc) * P +
                       static_cast<int64_t>(n) * ((cell / nc) % nc * P + static_cast<int64_t>(n) * (cell / (nc * nc) * P));
  const gptr<T> Y = to_global(static_cast<T*>(a.Y)) + static_cast<int64_t>(colc) * CF;
  const int i0 = wave * NPW;
  // row of owned node i (past the end: the last one, not used)
  auto row = [&](int i) {
    const int e = i0 + i < P3 ? i0 + i : P3 - 1;
    return (base + e % P + static_cast<int64_t>(n) * (e / P % P + static_cast<int64_t>(n) * (e / (P * P)))) * a.ldy * CF;
  };
  T yr[NPW], yi[CPLX ? NPW : 1];
#pragma unroll
  for (int i = 0; i < NPW; ++i) {
    const int64_t r = row(i);
    yr[i] = Y[r];
    if constexpr (CPLX) yi[i] = Y[r + 1];
  }
  const cptr<T> val = (cptr<T>)static_cast<const T*>(a.val);
  if (a.update) {
    const T al = static_cast<T>(a.alpha);
    for (int pr = p0; pr < p1; ++pr) {
      const gptr<const T> h = to_global(static_cast<const T*>(a.hP)) +
                              static_cast<int64_t>(a.pair_atom[pr]) * 4 * a.ldhp + static_cast<int64_t>(colc) * CF;
      T hr[4], hi[CPLX ? 4 : 1];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        hr[m] = al * h[m * a.ldhp];
        if constexpr (CPLX) hi[m] = al * h[m * a.ldhp + 1];
      }
#pragma unroll
      for (int i = 0; i < NPW; ++i) {
        if (P3 % NW != 0 && i0 + i >= P3) continue;
        const cptr<T> v = val + (static_cast<int64_t>(pr) * P3 + i0 + i) * 4 * CF;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if constexpr (CPLX) {
            yr[i] += v[2 * m] * hr[m];
            yr[i] -= v[2 * m + 1] * hi[m];
            yi[i] += v[2 * m] * hi[m];
            yi[i] += v[2 * m + 1] * hr[m];
          } else {
            yr[i] += v[m] * hr[m];
          }
        }
      }
    }
    if (ok) {
#pragma unroll
      for (int i = 0; i < NPW; ++i) {
        if (P3 % NW != 0 && i0 + i >= P3) continue;
        const int64_t r = row(i);
        Y[r] = yr[i];
        if constexpr (CPLX) Y[r + 1] = yi[i];
      }
    }
  }
  if (!a.part) return;
  const gptr<T> part = to_global(static_cast<T*>(a.part));
  for (int pr = p0; pr < p1; ++pr) {
    T acc[4 * CF];
#pragma unroll
    for (int m = 0; m < 4 * CF; ++m) acc[m] = T(0);
#pragma unroll
    for (int i = 0; i < NPW; ++i) {
      if (P3 % NW != 0 && i0 + i >= P3) continue;
      const cptr<T> v = val + (static_cast<int64_t>(pr) * P3 + i0 + i) * 4 * CF;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        if constexpr (CPLX) {   // conj(c) y
          acc[2 * m] += v[2 * m] * yr[i];
          acc[2 * m] += v[2 * m + 1] * yi[i];
          acc[2 * m + 1] += v[2 * m] * yi[i];
          acc[2 * m + 1] -= v[2 * m + 1] * yr[i];
        } else {
          acc[m] += v[m] * yr[i];
        }
      }
    }
    __syncthreads();   // the previous pair's sums are read
#pragma unroll
    for (int m = 0; m < 4 * CF; ++m) red[wave][m][lane] = acc[m];
    __syncthreads();
    for (int m = wave; m < 4 * CF; m += NW) {
      T s = red[0][m][lane];
#pragma unroll
      for (int w = 1; w < NW; ++w) s += red[w][m][lane];
      if (ok) part[(static_cast<int64_t>(pr) * 4 + m / CF) * a.ldhp + static_cast<int64_t>(col) * CF + m % CF] = s;
    }
  }
}

template <int P, typename T, bool CPLX>
__global__ void __launch_bounds__(512) nl_update_kernel(const NlUpdate a) {
  nl_update_item<P, T, CPLX>(a, blockIdx.x, blockIdx.y);
}

// hP[atom][m] = h sum over the atom's pairs of their partial projections
template <typename T>
__device__ __forceinline__ void nl_pair_reduce_item(const NlUpdate& a, const int am, const int jblk) {
  const int at = am / 4, m = am % 4;
  const int j = jblk * 256 + threadIdx.x;
  if (j >= a.ldhp) return;
  T s = T(0);
  if (j < a.nreal) {
    const gptr<const T> part = to_global(static_cast<const T*>(a.part)) + j + m * a.ldhp;
    const int e1 = a.atom_pair_ptr[at + 1];
#pragma unroll 8
    for (int e = a.atom_pair_ptr[at]; e < e1; ++e) s += part[static_cast<int64_t>(a.atom_pair[e]) * 4 * a.ldhp];
    s *= static_cast<T>(a.hcoef[am]);
  }
  to_global(static_cast<T*>(a.hP))[static_cast<int64_t>(am) * a.ldhp + j] = s;
}

template <typename T>
__global__ void __launch_bounds__(256) nl_pair_reduce_kernel(const NlUpdate a) {
  nl_pair_reduce_item<T>(a, blockIdx.x, blockIdx.y);
}

template <typename T, bool CPLX>
hipError_t nl_update_launch(const NlUpdate& a, int p, hipStream_t s) {
  const dim3 g(a.ncells, (a.ncols + 63) / 64);
  if (a.ncells > 0) {
    switch (p) {
      case 2: hipLaunchKernelGGL((nl_update_kernel<2, T, CPLX>), g, dim3(512), 0, s, a); break;
      case 3: hipLaunchKernelGGL((nl_update_kernel<3, T, CPLX>), g, dim3(512), 0, s, a); break;
      case 4: hipLaunchKernelGGL((nl_update_kernel<4, T, CPLX>), g, dim3(512), 0, s, a); break;
      case 5: hipLaunchKernelGGL((nl_update_kernel<5, T, CPLX>), g, dim3(512), 0, s, a); break;
      case 6: hipLaunchKernelGGL((nl_update_kernel<6, T, CPLX>), g, dim3(512), 0, s, a); break;
      case 7: hipLaunchKernelGGL((nl_update_kernel<7, T, CPLX>), g, dim3(512), 0, s, a); break;
      default: return hipErrorInvalidValue;
    }
  }
  if (a.part)
    hipLaunchKernelGGL((nl_pair_reduce_kernel<T>), dim3(a.natoms * 4, (a.ldhp + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---- elementwise helpers ----------------------------------------------------
template <typename T>
__global__ void fill_kernel(T* dst, int64_t rows, int64_t cols, int64_t ld) {
  const int64_t total = rows * cols;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < total;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t r = i / cols, c = i % cols;
    dst[r * ld + c] = T(0);
  }
}

// dst[r][c] = src[r][c] for a rows x cols block.  Blocks of at most 256
// columns: each workgroup step covers 256 / cols whole rows (thread = row in
// the step, column), so no thread divides a 64-bit index; wider blocks: one
// row per step, columns strided by 256.
template <typename TD, typename TS>
__global__ void __launch_bounds__(256) convert_kernel(TD* dst, int64_t ldd, const TS* src, int64_t lds,
                                                      int64_t rows, int ncol) {
  if (ncol <= 256) {
    const int rpb = 256 / ncol;
    const int tr = threadIdx.x / ncol, c = threadIdx.x % ncol;
    if (tr >= rpb) return;
    const int64_t step = static_cast<int64_t>(gridDim.x) * rpb;
#pragma unroll 4
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * rpb + tr; r < rows; r += step)
      dst[r * ldd + c] = static_cast<TD>(src[r * lds + c]);
  } else {
    for (int64_t r = blockIdx.x; r < rows; r += gridDim.x)
      for (int c = threadIdx.x; c < ncol; c += 256) dst[r * ldd + c] = static_cast<TD>(src[r * lds + c]);
  }
}

inline bool is_double(int prec) { return prec == CHFSI_F64 || prec == CHFSI_C128; }

unsigned grid_for(int64_t total) {
  int64_t g = (total + 255) / 256;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return static_cast<unsigned>(g);
}

}  // namespace

hipError_t launch_nl_project(const NlLaunch& L, int prec, hipStream_t s) {
  switch (prec) {
    case CHFSI_F64: return nl_launch<double, false>(L, s);
    case CHFSI_F32:
    case CHFSI_BF16: return nl_launch<float, false>(L, s);
    case CHFSI_C128: return nl_launch<double, true>(L, s);
    case CHFSI_C64: return nl_launch<float, true>(L, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_nl_update(const NlUpdate& a, int p, int prec, hipStream_t s) {
  switch (prec) {
    case CHFSI_F64: return nl_update_launch<double, false>(a, p, s);
    case CHFSI_F32: return nl_update_launch<float, false>(a, p, s);
    case CHFSI_C128: return nl_update_launch<double, true>(a, p, s);
    case CHFSI_C64: return nl_update_launch<float, true>(a, p, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_nl_project_batched(const NlBatch& b, int prec, hipStream_t s) {
  if (b.nprob <= 0 || b.total_chunks <= 0) return hipSuccess;
  const dim3 gp(static_cast<unsigned>(b.total_chunks), static_cast<unsigned>(b.max_col_tiles));
  const dim3 gr(static_cast<unsigned>(b.total_rows), static_cast<unsigned>(b.max_row_blocks));
  const NlLaunch* d = static_cast<const NlLaunch*>(b.descs);
  switch (prec) {
    case CHFSI_F64:
      hipLaunchKernelGGL((nl_partial_batched_kernel<double, false>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<double, false>), gr, dim3(256), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_F32:
      hipLaunchKernelGGL((nl_partial_batched_kernel<float, false>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<float, false>), gr, dim3(256), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_C128:
      hipLaunchKernelGGL((nl_partial_batched_kernel<double, true>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<double, true>), gr, dim3(256), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_C64:
      hipLaunchKernelGGL((nl_partial_batched_kernel<float, true>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<float, true>), gr, dim3(256), 0, s, d, b.row_off, b.nprob);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fill(void* dst, int64_t rows, int64_t cols, int64_t ld, int prec, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const unsigned g = grid_for(rows * cols);
  if (is_double(prec))
    hipLaunchKernelGGL(fill_kernel<double>, dim3(g), dim3(256), 0, s, static_cast<double*>(dst), rows, cols, ld);
  else
    hipLaunchKernelGGL(fill_kernel<float>, dim3(g), dim3(256), 0, s, static_cast<float*>(dst), rows, cols, ld);
  return hipGetLastError();
}

hipError_t launch_convert(void* dst, int64_t ldd, int dprec, const void* src, int64_t lds, int sprec,
                          int64_t rows, int64_t cols, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  if (cols > 0x7fffffff) return hipErrorInvalidValue;
  const unsigned g = grid_for(rows * cols);
  const bool dd = is_double(dprec), sd = is_double(sprec);
  const int ncol = static_cast<int>(cols);
  if (dd && sd)
    hipLaunchKernelGGL((convert_kernel<double, double>), dim3(g), dim3(256), 0, s, static_cast<double*>(dst), ldd,
                       static_cast<const double*>(src), lds, rows, ncol);
  else if (dd && !sd)
    hipLaunchKernelGGL((convert_kernel<double, float>), dim3(g), dim3(256), 0, s, static_cast<double*>(dst), ldd,
                       static_cast<const float*>(src), lds, rows, ncol);
  else if (!dd && sd)
    hipLaunchKernelGGL((convert_kernel<float, double>), dim3(g), dim3(256), 0, s, static_cast<float*>(dst), ldd,
                       static_cast<const double*>(src), lds, rows, ncol);
  else
    hipLaunchKernelGGL((convert_kernel<float, float>), dim3(g), dim3(256), 0, s, static_cast<float*>(dst), ldd,
                       static_cast<const float*>(src), lds, rows, ncol);
  return hipGetLastError();
}

// ---- fixed scratch for the allocation-free H~.X ------------------------------
// The projector partials and coefficients of chfsi_apply_noalloc() live in
// this file-scope device array instead of context workspace.  Each device the
// library runs on holds its own copy (kScratchBytes) until the process ends.
// Host code must never pass the array's name to a kernel: in host code it is
// a host-side stand-in, not a device address.  scratch_address() resolves the
// address for the current device.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

hipError_t scratch_address(void** out) {
  *out = nullptr;
  return hipGetSymbolAddress(out, HIP_SYMBOL(scratch));
}

}  // namespace chfsi
