// Node-level projector contraction of the nonlocal Hamiltonian (DFT-FE 1.0,
// Eq. nonlocalHamDiscrete and Algorithm 4, the steps that form the
// projections P_a = h_a sum_j conj(c~_{a,j}) X_j), and the elementwise
// helpers of the filter (zero fill, precision conversion of a block).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

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

// The same for blocks of up to 16 columns: a wave's lanes are 64 / W entries of
// the chunk by W >= ncols columns, and the entries' sums are added over the
// lanes in a fixed order.
template <typename T, bool CPLX>
__global__ void __launch_bounds__(256)
nl_partial_narrow_kernel(const int32_t* __restrict__ chunk_atom, const int64_t* __restrict__ chunk_begin,
                         const int64_t* __restrict__ atom_ptr, const int32_t* __restrict__ atom_node,
                         const double* __restrict__ atom_val, const T* __restrict__ X, int64_t ldx, int ncols,
                         T* __restrict__ partial, int64_t ldhp) {
  constexpr int NV = CPLX ? 8 : 4;
  __shared__ T red[4][NV][16];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, chunk = blockIdx.x;
  int W = 1;
  while (W < ncols) W *= 2;
  const int col = lane % W, colc = col < ncols ? col : ncols - 1;
  const int64_t e0 = chunk_begin[chunk], end = atom_ptr[chunk_atom[chunk] + 1];
  const int64_t e1 = e0 + kNlChunk < end ? e0 + kNlChunk : end;
  T acc[NV];
#pragma unroll
  for (int m = 0; m < NV; ++m) acc[m] = T(0);
#pragma unroll 4
  for (int64_t e = e0 + wave * (64 / W) + lane / W; e < e1; e += 4 * (64 / W)) {
    const int64_t j = atom_node[e] * ldx + colc;
    const double* v = atom_val + e * NV;
    if constexpr (CPLX) {
      const T xr = X[2 * j], xi = X[2 * j + 1];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const T cr = static_cast<T>(v[2 * m]), ci = static_cast<T>(v[2 * m + 1]);
        acc[2 * m] += cr * xr + ci * xi;       // conj(c) x
        acc[2 * m + 1] += cr * xi - ci * xr;
      }
    } else {
      const T x = X[j];
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[m] += static_cast<T>(v[m]) * x;
    }
  }
  for (int d = W; d < 64; d *= 2)
#pragma unroll
    for (int m = 0; m < NV; ++m) acc[m] += __shfl_xor(acc[m], d, 64);
  if (lane < W)
#pragma unroll
    for (int m = 0; m < NV; ++m) red[wave][m][lane] = acc[m];
  __syncthreads();
  if (static_cast<int>(threadIdx.x) < ncols) {
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const T s = ((red[0][m][col] + red[1][m][col]) + red[2][m][col]) + red[3][m][col];
      if constexpr (CPLX) partial[(static_cast<int64_t>(chunk) * 4 + m / 2) * ldhp + 2 * col + (m & 1)] = s;
      else partial[(static_cast<int64_t>(chunk) * 4 + m) * ldhp + col] = s;
    }
  }
}

// hP[atom][m] = h times the sum of the atom's chunks, 64 columns per workgroup:
// 8 waves take every 8th chunk, their sums are added in a fixed order.  (One
// thread per column over all chunks is a chain of dependent loads: 23 us
// for one column of 16 atoms on 12^3 cells, p = 5, 60 us for 128 columns of 64
// atoms on 24^3 cells, p = 6; this takes 4 and 7 us.)
template <typename T>
__device__ __forceinline__ void nl_reduce_item(const int am, const int jblk, gptr<const int32_t> atom_chunk_ptr,
                                               gptr<const double> hcoef, gptr<const T> partial, gptr<T> hP,
                                               int64_t ldhp, int nreal) {
  __shared__ T red[8][64];
  const int at = am / 4, m = am % 4;   // am = atom * 4 + component
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int64_t j = jblk * 64 + lane;  // ldhp is a multiple of 64
  T s = T(0);
  if (j < nreal) {
    const int c1 = atom_chunk_ptr[at + 1];
#pragma unroll 4
    for (int ch = atom_chunk_ptr[at] + wave; ch < c1; ch += 8) s += partial[(static_cast<int64_t>(ch) * 4 + m) * ldhp + j];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[w][lane];
  hP[static_cast<int64_t>(am) * ldhp + j] = s * static_cast<T>(hcoef[am]);
}

template <typename T>
__global__ void __launch_bounds__(512)
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
__global__ void __launch_bounds__(512)
nl_reduce_batched_kernel(const NlLaunch* __restrict__ d, const int64_t* __restrict__ am_off, const int nprob) {
  const int q = problem_of(am_off, nprob, blockIdx.x);
  const NlLaunch& L = d[q];
  if (static_cast<int64_t>(blockIdx.y) * 64 >= L.ldhp) return;   // the grid is the widest problem's
  nl_reduce_item<T>(static_cast<int>(blockIdx.x - am_off[q]), blockIdx.y, to_global(L.atom_chunk_ptr),
                    to_global(L.hcoef), to_global(static_cast<const T*>(L.partial)),
                    to_global(static_cast<T*>(L.hP)), L.ldhp, CPLX ? 2 * L.ncols : L.ncols);
}

template <typename T, bool CPLX>
hipError_t nl_launch(const NlLaunch& L, hipStream_t s) {
  if (L.nchunks <= 0) return hipSuccess;
  const int nct = (L.ncols + 63) / 64;
  // up to 16 columns the lanes of a wave take several entries at a time (one
  // column, 16 atoms, 12^3 cells, p = 5: 26 -> 7 us)
  if (L.ncols <= 16)
    hipLaunchKernelGGL((nl_partial_narrow_kernel<T, CPLX>), dim3(L.nchunks), dim3(256), 0, s, L.chunk_atom,
                       L.chunk_begin, L.atom_ptr, L.atom_node, L.atom_val, static_cast<const T*>(L.X), L.ldx, L.ncols,
                       static_cast<T*>(L.partial), L.ldhp);
  else
    hipLaunchKernelGGL((nl_partial_kernel<T, CPLX>), dim3(L.nchunks, nct), dim3(256), 0, s,
                       L.chunk_atom, L.chunk_begin, L.atom_ptr, L.atom_node, L.atom_val,
                       static_cast<const T*>(L.X), L.ldx, L.ncols, static_cast<T*>(L.partial), L.ldhp);
  const int nreal = CPLX ? 2 * L.ncols : L.ncols;
  hipLaunchKernelGGL((nl_reduce_kernel<T>), dim3(L.natoms * 4, L.ldhp / 64), dim3(512), 0, s,
                     L.atom_chunk_ptr, L.hcoef, static_cast<const T*>(L.partial), static_cast<T*>(L.hP),
                     L.ldhp, nreal);
  return hipGetLastError();
}

// ---- nonlocal update fused with the next projection -----------------------------
// Y += alpha C (h P) on the nodes that the projectors touch, and, from the
// updated values while they are in registers, the partial projections
// C^H Y of the next step (Algorithm 4 steps 1-6 around one Chebyshev step).
// The tensor-product kernel leaves the nonlocal term out: its waves have no
// registers left for it, and reading and writing the touched rows here costs
// little more than reading them for the projection alone.
// Bound by memory: the touched rows are read and written once.  On the
// 24^3-cell p = 6 operator with 64 atoms, 128 columns, FP64, most of a 3.06 GB
// block and 1.06 ms per step; rows in registers of an 8-wave workgroup with the
// projections on vector FMAs and a sum over the waves took 1.10 ms there, and
// 0.21 against 0.16 ms on 12^3 cells, p = 5, 160 columns, where the chains of
// dependent loads show.
// One wave per (cell that owns touched nodes, 32 real columns): no barriers.
// It walks over the cell's owned nodes in tiles of 16, the next tile's rows in
// flight.  Both products run on the 16x16x4 MFMA: the accumulator layout of a
// tile (16 nodes x 16 columns) is also the layout in which its values enter
// the projection as an operand (16 columns x 4 nodes per step), and the
// projectors of 4 atoms fill its other 16 rows.  Cells with more than 4 atoms
// read their rows again for the further atoms' projections.  32 columns: with
// 16 the projector values are read twice as often (3 % of a filter), with 64
// two waves per SIMD fit instead of four (3 % on the 12^3 box).  Requesting a
// tile's projector values together takes 3 % off the filter on the 12^3 box;
// complex FP64 and the batched kernel are 6-8 % slower that way.
// The atoms' terms are summed from zero and the sum is added to the row.  With
// the row as the MFMAs' accumulator it would be rounded in each of their four
// steps, at its own size: a degree-10 FP32 filter with three atoms over the box
// then was off by 4.6e-7 (p = 7; the dense kernel: 4.0e-7), now by 2.8e-7.  In the
// batched FP64 kernels, whose registers do not hold the sums, every atom's term
// is added on its own.  FP64 takes all 128 registers and up to 16 bytes per lane
// of scratch memory (real, p = 2, 6 and 7), batched up to 28 (complex, p = 7).
constexpr int kNlGroups = 2;   // groups of 16 real columns per wave
typedef double nd4 __attribute__((ext_vector_type(4)));
typedef float nf4 __attribute__((ext_vector_type(4)));
template <typename T> struct NlMma;
template <> struct NlMma<double> {
  typedef nd4 acc;
  static __device__ __forceinline__ acc run(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  // row of the accumulator's register i in lane group q
  static __device__ __forceinline__ int row(int i, int q) { return 4 * i + q; }
};
template <> struct NlMma<float> {
  typedef nf4 acc;
  static __device__ __forceinline__ acc run(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int i, int q) { return 4 * q + i; }
};
// (re, im) -> (im, -re) of interleaved columns, one real column per lane
__device__ __forceinline__ int nl_swap(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ double nl_rot(double v, int lane) {
  const double o = __hiloint2double(nl_swap(__double2hiint(v)), nl_swap(__double2loint(v)));
  return (lane & 1) ? -o : o;
}
__device__ __forceinline__ float nl_rot(float v, int lane) {
  const float o = __int_as_float(nl_swap(__float_as_int(v)));
  return (lane & 1) ? -o : o;
}

// The index tables and a batch's descriptors are read with scalar loads: they
// are the same for a whole wave, and no vector registers are left for them.
template <typename T> using cptr = const __attribute__((address_space(4))) T*;
template <typename T> __device__ __forceinline__ cptr<T> to_const(const T* p) { return (cptr<T>)p; }

template <int P, typename T, bool CPLX, bool TOGETHER, bool ACROSS>
__device__ __forceinline__ void nl_update_item(const NlUpdate& a, const int item, const int ctile,
                                               const int32_t* noff, const int part_z = 0, const int parts = 1) {
    constexpr int P3 = P * P * P, NT = (P3 + 15) / 16, CV = CPLX ? 2 : 1, NC = kNlGroups;
  typedef typename NlMma<T>::acc acc_t;
  const int lane = threadIdx.x % 64, q = lane / 16, cl = lane % 16;
  const auto pair_ptr = to_const(a.pair_ptr);
  const int cell = to_const(a.cells)[item];
  const int p0 = pair_ptr[item], np = pair_ptr[item + 1] - p0;
  const int nc = a.nc, n = nc * P;
  const int64_t base = static_cast<int64_t>(cell % nc) * P +
                       static_cast<int64_t>(n) * ((cell / nc) % nc * P + static_cast<int64_t>(n) * (cell / (nc * nc) * P));
  const int64_t ld = a.ldy * (CPLX ? 2 : 1);
  const gptr<T> Y = to_global(static_cast<T*>(a.Y)) + base * ld;
  int col[NC];
  bool ok[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    col[c] = ctile * (16 * NC) + c * 16 + cl;
    ok[c] = col[c] < a.nreal;
    if (!ok[c]) col[c] = CPLX ? a.nreal - 2 + (cl & 1) : a.nreal - 1;
  }
  struct Tile {
    int32_t off[4];   // nodes from the cell's first node
    T y[NC][4];
  };
  auto load = [&](int t, Tile& u) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u.off[i] = noff[t * 16 + NlMma<T>::row(i, q)];
#pragma unroll
      for (int c = 0; c < NC; ++c) u.y[c][i] = Y[u.off[i] * ld + col[c]];
    }
  };
  const gptr<const T> val = to_global(static_cast<const T*>(a.val)) + static_cast<int64_t>(p0) * NT * CV * 64;
  const gptr<const T> hp = to_global(static_cast<const T*>(a.hP));
  const T al = static_cast<T>(a.alpha), al_lo = static_cast<T>(a.alpha - static_cast<double>(al));
  T hb[4][NC];   // alpha h P of the first four atoms, B operands
  auto load_h = [&](int g, T (&h)[NC]) {
    const gptr<const T> r = hp + (static_cast<int64_t>(to_const(a.pair_atom)[p0 + g]) * 4 + q) * a.ldhp;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const T v = r[col[c]];
      h[c] = al * v;
      if constexpr (sizeof(T) == 4) h[c] += al_lo * v;
    }
  };
#pragma unroll
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int c = 0; c < NC; ++c) hb[g][c] = T(0);
    if (g < np) load_h(g, hb[g]);
  }
  auto load_c = [&](int g, int t, T (&cv)[CV]) {
#pragma unroll
    for (int v = 0; v < CV; ++v) cv[v] = val[((static_cast<int64_t>(g) * NT + t) * CV + v) * 64 + lane];
  };
  // d += one atom's term at the tile's rows
  auto term = [&](const T (&cv)[CV], const T h, acc_t& d) {
    d = NlMma<T>::run(cv[0], h, d);
    if constexpr (CPLX) d = NlMma<T>::run(cv[1], -nl_rot(h, lane), d);
  };
  auto add = [&](const acc_t& d, T (&y)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] += d[i];
  };
  // one atom's term on its own
  auto one = [&](const T (&cv)[CV], const T (&h)[NC], Tile& u) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      acc_t d = {0, 0, 0, 0};
      term(cv, h[c], d);
      add(d, u.y[c]);
    }
  };
  acc_t pj[NC];   // projections: 16 columns x 4 projectors of 4 atoms
  auto clear = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c) pj[c] = acc_t{0, 0, 0, 0};
  };
  // projections of atoms g0 .. g0 + 3 from the rows of tile t
  auto load_p = [&](int g0, int t, T (&b)[4][CV]) {
    const int g = g0 + cl / 4;
    const bool in = g < np;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < CV; ++v) {
        const T e = val[((static_cast<int64_t>(in ? g : 0) * NT + t) * CV + v) * 64 + cl % 4 * 16 + NlMma<T>::row(i, q)];
        b[i][v] = in ? e : T(0);
      }
  };
  auto project = [&](const T (&b)[4][CV], const Tile& u) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        pj[c] = NlMma<T>::run(u.y[c][i], b[i][0], pj[c]);
        if constexpr (CPLX) pj[c] = NlMma<T>::run(nl_rot(u.y[c][i], lane), b[i][1], pj[c]);
      }
  };
  const gptr<T> part = to_global(static_cast<T*>(a.part));
  // accumulator rows are columns of Y, its columns (lane % 16) atom and projector
  auto put = [&](int g0) {
    const int g = g0 + cl / 4;
    if (g >= np) return;
    const gptr<T> o = part + (static_cast<int64_t>(p0 + g) * 4 + cl % 4) * a.ldhp;
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = ctile * (16 * NC) + c * 16 + NlMma<T>::row(i, q);
        if (j < a.nreal) o[j] = pj[c][i];
      }
  };
  Tile ta, tb;
  // TOGETHER: the projector values of a tile are requested at once (past the
  // cell's last atom: its first one's), not one atom after the other
  auto step = [&](int t, Tile& u) {
    T cv[4][CV], b[4][CV];
    if constexpr (TOGETHER) {
#pragma unroll
      for (int g = 0; g < 4; ++g) load_c(g < np ? g : 0, t, cv[g]);
      load_p(0, t, b);
    }
    if constexpr (TOGETHER) {
      acc_t d[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) d[c] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int c = 0; c < NC; ++c) term(cv[g], hb[g][c], d[c]);
#pragma unroll
      for (int c = 0; c < NC; ++c) add(d[c], u.y[c]);
    } else if constexpr (ACROSS) {
      acc_t d[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) d[c] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (g < np) {
          load_c(g, t, cv[0]);
#pragma unroll
          for (int c = 0; c < NC; ++c) term(cv[0], hb[g][c], d[c]);
        }
#pragma unroll
      for (int c = 0; c < NC; ++c) add(d[c], u.y[c]);
    } else {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (g < np) {
          load_c(g, t, cv[0]);
          one(cv[0], hb[g], u);
        }
    }
#pragma unroll 1
    for (int g = 4; g < np; ++g) {
      T h[NC], c1[CV];
      load_h(g, h);
      load_c(g, t, c1);
      one(c1, h, u);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (t * 16 + NlMma<T>::row(i, q) < P3) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (ok[c]) Y[u.off[i] * ld + col[c]] = u.y[c][i];
      }
    if (a.part) {
      if constexpr (!TOGETHER) load_p(0, t, b);
      project(b, u);
    }
  };
  clear();
  const int t0 = NT * part_z / parts, t1 = NT * (part_z + 1) / parts;
  if (t0 == t1) return;
  load(t0, ta);
#pragma unroll 1
  for (int t = t0; t < t1; t += 2) {
    if (t + 1 < t1) load(t + 1, tb);
    step(t, ta);
    if (t + 2 < t1) load(t + 2, ta);
    if (t + 1 < t1) step(t + 1, tb);
  }
  if (!a.part) return;
  put(0);
#pragma unroll 1
  for (int g0 = 4; g0 < np; g0 += 4) {
    clear();
#pragma unroll 1
    for (int t = 0; t < NT; ++t) {
      T b[4][CV];
      load(t, ta);
      load_p(g0, t, b);
      project(b, ta);
    }
    put(g0);
  }
}

// Offsets of the owned nodes of a cell from its first (past the end: the last one).
template <int P> __device__ __forceinline__ void nl_node_offsets(int nc, int32_t* noff) {
  constexpr int P3 = P * P * P, NT = (P3 + 15) / 16;
  const int n = nc * P;
  for (int i = threadIdx.x; i < NT * 16; i += 256) {
    const int e = i < P3 ? i : P3 - 1;
    noff[i] = e % P + n * (e / P % P + n * (e / (P * P)));
  }
  __syncthreads();
}

constexpr int kNlCells = 4;    // cells (waves) per workgroup

template <int P, typename T, bool CPLX>
__global__ void __launch_bounds__(256, 4) nl_update_kernel(const NlUpdate a) {
  __shared__ int32_t noff[(P * P * P + 15) / 16 * 16];
  nl_node_offsets<P>(a.nc, noff);
  const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * kNlCells + threadIdx.x / 64);
  if (item < a.ncells) nl_update_item<P, T, CPLX, !(CPLX && sizeof(T) == 8), true>(a, item, blockIdx.y, noff, blockIdx.z, gridDim.z);
}

// The update of many problems (batched filter): descriptors in device memory.
__device__ __forceinline__ NlUpdate load_update(const NlUpdate* p) {
  struct Words { uint64_t w[sizeof(NlUpdate) / 8]; } v;
  static_assert(sizeof(Words) == sizeof(NlUpdate), "whole words");
  const cptr<uint64_t> s = to_const(reinterpret_cast<const uint64_t*>(p));
#pragma unroll
  for (unsigned i = 0; i < sizeof(NlUpdate) / 8; ++i) v.w[i] = s[i];
  return __builtin_bit_cast(NlUpdate, v);
}

template <int P, typename T, bool CPLX>
__global__ void __launch_bounds__(256, 4)
nl_update_batched_kernel(const NlUpdate* __restrict__ d, const int64_t* __restrict__ cell_off, const int nprob) {
  __shared__ int32_t noff[(P * P * P + 15) / 16 * 16];
  const int q = __builtin_amdgcn_readfirstlane(problem_of(cell_off, nprob, blockIdx.x));
  const NlUpdate a = load_update(d + q);
  if (static_cast<int>(blockIdx.y) * 16 * kNlGroups >= a.nreal) return;
  nl_node_offsets<P>(a.nc, noff);
  const int item =
      __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x - cell_off[q]) * kNlCells + threadIdx.x / 64);
  if (item < a.ncells) nl_update_item<P, T, CPLX, false, sizeof(T) == 4>(a, item, blockIdx.y, noff);
}

// hP[atom][m] = h sum over the atom's pairs of their partial projections, 64
// columns per workgroup: 8 waves take every 8th pair, their sums are added in
// a fixed order, in double (hundreds of pairs per atom).
template <typename T>
__device__ __forceinline__ void nl_pair_reduce_item(const NlUpdate& a, const int am, const int jblk) {
  __shared__ double red[8][64];
  const int at = am / 4, m = am % 4;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int64_t j = jblk * 64 + lane;   // ldhp is a multiple of 64
  double s = 0.0;
  if (j < a.nreal) {
    const gptr<const T> part = to_global(static_cast<const T*>(a.part)) + j + m * a.ldhp;
    const gptr<const int32_t> list = to_global(a.atom_pair);
    const int e1 = a.atom_pair_ptr[at + 1];
#pragma unroll 8
    for (int e = a.atom_pair_ptr[at] + wave; e < e1; e += 8) s += part[static_cast<int64_t>(list[e]) * 4 * a.ldhp];
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave != 0) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[w][lane];
  to_global(static_cast<T*>(a.hP))[static_cast<int64_t>(am) * a.ldhp + j] = static_cast<T>(s * a.hcoef[am]);
}

template <typename T>
__global__ void __launch_bounds__(512) nl_pair_reduce_kernel(const NlUpdate a) {
  nl_pair_reduce_item<T>(a, blockIdx.x, blockIdx.y);
}

template <typename T>
__global__ void __launch_bounds__(512)
nl_pair_reduce_batched_kernel(const NlUpdate* __restrict__ d, const int64_t* __restrict__ row_off, const int nprob) {
  const int q = __builtin_amdgcn_readfirstlane(problem_of(row_off, nprob, blockIdx.x));
  const NlUpdate& a = d[q];
  if (static_cast<int64_t>(blockIdx.y) * 64 >= a.ldhp) return;
  nl_pair_reduce_item<T>(a, static_cast<int>(blockIdx.x - row_off[q]), blockIdx.y);
}

// Parts of a cell's tiles, each a wave of its own, where no projections are
// summed over them: as many as make 8192 waves, of two tiles or more (one
// column, 12^3 cells, p = 5: 28 us by 1728 waves, 18 us by four times as many).
unsigned nl_update_parts(const NlUpdate& a, int p) {
  if (a.part || a.ncells <= 0) return 1;
  const int64_t waves = static_cast<int64_t>(a.ncells) * ((a.nreal + 16 * kNlGroups - 1) / (16 * kNlGroups));
  const int64_t pairs = (p * p * p + 15) / 16 / 2;
  return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(8192 / waves, pairs)));
}

template <typename T, bool CPLX>
hipError_t nl_update_launch(const NlUpdate& a, int p, hipStream_t s) {
  const dim3 g((a.ncells + kNlCells - 1) / kNlCells, (a.nreal + 16 * kNlGroups - 1) / (16 * kNlGroups),
               nl_update_parts(a, p));
  if (a.ncells > 0) {
    switch (p) {
      case 2: hipLaunchKernelGGL((nl_update_kernel<2, T, CPLX>), g, dim3(256), 0, s, a); break;
      case 3: hipLaunchKernelGGL((nl_update_kernel<3, T, CPLX>), g, dim3(256), 0, s, a); break;
      case 4: hipLaunchKernelGGL((nl_update_kernel<4, T, CPLX>), g, dim3(256), 0, s, a); break;
      case 5: hipLaunchKernelGGL((nl_update_kernel<5, T, CPLX>), g, dim3(256), 0, s, a); break;
      case 6: hipLaunchKernelGGL((nl_update_kernel<6, T, CPLX>), g, dim3(256), 0, s, a); break;
      case 7: hipLaunchKernelGGL((nl_update_kernel<7, T, CPLX>), g, dim3(256), 0, s, a); break;
      default: return hipErrorInvalidValue;
    }
  }
  if (a.part)
    hipLaunchKernelGGL((nl_pair_reduce_kernel<T>), dim3(a.natoms * 4, a.ldhp / 64), dim3(512), 0, s, a);
  return hipGetLastError();
}

__global__ void __launch_bounds__(256)
own_table_kernel(const int32_t* __restrict__ own_pair, int p, int rts, const double* __restrict__ pair_re,
                 const double* __restrict__ pair_im, int per, double* __restrict__ out64, float* __restrict__ out32) {
  const int64_t src = static_cast<int64_t>(own_pair[blockIdx.x]) * rts;
  const int vw = pair_im ? 8 : 4;
  for (int i = threadIdx.x; i < per; i += 256) {
    const int l = i / (16 * vw) * 16 + i % 16, v = i / 16 % vw, m = v % 4;
    double x = 0.0;
    if (l < p * p * p) {
      const int ax = l % p, ay = l / p % p, az = l / (p * p);
      const int lid = ax + (p + 1) * (ay + (p + 1) * az);
      const int mult = (ax ? 1 : 2) * (ay ? 1 : 2) * (az ? 1 : 2);
      x = (v < 4 ? pair_re : pair_im)[(src + lid / 16) * 64 + m * 16 + lid % 16] * mult;
    }
    const int64_t o = static_cast<int64_t>(blockIdx.x) * per + i;
    out64[o] = x;
    out32[o] = static_cast<float>(x);
  }
}

template <typename T, bool CPLX>
hipError_t nl_update_batched(const NlUpdateBatch& b, int p, hipStream_t s) {
  const NlUpdate* d = static_cast<const NlUpdate*>(b.descs);
  const dim3 g(static_cast<unsigned>(b.total_blocks), (b.max_real + 16 * kNlGroups - 1) / (16 * kNlGroups));
  if (b.total_blocks > 0) {
    switch (p) {
      case 2: hipLaunchKernelGGL((nl_update_batched_kernel<2, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      case 3: hipLaunchKernelGGL((nl_update_batched_kernel<3, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      case 4: hipLaunchKernelGGL((nl_update_batched_kernel<4, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      case 5: hipLaunchKernelGGL((nl_update_batched_kernel<5, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      case 6: hipLaunchKernelGGL((nl_update_batched_kernel<6, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      case 7: hipLaunchKernelGGL((nl_update_batched_kernel<7, T, CPLX>), g, dim3(256), 0, s, d, b.cell_off, b.nprob); break;
      default: return hipErrorInvalidValue;
    }
  }
  if (b.project && b.total_rows > 0)
    hipLaunchKernelGGL((nl_pair_reduce_batched_kernel<T>), dim3(static_cast<unsigned>(b.total_rows), b.max_ldhp / 64),
                       dim3(512), 0, s, d, b.row_off, b.nprob);
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

int nl_update_cells() { return kNlCells; }

size_t own_table_entries(int p, bool cplx) { return static_cast<size_t>((p * p * p + 15) / 16 * 16) * (cplx ? 8 : 4); }

hipError_t launch_own_table(const int32_t* own_pair, int nown, int p, int mpad, const double* pair_re,
                            const double* pair_im, double* out64, float* out32, hipStream_t s) {
  if (nown <= 0) return hipSuccess;
  hipLaunchKernelGGL(own_table_kernel, dim3(nown), dim3(256), 0, s, own_pair, p, mpad / 16, pair_re, pair_im,
                     static_cast<int>(own_table_entries(p, pair_im != nullptr)), out64, out32);
  return hipGetLastError();
}

hipError_t launch_nl_update_batched(const NlUpdateBatch& b, int p, int prec, hipStream_t s) {
  switch (prec) {
    case CHFSI_F64: return nl_update_batched<double, false>(b, p, s);
    case CHFSI_F32: return nl_update_batched<float, false>(b, p, s);
    case CHFSI_C128: return nl_update_batched<double, true>(b, p, s);
    case CHFSI_C64: return nl_update_batched<float, true>(b, p, s);
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
      hipLaunchKernelGGL((nl_reduce_batched_kernel<double, false>), gr, dim3(512), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_F32:
      hipLaunchKernelGGL((nl_partial_batched_kernel<float, false>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<float, false>), gr, dim3(512), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_C128:
      hipLaunchKernelGGL((nl_partial_batched_kernel<double, true>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<double, true>), gr, dim3(512), 0, s, d, b.row_off, b.nprob);
      break;
    case CHFSI_C64:
      hipLaunchKernelGGL((nl_partial_batched_kernel<float, true>), gp, dim3(256), 0, s, d, b.chunk_off, b.nprob);
      hipLaunchKernelGGL((nl_reduce_batched_kernel<float, true>), gr, dim3(512), 0, s, d, b.row_off, b.nprob);
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
