// H~.X on gfx950 through the tensor-product form of the cell matrix, fused
// with one step of the scaled Chebyshev recurrence (DFT-FE 1.0, Section 4.3,
// Eq. celldgemm, Algorithm 4; Section 3.1).
//
// On the uniform mesh of cubes the Loewdin-scaled cell matrix is
//   A = kappa [ B_x (x) M (x) M + M (x) B_y (x) M + M (x) M (x) B_z ],
// M the scaled consistent 1D mass, B_d = K - i (k_d h) S (K half the scaled 1D
// stiffness, S the skew derivative), kappa = 1 / h^2; M, K and S depend on the
// order alone.  The GLL rule integrates every product of two polynomials of
// degree p exactly except that of the two leading terms, so the consistent
// mass is the lumped one less a rank-one term,
//   M = diag(1/2, 1, .., 1, 1/2) - m m^T,  m_i ~ sqrt(w_i) P_p(x_i),
// whose diagonal assembles to the identity.  Applied axis by axis, A takes 5
// products with (p+1) x (p+1) matrices per cell (B_x, three in y: M twice and
// B_y, and B_z), and M in x and in z by its rank-one form, instead of one product
// with a (p+1)^3 x (p+1)^3 matrix: about 2 (5 (p+1) + 5) operations per cell node
// and column instead of 2 (p+1)^3, 8.6 times fewer at p = 6 (complex data: B by
// two products).  That leaves memory as the bound.  The 1D products are too small
// for MFMA tiles (and FP64 runs at the same rate on the vector units).
//
// Each node is computed by one thread and written once: nothing is zeroed
// beforehand, no atomics are needed, every node's sum has a fixed order.  A
// workgroup owns TX columns of cells in z (a chunk of nz cells high), the
// TX p x p nodes per plane with local indices < p, and one 128-byte line per
// node: 16 lanes of one double or two floats.  It marches through the planes.
//   Producer waves take the 2p + 1 rows of a plane (the owned row 0 of a cell
//   also belongs to the neighbour below it) and form the x products M u and
//   B_x u at the owned x positions, reading the left neighbour's nodes too;
//   they hold two planes in flight in registers and no accumulators.
//   Consumer waves take 4 x positions and about half of the y positions, form
//   c = M_y M_x u and d = M_y B_x u + B_y M_x u from LDS, and add the plane's
//   contribution B_z c + M_z d to the p + 1 planes of its cell in registers.
//   At a plane's own step they add the potential and -beta X_{k-1}.  Complete
//   planes are stored, in place over X_{k-1} in the filter.
// The nonlocal term is added by nl_update_kernel.
// Bound by memory: on 24^3 cells, p = 6, 128 columns, FP64, a filter step moves
// 11.2 GB (9.2 GB needed) in 3.05 ms, where a three-stream add over as much
// runs at 5.5 TB/s.  The first step (no X_{k-1}): 2.56 ms; FP32 1.34 ms; 12^3
// cells, p = 5, 160 columns: 0.258 ms; 20^3 cells, p = 5, complex FP64: 1.98 ms.
// All without the nonlocal term.  A whole step with the update and its sums, and
// one by the dense cell kernel with the projections before it: 4.20 and 8.60 ms;
// 0.42 and 0.88 ms on the 12^3 cells; a complex product of its own 3.15 and
// 7.66 ms.
// LDS is double buffered with one barrier per plane; a chunk starts with the
// cell below it, whose top plane it shares.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "device_util.h"
#include "internal.h"

namespace chfsi {
namespace {

constexpr int kL = 16;        // lanes per node
constexpr int kNt = 2;        // non-temporal: results are not read again before the caches turn over
constexpr int kU = 4;         // slots (x positions, rows) per wave

// Tables in device memory: the distinct entries of K, M and S (20 each), m
// (8), then for every k the columns K[.][k] and S[.][k] (8 entries each) and
// m_k.
constexpr int kTabMass = 20, kTabS = 40, kTabM = 60, kTabCol = 68, kTabStep = 24;

// Lane values: one double, or two adjacent floats (for complex data the real
// and imaginary parts of one entry).
typedef float f2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <typename T> struct Lane;
template <> struct Lane<double> { typedef double V; };
template <> struct Lane<float> { typedef f2 V; };

template <typename T>
struct TsArgs {
  const T* Xk;
  const T* Xp;
  T* Tg;
  int64_t ldx, ldp, ldt;        // real entries
  const double* vdiag;
  const T* tab;                 // 1D factors
  int ncols, nc, nz;            // real columns, cells per side, cells per chunk in z
  int has_prev;
  // alpha kappa and beta / (alpha kappa), each in two parts; c / kappa, 1 / kappa
  T ak, ak_lo, bk, bk_lo;
  double ck, ikap;
  T sx, sy, sz;                 // k_d h (complex operators)
};

// Uniform read-only data (the arguments, the 1D factors) is read with scalar
// loads where it is used: held for the whole march it would not fit in the
// scalar registers, and the compiler would spill it to lanes of vector
// registers.  reload() keeps it from hoisting the loads behind the pointer
// out of a step.
template <typename T> using cptr = const __attribute__((address_space(4))) T*;
template <typename T> __device__ __forceinline__ cptr<T> to_const(const T* p) { return (cptr<T>)p; }
template <typename T> __device__ __forceinline__ cptr<T> reload(cptr<T> p) {
  uint64_t v = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(v));
  return reinterpret_cast<cptr<T>>(v);
}

// Position of entry (i, j) in a packed table: a matrix that is symmetric (or
// skew) and symmetric (skew) under i -> p - i is given by its entries with
// i <= j, i + j <= p.
__host__ __device__ constexpr int tab_index(int p, int i, int j) {
  if (i > j) {
    const int t = i;
    i = j;
    j = t;
  }
  if (i + j > p) {
    const int t = p - j;
    j = p - i;
    i = t;
  }
  return i * (p + 1) - i * (i - 1) + (j - i);
}

// Plane `gz` of a block whose planes hold `plane` entries.  Offsets in a plane
// stay below 2 GB; loads beyond `bytes` return 0.
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const T* p, int64_t plane, int gz,
                                                             uint32_t bytes = 0x7fffffffu) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p + gz * plane), 0, bytes, 0x00020000);
}
template <typename V> __device__ __forceinline__ V bl(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  static_assert(sizeof(V) == 8, "8 bytes per lane");
  return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
}
template <typename V> __device__ __forceinline__ void bs(V v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, kNt);
}

// (re, im) -> (im, -re) times s: the imaginary products of a complex entry,
// spread over two lanes (double; `s` carries the lane's sign) or in one.
__device__ __forceinline__ int swap_lane(int v) { return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true); }
__device__ __forceinline__ double imul(double v, double s) {
  return s * __hiloint2double(swap_lane(__double2hiint(v)), swap_lane(__double2loint(v)));
}
__device__ __forceinline__ f2 imul(f2 v, float s) { return f2{v.y, -v.x} * s; }
__device__ __forceinline__ double lane_sign(double s, int lane) { return (lane & 1) ? -s : s; }
__device__ __forceinline__ float lane_sign(float s, int) { return s; }

// a += s in the branch of plane q.  Written as distinct asm so that the
// compiler does not merge the branches into one indexed access, which would
// put the accumulators into scratch memory.
__device__ __forceinline__ void add_plane(double& a, double s, int q) {
  asm volatile("v_add_f64 %0, %0, %1 ; plane %2" : "+v"(a) : "v"(s), "i"(q));
}
__device__ __forceinline__ void add_plane(f2& a, f2 s, int q) {
  float x = a.x, y = a.y;
  asm volatile("v_add_f32 %0, %0, %1 ; plane %2" : "+v"(x) : "v"(s.x), "i"(q));
  asm volatile("v_add_f32 %0, %0, %1 ; plane %2" : "+v"(y) : "v"(s.y), "i"(q));
  a = f2{x, y};
}

// Shape of a workgroup: a tile of TX x 1 cells.  A producer slot takes one row
// of the plane, a consumer slot one x position and one half of the y
// positions; the slots of a consumer wave share the y half, so that the 1D
// coefficients are uniform over a wave.
template <int P, typename T, bool CPLX, int TX> struct TsShape {
  static constexpr int R = 2 * P + 1;               // rows per plane
  static constexpr int RW = (TX + 1) * P + 1;       // nodes per row
  static constexpr int XN = TX * P;                 // owned x positions
  static constexpr int JH = (P + 1) / 2;            // y positions of the first half (at most 4)
  static constexpr int XG = (XN + kU - 1) / kU;     // consumer waves per y half
  static constexpr int PW = (R + kU - 1) / kU;      // producer waves
  static constexpr int WAVES = PW + 2 * XG;
  static constexpr int LROW = 2 * XN * kL;          // LDS entries per row (M and B parts)
  static constexpr int LBUF = R * LROW;
  // workgroups per compute unit the registers are cut for: two where the LDS
  // holds them, one for complex operators, whose waves need the registers
  static constexpr int NWG = CPLX || 2 * LBUF * 16 > 160 * 1024 ? 1 : 2;
  static constexpr int WPE = (WAVES * NWG + 3) / 4; // waves per SIMD
  static constexpr bool BATCH = WPE <= 4;
};

struct TsTile {
  int tx, ty;       // first cell of the tile in x, cell in y
  int zc0, zcn;     // cells of the chunk in z
  int col0;
};

// Producer waves: the x products of every row of every plane.
template <int P, typename T, bool CPLX, int TX>
__device__ __forceinline__ void ts_produce(const cptr<TsArgs<T>> args, const TsTile& t, typename Lane<T>::V* lds) {
  using Sh = TsShape<P, T, CPLX, TX>;
  typedef typename Lane<T>::V V;
  constexpr int Q = P + 1, RW = Sh::RW;
  constexpr int ES = sizeof(T), CL = 8 / ES;        // columns per lane
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lane = threadIdx.x % 64;
  const int n = args->nc * P;
  const uint32_t lxb = static_cast<uint32_t>(args->ldx) * ES;   // bytes per node
  const uint32_t range = (static_cast<uint32_t>(n) * n - 1) * lxb + args->ncols * ES;
  // lanes beyond the last column read 0 or the next row's entries, not used
  const int col = t.col0 + lane % kL * CL;
  const int slot = wave * kU + lane / kL;
  const bool rowok = slot < Sh::R;
  const int row = rowok ? slot : Sh::R - 1;
  int gy = t.ty * P - P + row;
  if (gy < 0) gy += n;
  if (gy >= n) gy -= n;
  const uint32_t vrow = static_cast<uint32_t>(gy) * n * lxb + col * ES;
  V* const wr = lds + row * Sh::LROW + lane % kL;
  const int x0 = t.tx * P;
  // the left neighbour's nodes, then the tile's (wrapped past the end)
  auto load = [&](V (&u)[RW], int gz) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t r = plane_rsrc(args->Xk, static_cast<int64_t>(n) * n * args->ldx, gz, range);
    uint32_t so = (x0 == 0 ? n - P : x0 - P) * lxb;
#pragma unroll
    for (int i = 0; i < P; ++i, so += lxb) u[i] = bl<V>(r, vrow, so);
    int x = x0;
    so = x0 * lxb;
#pragma unroll
    for (int i = P; i < RW; ++i) {
      u[i] = bl<V>(r, vrow, so);
      ++x;
      so += lxb;
      if ((i - P) % P == P - 1 && x >= n) {   // past a cell's last owned node
        x = 0;
        so = 0;
      }
    }
  };
  auto xprod = [&](const V (&u)[RW], int buf) __attribute__((always_inline)) {
    const cptr<T> tab = reload(to_const(args->tab));
    V* o = wr + buf * Sh::LBUF;
    V w[CPLX ? RW : 1];
    if constexpr (CPLX) {
      const T ss = lane_sign(args->sx, lane);
#pragma unroll
      for (int i = 0; i < RW; ++i) w[i] = imul(u[i], ss);
    }
    V sl = V(0);          // m . u of the cell to the left
#pragma unroll
    for (int j = 0; j < Q; ++j) sl += tab[kTabM + j] * u[j];
#pragma unroll
    for (int c = 0; c < TX; ++c) {
      const int b = (c + 1) * P;
      V s = V(0);
#pragma unroll
      for (int j = 0; j < Q; ++j) s += tab[kTabM + j] * u[b + j];
#pragma unroll
      for (int i = 0; i < P; ++i) {
        // local index 0 also belongs to the left neighbour, mirrored
        V va = u[b + i] - tab[kTabM + i] * s;
        if (i == 0) va -= tab[kTabM + P] * sl;
        V vb = V(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          const V v = i > 0 ? u[b + j] : (j > 0 ? u[b + j] + u[b - j] : u[b] + u[b]);
          vb += tab[tab_index(P, i, j)] * v;
          if constexpr (CPLX) {
            if (i != j) {
              // S is skew, and skew under the mirror
              const V x = i > 0 ? w[b + j] : w[b + j] - w[b - j];
              const T e = tab[kTabS + tab_index(P, i, j)];
              if (i > j) vb -= e * x;
              else vb += e * x;
            }
          }
        }
        if (rowok) {
          o[(c * P + i) * kL] = va;
          o[(Sh::XN + c * P + i) * kL] = vb;
        }
      }
      sl = s;
    }
  };
  const int npl = (t.zcn + 1) * P + 1;
  int gz = (t.zc0 == 0 ? args->nc - 1 : t.zc0 - 1) * P;
  auto next = [&]() __attribute__((always_inline)) {
    const int g = gz;
    if (++gz >= n) gz = 0;
    return g;
  };
  // two planes in flight in registers; loads past the last plane read the
  // next planes of the periodic mesh and are not used
  V ua[RW], ub[RW];
  load(ua, next());
  load(ub, next());
  xprod(ua, 0);
  load(ua, next());
  __syncthreads();
  for (int q = 1; q < npl; q += 2) {
    xprod(ub, 1);
    __builtin_amdgcn_sched_barrier(0);
    load(ub, next());
    __syncthreads();
    if (q + 1 < npl) {
      xprod(ua, 0);
      __builtin_amdgcn_sched_barrier(0);
      load(ua, next());
      __syncthreads();
    }
  }
}

// Consumer waves: y products, z accumulation, the terms of the owned nodes.
template <int P, typename T, bool CPLX, int TX, int YH>
__device__ __forceinline__ void ts_consume(const cptr<TsArgs<T>> args, const TsTile& t,
                                           const typename Lane<T>::V* lds) {
  using Sh = TsShape<P, T, CPLX, TX>;
  typedef typename Lane<T>::V V;
  constexpr int Q = P + 1;
  constexpr int J0 = YH == 0 ? 0 : Sh::JH, JN = YH == 0 ? Sh::JH : P - Sh::JH;
  constexpr int ES = sizeof(T), CL = 8 / ES;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64) - Sh::PW;
  const int lane = threadIdx.x % 64;
  const int n = args->nc * P;
  const int64_t n2 = static_cast<int64_t>(n) * n;
  const int col = t.col0 + lane % kL * CL;
  const int xg = wave % Sh::XG, xw = xg * kU;  // x positions xw .. xw + 3 of the tile
  int xi = xw + lane / kL;
  if (xi >= Sh::XN) xi = Sh::XN - 1;
  const int gx = t.tx * P + xi;                // a ragged last tile has no nodes beyond n
  const bool ok = col < args->ncols && xw + lane / kL < Sh::XN && gx < n;
  const uint32_t node0 = static_cast<uint32_t>(gx < n ? gx : 0) + static_cast<uint32_t>(n) * (t.ty * P + J0);
  const uint32_t vx = node0 * static_cast<uint32_t>(args->ldx * ES) + col * ES;
  const uint32_t vp = node0 * static_cast<uint32_t>(args->ldp * ES) + col * ES;
  const uint32_t vt = node0 * static_cast<uint32_t>(args->ldt * ES) + col * ES;
  const V* const rd = lds + xi * kL + lane % kL;
  const V* const rds = lds + xi * kL + (lane % kL ^ 1);   // partner lane

  V acc[Q][JN], sz[JN];
#pragma unroll
  for (int j = 0; j < JN; ++j) {
    sz[j] = V(0);
#pragma unroll
    for (int k = 0; k < Q; ++k) acc[k][j] = V(0);
  }
  V cv[JN], dv[JN], cs[CPLX ? JN : 1];
  auto yprod = [&](const cptr<T> tab, int buf) __attribute__((always_inline)) {
    const V* r0 = rd + buf * Sh::LBUF;
    const V* r1 = rds + buf * Sh::LBUF;
    const T ss = CPLX ? lane_sign(args->sy, lane) : T(0);
#pragma unroll
    for (int j = 0; j < JN; ++j) cv[j] = dv[j] = V(0);
    // where the registers allow it, all reads of the cell's rows before their products
    V ra[Sh::BATCH ? Q : 1], rb[Sh::BATCH ? Q : 1];
    if constexpr (Sh::BATCH) {
#pragma unroll
      for (int r = 0; r < Q; ++r) {
        ra[r] = r0[(P + r) * Sh::LROW];
        rb[r] = r0[(P + r) * Sh::LROW + Sh::XN * kL];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < Q; ++r) {
      V av = Sh::BATCH ? ra[Sh::BATCH ? r : 0] : r0[(P + r) * Sh::LROW];
      V bv = Sh::BATCH ? rb[Sh::BATCH ? r : 0] : r0[(P + r) * Sh::LROW + Sh::XN * kL];
      V as = V(0);
      if constexpr (CPLX) {
        if constexpr (sizeof(T) == 8) as = ss * r1[(P + r) * Sh::LROW];
        else as = imul(av, ss);
      }
#pragma unroll
      for (int j = JN - 1; j >= 0; --j) {
        const int i = J0 + j;
        if (i == 0) {   // also the lower neighbour's row at distance r, mirrored
          const V al = r > 0 ? r0[(P - r) * Sh::LROW] : av;
          if constexpr (CPLX) {
            if (r > 0) {
              if constexpr (sizeof(T) == 8) as -= ss * r1[(P - r) * Sh::LROW];
              else as -= imul(al, ss);
            }
          }
          bv += r > 0 ? r0[(P - r) * Sh::LROW + Sh::XN * kL] : bv;
          av += al;
        }
        const T m = tab[kTabMass + tab_index(P, i, r)];
        cv[j] += m * av;
        dv[j] += m * bv;
        dv[j] += tab[tab_index(P, i, r)] * av;
        if constexpr (CPLX) {
          if (i != r) {
            const T e = tab[kTabS + tab_index(P, i, r)];
            if (i > r) dv[j] -= e * as;
            else dv[j] += e * as;
          }
        }
      }
    }
    if constexpr (CPLX) {
      const T s = lane_sign(args->sz, lane);
#pragma unroll
      for (int j = 0; j < JN; ++j) cs[j] = imul(cv[j], s);
    }
  };
  // contribution of plane k of a cell to the cell's planes
  T zk[Q], zs[CPLX ? Q : 1], zm;
  auto zload = [&](int k) __attribute__((always_inline)) {
    const cptr<T> col_ = reload(to_const(args->tab)) + kTabCol + k * kTabStep;
    zm = col_[16];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      zk[q] = col_[q];
      if constexpr (CPLX) zs[q] = col_[8 + q];
    }
  };
  auto zadd = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < JN; ++j) sz[j] += zm * dv[j];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        acc[q][j] += zk[q] * cv[j];
        if constexpr (CPLX) acc[q][j] += zs[q] * cs[j];
      }
  };
  // terms of the owned nodes of plane gz (plane k of its cell): potential and
  // previous iterate (loaded ahead), projectors
  V xo[JN], xp[JN];
  double vo[JN];
  const uint32_t nm1 = static_cast<uint32_t>(n) * n - 1;
  auto load_own = [&](int gz) __attribute__((always_inline)) {
    const cptr<TsArgs<T>> A = reload(args);
    const uint32_t lx = static_cast<uint32_t>(A->ldx * ES), lp = static_cast<uint32_t>(A->ldp * ES);
    const __amdgpu_buffer_rsrc_t rx = plane_rsrc(A->Xk, n2 * A->ldx, gz, nm1 * lx + A->ncols * ES);
    const __amdgpu_buffer_rsrc_t rv = plane_rsrc(A->vdiag, n2, gz);
    // without a previous iterate the range is empty and the loads return 0
    const __amdgpu_buffer_rsrc_t rp = plane_rsrc(A->Xp, n2 * A->ldp, gz, A->has_prev ? nm1 * lp + A->ncols * ES : 0u);
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      xo[j] = bl<V>(rx, vx, j * n * lx);
      vo[j] = bl<double>(rv, node0 * 8, j * n * 8);
      xp[j] = bl<V>(rp, vp, j * n * lp);
    }
  };
  V os[JN];
  auto own = [&]() __attribute__((always_inline)) {
    const cptr<TsArgs<T>> A = reload(args);
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const double w = vo[j] * A->ikap - A->ck;
      os[j] = static_cast<T>(w) * xo[j];
      if constexpr (sizeof(T) == 4) os[j] += static_cast<T>(w - static_cast<T>(w)) * xo[j];
      os[j] -= A->bk * xp[j];
      os[j] -= A->bk_lo * xp[j];
    }
  };
  auto own_add = [&](int k) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < P; ++q)
      if (q == k) {   // uniform
#pragma unroll
        for (int j = 0; j < JN; ++j) add_plane(acc[q][j], os[j] + dv[j], q);
      }
  };
  // stores the completed planes 0 .. P - 1 of cell zc
  auto emit = [&](int zc) __attribute__((always_inline)) {
    const cptr<TsArgs<T>> A = reload(args);
    const uint32_t lt = static_cast<uint32_t>(A->ldt * ES);
    const T ak = A->ak, ak_lo = A->ak_lo;
    if (ok) {
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const __amdgpu_buffer_rsrc_t r = plane_rsrc(A->Tg, n2 * A->ldt, zc * P + k);
#pragma unroll
        for (int j = 0; j < JN; ++j) {
          const V v = ak * acc[k][j] + ak_lo * acc[k][j];
          if constexpr (CL == 1) {
            bs(v, r, vt, j * n * lt);
          } else {
            if (col + 1 < A->ncols) bs(v, r, vt, j * n * lt);
            else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v.x), r, vt, j * n * lt, kNt);
          }
        }
      }
    }
  };

  const int npl = (t.zcn + 1) * P + 1;
  int k = 0, zc = t.zc0 - 1;      // plane q is plane k of cell zc (the first cell is the one below the chunk)
  __syncthreads();
  for (int q = 0;; ++q) {
    const bool owned = zc >= t.zc0 && q < npl - 1;
    load_own(owned ? zc * P + k : t.zc0 * P);   // unused where not owned
    __builtin_amdgcn_sched_barrier(0);
    yprod(reload(to_const(args->tab)), q & 1);
    __builtin_amdgcn_sched_barrier(0);
    own();   // before this step's stores: a wait for loads also waits for older stores
    __builtin_amdgcn_sched_barrier(0);
    if (k == 0 && q > 0) {
      // top plane of the cell below, which completes its planes
      zload(P);
      zadd();
      const cptr<T> tab = reload(to_const(args->tab));
#pragma unroll
      for (int r = 0; r < Q; ++r)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[r][j] -= tab[kTabM + r] * sz[j];
      if (zc > t.zc0) emit(zc - 1);
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        acc[0][j] = acc[P][j];
        sz[j] = V(0);
      }
#pragma unroll
      for (int r = 1; r < Q; ++r)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[r][j] = V(0);
    }
    zload(k);
    zadd();
    if (owned) own_add(k);
    if (++k == P) {
      k = 0;
      ++zc;
    }
    if (q == npl - 1) break;
    __syncthreads();
  }
}

// Workgroup w of a problem: its tile, chunk and columns, then its wave's role.
// Tiles come fastest, then chunks in z, then column tiles.
template <int P, typename T, bool CPLX, int TX>
__device__ __forceinline__ void ts_workgroup(const cptr<TsArgs<T>> args, const int w, typename Lane<T>::V* lds) {
  using Sh = TsShape<P, T, CPLX, TX>;
  constexpr int NCOL = kL * 8 / static_cast<int>(sizeof(T));
  const int nc = args->nc, nz = args->nz;
  const int ntx = (nc + TX - 1) / TX, nt = ntx * nc, nzc = (nc + nz - 1) / nz;
  const int tile = w % nt;
  const int zch = (w / nt) % nzc;
  TsTile t;
  t.tx = tile % ntx * TX;
  t.ty = tile / ntx;
  t.zc0 = zch * nz;
  t.zcn = nc - t.zc0 < nz ? nc - t.zc0 : nz;
  t.col0 = w / (nt * nzc) * NCOL;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  if (wave < Sh::PW) ts_produce<P, T, CPLX, TX>(args, t, lds);
  else if (wave < Sh::PW + Sh::XG) ts_consume<P, T, CPLX, TX, 0>(args, t, lds);
  else ts_consume<P, T, CPLX, TX, 1>(args, t, lds);
}

// Workgroups are dispatched round-robin over the 8 XCDs; remap so that each
// XCD works on neighbouring cell columns, which share rows in its L2.
__device__ __forceinline__ int xcd_order(int pid, int nblk) {
  const int q = nblk / 8, r = nblk % 8;
  const int xcd = pid % 8, slot = pid / 8;
  return (xcd < r) ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}

template <int P, typename T, bool CPLX, int TX>
__global__ void __attribute__((amdgpu_flat_work_group_size(64 * TsShape<P, T, CPLX, TX>::WAVES,
                                                           64 * TsShape<P, T, CPLX, TX>::WAVES),
                               amdgpu_waves_per_eu(TsShape<P, T, CPLX, TX>::WPE)))
tensor_hx_kernel(const TsArgs<T> kernel_args, const TsArgs<T>* descs, const int64_t* item_off, const int nprob) {
  using Sh = TsShape<P, T, CPLX, TX>;
  __shared__ typename Lane<T>::V lds[2 * Sh::LBUF];
  int pid = blockIdx.x, nblk = gridDim.x;
  cptr<TsArgs<T>> args = (cptr<TsArgs<T>>)__builtin_amdgcn_kernarg_segment_ptr();
  if (nprob > 0) {   // the arguments come first in the segment; a batch has them in a device table
    const int q = __builtin_amdgcn_readfirstlane(problem_of(item_off, nprob, pid));
    const int first = static_cast<int>(item_off[q]);
    nblk = static_cast<int>(item_off[q + 1]) - first;
    pid -= first;    // every problem over all XCDs: their workgroups differ in length
    args = to_const(descs + q);
  }
  ts_workgroup<P, T, CPLX, TX>(args, xcd_order(pid, nblk), lds);
}

// Cells per chunk in z.  A chunk repeats the planes of the cell below it, so
// long chunks save work, but the launch should end in full rounds of
// workgroups: the fewest rounds times cells marched.
int chunk_cells(int64_t columns, int nc, int slots) {
  int best = nc;
  int64_t cost = -1;
  for (int chunks = 1; chunks <= nc; ++chunks) {
    const int nz = (nc + chunks - 1) / chunks;
    const int64_t wgs = columns * ((nc + nz - 1) / nz);
    const int64_t c = (wgs + slots - 1) / slots * (nz + 1);
    if (cost < 0 || c < cost) {
      cost = c;
      best = nz;
    }
  }
  return best;
}

// Workgroups of one problem and its argument block.
template <int P, typename T, bool CPLX, int TX>
int64_t ts_pack(const TensorLaunch& L, double share, TsArgs<T>& a) {
  using Sh = TsShape<P, T, CPLX, TX>;
  a.Xk = static_cast<const T*>(L.Xk);
  a.Xp = static_cast<const T*>(L.Xp ? L.Xp : L.Xk);
  a.Tg = static_cast<T*>(L.T);
  a.ldx = L.ldx;
  a.ldp = L.Xp ? L.ldp : L.ldx;
  a.ldt = L.ldt;
  a.vdiag = L.vdiag;
  a.ncols = L.ncols;
  a.nc = L.nc;
  a.tab = static_cast<const T*>(L.tab);
  a.has_prev = L.Xp != nullptr;
  // the scalars of the recurrence, divided by alpha kappa.  Rounded once, each of
  // them would be another polynomial, the same way at every node and in every
  // step: up to 9e-7 of a degree-10 filter in single precision, where the
  // roundings of its sums come to 3e-7.  The second part holds what the first
  // one leaves; (V - c) / kappa is formed in double and applied in two parts.
  const double hh = L.h * L.h, bh = L.beta * hh;
  a.ikap = hh;
  a.ck = L.c * hh;
  a.ak = static_cast<T>(L.alpha / hh);
  a.ak_lo = static_cast<T>(std::fma(-static_cast<double>(a.ak), hh, L.alpha) / hh);
  a.bk = static_cast<T>(bh / L.alpha);
  a.bk_lo = static_cast<T>((std::fma(-static_cast<double>(a.bk), L.alpha, bh) + std::fma(L.beta, hh, -bh)) / L.alpha);
  a.sx = static_cast<T>(L.kh[0]);
  a.sy = static_cast<T>(L.kh[1]);
  a.sz = static_cast<T>(L.kh[2]);
  constexpr int NCOL = kL * 8 / static_cast<int>(sizeof(T));
  const int64_t columns = static_cast<int64_t>((L.ncols + NCOL - 1) / NCOL) * L.nc * ((L.nc + TX - 1) / TX);
  a.nz = chunk_cells(columns, L.nc, std::max(1, static_cast<int>(share * L.ncu * Sh::NWG)));
  return columns * ((L.nc + a.nz - 1) / a.nz);
}

// Cells in x per workgroup: a wide tile reads fewer neighbour nodes per owned
// node (3 cells against 2 at p = 6, 24^3 cells, 128 columns: 2.56 against
// 2.71 ms in FP64, 1.31 against 1.53 ms in FP32), as far as the LDS and, for
// complex p = 6, the registers allow; two cells where the wide tile would
// leave more than an eighth of its cells beyond the mesh, and in launches of
// their own that are short of workgroups (launch_tensor_hx): without projectors,
// 3^3 cells, p = 3, 33 columns, 9.8 against 11.6 us in single complex precision,
// 7.8 against 8.6 in FP64.
constexpr int wide_tile(int p, bool cplx) { return p <= 3 ? 4 : (p <= 5 || (p == 6 && !cplx) ? 3 : 2); }
inline bool use_wide(const int* nc, int n, int wide) {
  double w = 0, two = 0;
  for (int i = 0; i < n; ++i) {
    const double rows = static_cast<double>(nc[i]) * nc[i];
    w += rows * ((nc[i] + wide - 1) / wide * wide);
    two += rows * ((nc[i] + 1) / 2 * 2);
  }
  return w * 8 <= two * 9;
}

// f(Tag) with the kernel's template arguments.
template <int P, typename T, bool CPLX, int TX> struct TsTag {
  typedef T real;
  static int64_t pack(const TensorLaunch& L, double share, TsArgs<T>& a) { return ts_pack<P, T, CPLX, TX>(L, share, a); }
  static hipError_t launch(int64_t nblk, const TsArgs<T>& a, const TsArgs<T>* descs, const int64_t* off, int nprob,
                           hipStream_t s) {
    if (nblk <= 0) return hipSuccess;
    if (nblk > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((tensor_hx_kernel<P, T, CPLX, TX>), dim3(static_cast<unsigned>(nblk)),
                       dim3(64 * TsShape<P, T, CPLX, TX>::WAVES), 0, s, a, descs, off, nprob);
    return hipGetLastError();
  }
};
template <int P, typename T, bool CPLX, typename F> auto ts_tile(bool wide, F f) {
  constexpr int W = wide_tile(P, CPLX);
  return wide ? f(TsTag<P, T, CPLX, W>{}) : f(TsTag<P, T, CPLX, 2>{});
}
template <typename T, bool CPLX, typename F> auto ts_order(int p, bool wide, F f) {
  switch (p) {
    case 2: return ts_tile<2, T, CPLX>(wide, f);
    case 3: return ts_tile<3, T, CPLX>(wide, f);
    case 4: return ts_tile<4, T, CPLX>(wide, f);
    case 5: return ts_tile<5, T, CPLX>(wide, f);
    case 6: return ts_tile<6, T, CPLX>(wide, f);
    default: return ts_tile<7, T, CPLX>(wide, f);
  }
}
template <typename F> auto ts_dispatch(int p, int prec, bool wide, F f) {
  switch (prec) {
    case CHFSI_F64: return ts_order<double, false>(p, wide, f);
    case CHFSI_F32: return ts_order<float, false>(p, wide, f);
    case CHFSI_C128: return ts_order<double, true>(p, wide, f);
    default: return ts_order<float, true>(p, wide, f);
  }
}
bool ts_valid(int p, int prec) {
  return p >= 2 && p <= 7 && (prec == CHFSI_F64 || prec == CHFSI_F32 || prec == CHFSI_C128 || prec == CHFSI_C64);
}

}  // namespace

void pack_tensor_tables(int p, const double* K1, const double* S1, const double* m1, double* out) {
  for (int i = 0; i < kTensorTab; ++i) out[i] = 0.0;
  for (int i = 0; i <= p; ++i) {
    out[kTabM + i] = m1[i];
    for (int j = i; j <= p - i; ++j) {
      const int e = tab_index(p, i, j), m = i * (p + 1) + j;
      out[e] = K1[m];
      out[kTabMass + e] = (i != j ? 0.0 : (i == 0 || i == p ? 0.5 : 1.0)) - m1[i] * m1[j];
      out[kTabS + e] = S1[m];
    }
  }
  for (int k = 0; k <= p; ++k) {
    double* c = out + kTabCol + kTabStep * k;
    for (int q = 0; q <= p; ++q) {
      const int e = tab_index(p, q, k);
      c[q] = out[e];
      c[8 + q] = q == k ? 0.0 : (q > k ? -out[kTabS + e] : out[kTabS + e]);
    }
    c[16] = m1[k];
  }
}

hipError_t launch_tensor_hx(const TensorLaunch& L, int prec, hipStream_t s) {
  if (!ts_valid(L.p, prec)) return hipErrorInvalidValue;
  // a launch whose two-cell tiles, one cell high, all run at once is as long as
  // one of them: the wide ones, with more work in each, only lengthen it
  const int ncol = prec == CHFSI_F64 || prec == CHFSI_C128 ? kL : 2 * kL;
  const bool few = static_cast<int64_t>((L.ncols + ncol - 1) / ncol) * L.nc * L.nc * ((L.nc + 1) / 2) <= L.ncu;
  return ts_dispatch(L.p, prec, !few && tensor_batch_wide(L.p, prec, {L.nc}), [&](auto tag) {
    typedef decltype(tag) Tag;
    TsArgs<typename Tag::real> a;
    const int64_t nblk = Tag::pack(L, 1.0, a);
    return Tag::launch(nblk, a, nullptr, nullptr, 0, s);
  });
}

size_t tensor_desc_bytes(int prec) {
  return prec == CHFSI_F64 || prec == CHFSI_C128 ? sizeof(TsArgs<double>) : sizeof(TsArgs<float>);
}

bool tensor_batch_wide(int p, int prec, const std::vector<int>& nc) {
  return use_wide(nc.data(), static_cast<int>(nc.size()), wide_tile(p, prec == CHFSI_C128 || prec == CHFSI_C64));
}

int64_t pack_tensor_desc(const TensorLaunch& L, int prec, bool wide, double share, void* out) {
  return ts_dispatch(L.p, prec, wide, [&](auto tag) {
    typedef decltype(tag) Tag;
    return Tag::pack(L, share, *static_cast<TsArgs<typename Tag::real>*>(out));
  });
}

hipError_t launch_tensor_batched(const TensorBatch& b, int prec, hipStream_t s) {
  if (!ts_valid(b.p, prec)) return hipErrorInvalidValue;
  return ts_dispatch(b.p, prec, b.wide, [&](auto tag) {
    typedef decltype(tag) Tag;
    typedef TsArgs<typename Tag::real> A;
    return Tag::launch(b.nblk, A{}, static_cast<const A*>(b.descs), b.item_off, b.nprob, s);
  });
}

}  // namespace chfsi
