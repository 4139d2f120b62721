// HIP kernels of the CutFEM vertex-patch multigrid for gfx950 (MI355X).
//
// Data layout: every level keeps its vectors on the full (kN+1)^d node lattice,
// x fastest, with exact zeros at inactive nodes.  Lattice indexing needs no DoF
// index lists inside the patch kernels, and the patches of one colour read
// neighbouring x-rows, which keeps the HBM streams coalesced.  Compact vectors
// (canonical DoF order) exist only at the library boundary.
//
// Operator (paper eq. (cutfem_nitsche) + eq. (cutfem-ghost)), evaluated row by
// row for a node i:
//   (A x)_i = sum_{active cells T containing i} row_i(E_T) x_T
//           + sum_{ghost faces F of those cells} row_i(G_F) x_{T1 u T2}
// with E_T the uncut stiffness (shared, kept in LDS) or the dense matrix of a
// cut cell, and G_F = sum_m c_m (d^m-jump) x (1-D mass on the face) built from
// 1-D tables: a face needs no stored data.  The operator kernel takes the
// terms of the special cells (cut, or with a ghost face) from two pre-passes:
// the mass-contracted jumps of every ghost face, then one value per special
// cell and node.
//
// Smoother colour steps (paper eqs. (local-solver), (smoother-split)):
//   interior patches: one fused kernel - x on the patch closure is staged in
//     LDS, the residual on the (2k-1)^d internal nodes uses the Cartesian
//     stiffness, the local solve is fast diagonalisation (S (x) S (x) S) D^-1
//     (S^T (x) S^T (x) S^T), and the internal values are updated in place.  Same
//     coloured interior patches read only their own closure, so the fused
//     update is race free.
//   cut patches: residual (general rows incl. ghost faces, which may reach into
//     a same-coloured neighbour) and dense inverse GEMV; every patch of the
//     colour must see the state at the start of the step, so the steps of a
//     smoothing pass alternate between two x buffers (read one, write x + d
//     and the previous colour's DoFs into the other); an odd last step writes
//     the corrections to a buffer that a second kernel adds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "kernels.h"

namespace cmg {
namespace dev {

template <int B, int E>
struct Pow { static constexpr int v = B * Pow<B, E - 1>::v; };
template <int B>
struct Pow<B, 0> { static constexpr int v = 1; };

template <int D, int K>
struct Shape {
  static constexpr int N1 = K + 1;                 // nodes per cell and direction
  static constexpr int NL = Pow<N1, D>::v;         // nodes per cell
  static constexpr int NP1 = 2 * K - 1;            // internal patch nodes per direction
  static constexpr int NP = Pow<NP1, D>::v;        // internal patch nodes
  static constexpr int NC1 = 2 * K + 1;            // patch closure nodes per direction
  static constexpr int NC = Pow<NC1, D>::v;
  // patches per 256-thread block of the interior step; Q1 (one node a patch)
  // stays at 64: 256 make few blocks (in 3-D 13 at 64^3 cells, with 111 KB of LDS
  // each).  Off-centre ball, 64^3 cells: step 10.3 -> 7.1 us; off-centre disc, with
  // 256, 128, 64, 32, 16 patches a block: 1024^2 cells 8.2, 7.7, 7.8, 8.7, 11.3 us
  // (V-cycle 611, 595, 586, 594, 616 us), 256^2 cells 7.1, 6.5, 6.5, 6.6, 6.5 us
  static constexpr int PPB = NP == 1 ? 64 : 256 / NP;
  // table layout (doubles), see LevelTables on the host
  static constexpr int T_KCELL = 0;
  static constexpr int T_MHAT = T_KCELL + NL * NL;
  static constexpr int T_D0 = T_MHAT + N1 * N1;
  static constexpr int T_D1 = T_D0 + K * N1;
  static constexpr int T_GC = T_D1 + K * N1;
  static constexpr int T_FDS = T_GC + K;
  static constexpr int T_FDD = T_FDS + NP1 * NP1;
  static constexpr int T_P1D = T_FDD + NP;
  static constexpr int T_K1S = T_P1D + NC1 * N1;
  static constexpr int T_JM = T_K1S + N1 * N1;      // jump weights j_m(s) of the m-th derivative, K x (2K+1)
  static constexpr int T_GJ = T_JM + K * NC1;       // the same times the ghost coefficient
  static constexpr int T_SIZE = T_GJ + K * NC1;
};

// Work index of block b out of n such that the blocks of one XCD take one
// contiguous range of work items.  The chip dispatches workgroups to its 8
// XCDs round-robin by block index and every XCD has its own L2, so without
// the remap consecutive (spatially neighbouring) cut patches land on
// different XCDs and each XCD fetches the x-lines they share separately
// (measured: finest cut steps 2.5% faster in FP64 and FP32).  The grid-stride
// operator and interior-patch kernels keep the plain order, which measured
// faster for them (the remap cost them 8% and 20%).
// Bijective on [0, n): XCD x < n % 8 takes n / 8 + 1 items, the others n / 8.
__device__ __forceinline__ int xcd_block(int b, int n) {
  constexpr int NX = 8;
  const int q = n / NX, r = n % NX, xc = b % NX, s = b / NX;
  return xc < r ? xc * (q + 1) + s : r * (q + 1) + (xc - r) * q + s;
}

// Grouped launch: one launch runs the same kernel for several problems, the
// problem's argument record being entry blockIdx.z of a device table.  The
// grid is the largest of the members' grids, so every kernel with a grouped
// form lets the blocks beyond its own work return (grid-stride loops, index
// bounds, or a patch index past the colour's patches).
template <int LB, typename A>
__global__ __launch_bounds__(LB) void k_grouped(const A* __restrict__ tab) {
  tab[blockIdx.z].run();
}

__device__ __forceinline__ int64_t lat(int D, int nn, const int* I) {
  return D == 2 ? I[0] + (int64_t)nn * I[1] : I[0] + (int64_t)nn * (I[1] + (int64_t)nn * I[2]);
}

__device__ __forceinline__ int64_t cell_lin(int D, int N, const int* c) {
  return D == 2 ? c[0] + (int64_t)N * c[1] : c[0] + (int64_t)N * (c[1] + (int64_t)N * c[2]);
}

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// One 16x16x4 matrix-core product: lane l holds A(l%16, l/16) and B(l/16,
// l%16); of D it holds column l%16 and, as element v, row mfma_row(l, v).
__device__ __forceinline__ floatx4 mfma16(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ doublex4 mfma16(double a, double b, doublex4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
template <typename T>
struct Mfma;
template <>
struct Mfma<float> {
  using Acc = floatx4;
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane / 16) + v; }
};
template <>
struct Mfma<double> {
  using Acc = doublex4;
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * v + lane / 16; }
};

// Ghost-face pre-pass of the operator: for every ghost face and derivative order
// m, the jump J_m(b_t) = sum_bd psi_bd^(m)(1) x_lower - psi_bd^(m)(0) x_upper at the
// tangential face nodes b_t, contracted with the reference face mass:
// W_m(i_t) = sum_{b_t} prod_j Mhat[i_t,j, b_t,j] J_m(b_t).  A row of a node i of
// a cell adjacent to the face then only needs gc_m * trace_m(i_dir) * W_m(i_t).
// One thread per face and column: the 2 (k+1) nodes along the normal at each
// tangential node are read once for all k orders.
template <int D, int K, typename T>
__device__ __forceinline__ void face_w_body(KLevel L, const T* __restrict__ x, T* __restrict__ W) {
  using S = Shape<D, K>;
  constexpr int N1 = S::N1;
  constexpr int NT = Pow<N1, D - 1>::v;
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  W += blockIdx.y * L.n_faces * K * NT;
  const int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (f >= L.n_faces) return;
  const double* mh = L.tables + S::T_MHAT;
  const double* d0 = L.tables + S::T_D0;
  const double* d1 = L.tables + S::T_D1;
  const int dir = L.face_dir[f];
  int c[3];
  {
    int64_t r = L.face_lower[f];
#pragma unroll
    for (int a = 0; a < D; ++a) { c[a] = static_cast<int>(r % L.N); r /= L.N; }
  }
  // first node of the lower cell and the lattice strides
  int64_t base = 0, sn = 1, st0 = 0, st1 = 0;
  {
    int64_t sa = 1;
    int tb = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      base += K * c[a] * sa;
      if (a == dir) sn = sa;
      else if (tb++ == 0) st0 = sa;
      else st1 = sa;
      sa *= L.nn;
    }
  }
  T J[K][NT];
#pragma unroll
  for (int bt = 0; bt < NT; ++bt) {
    const int64_t el = base + (bt % N1) * st0 + (D == 3 ? (bt / N1) * st1 : 0);
    T xl[N1], xu[N1];
#pragma unroll
    for (int bd = 0; bd <= K; ++bd) {
      xl[bd] = x[el + bd * sn];
      xu[bd] = x[el + (bd + K) * sn];
    }
#pragma unroll
    for (int m = 0; m < K; ++m) {
      T acc = 0;
#pragma unroll
      for (int bd = 0; bd <= K; ++bd) acc += (T)d1[m * N1 + bd] * xl[bd] - (T)d0[m * N1 + bd] * xu[bd];
      J[m][bt] = acc;
    }
  }
#pragma unroll
  for (int m = 0; m < K; ++m) {
    T* out = W + (f * K + m) * NT;
    if (D == 2) {
#pragma unroll
      for (int it = 0; it < N1; ++it) {
        T acc = 0;
#pragma unroll
        for (int bt = 0; bt < N1; ++bt) acc += (T)mh[it * N1 + bt] * J[m][bt];
        out[it] = acc;
      }
      continue;
    }
    T H[NT];  // (Mhat x Mhat) J by two 1-D contractions
#pragma unroll
    for (int b1 = 0; b1 < N1; ++b1)
#pragma unroll
      for (int i0 = 0; i0 < N1; ++i0) {
        T acc = 0;
#pragma unroll
        for (int b0 = 0; b0 < N1; ++b0) acc += (T)mh[i0 * N1 + b0] * J[m][b0 + N1 * b1];
        H[i0 + N1 * b1] = acc;
      }
#pragma unroll
    for (int i1 = 0; i1 < N1; ++i1)
#pragma unroll
      for (int i0 = 0; i0 < N1; ++i0) {
        T acc = 0;
#pragma unroll
        for (int b1 = 0; b1 < N1; ++b1) acc += (T)mh[i1 * N1 + b1] * H[i0 + N1 * b1];
        out[i0 + N1 * i1] = acc;
      }
  }
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_face_w(KLevel L, const T* __restrict__ x, T* __restrict__ W) {
  face_w_body<D, K, T>(L, x, W);
}

// argument record of k_face_w for grouped launches (k_grouped)
template <int D, int K, typename T>
struct FaceWArgs {
  KLevel L;
  const T* x;
  T* W;
  __device__ void run() const { face_w_body<D, K, T>(L, x, W); }
};

// Special-cell pre-pass of the operator.  A special cell T is cut or has a
// ghost face; for each of them and every column it forms the contribution of T
// to the rows of its nodes,
//   C_T(i) = (E_T x_T)_i + sum_{ghost faces F of T} sum_m gc_m trace_m(i_dir) W_m(F)(i_t),
// with E_T the cut-cell matrix or the uncut stiffness and W the face pre-pass
// output, so that the operator kernel adds one value per special cell and
// node.  CPB cells per block, one thread per cell node and CT of the NCOL
// columns, the NCOL / CT column slots in waves of their own.  A cut cell's E_T
// is symmetric and read as its packed upper triangle, (k+1)^d ((k+1)^d + 1) / 2
// entries instead of (k+1)^{2d}, staged in LDS by the cell's threads of all
// slots (consecutive threads, consecutive entries).  The matrices' bytes bound
// the kernel; a cell's own chain (its record, its matrix, its ghost terms) hides
// only behind other waves and behind loads in flight, hence 4 waves on a
// matrix where there are columns for them, and the ghost terms of a direction
// read at once, a side without a face read as face 0 and dropped.
// 8 columns, Q3, 16 569 special cells (275 MB of FP64 matrices): FP64 497 -> 231 us,
// FP32 220 -> 123 us; Q2 disc of 512^2, one column: 6.2 -> 4.7 us.
template <int D, int K, int NCOL>
struct CellShape {
  static constexpr int NL = Shape<D, K>::NL;
  static constexpr int CPB = 64 / NL;
  static constexpr int NW = NCOL < 4 ? 1 : 4;  // column slots, a wave each
  static constexpr int CT = NCOL / NW;         // columns of a slot
  static constexpr int TH = 64 * NW;
  static_assert(CPB >= 1 && CT * NW == NCOL, "one thread per cell node and slot");
};

template <int D, int K, typename T, int NCOL>
__device__ __forceinline__ void cell_ax_body(KLevel L, const T* __restrict__ x, const T* __restrict__ W,
                                             T* __restrict__ C, int ncol) {
  using S = Shape<D, K>;
  using H = CellShape<D, K, NCOL>;
  constexpr int N1 = S::N1, NL = S::NL, CPB = H::CPB, CT = H::CT, NF = 2 * D;
  constexpr int NT = Pow<N1, D - 1>::v;
  constexpr int NPK = NL * (NL + 1) / 2;  // entries of a packed symmetric cell matrix
  // column group blockIdx.y of at most NCOL columns
  x += (int64_t)blockIdx.y * NCOL * L.n_nodes;
  W += (int64_t)blockIdx.y * NCOL * L.n_faces * K * NT;
  C += (int64_t)blockIdx.y * NCOL * L.n_spec * NL;
  ncol = ncol - (int)blockIdx.y * NCOL < NCOL ? ncol - (int)blockIdx.y * NCOL : NCOL;
  __shared__ T xs[CPB][NL][NCOL];
  __shared__ T epk[CPB][NPK];
  const int slot = H::NW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int c0 = slot * CT, nc = ncol - c0;  // the slot's columns (none if nc <= 0)
  const int lc = threadIdx.x % 64 / NL;
  const int i = threadIdx.x % 64 % NL;
  const int64_t t = (int64_t)blockIdx.x * CPB + lc;
  const bool on = lc < CPB && t < L.n_spec;
  int il[3] = {0, 0, 0};
  int32_t info[1 + NF];
  if (on) {
    int64_t r = L.spec_cells[t];
#pragma unroll
    for (int j = 0; j <= NF; ++j) info[j] = L.spec_info[t * (1 + NF) + j];
    int I[3];
    int q = i;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      il[a] = q % N1;
      q /= N1;
      I[a] = K * static_cast<int>(r % L.N) + il[a];
      r /= L.N;
    }
    const int64_t node = lat(D, L.nn, I);
#pragma unroll
    for (int c = 0; c < CT; ++c) xs[lc][i][c0 + c] = c < nc ? x[(c0 + c) * L.n_nodes + node] : (T)0;
    // a cut cell's matrix, read once as its packed upper triangle (the cell's
    // threads read consecutive entries, G loads in flight per thread) and
    // staged for all rows
    if (info[0] >= 0) {
      const T* P = L.cut_packed_t<T>() + (int64_t)info[0] * NPK;
      constexpr int RT = NL * H::NW, NR = (NPK + RT - 1) / RT, G = NR < 16 ? NR : 8;
      const int e0 = slot * NL + i;
#pragma unroll
      for (int r0 = 0; r0 < NR; r0 += G) {
        T v[G];
#pragma unroll
        for (int r = 0; r < G; ++r) {
          const int e = (r0 + r) * RT + e0;
          v[r] = P[e < NPK ? e : NPK - 1];
        }
#pragma unroll
        for (int r = 0; r < G; ++r) {
          const int e = (r0 + r) * RT + e0;
          if (e < NPK) epk[lc][e] = v[r];
        }
      }
    }
  }
  // ghost terms before the barrier: their loads do not wait for the staged x
  T acc[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) acc[c] = 0;
  if (on && nc > 0 && L.n_faces > 0) {
    const int64_t wcol = L.n_faces * K * NT;
    const double* d0 = L.tables + S::T_D0;
    const double* d1 = L.tables + S::T_D1;
    const double* gc = L.tables + S::T_GC;
#pragma unroll
    for (int dir = 0; dir < D; ++dir) {
      int it = 0, st = 1;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        if (a == dir) continue;
        it += il[a] * st;
        st *= N1;
      }
      T w[2][K][CT];
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const int fid = info[1 + 2 * dir + side];
        const T* p = W + (int64_t)(fid < 0 ? 0 : fid) * K * NT + it + c0 * wcol;
#pragma unroll
        for (int m = 0; m < K; ++m)
#pragma unroll
          for (int c = 0; c < CT; ++c) w[side][m][c] = p[(c < nc ? c : 0) * wcol + m * NT];
      }
#pragma unroll
      for (int side = 0; side < 2; ++side) {
        const bool face = info[1 + 2 * dir + side] >= 0;
#pragma unroll
        for (int m = 0; m < K; ++m) {
          const T sg = (T)(gc[m] * (side == 1 ? d1[m * N1 + il[dir]] : -d0[m * N1 + il[dir]]));
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[c] = face ? acc[c] + sg * w[side][m][c] : acc[c];
        }
      }
    }
  }
  __syncthreads();
  if (!on || nc <= 0) return;
  T cell[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) cell[c] = 0;
  if (info[0] >= 0) {
    // entry (a, b), a <= b, of the packed upper triangle sits at a (2 NL - a + 1) / 2 + b - a;
    // row i of E is (j, i) for j < i and (i, j) from the diagonal on
    const int rowi = i * (2 * NL - i + 1) / 2;
#pragma unroll 4
    for (int j = 0; j < NL; ++j) {
      const int q = j < i ? j * (2 * NL - j + 1) / 2 + (i - j) : rowi + (j - i);
      const T e = epk[lc][q];
#pragma unroll
      for (int c = 0; c < CT; ++c) cell[c] += e * xs[lc][j][c0 + c];
    }
  } else {
    const T* row = L.kcell_t<T>() + S::T_KCELL + i * NL;
#pragma unroll 4
    for (int j = 0; j < NL; ++j) {
      const T e = row[j];
#pragma unroll
      for (int c = 0; c < CT; ++c) cell[c] += e * xs[lc][j][c0 + c];
    }
  }
#pragma unroll
  for (int c = 0; c < CT; ++c)
    if (c < nc) C[(c0 + c) * L.n_spec * NL + t * NL + i] = cell[c] + acc[c];
}

template <int D, int K, typename T, int NCOL>
__global__ __launch_bounds__((CellShape<D, K, NCOL>::TH)) void k_cell_ax(KLevel L, const T* __restrict__ x, const T* __restrict__ W,
                                                T* __restrict__ C, int ncol) {
  cell_ax_body<D, K, T, NCOL>(L, x, W, C, ncol);
}

// argument record of k_cell_ax for grouped launches (k_grouped)
template <int D, int K, typename T, int NCOL>
struct CellAxArgs {
  KLevel L;
  const T* x;
  const T* W;
  T* C;
  int ncol;
  __device__ void run() const { cell_ax_body<D, K, T, NCOL>(L, x, W, C, ncol); }
};

template <int D, int K>
struct ApplyShape {
  static constexpr int B = (D == 3 && K == 3) ? 2 : 4;   // cells per tile and direction
  static constexpr int R1 = (B + 1) * K + 1;             // staged nodes per direction: cells -1 .. B-1
  static constexpr int NR = Pow<R1, D>::v;
  static constexpr int C1 = B + 1;                       // staged cells per direction
  static constexpr int NCC = Pow<C1, D>::v;
  static constexpr int O1 = B * K + 1;                   // owned nodes per direction (last tile: + 1)
  static constexpr int NO = Pow<O1, D>::v;
};

// y = A x (b == nullptr) or y = b - A x on the active nodes of a tile of B^d
// cells.  x on the cells -1 .. B-1 around the tile is staged in LDS; every
// owned node sums, over the cells that contain it, the uncut stiffness row
// (from LDS) or the special-cell value of the pre-pass (from C).  The C loads
// of a node's cells are independent and issued together before the LDS rows.
template <int D, int K, typename T>
__device__ __forceinline__ void apply_rows_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                                T* __restrict__ y, const T* __restrict__ C) {
  using S = Shape<D, K>;
  using A = ApplyShape<D, K>;
  constexpr int N1 = S::N1, NL = S::NL, B = A::B, R1 = A::R1, C1 = A::C1, O1 = A::O1;
  constexpr int NCB = 1 << D;
  constexpr int NRW = N1 * (D == 3 ? N1 : 1);
  __shared__ T tab[S::T_MHAT];  // uncut stiffness, in the path's precision
  __shared__ T xs[A::NR];
  __shared__ int32_t csid[A::NCC];
  for (int i = threadIdx.x; i < S::T_MHAT; i += blockDim.x) tab[i] = L.kcell_t<T>()[i];
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  if (b) b += blockIdx.y * L.n_nodes;
  y += blockIdx.y * L.n_nodes;
  C += blockIdx.y * L.n_spec * NL;
  const int NTd = (L.N + B - 1) / B;
  for (int ti = blockIdx.x; ti < L.n_tiles; ti += gridDim.x) {
    __syncthreads();
    int tc[3] = {0, 0, 0};
    {
      int r = L.tiles[ti];
#pragma unroll
      for (int a = 0; a < D; ++a) { tc[a] = r % NTd; r /= NTd; }
    }
    for (int e = threadIdx.x; e < A::NCC; e += blockDim.x) {
      int c[3];
      bool in = true;
      int r = e;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        c[a] = B * tc[a] - 1 + r % C1;
        r /= C1;
        in = in && c[a] >= 0 && c[a] < L.N;
      }
      csid[e] = in ? L.cell_sid[cell_lin(D, L.N, c)] : -2;
    }
    for (int e = threadIdx.x; e < A::NR; e += blockDim.x) {
      int I[3];
      bool in = true;
      int r = e;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        I[a] = K * (B * tc[a] - 1) + r % R1;
        r /= R1;
        in = in && I[a] >= 0 && I[a] < L.nn;
      }
      xs[e] = in ? x[lat(D, L.nn, I)] : (T)0;
    }
    __syncthreads();
    // the node's cells along each direction: a node on a cell boundary
    // (q % K == 0) lies in staged cells q/K (local index K) and q/K + 1 (local
    // index 0), any other node only in q/K + 1; comb bit a selects the upper one
    auto cell_of = [&](const int* q, int comb, int* c, int* il) {
      bool ok = true;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const int sel = (comb >> a) & 1;
        if (q[a] % K == 0) {
          c[a] = q[a] / K + sel;
          il[a] = sel ? 0 : K;
        } else {
          ok = ok && sel == 0;
          c[a] = q[a] / K + 1;
          il[a] = q[a] % K;
        }
        ok = ok && c[a] < C1;  // beyond the background box
      }
      return ok;
    };
#pragma unroll 1
    for (int e = threadIdx.x; e < A::NO; e += blockDim.x) {
      int q[3], I[3];
      bool own = true;
      int r = e;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        q[a] = r % O1;
        r /= O1;
        I[a] = K * B * tc[a] + q[a];
        // the layer q = B K belongs to the next tile unless this is the last one
        own = own && I[a] < L.nn && (q[a] < B * K || tc[a] == NTd - 1);
      }
      if (!own) continue;
      const int64_t node = lat(D, L.nn, I);
      const T bv = b ? b[node] : (T)0;
      // pass 1: the special-cell values, all loads in flight together
      T cv[NCB];
      bool act = false;  // the node lies in an active cell
#pragma unroll
      for (int comb = 0; comb < NCB; ++comb) {
        cv[comb] = 0;
        int c[3], il[3];
        if (!cell_of(q, comb, c, il)) continue;
        int ce = c[0] + C1 * c[1];
        if (D == 3) ce += C1 * C1 * c[2];
        const int sid = csid[ce];
        if (sid == -2) continue;  // inactive cell
        act = true;
        if (sid < 0) continue;
        int iloc = il[0] + N1 * il[1];
        if (D == 3) iloc += N1 * N1 * il[2];
        cv[comb] = C[(int64_t)sid * NL + iloc];
      }
      if (!act) continue;
      // pass 2: uncut stiffness rows of the regular cells from LDS
      T ax = 0;
#pragma unroll 1
      for (int comb = 0; comb < NCB; ++comb) {
        int c[3], il[3];
        if (!cell_of(q, comb, c, il)) continue;
        int ce = c[0] + C1 * c[1];
        if (D == 3) ce += C1 * C1 * c[2];
        if (csid[ce] != -1) continue;
        int iloc = il[0] + N1 * il[1];
        if (D == 3) iloc += N1 * N1 * il[2];
        int xb = K * c[0] + R1 * K * c[1];
        if (D == 3) xb += R1 * R1 * K * c[2];
        const T* row = tab + iloc * NL;
        T acc[NRW];
#pragma unroll
        for (int a = 0; a < NRW; ++a) acc[a] = 0;
#pragma unroll
        for (int bq = 0; bq < NL; ++bq) {
          const int b0 = bq % N1, b12 = bq / N1;
          const int xi = xb + b0 + R1 * (b12 % N1) + (D == 3 ? R1 * R1 * (b12 / N1) : 0);
          acc[b12] += row[bq] * xs[xi];
        }
        T sacc = 0;
#pragma unroll
        for (int a = 0; a < NRW; ++a) sacc += acc[a];
        ax += sacc;
      }
#pragma unroll
      for (int comb = 0; comb < NCB; ++comb) ax += cv[comb];
      y[node] = b ? bv - ax : ax;
    }
  }
}

// The same for Q2 and Q3 in 3-D, the regular cells on the matrix cores: they all
// have one stiffness matrix, so the products of 16 cells are 16x16x4 products
// of its rows (kept in a wave's registers for all tiles of the block) with the
// cells' x as columns, left in LDS as one value per cell and node; every owned
// node then sums its up to 2^d cells' values (from LDS, or the pre-pass's from
// C) with all reads in flight.  Dense rows node by node made every wave walk
// 8 (k+1)^3 terms for the few nodes that lie in 8 cells, at two LDS reads a
// term.  128^3 ball, Q2, FP64: product 229 -> 181 us; ball at 32^3 51 -> 38 us; Q3
// union at 32^3, residual of 8 columns 314 -> 232 us.
template <int K, typename T>
__device__ __forceinline__ void apply_mfma_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                                T* __restrict__ y, const T* __restrict__ C) {
  using S = Shape<3, K>;
  using A = ApplyShape<3, K>;
  using Acc = typename Mfma<T>::Acc;
  constexpr int N1 = S::N1, NL = S::NL, B = A::B, R1 = A::R1, C1 = A::C1, O1 = A::O1, NCC = A::NCC;
  constexpr int NRT = (NL + 15) / 16, NKS = (NL + 3) / 4, YS = NL | 1;
  static_assert(4 % NRT == 0 && NCC <= 128, "row tiles per wave, cells per block");
  __shared__ T xs[A::NR];
  __shared__ T Y[NCC][YS];        // cell products of the regular cells, in list order
  __shared__ int32_t csid[NCC];   // special id; the cells of the list: -3 - place in it
  __shared__ int16_t list[NCC];   // first staged node of every regular cell
  __shared__ int nreg;
  const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int lr = lane % 16, lk = lane / 16, rt = wave % NRT;
  T a[NKS];  // rows 16 rt .. of the uncut stiffness
  {
    const int r = rt * 16 + lr;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int q = 4 * ks + lk;
      const T e = L.kcell_t<T>()[S::T_KCELL + (r < NL ? r : 0) * NL + (q < NL ? q : 0)];
      a[ks] = r < NL && q < NL ? e : (T)0;
    }
  }
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  if (b) b += blockIdx.y * L.n_nodes;
  y += blockIdx.y * L.n_nodes;
  C += blockIdx.y * L.n_spec * NL;
  const int NTd = (L.N + B - 1) / B;
  for (int ti = blockIdx.x; ti < L.n_tiles; ti += gridDim.x) {
    __syncthreads();
    const int tile = L.tiles[ti];
    const int tc[3] = {tile % NTd, (tile / NTd) % NTd, tile / (NTd * NTd)};
    {
      constexpr int NIT = (A::NR + 255) / 256;
      T v[NIT];
#pragma unroll
      for (int u = 0; u < NIT; ++u) {
        const int e = threadIdx.x + 256 * u;
        int I[3], r = e;
        bool in = e < A::NR;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          I[d] = K * (B * tc[d] - 1) + r % R1;
          r /= R1;
          in = in && I[d] >= 0 && I[d] < L.nn;
        }
        v[u] = in ? x[lat(3, L.nn, I)] : (T)0;
      }
      if (wave == 0) {
        // the cells' special ids, and the list of the regular ones in cell order
        int n = 0;
#pragma unroll
        for (int h = 0; h < (NCC + 63) / 64; ++h) {
          const int e = lane + 64 * h;
          int c[3], r = e;
          bool in = e < NCC;
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            c[d] = B * tc[d] - 1 + r % C1;
            r /= C1;
            in = in && c[d] >= 0 && c[d] < L.N;
          }
          const int sid = in ? L.cell_sid[cell_lin(3, L.N, c)] : -2;
          const uint64_t m = __ballot(sid == -1);
          const int at = n + __popcll(m & ((1ull << lane) - 1));
          if (e < NCC) csid[e] = sid == -1 ? -3 - at : sid;
          if (sid == -1) list[at] = static_cast<int16_t>(K * (e % C1 + R1 * ((e / C1) % C1 + R1 * (e / (C1 * C1)))));
          n += __popcll(m);
        }
        if (lane == 0) nreg = n;
      }
#pragma unroll
      for (int u = 0; u < NIT; ++u) {
        const int e = threadIdx.x + 256 * u;
        if (e < A::NR) xs[e] = v[u];
      }
    }
    __syncthreads();
    const int nr = nreg;
    for (int g = wave / NRT; g * 16 < nr; g += 4 / NRT) {  // wave-uniform: every lane takes part in the products
      const int slot = g * 16 + lr;
      const T* xc = xs + list[slot < nr ? slot : 0];
      Acc acc = {0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int q = 4 * ks + lk;
        const int at = q % N1 + R1 * ((q / N1) % N1 + R1 * (q / (N1 * N1)));
        acc = mfma16(a[ks], q < NL ? xc[at] : (T)0, acc);
      }
      if (slot < nr) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int r = rt * 16 + Mfma<T>::row(lane, v);
          if (r < NL) Y[slot][r] = acc[v];
        }
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int e = threadIdx.x; e < A::NO; e += 256) {
      const int q[3] = {e % O1, (e / O1) % O1, e / (O1 * O1)};
      bool own = true;
      int I[3];
      // the node's cells along each direction: a node on a cell boundary lies in
      // the staged cells q/K (local index K) and q/K + 1 (0), any other in q/K + 1
      int cc[3][2], il[3][2], two[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        I[d] = K * B * tc[d] + q[d];
        // the layer q = B K belongs to the next tile unless this is the last one
        own = own && I[d] < L.nn && (q[d] < B * K || tc[d] == NTd - 1);
        const bool edge = q[d] % K == 0;
        cc[d][0] = edge ? q[d] / K : q[d] / K + 1;
        il[d][0] = edge ? K : q[d] % K;
        two[d] = edge && q[d] / K + 1 < C1;  // (not beyond the background box)
        cc[d][1] = two[d] ? q[d] / K + 1 : cc[d][0];
        il[d][1] = two[d] ? 0 : il[d][0];
      }
      if (!own) continue;
      const int64_t node = lat(3, L.nn, I);
      const T bv = b ? b[node] : (T)0;
      T cv[8], yv[8];
      bool act = false;  // the node lies in an active cell
#pragma unroll
      for (int comb = 0; comb < 8; ++comb) {
        const int s0 = comb & 1, s1 = (comb >> 1) & 1, s2 = comb >> 2;
        const bool has = (!s0 || two[0]) && (!s1 || two[1]) && (!s2 || two[2]);
        const int sid = csid[cc[0][s0] + C1 * (cc[1][s1] + C1 * cc[2][s2])];
        const int iloc = il[0][s0] + N1 * (il[1][s1] + N1 * il[2][s2]);
        act = act || (has && sid != -2);
        cv[comb] = has && sid >= 0 ? C[(int64_t)sid * NL + iloc] : (T)0;
        const T r = Y[sid <= -3 ? -3 - sid : 0][iloc];
        yv[comb] = has && sid <= -3 ? r : (T)0;
      }
      if (!act) continue;
      T ax = 0;
#pragma unroll
      for (int comb = 0; comb < 8; ++comb) ax += yv[comb];
#pragma unroll
      for (int comb = 0; comb < 8; ++comb) ax += cv[comb];
      y[node] = b ? bv - ax : ax;
    }
  }
}

template <int D, int K, typename T>
__device__ __forceinline__ void apply_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                           T* __restrict__ y, const T* __restrict__ C) {
  // Q1 rows have 8 entries, too few for a row tile, and 2-D meshes few mixed tiles
  if constexpr (D == 3 && K > 1)
    apply_mfma_body<K, T>(L, x, b, y, C);
  else
    apply_rows_body<D, K, T>(L, x, b, y, C);
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_apply(KLevel L, const T* __restrict__ x, const T* __restrict__ b,
                                               T* __restrict__ y, const T* __restrict__ C) {
  apply_body<D, K, T>(L, x, b, y, C);
}

// argument record of k_apply for grouped launches (k_grouped)
template <int D, int K, typename T>
struct ApplyArgs {
  KLevel L;
  const T* x;
  const T* b;
  T* y;
  const T* C;
  __device__ void run() const { apply_body<D, K, T>(L, x, b, y, C); }
};

// Entry (s, j) of the 1-D matrix assembled from the element matrix e ((k+1) x
// (k+1), row-major) over the NCELL staged cells of an operator tile along one
// direction (cell c holds staged nodes K c .. K c + K).  tile1d_nz tells
// whether some cell holds both nodes; with compile-time s and j both fold.
template <int K, int NCELL>
__host__ __device__ constexpr bool tile1d_nz(int s, int j) {
  for (int c = 0; c < NCELL; ++c)
    if (s >= K * c && s <= K * c + K && j >= K * c && j <= K * c + K) return true;
  return false;
}
template <int K, int NCELL>
__device__ __forceinline__ double tile1d(const double* e, int s, int j) {
  double v = 0;
#pragma unroll
  for (int c = 0; c < NCELL; ++c)
    if (s >= K * c && s <= K * c + K && j >= K * c && j <= K * c + K) v += e[(s - K * c) * (K + 1) + (j - K * c)];
  return v;
}
// A run-time row s >= K of the assembled 1-D matrices of a tile: 2k+1 taps from
// column first on, the last k of them step apart.  A cell boundary couples
// with both its cells (step 1); any other node, and the line's last one, only
// with the k+1 nodes of one cell: its further taps repeat that cell's last
// node with zero entries, so no node outside its cells is ever read.
template <int K, int NCELL, typename T>
struct TileRow {
  int first, step;
  T m[2 * K + 1], k[2 * K + 1];
  __device__ __forceinline__ void load(const double* em, const double* ek, int s) {
    const bool wide = s % K == 0 && s < NCELL * K;
    const int i = wide || s == NCELL * K ? K : s % K;  // row of the (lower) cell's element matrix
    first = s - i;
    step = wide ? 1 : 0;
#pragma unroll
    for (int t = 0; t <= 2 * K; ++t) {
      T vm = t <= K ? (T)em[i * (K + 1) + (t <= K ? t : 0)] : (T)0, vk = t <= K ? (T)ek[i * (K + 1) + (t <= K ? t : 0)] : (T)0;
      if (t >= K) {  // the upper cell's first row
        const double um = em[t >= K ? t - K : 0], uk = ek[t >= K ? t - K : 0];
        vm = wide ? (T)((t == K ? em[i * (K + 1) + K] : 0.0) + um) : vm;
        vk = wide ? (T)((t == K ? ek[i * (K + 1) + K] : 0.0) + uk) : vk;
      }
      m[t] = vm;
      k[t] = vk;
    }
  }
  __device__ __forceinline__ int at(int t) const { return first + (t <= K ? t : K + (t - K) * step); }
};

// y = A x (b == nullptr) or y = b - A x on the active nodes of a tile whose
// staged cells -1 .. B-1 are all active and regular.  There A is the sum over
// directions a of tensor products of the assembled 1-D stiffness h^(d-2) K1
// along a and the assembled 1-D mass along the others (the uncut cell
// stiffness has this form, summed over the staged cells), applied by one pass
// per direction: along the slowest direction every staged line gives Mhat x
// and Khat x on the owned rows; in 3-D the next direction gives Mhat Mhat x and
// Khat Mhat x + Mhat Khat x; every owned node contracts direction 0 at its own
// position.  Only the band of the 1-D matrices is applied.
//
// 2-D: a thread keeps one (line, row) of the first pass and one owned node of
// the second for all tiles of its block, so the entries of both rows stay in
// its registers; a block works on as many tiles at once as its threads cover,
// and the next tiles' x is on its way while the current ones are contracted.
// The former form gave the first pass one thread per line, 16 of 256 for Q3.
// Circle, Q3, 1024^2 cells (6.1 million DoFs), FP64: 298 -> 75 us; now bound by
// the 22 LDS reads of a node (one 8-byte word a clock and bank pair).
template <int K, typename T>
__device__ __forceinline__ void apply_sf2_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                               T* __restrict__ y) {
  using S = Shape<2, K>;
  using A = ApplyShape<2, K>;
  constexpr int B = A::B, R1 = A::R1, C1 = A::C1, O1 = A::O1, NR = R1 * R1, TP = 256 / NR;
  static_assert(TP >= 1, "a thread per staged node");
  __shared__ T xv[TP][NR];
  __shared__ T um[TP][O1 * R1], uk[TP][O1 * R1];
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  if (b) b += blockIdx.y * L.n_nodes;
  y += blockIdx.y * L.n_nodes;
  const int NTd = (L.N + B - 1) / B;
  const int p = threadIdx.x / NR, r = threadIdx.x % NR;
  const int i0 = r % R1, i1 = r / R1;  // staged node, and (line, row) of the first pass
  const int q0 = r % O1, q1 = r / O1;  // owned node
  constexpr int NE = S::N1 * S::N1;
  __shared__ double em[NE], ek[NE];  // element mass and stiffness: one load, then the rows out of LDS
  for (int i = threadIdx.x; i < NE; i += 256) {
    em[i] = L.tables[S::T_MHAT + i];
    ek[i] = L.tables[S::T_K1S + i];
  }
  __syncthreads();
  TileRow<K, C1, T> r1, r0;
  r1.load(em, ek, K + (i1 < O1 ? i1 : 0));
  r0.load(em, ek, K + q0);
  const int step = gridDim.x * TP;
  auto load = [&](int ti, int& tile) {
    tile = p < TP && ti < L.n_tiles_sf ? L.tiles_sf[ti] : -1;
    if (tile < 0) return (T)0;
    return x[K * (B * (tile % NTd) - 1) + i0 + (int64_t)L.nn * (K * (B * (tile / NTd) - 1) + i1)];
  };
  int tile;
  T v = load(blockIdx.x * TP + p, tile);
  for (int t0 = blockIdx.x * TP; t0 < L.n_tiles_sf; t0 += step) {
    const int tc = tile;
    if (p < TP) xv[p][r] = v;
    __syncthreads();  // x staged, and the previous tiles' second pass is done
    v = load(t0 + step + p, tile);
    if (tc >= 0 && i1 < O1) {
      T am = 0, ak = 0;
#pragma unroll
      for (int t = 0; t <= 2 * K; ++t) {
        const T xt = xv[p][i0 + R1 * r1.at(t)];
        am += r1.m[t] * xt;
        ak += r1.k[t] * xt;
      }
      um[p][i0 + R1 * i1] = am;
      uk[p][i0 + R1 * i1] = ak;
    }
    __syncthreads();
    if (tc >= 0 && q1 < O1) {
      const int c0 = tc % NTd, c1 = tc / NTd;
      // the layer q = B K belongs to the next tile unless this is the last one
      if ((q0 < B * K || c0 == NTd - 1) && (q1 < B * K || c1 == NTd - 1)) {
        const int64_t node = K * B * c0 + q0 + (int64_t)L.nn * (K * B * c1 + q1);
        const T bv = b ? b[node] : (T)0;
        T ax = 0;
#pragma unroll
        for (int t = 0; t <= 2 * K; ++t) {
          const int at = r0.at(t) + R1 * q1;
          ax += r0.k[t] * um[p][at];
          ax += r0.m[t] * uk[p][at];
        }
        y[node] = b ? bv - ax : ax;
      }
    }
  }
}

// 3-D: the entries of the first two passes are read at compile-time places of
// the level tables (scalar registers), those of the last from a table of the
// owned rows in LDS, where they were summed again at every use.  Finest
// level of the 128^3 ball, Q2, FP64: 63.6 -> 48.6 us.
template <int K, typename T>
__device__ __forceinline__ void apply_sf3_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                               T* __restrict__ y) {
  using S = Shape<3, K>;
  using A = ApplyShape<3, K>;
  constexpr int B = A::B, R1 = A::R1, C1 = A::C1, O1 = A::O1;
  constexpr int NW = R1 * O1 * O1;                       // values per second-pass array
  constexpr int NXV = A::NR > 2 * NW ? A::NR : 2 * NW;
  constexpr int NU = R1 * R1 * O1;                       // values per first-pass array
  __shared__ T xv[NXV];     // x staged, then the second pass: [0, NW) and [NW, 2 NW)
  __shared__ __align__(16) T ua[2][NU];  // first pass: Mhat x and Khat x along the slowest direction
  __shared__ TileRow<K, C1, T> rows[O1];
  const double* m1 = L.tables + S::T_MHAT;
  const double* k1 = L.tables + S::T_K1S;
  {
    constexpr int NE = S::N1 * S::N1;
    double* e = reinterpret_cast<double*>(&ua[0][0]);  // free until the first tile's first pass
    static_assert(sizeof(ua) >= 2 * NE * sizeof(double), "the element matrices fit");
    for (int i = threadIdx.x; i < NE; i += 256) {
      e[i] = m1[i];
      e[NE + i] = k1[i];
    }
    __syncthreads();
    if (threadIdx.x < O1) rows[threadIdx.x].load(e, e + NE, K + threadIdx.x);
  }
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  if (b) b += blockIdx.y * L.n_nodes;
  y += blockIdx.y * L.n_nodes;
  const int NTd = (L.N + B - 1) / B;
  const int64_t nn = L.nn;
  for (int ti = blockIdx.x; ti < L.n_tiles_sf; ti += gridDim.x) {
    __syncthreads();  // tables, and the previous tile finished with the LDS buffers
    const int tile = L.tiles_sf[ti];
    const int tc[3] = {tile % NTd, (tile / NTd) % NTd, tile / (NTd * NTd)};
    const T* xt = x + K * (B * tc[0] - 1) + nn * (K * (B * tc[1] - 1) + nn * (K * (B * tc[2] - 1)));
    {
      constexpr int NIT = (A::NR + 255) / 256;
      T v[NIT];
#pragma unroll
      for (int u = 0; u < NIT; ++u) {
        const int e = threadIdx.x + 256 * u;
        v[u] = e < A::NR ? xt[e % R1 + nn * ((e / R1) % R1 + nn * (e / (R1 * R1)))] : (T)0;
      }
#pragma unroll
      for (int u = 0; u < NIT; ++u) {
        const int e = threadIdx.x + 256 * u;
        if (e < A::NR) xv[e] = v[u];
      }
    }
    __syncthreads();
    // slowest direction: every staged line, rows K .. K + O1 - 1
    constexpr int NLA = R1 * R1;
    for (int l = threadIdx.x; l < NLA; l += blockDim.x) {
      T xl[R1];
#pragma unroll
      for (int j = 0; j < R1; ++j) xl[j] = xv[l + NLA * j];
#pragma unroll
      for (int q = 0; q < O1; ++q) {
        T um = 0, uk = 0;
#pragma unroll
        for (int j = 0; j < R1; ++j) {
          if (!tile1d_nz<K, C1>(K + q, j)) continue;
          um += (T)tile1d<K, C1>(m1, K + q, j) * xl[j];
          uk += (T)tile1d<K, C1>(k1, K + q, j) * xl[j];
        }
        ua[0][l * O1 + q] = um;
        ua[1][l * O1 + q] = uk;
      }
    }
    __syncthreads();
    // direction 1 on the lines (s0, q2): Mhat Mhat x into [0, NW), Khat Mhat x + Mhat Khat x into [NW, 2 NW)
    for (int t = threadIdx.x; t < R1 * O1; t += blockDim.x) {
      const int s0 = t % R1, q2 = t / R1;
      T ul[R1], kl[R1];
#pragma unroll
      for (int j = 0; j < R1; ++j) {
        ul[j] = ua[0][(s0 + R1 * j) * O1 + q2];
        kl[j] = ua[1][(s0 + R1 * j) * O1 + q2];
      }
#pragma unroll
      for (int q = 0; q < O1; ++q) {
        T vmm = 0, vxx = 0;
#pragma unroll
        for (int j = 0; j < R1; ++j) {
          if (!tile1d_nz<K, C1>(K + q, j)) continue;
          vmm += (T)tile1d<K, C1>(m1, K + q, j) * ul[j];
          vxx += (T)tile1d<K, C1>(k1, K + q, j) * ul[j];
          vxx += (T)tile1d<K, C1>(m1, K + q, j) * kl[j];
        }
        xv[s0 + R1 * (q + O1 * q2)] = vmm;
        xv[NW + s0 + R1 * (q + O1 * q2)] = vxx;
      }
    }
    __syncthreads();
    // direction 0 at every owned node: Khat (first array) + Mhat (second array)
#pragma unroll 1
    for (int e = threadIdx.x; e < A::NO; e += blockDim.x) {
      const int q[3] = {e % O1, (e / O1) % O1, e / (O1 * O1)};
      bool own = true;
      // the layer q = B K belongs to the next tile unless this is the last one
#pragma unroll
      for (int a = 0; a < 3; ++a) own = own && (q[a] < B * K || tc[a] == NTd - 1);
      if (!own) continue;
      const int64_t node = K * B * tc[0] + q[0] + nn * (K * B * tc[1] + q[1] + nn * (K * B * tc[2] + q[2]));
      const T bv = b ? b[node] : (T)0;
      const TileRow<K, C1, T>& rw = rows[q[0]];
      const int rest = R1 * (q[1] + O1 * q[2]);
      T ax = 0;
#pragma unroll
      for (int t = 0; t <= 2 * K; ++t) {
        const int at = rw.at(t) + rest;
        ax += rw.k[t] * xv[at];
        ax += rw.m[t] * xv[NW + at];
      }
      y[node] = b ? bv - ax : ax;
    }
  }
}

template <int D, int K, typename T>
__device__ __forceinline__ void apply_sf_body(const KLevel& L, const T* __restrict__ x, const T* __restrict__ b,
                                              T* __restrict__ y) {
  if constexpr (D == 2)
    apply_sf2_body<K, T>(L, x, b, y);
  else
    apply_sf3_body<K, T>(L, x, b, y);
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_apply_sf(KLevel L, const T* __restrict__ x, const T* __restrict__ b,
                                                  T* __restrict__ y) {
  apply_sf_body<D, K, T>(L, x, b, y);
}

// argument record of k_apply_sf for grouped launches (k_grouped)
template <int D, int K, typename T>
struct ApplySfArgs {
  KLevel L;
  const T* x;
  const T* b;
  T* y;
  __device__ void run() const { apply_sf_body<D, K, T>(L, x, b, y); }
};

// Entry (r, j) of a 1-D matrix assembled on the 2k+1 closure nodes of a patch
// from the element matrix e ((k+1) x (k+1), row-major) of its two cells, the
// second cell starting at node k.  patch1d_nz tells whether some cell holds
// both nodes; with compile-time r and j both fold to constants.
template <int K>
__device__ __forceinline__ constexpr bool patch1d_nz(int r, int j) {
  return (r <= K && j <= K) || (r >= K && j >= K);
}
template <int K, typename E>
__device__ __forceinline__ E patch1d(const E* e, int r, int j) {
  E v = 0;
  if (r <= K && j <= K) v += e[r * (K + 1) + j];
  if (r >= K && j >= K) v += e[(r - K) * (K + 1) + (j - K)];
  return v;
}
// The same with a run-time row r: each term is read when its cell holds both nodes.
template <int K, typename E>
__device__ __forceinline__ E patch1d_rt(const E* e, int r, int j) {
  const E lo = (r <= K && j <= K) ? e[(r <= K ? r : 0) * (K + 1) + (j <= K ? j : 0)] : E(0);
  const E hi = (r >= K && j >= K) ? e[(r >= K ? r - K : 0) * (K + 1) + (j >= K ? j - K : 0)] : E(0);
  return lo + hi;
}

// Fused colour step over interior patches.
template <int D, int K, typename T>
__device__ __forceinline__ void interior_step_body(KLevel L, const int32_t* __restrict__ verts, int nv,
                                                   T* __restrict__ x, const T* __restrict__ b) {
  using S = Shape<D, K>;
  constexpr int NP = S::NP, NP1 = S::NP1, NC = S::NC, NC1 = S::NC1, PPB = S::PPB, N1 = S::N1;
  // the level tables this kernel reads, in the precision of the path: 1-D mass,
  // scaled 1-D stiffness, fast-diagonalisation eigenvectors and inverse sums
  __shared__ T cm1[N1 * N1], ck1[N1 * N1], cfs[NP1 * NP1], cfd[NP];
  __shared__ T xs[PPB][NC];
  __shared__ T ra[PPB][NP];
  __shared__ T rb[PPB][NP];
  __shared__ int64_t pbase[PPB];  // lattice index of each patch's closure corner (-1: no patch)
  // sum-factorisation intermediates: after the slowest direction (3-D only) and
  // after the next one, per closure line of the remaining directions
  __shared__ T su[D == 3 ? PPB : 1][D == 3 ? NC1 * NC1 : 1][NP1];
  __shared__ T sk[D == 3 ? PPB : 1][D == 3 ? NC1 * NC1 : 1][NP1];
  __shared__ T vm[PPB][NC1][D == 3 ? NP1 * NP1 : NP1];
  __shared__ T vx[PPB][NC1][D == 3 ? NP1 * NP1 : NP1];
  for (int i = threadIdx.x; i < N1 * N1; i += blockDim.x) {
    cm1[i] = (T)L.tables[S::T_MHAT + i];
    ck1[i] = (T)L.tables[S::T_K1S + i];
  }
  for (int i = threadIdx.x; i < NP1 * NP1; i += blockDim.x) cfs[i] = (T)L.tables[S::T_FDS + i];
  for (int i = threadIdx.x; i < NP; i += blockDim.x) cfd[i] = (T)L.tables[S::T_FDD + i];
  x += blockIdx.y * L.n_nodes;  // column blockIdx.y
  b += blockIdx.y * L.n_nodes;
  const int p = threadIdx.x / NP, i = threadIdx.x % NP;
  const int NV = L.N + 1;
  const int64_t nn = L.nn, nn2 = nn * nn;
  const int ngroups = (nv + PPB - 1) / PPB;
  // lattice offset of the thread's internal node from the closure corner
  int pi[3] = {0, 0, 0};
  int64_t ioff = 0;
  {
    int ri = i;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      pi[a] = ri % NP1 + 1;
      ri /= NP1;
    }
    ioff = pi[0] + nn * pi[1] + (D == 3 ? nn2 * pi[2] : 0);
  }
  for (int grp = blockIdx.x; grp < ngroups; grp += gridDim.x) {
  const int gp0 = grp * PPB;
  __syncthreads();  // previous group finished with the LDS buffers
  if (threadIdx.x < PPB) {
    int64_t base = -1;
    if (gp0 + (int)threadIdx.x < nv) {
      int vr = verts[gp0 + threadIdx.x];
      int J[3];
#pragma unroll
      for (int a = 0; a < D; ++a) {
        J[a] = K * (vr % NV) - K;
        vr /= NV;
      }
      base = lat(D, L.nn, J);
    }
    pbase[threadIdx.x] = base;
  }
  __syncthreads();
  // stage the closures of all patches of this block: all loads first, then the LDS stores
  {
    constexpr int NST = PPB * NC, NIT = (NST + 255) / 256;
    T v[NIT];
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
      const int e = threadIdx.x + 256 * u;
      v[u] = 0;
      if (e < NST) {
        const int pp = e / NC, q = e % NC;
        const int64_t base = pbase[pp];
        if (base >= 0) {
          const int q0 = q % NC1, q1 = (q / NC1) % NC1, q2 = q / (NC1 * NC1);
          v[u] = x[base + q0 + nn * q1 + (D == 3 ? nn2 * q2 : 0)];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < NIT; ++u) {
      const int e = threadIdx.x + 256 * u;
      if (e < NST) xs[e / NC][e % NC] = v[u];
    }
  }
  __syncthreads();
  const bool active = p < PPB && gp0 + p < nv;
  int64_t node = 0;
  T bnode = 0;
  if (active) {
    node = pbase[p] + ioff;
    bnode = b[node];
  }
  // residual b - A x at the internal nodes by sum factorisation on the closure.
  // An interior patch's 2^d cells are all uncut, so A restricted to it is the
  // sum over directions a of tensor products with the assembled 1-D stiffness
  // (h^(d-2) K1) along a and the assembled 1-D mass along the others (each 1-D
  // matrix on the 2k+1 closure nodes is the sum of the two cells' element
  // matrices).  Contractions run from the slowest direction to the fastest;
  // only the internal rows 1..2k-1 of each direction are formed.
  {
    const T* m1 = cm1;
    const T* k1 = ck1;
    if constexpr (D == 3) {
      // direction 2: um = Mhat_2 x, uk = Khat_2 x on every (q0, q1) line
      for (int t = threadIdx.x; t < PPB * NC1 * NC1; t += blockDim.x) {
        const int pp = t / (NC1 * NC1), l = t % (NC1 * NC1);
        if (gp0 + pp >= nv) continue;
        T xv[NC1];
#pragma unroll
        for (int j = 0; j < NC1; ++j) xv[j] = xs[pp][l + NC1 * NC1 * j];
#pragma unroll
        for (int r = 1; r <= NP1; ++r) {
          T um = 0, uk = 0;
#pragma unroll
          for (int j = 0; j < NC1; ++j) {
            if (!patch1d_nz<K>(r, j)) continue;
            um += (T)patch1d<K>(m1, r, j) * xv[j];
            uk += (T)patch1d<K>(k1, r, j) * xv[j];
          }
          su[pp][l][r - 1] = um;
          sk[pp][l][r - 1] = uk;
        }
      }
      __syncthreads();
      // direction 1: vm = Mhat_1 um, vx = Khat_1 um + Mhat_1 uk on every (q0, r2) line
      for (int t = threadIdx.x; t < PPB * NC1 * NP1; t += blockDim.x) {
        const int pp = t / (NC1 * NP1), q0 = (t / NP1) % NC1, r2 = t % NP1;
        if (gp0 + pp >= nv) continue;
        T uv[NC1], kv[NC1];
#pragma unroll
        for (int j = 0; j < NC1; ++j) {
          uv[j] = su[pp][q0 + NC1 * j][r2];
          kv[j] = sk[pp][q0 + NC1 * j][r2];
        }
#pragma unroll
        for (int r = 1; r <= NP1; ++r) {
          T vmv = 0, vxv = 0;
#pragma unroll
          for (int j = 0; j < NC1; ++j) {
            if (!patch1d_nz<K>(r, j)) continue;
            vmv += (T)patch1d<K>(m1, r, j) * uv[j];
            vxv += (T)patch1d<K>(k1, r, j) * uv[j];
            vxv += (T)patch1d<K>(m1, r, j) * kv[j];
          }
          vm[pp][q0][(r - 1) + NP1 * r2] = vmv;
          vx[pp][q0][(r - 1) + NP1 * r2] = vxv;
        }
      }
    } else {
      // direction 1: um = Mhat_1 x, uk = Khat_1 x on every q0 line
      for (int t = threadIdx.x; t < PPB * NC1; t += blockDim.x) {
        const int pp = t / NC1, q0 = t % NC1;
        if (gp0 + pp >= nv) continue;
        T xv[NC1];
#pragma unroll
        for (int j = 0; j < NC1; ++j) xv[j] = xs[pp][q0 + NC1 * j];
#pragma unroll
        for (int r = 1; r <= NP1; ++r) {
          T um = 0, uk = 0;
#pragma unroll
          for (int j = 0; j < NC1; ++j) {
            if (!patch1d_nz<K>(r, j)) continue;
            um += (T)patch1d<K>(m1, r, j) * xv[j];
            uk += (T)patch1d<K>(k1, r, j) * xv[j];
          }
          vm[pp][q0][r - 1] = um;
          vx[pp][q0][r - 1] = uk;
        }
      }
    }
    __syncthreads();
    // direction 0, at the thread's own node: (A x)(node) = Khat_0 vm + Mhat_0 vx
    if (active) {
      const int rw = (pi[1] - 1) + (D == 3 ? NP1 * (pi[2] - 1) : 0);
      T ax = 0;
#pragma unroll
      for (int j = 0; j < NC1; ++j) {
        if (j < pi[0] - K || j > pi[0] + K) continue;
        ax += (T)patch1d_rt<K>(k1, pi[0], j) * vm[p][j][rw];
        ax += (T)patch1d_rt<K>(m1, pi[0], j) * vx[p][j][rw];
      }
      ra[p][i] = bnode - ax;
    }
  }
  __syncthreads();
  // fast diagonalisation: apply S^T along every direction, scale, apply S
  const T* fs = cfs;
  T* src = &ra[0][0];
  T* dst = &rb[0][0];
  for (int stage = 0; stage < 2 * D; ++stage) {
    const int a = stage % D;
    const bool transpose = stage < D;
    if (active) {
      int ia[3];
      int rr = i;
#pragma unroll
      for (int j = 0; j < D; ++j) { ia[j] = rr % NP1; rr /= NP1; }
      int strideA = 1;
      for (int j = 0; j < a; ++j) strideA *= NP1;
      const int baseIdx = i - ia[a] * strideA;
      T s = 0;
#pragma unroll
      for (int q = 0; q < NP1; ++q) {
        const T m = transpose ? fs[q * NP1 + ia[a]] : fs[ia[a] * NP1 + q];
        s += m * src[p * NP + baseIdx + q * strideA];
      }
      if (stage == D - 1) s *= cfd[i];
      dst[p * NP + i] = s;
    }
    __syncthreads();
    T* t = src;
    src = dst;
    dst = t;
  }
  // x at the node is still in the staged closure: no second read of HBM
  if (active) x[node] = xs[p][pi[0] + NC1 * pi[1] + (D == 3 ? NC1 * NC1 * pi[2] : 0)] + src[p * NP + i];
  }
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_interior_step(KLevel L, const int32_t* __restrict__ verts, int nv,
                                                       T* __restrict__ x, const T* __restrict__ b) {
  interior_step_body<D, K, T>(L, verts, nv, x, b);
}

// argument record of k_interior_step for grouped launches (k_grouped)
template <int D, int K, typename T>
struct InteriorStepArgs {
  KLevel L;
  const int32_t* verts;
  int nv;
  T* x;
  const T* b;
  __device__ void run() const { interior_step_body<D, K, T>(L, verts, nv, x, b); }
};

// The value that the DPP pattern CTRL brings to this lane: 0x55 q the lane q of
// its quad, 0x120 + n the lane n below it in its row of 16 (cyclic).
template <int CTRL>
__device__ __forceinline__ float lane_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_dpp(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}

// Threads of a large cut-patch launch: a thread per internal node at least.
template <int D, int K>
struct CutThreads {
  static constexpr int v = Shape<D, K>::NP <= 64 ? 64 : 128;
};

// Sizes of the one-column cut step (one block per patch).
template <int D, int K, typename T, int TH_>
struct CutShape {
  using S = Shape<D, K>;
  static constexpr int TH = TH_, NWV = TH / 64;
  static constexpr int COPY = 8;                          // copy-job items per thread of a copy block
  static constexpr int NTC = 1 << (D - 1);                // tangential cells of a direction
  static constexpr int NPAIR = Pow<2 * K, D>::v;          // (node, cell) pairs
  static constexpr int SLABS = S::N1;                     // slabs of a cell row along the slowest direction
  static constexpr int SL = S::NL / SLABS;                // entries per slab
  static constexpr bool SPLIT = TH > CutThreads<D, K>::v;      // a lane per slab instead of one per pair
  static constexpr int PS = SPLIT ? SLABS : 1;            // lanes per pair
  static constexpr int EPT = S::NL / PS;                  // row entries per task
  static constexpr int NRND = (NPAIR * PS + TH - 1) / TH; // rounds of row tasks
  static constexpr bool PRE = NRND * EPT * (int)sizeof(T) <= 40 * 4;  // row loads issued before x is staged (more cost a wave per SIMD)
  static constexpr int GS = SPLIT && S::NP > 1 ? 4 : 1;   // lanes per row of the local solve
  static constexpr int NACC = S::NP <= 32 ? 4 : 8;        // partial sums of a row of the local solve
  static constexpr int JP = (S::NP + NACC - 1) / NACC * NACC / GS;  // entries of a row per lane
  static constexpr int RSN = (S::NP + 31) / 32 * 32;      // residual rows, padded with zeros
  static constexpr int HT = Pow<2 * K, D - 1>::v;         // (tangential cell, internal node) choices
  static constexpr int HS = S::NP1 * HT;                  // ghost rows per direction
  static constexpr int GR = D == 3 ? (3 + NWV - 1) / NWV : 1;  // directions per wave
  static_assert(S::NP * GS <= TH, "a cut-patch block needs the lanes of every row of the local solve");
};

template <int D, int K, typename T, int TH>
struct CutSmem {
  using S = Shape<D, K>;
  using C = CutShape<D, K, T, TH>;
  T xs[S::NC];                    // x on the patch closure
  T parts[C::NPAIR * C::PS];      // cell rows
  T H[D][C::HS];                  // ghost rows
  T rs[C::RSN];                   // residual rows
  T jg[2 * K * S::NC1];           // jump weights j_m, gc_m j_m
  int16_t pos[S::NP];             // closure index of every row
};

// Cut patches, phase 1: residual on the internal nodes and dense local solve
// d_j = A_j^{-1} r_j (GEMV with the symmetric inverse), one block per patch
// and one column per blockIdx.y (columns are n_nodes apart in x, b and xb and
// n_nodes of the colour apart in dbuf).  With xb == nullptr d_j goes to dbuf;
// otherwise xb = x + d_j on the patch's internal DoFs (same-coloured patches
// share none), and the first cj.nblk blocks copy the nodes of the copy job
// from x to xb instead of solving a patch.
//
// One patch is a chain of short phases, so what counts is its length and the
// instructions in it:
//   - the patch's record (offsets, vertex, flags, cut ids) is scalar loads of
//     one round trip; x, b, the node layers beyond the closure that ghost faces
//     reach and (where they fit in registers) the cell rows are requested
//     before anything is waited for;
//   - cell rows: along each direction an internal node at patch coordinate p in
//     1..2k-1 lies in cell layer 0 (p <= k) and/or 1 (p >= k), which gives 2k
//     (p, layer) choices per direction and (2k)^d (node, cell) pairs, a lane each;
//   - ghost faces by sum factorisation as in k_cut_cols: a wave takes a
//     direction, 16 lanes a tangential cell, a lane one node line;
//   - every node sums its pairs and ghost rows in a fixed order with all LDS
//     reads in flight, and a lane takes a row of the local solve.
// Launches that leave CUs idle (coarse levels) take more threads: a lane per
// slab of a pair's cell row and 4 lanes per row of the local solve, whose
// entries are requested at the start.  Every sum keeps its order, so results
// do not depend on the choice.  128^3 ball, Q2, finest step (11,866 patches): FP64
// 58.5 -> 48.1 us, FP32 38.3 -> 28.7 us; 740 patches FP64 10.7 -> 8.8 us; union of 8
// spheres, Q3, 40 patches 25.0 -> 13.9 us.  The finest step is bound by its reads
// (cut-cell rows in 216-byte pieces and inverses, 180 MB), a small one by four
// dependent round trips to memory and the launch.
template <int D, int K, typename T, int TH>
__global__ __launch_bounds__(TH) void k_cut_solve(KLevel L, CutGroupDev G, const T* __restrict__ x,
                                                  const T* __restrict__ b, T* __restrict__ dbuf, T* __restrict__ xb,
                                                  CopyJob cj) {
  using S = Shape<D, K>;
  using C = CutShape<D, K, T, TH>;
  constexpr int N1 = S::N1, NL = S::NL, NC = S::NC, W1 = S::NC1, NP = S::NP, NP1 = S::NP1, NCELL = 1 << D;
  constexpr int NTC = C::NTC;
  __shared__ CutSmem<D, K, T, TH> sm;
  const int tid = threadIdx.x;
  x += blockIdx.y * L.n_nodes;
  b += blockIdx.y * L.n_nodes;
  dbuf += blockIdx.y * G.n_nodes;
  if (xb) xb += blockIdx.y * L.n_nodes;
  if ((int)blockIdx.x < cj.nblk) {
    // copy block: C::COPY items per thread, index loads first, then the values
    int32_t nd[C::COPY];
#pragma unroll
    for (int u = 0; u < C::COPY; ++u) {
      const int64_t i = ((int64_t)blockIdx.x * C::COPY + u) * TH + tid;
      nd[u] = (i < cj.n && !(cj.skip[i] & cj.mask)) ? cj.nodes[i] : -1;
    }
    T v[C::COPY];
#pragma unroll
    for (int u = 0; u < C::COPY; ++u) v[u] = nd[u] >= 0 ? x[nd[u]] : (T)0;
#pragma unroll
    for (int u = 0; u < C::COPY; ++u)
      if (nd[u] >= 0) xb[nd[u]] = v[u];
    return;
  }
  const int gp = xcd_block(blockIdx.x - cj.nblk, gridDim.x - cj.nblk);
  // the patch's record
  const int off = G.off[gp], nj = G.off[gp + 1] - off;
  const int64_t ioff = G.inv_off[gp];
  const uint64_t vp = G.vpack[gp];
  // flags of the 2^d cells, 4 cells a word
  const uint64_t fga = reinterpret_cast<const uint64_t*>(G.cell_fg)[(int64_t)gp * (NCELL / 4)];
  const uint64_t fgb = reinterpret_cast<const uint64_t*>(G.cell_fg)[(int64_t)gp * (NCELL / 4) + NCELL / 4 - 1];
  auto cell_fg = [fga, fgb](int o) { return static_cast<int>((o >= 4 ? fgb : fga) >> (16 * (o & 3))) & 0xffff; };
  const int nn = L.nn, nn2 = nn * nn;
  int V[3] = {1, 1, 1};
  bool inside = true;  // the closure lies in the lattice
#pragma unroll
  for (int a = 0; a < D; ++a) {
    V[a] = static_cast<int>(vp >> (21 * a)) & 0x1fffff;
    inside = inside && V[a] >= 1 && V[a] < L.N;
  }
  const int cbase = K * (V[0] - 1) + nn * (K * (V[1] - 1)) + (D == 3 ? nn2 * (K * (V[2] - 1)) : 0);
  x += cbase;  // from here on relative to the closure's corner
  b += cbase;
  // lattice offset of a closure node
  auto loff = [&](int q) {
    return q % W1 + nn * ((q / W1) % W1) + (D == 3 ? nn2 * (q / (W1 * W1)) : 0);
  };
  // closure
  constexpr int NIT = (NC + TH - 1) / TH;
  T v[NIT];
#pragma unroll
  for (int u = 0; u < NIT; ++u) {
    const int e = tid + TH * u < NC ? tid + TH * u : NC - 1;
    if (inside) {
      v[u] = x[loff(e)];
    } else {  // nodes beyond the lattice count as zero
      int r = e;
      bool in = true;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const int I = K * (V[a] - 1) + r % W1;
        r /= W1;
        in = in && I >= 0 && I < nn;
      }
      v[u] = in ? x[loff(e)] : (T)0;
    }
  }
  const int bsafe = K + nn * K + (D == 3 ? nn2 * K : 0);  // the patch's vertex node
  // ghost faces: a wave per direction in 3-D (lane: tangential cell, b1, b0), all of them in the first wave in 2-D
  const int lane = tid % 64, wave = C::NWV == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / 64);
  const int b0 = lane % 4, b1 = D == 3 ? (lane / 4) % 4 : 0;
  const int t0 = D == 3 ? (lane / 16) & 1 : (lane / 4) & 1, t1 = D == 3 ? lane / 32 : 0;
  T lo[C::GR][K], hi[C::GR][K];
  bool gf[C::GR][3];
#pragma unroll
  for (int g = 0; g < C::GR; ++g) {
    const int dir = D == 3 ? wave + g * C::NWV : (lane / 8) & 1;
    const bool mine = D == 3 ? dir < 3 : tid < 16;
    const int d0 = dir == 0 ? 1 : 0, d1 = dir == 2 ? 1 : 2;  // tangential directions (d1: 3-D only)
    const int o = (t0 << d0) | (D == 3 ? t1 << d1 : 0);
    const int glo = cell_fg(o) >> 8, ghi = cell_fg((o | 1 << dir) & (NCELL - 1)) >> 8;
    const bool on = mine && b0 < N1 && b1 < N1;
    gf[g][0] = on && (glo & (1 << (2 * dir)));
    gf[g][1] = on && (glo & (2 << (2 * dir)));
    gf[g][2] = on && (ghi & (2 << (2 * dir)));
    const int gd = dir == 0 ? 1 : dir == 1 ? nn : nn2, g0 = d0 == 0 ? 1 : nn, g1 = D == 3 ? (d1 == 1 ? nn : nn2) : 0;
    const T* xg = x + ((K * t0 + b0) * g0 + (K * t1 + b1) * g1);
    // patch-local residual: x beyond the closure counts as zero
    const bool flo = gf[g][0] && !L.ghost_local, fhi = gf[g][2] && !L.ghost_local;
#pragma unroll
    for (int q = 0; q < K; ++q) {
      // a lane without the face reads a node that is in the lattice anyway
      const T l = *(flo ? xg + (q - K) * gd : b + bsafe), h = *(fhi ? xg + (2 * K + 1 + q) * gd : b + bsafe);
      lo[g][q] = flo ? l : (T)0;
      hi[g][q] = fhi ? h : (T)0;
    }
  }
  // entries of the 1-D mass for the tangential directions (see k_cut_cols)
  const T* tab = L.tables_t<T>();
  constexpr int NJG = 2 * K * W1;  // jump weights, plain and times the ghost coefficients
  const T jgv = tab[S::T_JM + (tid < NJG ? tid : 0)];
  T w0[4], w1[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int q1 = (b1 - q) & 3, r0 = b0 < N1 ? b0 : 0, r1 = b1 < N1 ? b1 : 0;
    const T e0 = tab[S::T_MHAT + r0 * N1 + (q < N1 ? q : 0)], e1 = tab[S::T_MHAT + r1 * N1 + (q1 < N1 ? q1 : 0)];
    w0[q] = b0 < N1 && q < N1 ? e0 : (T)0;
    w1[q] = b1 < N1 && q1 < N1 ? e1 : (T)0;
  }
  // row tasks: pair t / PS, slabs from (t % PS) SLABS / PS on
  auto pair_of = [&](int pt, int& o, int& iloc) {
    o = 0;
    iloc = 0;
    int r = pt, st = 1;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const int j = r % (2 * K);
      r /= 2 * K;
      o |= (j >= K ? 1 : 0) << a;
      iloc += (j < K ? j + 1 : j - K) * st;
      st *= N1;
    }
  };
  auto row_ptr = [&](int t) {
    int o, iloc;
    pair_of(t / C::PS, o, iloc);
    const int cut = G.cell_cut[(int64_t)gp * NCELL + o];
    const T* m = cell_fg(o) & 2 ? L.cut_mats_t<T>() + (int64_t)cut * NL * NL : L.kcell_t<T>() + S::T_KCELL;
    return m + iloc * NL + (C::PS > 1 ? (t % C::PS) * C::SL : 0);
  };
  T row[C::PRE ? C::NRND : 1][C::EPT];
  if constexpr (C::PRE) {
#pragma unroll
    for (int u = 0; u < C::NRND; ++u) {
      const int t = tid + TH * u;
      if (t < C::NPAIR * C::PS) {
        const T* m = row_ptr(t);
#pragma unroll
        for (int e = 0; e < C::EPT; ++e) row[u][e] = m[e];
      }
    }
  }
  // the thread's node: closure index (from the record unless the patch is full), b
  int pos = 0;
  T bval = 0;
  if (tid < nj) {
    if (nj == NP)  // uniform
      pos = tid % NP1 + 1 + W1 * ((tid / NP1) % NP1 + 1) + (D == 3 ? W1 * W1 * (tid / (NP1 * NP1) + 1) : 0);
    else
      pos = G.pos[off + tid];
    bval = b[loff(pos)];
    sm.pos[tid] = static_cast<int16_t>(pos);
  }
  // the lane's part of its row of the local solve
  const int gi = tid / C::GS, gu = tid % C::GS;
  const T* inv = G.inv_t<T>() + ioff + (gi < nj ? gi : 0);
  T iv[C::SPLIT ? C::JP : 1];
  if constexpr (C::SPLIT) {
#pragma unroll
    for (int e = 0; e < C::JP; ++e) {
      const int j = gu + C::GS * e;
      iv[e] = inv[(int64_t)(j < nj ? j : nj - 1) * nj];
    }
  }
#pragma unroll
  for (int u = 0; u < NIT; ++u) {
    const int e = tid + TH * u;
    if (e < NC) sm.xs[e] = v[u];
  }
  if (tid < NJG) sm.jg[tid] = jgv;
  __syncthreads();
  // ghost rows
  uint32_t gmask = 0;  // bit dir 2^(d-1) + t: that (direction, tangential cell) has a face
#pragma unroll
  for (int dt = 0; dt < D * NTC; ++dt) {
    const int dir = dt / NTC, t = dt % NTC;
    const int d0 = dir == 0 ? 1 : 0, d1 = dir == 2 ? 1 : 2;
    const int o = ((t & 1) << d0) | (D == 3 ? (t >> 1) << d1 : 0);
    if (((cell_fg(o) >> 8) & (3 << (2 * dir))) || ((cell_fg(o | 1 << dir) >> 8) & (2 << (2 * dir)))) gmask |= 1u << dt;
  }
#pragma unroll
  for (int g = 0; g < C::GR; ++g) {
    const int dir = D == 3 ? wave + g * C::NWV : (lane / 8) & 1;
    if (D == 3 ? (dir >= 3 || !((gmask >> (4 * dir)) & 15)) : (wave > 0 || !gmask)) continue;  // wave-uniform
    const int d0 = dir == 0 ? 1 : 0, d1 = dir == 2 ? 1 : 2;
    const int sd = dir == 0 ? 1 : dir == 1 ? W1 : W1 * W1;
    const int s0 = d0 == 0 ? 1 : W1, s1 = D == 3 ? (d1 == 1 ? W1 : W1 * W1) : 0;
    T y[NP1];
#pragma unroll
    for (int p = 0; p < NP1; ++p) y[p] = 0;
    const T* xl = sm.xs + (K * t0 + (b0 < N1 ? b0 : 0)) * s0 + (K * t1 + (b1 < N1 ? b1 : 0)) * s1;
    T xv[2 * K + 1];
#pragma unroll
    for (int q = 0; q <= 2 * K; ++q) xv[q] = xl[q * sd];
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const T* jm = sm.jg + m * W1;
      const T* gj = sm.jg + (K + m) * W1;
      T J0 = 0, J1 = 0, J2 = 0;
#pragma unroll
      for (int q = 0; q <= 2 * K; ++q) {
        J0 += jm[q] * (q < K ? lo[g][q < K ? q : 0] : xv[q < K ? 0 : q - K]);
        J1 += jm[q] * xv[q];
        J2 += jm[q] * (q <= K ? xv[q <= K ? q + K : 0] : hi[g][q <= K ? 0 : q - K - 1]);
      }
      J0 = gf[g][0] ? J0 : (T)0;
      J1 = gf[g][1] ? J1 : (T)0;
      J2 = gf[g][2] ? J2 : (T)0;
#pragma unroll
      for (int p = 1; p < 2 * K; ++p) {
        y[p - 1] += gj[p] * J1;
        if (p <= K) y[p - 1] += gj[p <= K ? p + K : 0] * J0;
        if (p >= K) y[p - 1] += gj[p >= K ? p - K : 0] * J2;
      }
    }
    const int i0 = b0 - 1 + t0, i1 = b1 - 1 + t1;  // internal rows 0..k-1 of the tangential cell
    const bool put = (D == 3 || tid < 16) && b0 < N1 && b1 < N1 && i0 >= 0 && i0 < K && (D == 2 || (i1 >= 0 && i1 < K));
    T* h = sm.H[dir] + (D == 3 ? (t0 * K + i0) * 2 * K + t1 * K + i1 : t0 * K + i0);
#pragma unroll
    for (int p = 0; p < NP1; ++p) {
      T s = w0[0] * lane_dpp<0x00>(y[p]) + w0[1] * lane_dpp<0x55>(y[p]);
      if (N1 > 2) s += w0[2] * lane_dpp<0xaa>(y[p]);
      if (N1 > 3) s += w0[3] * lane_dpp<0xff>(y[p]);
      if (D == 3)
        s = (w1[0] * s + w1[1] * lane_dpp<0x124>(s)) + (w1[2] * lane_dpp<0x128>(s) + w1[3] * lane_dpp<0x12c>(s));
      if (put) h[p * C::HT] = s;
    }
  }
  // cell rows: one partial sum per slab, the slabs in order
#pragma unroll
  for (int u = 0; u < C::NRND; ++u) {
    const int t = tid + TH * u;
    if (t >= C::NPAIR * C::PS) break;
    int o, iloc;
    pair_of(t / C::PS, o, iloc);
    const T* xc = sm.xs + K * (o & 1) + W1 * K * ((o >> 1) & 1) + (D == 3 ? W1 * W1 * K * ((o >> 2) & 1) : 0);
    if (C::PS > 1) xc += (t % C::PS) * (D == 3 ? W1 * W1 : W1);
    const T* m = C::PRE ? nullptr : row_ptr(t);
    T part = 0;
#pragma unroll
    for (int z = 0; z < C::SLABS / C::PS; ++z) {
      T r[C::SL];
#pragma unroll
      for (int e = 0; e < C::SL; ++e) r[e] = C::PRE ? row[C::PRE ? u : 0][C::PRE ? z * C::SL + e : 0] : m[z * C::SL + e];
      T s = 0;
#pragma unroll
      for (int e = 0; e < C::SL; ++e) s += r[e] * xc[e % N1 + W1 * (e / N1) + z * (D == 3 ? W1 * W1 : W1)];
      part = z == 0 ? s : part + s;
    }
    sm.parts[t] = cell_fg(o) & 1 ? part : (T)0;
  }
  __syncthreads();
  // residual rows
  if (tid < nj) {
    const int pi[3] = {pos % W1, (pos / W1) % W1, D == 3 ? pos / (W1 * W1) : 0};
    // the node's pairs: per direction index j = p - 1 (layer 0, p <= k) and
    // j = p (layer 1, p >= k); every choice is read, so that the reads are in
    // flight together, and those that the node does not have are dropped
    int jlo[3] = {0, 0, 0}, jn[3] = {1, 1, 1};
#pragma unroll
    for (int a = 0; a < D; ++a) {
      jlo[a] = pi[a] <= K ? pi[a] - 1 : pi[a];
      jn[a] = pi[a] == K ? 2 : 1;
    }
    T ax = 0;
#pragma unroll
    for (int e = 0; e < NCELL; ++e) {
      int t = 0, st = 1;
      bool has = true;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const int ea = (e >> a) & 1;
        has = has && ea < jn[a];
        t += (jlo[a] + (ea & (jn[a] - 1))) * st;
        st *= 2 * K;
      }
      T p = sm.parts[t * C::PS];
#pragma unroll
      for (int z = 1; z < C::PS; ++z) p += sm.parts[t * C::PS + z];
      ax += has ? p : (T)0;
    }
#pragma unroll
    for (int dir = 0; dir < D; ++dir) {
      constexpr int D1[3] = {2, 2, 1};
      const int d0 = dir == 0 ? 1 : 0, d1 = D1[dir];
#pragma unroll
      for (int e = 0; e < NTC; ++e) {
        const int e0 = e & 1, e1 = e >> 1;
        const int j0 = jlo[d0] + (e0 & (jn[d0] - 1)), j1 = D == 3 ? jlo[d1] + (e1 & (jn[d1] - 1)) : 0;
        const int t = (j0 >= K ? 1 : 0) | (j1 >= K ? 2 : 0);
        const bool has = e0 < jn[d0] && (D == 2 || e1 < jn[d1]) && ((gmask >> (dir * NTC + t)) & 1);
        const T h = sm.H[dir][(pi[dir] - 1) * C::HT + (D == 3 ? j0 * 2 * K + j1 : j0)];
        ax += has ? h : (T)0;
      }
    }
    sm.rs[tid] = bval - ax;
  }
  for (int e = nj + tid; e < C::RSN; e += TH) sm.rs[e] = 0;
  __syncthreads();
  // d = A_j^{-1} r: row i as column i (the inverse is symmetric), so that
  // neighbouring rows read neighbouring entries; entry j goes to partial sum
  // j % NACC.  Loads past the last entry re-read it (their residual is zero).
  if (gi >= nj) return;
  T dv;
  T acc[C::NACC / C::GS];
#pragma unroll
  for (int u = 0; u < C::NACC / C::GS; ++u) acc[u] = 0;
  if constexpr (C::SPLIT) {
#pragma unroll
    for (int e = 0; e < C::JP; ++e) acc[e % (C::NACC / C::GS)] += iv[e] * sm.rs[gu + C::GS * e];
  } else {
    constexpr int NB = NP <= 32 ? C::JP : (sizeof(T) == 4 ? 32 : 16);  // independent loads in flight
    for (int j = 0; j < (NP <= 32 ? 1 : nj); j += NB) {
      T r[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) r[u] = inv[(int64_t)(j + u < nj ? j + u : nj - 1) * nj];
#pragma unroll
      for (int u = 0; u < NB; ++u) acc[u % C::NACC] += r[u] * sm.rs[j + u];
    }
  }
  if constexpr (C::GS == 4) {
    // lane u of the quad holds the partial sums u and (for 8) u + 4
    T s[2];
#pragma unroll
    for (int u = 0; u < C::NACC / 4; ++u)
      s[u] = (lane_dpp<0x00>(acc[u]) + lane_dpp<0x55>(acc[u])) + (lane_dpp<0xaa>(acc[u]) + lane_dpp<0xff>(acc[u]));
    dv = C::NACC == 8 ? s[0] + s[C::NACC / 4 - 1] : s[0];
  } else if constexpr (C::NACC == 8) {
    dv = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
  } else {
    dv = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
  if (gu != 0) return;
  const int ps = sm.pos[gi];
  if (xb)
    xb[cbase + loff(ps)] = sm.xs[ps] + dv;
  else
    dbuf[off + gi] = dv;
}

// Cut colour step for up to kMaxCols columns, one block per patch: residual
// rows of all columns, dense local solve, and the update (two-buffer form, see
// k_cut_solve) in one launch.
//   1. x on the patch closure is staged in LDS, column by column.
//   2. Cell rows on the matrix cores: every active cell of the patch
//      multiplies the k^d rows of its matrix (cut-cell matrix or uncut
//      stiffness) that belong to internal nodes with the cell's part of the
//      closure, 16 rows x 4 nodes x (8 of 16) columns an instruction, so a
//      matrix entry is loaded once for all columns and x comes out of LDS once
//      per 16 rows.  A wave takes whole cells; its matrix loads do not depend
//      on x and are issued before the closure has arrived.
//   3. Ghost faces by sum factorisation: for a direction, the faces on the
//      planes 0, 1, 2 of one tangential cell act on the node lines along the
//      direction with the rank-k matrix sum_m gc_m j_m j_m^T (j_m: the jump of
//      the m-th derivative as weights of the 2k+1 nodes), then with the 1-D
//      mass in each tangential direction.  A wave takes one (direction,
//      tangential cell), so whether a plane has a face is a scalar branch; a
//      lane takes one node line of one column, and the tangential contractions
//      exchange values between the 4 lanes of a quad and the 4 quads of a row
//      of 16 lanes.  Faces on the patch boundary read their k node layers
//      beyond the closure from memory.
//   4. A thread sums, per (node, column), the cell rows and the ghost rows in
//      a fixed order.
//   5. d = A_j^{-1} r on the matrix cores; FP32 reads the inverse in tile
//      order (CutGroupDev::inv_tiles), FP64 the symmetric dense inverse.
// A column's arithmetic does not depend on the other columns or their number.
// The former form (a jump pre-pass over all faces of the level, one thread per
// cell row with 8 accumulators, a separate update) was bound by one patch's
// serial chain and by LDS reads (one 8-column row of x per matrix entry).
// Union of 8 spheres, Q3, 64^3 cells, 8 columns, FP32: finest step with jumps
// and update 317 -> 144 us, V-cycle 23.0 -> 9.3 ms.  That step is bound by what it
// moves: 508 MB (287 MB with every closure, cell and inverse read once) at 3.5
// TB/s, three quarters of a copy's rate, with 4 blocks a CU (LDS) to keep loads in
// flight; texture units 55%, LDS 19%, matrix cores 11% busy.  FP64: 896 MB (570) in
// 256 us, also 3.5 TB/s, at 2 blocks a CU.  A small launch is bound by one patch's
// chain of loads, LDS exchanges and dependent products.
template <int D, int K, typename T, int NW_>
struct ColsShape {
  using S = Shape<D, K>;
  static constexpr int NW = NW_;                         // waves per block
  static constexpr int TH = 64 * NW;
  static constexpr int NCELL = 1 << D;
  static constexpr int KD = Pow<K, D>::v;                // internal rows per cell
  static constexpr int NRT = (KD + 15) / 16;             // row tiles per cell
  static constexpr bool VEC = S::NL % 16 == 0;           // cell rows in runs of 4 entries per lane
  static constexpr int NKS = (S::NL + 3) / 4;            // matrix-core steps per row tile
  static constexpr int NPAIR = Pow<2 * K, D>::v | 1;     // (node, cell) pairs, odd column stride
  static constexpr int NPP = (S::NP + 15) / 16 * 16;     // residual rows, padded
  static constexpr int HT = Pow<2 * K, D - 1>::v;        // (tangential cell, internal node) choices
  static constexpr int HS = (S::NP1 * HT) | 1;           // ghost rows per direction and column, odd stride
  static constexpr int LPC = D == 3 ? 16 : 4;            // lanes of one column in a ghost task
  static constexpr int CPW = 64 / LPC;                   // columns of one ghost task
  static constexpr int NGT = (kMaxCols + CPW - 1) / CPW; // ghost tasks per (direction, tangential cell)
  static constexpr int NPT = S::NP <= 1 ? 1 : S::NP <= 4 ? 4 : S::NP <= 16 ? 16 : S::NP <= 32 ? 32 : S::NP <= 64 ? 64 : 128;
  static constexpr int CPI = TH / NPT;                   // columns per round of (node, column) tasks
  static constexpr int NRD = (kMaxCols + CPI - 1) / CPI; // rounds
  static constexpr int COPY = 8;                         // copy-job items per thread of a copy block
  // column of round u of a task with first column tc, kept in range where the task has none
  static __device__ __forceinline__ int col(int tc, int u) {
    const int c = tc + CPI * u;
    return CPI * NRD > kMaxCols && c >= kMaxCols ? kMaxCols - 1 : c;
  }
};

template <int D, int K, typename T, int NW>
struct ColsSmem {
  using S = Shape<D, K>;
  using C = ColsShape<D, K, T, NW>;
  T xs[kMaxCols][S::NC];             // x on the closure (the node count is odd)
  T parts[kMaxCols][C::NPAIR];       // cell rows
  T H[D][kMaxCols][C::HS];           // ghost rows
  T rs[kMaxCols][C::NPP + 1];        // residual rows
  T jm[K][2 * K + 1], gj[K][2 * K + 1], mh[S::N1][S::N1];  // jump weights j_m, gc_m j_m, 1-D mass
  int32_t node[C::NPP];              // lattice node and closure index of every row
  int16_t pos[C::NPP];
};

template <int D, int K, typename T, int NW>
__device__ __forceinline__ void cut_cols_body(const KLevel& L, const CutGroupDev& G, const T* __restrict__ x,
                                              const T* __restrict__ b, T* __restrict__ dbuf, T* __restrict__ xb,
                                              const CopyJob& cj, int ncol) {
  // column group blockIdx.y of at most kMaxCols columns
  x += (int64_t)blockIdx.y * kMaxCols * L.n_nodes;
  b += (int64_t)blockIdx.y * kMaxCols * L.n_nodes;
  if (xb) xb += (int64_t)blockIdx.y * kMaxCols * L.n_nodes;
  if (dbuf) dbuf += (int64_t)blockIdx.y * kMaxCols * G.n_nodes;
  ncol = ncol - (int)blockIdx.y * kMaxCols < kMaxCols ? ncol - (int)blockIdx.y * kMaxCols : kMaxCols;
  using S = Shape<D, K>;
  using C = ColsShape<D, K, T, NW>;
  using Acc = typename Mfma<T>::Acc;
  constexpr int N1 = S::N1, NL = S::NL, NC = S::NC, W1 = S::NC1, NP1 = S::NP1, KD = C::KD, NKS = C::NKS;
  constexpr int NCELL = C::NCELL, TH = C::TH;
  __shared__ ColsSmem<D, K, T, NW> sm;
  const int tid = threadIdx.x;
  if ((int)blockIdx.x < cj.nblk) {
    // copy block (see k_cut_solve): the items once for all columns
#pragma unroll
    for (int u = 0; u < C::COPY; ++u) {
      const int64_t i = ((int64_t)blockIdx.x * C::COPY + u) * TH + tid;
      if (i >= cj.n || (cj.skip[i] & cj.mask)) continue;
      const int64_t nd = cj.nodes[i];
      for (int c = 0; c < ncol; ++c) xb[c * L.n_nodes + nd] = x[c * L.n_nodes + nd];
    }
    return;
  }
  if ((int)blockIdx.x - cj.nblk >= G.n_patch) return;  // grouped launches: a block beyond this problem's work
  const int gp = xcd_block(blockIdx.x - cj.nblk, G.n_patch);
  const int lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int lr = lane % 16, lk = lane / 16;
  const int off = G.off[gp], nj = G.off[gp + 1] - off;
  const int64_t nn = L.nn, nn2 = nn * nn;
  int V[3] = {0, 0, 0};
  {
    const uint64_t vp = G.vpack[gp];
#pragma unroll
    for (int a = 0; a < D; ++a) V[a] = static_cast<int>(vp >> (21 * a)) & 0x1fffff;
  }
  const int64_t cbase = K * (V[0] - 1) + nn * (K * (V[1] - 1)) + (D == 3 ? nn2 * (K * (V[2] - 1)) : 0);
  // local index of row r (of the k^d internal rows of cell o), and its pair index
  auto row_of = [&](int o, int r, int& iloc, int& pair) {
    iloc = 0;
    pair = 0;
    int s1 = 1, s2 = 1;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const int i = r % K, layer = (o >> a) & 1;
      r /= K;
      iloc += (i + 1 - layer) * s1;
      pair += (layer * K + i) * s2;
      s1 *= N1;
      s2 *= 2 * K;
    }
  };
  // matrix entries of the wave's cell o for one row tile: VEC: lane (lr, lk)
  // holds nodes 16 kk + 4 lk + s (kk, s < 4) of row lr, used in step 4 kk + s;
  // else node 4 ks + lk in step ks
  auto load_rows = [&](int rt, uint16_t fg, int cut, T* a, int o) {
    const int r = rt * 16 + lr;
    int iloc, pair;
    row_of(o, r < KD ? r : KD - 1, iloc, pair);
    const T* m = (fg & 2) ? L.cut_mats_t<T>() + (int64_t)cut * NL * NL : L.kcell_t<T>() + S::T_KCELL;
    m += iloc * NL;
    if constexpr (C::VEC) {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) a[ks] = m[16 * (ks / 4) + 4 * lk + ks % 4];
    } else {
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int q = 4 * ks + lk;
        a[ks] = q < NL ? m[q] : (T)0;
      }
    }
  };
  auto node_of = [&](int ks) { return C::VEC ? 16 * (ks / 4) + 4 * lk + ks % 4 : 4 * ks + lk; };
  // products of one row tile, the rows stored as pairs
  auto mul_rows = [&](int o, int rt, const T* a) {
    int xo = K * (o & 1) + W1 * K * ((o >> 1) & 1);
    if (D == 3) xo += W1 * W1 * K * ((o >> 2) & 1);
    const T* xc = sm.xs[lr % kMaxCols] + xo;
    Acc acc = {0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int q = node_of(ks), b12 = q / N1;
      const int xi = q % N1 + W1 * (b12 % N1) + (D == 3 ? W1 * W1 * (b12 / N1) : 0);
      const T bb = q < NL ? xc[xi] : (T)0;
      acc = mfma16(a[ks], bb, acc);
    }
    if (lr < kMaxCols) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = rt * 16 + Mfma<T>::row(lane, v);
        if (r < KD) {
          int iloc, pair;
          row_of(o, r, iloc, pair);
          sm.parts[lr][pair] = acc[v];
        }
      }
    }
  };
  // the wave's cells: flags, and matrix loads in flight while x is staged (the
  // first cell only where all of them would take more than 64 registers)
  constexpr int NCW = NCELL / NW;
  constexpr bool ALL = NCW * C::NRT * NKS * (int)sizeof(T) <= 64 * 4;
  // flags of the 2^d cells, 4 cells a word
  const uint64_t fga = reinterpret_cast<const uint64_t*>(G.cell_fg)[(int64_t)gp * (NCELL / 4)];
  const uint64_t fgb = reinterpret_cast<const uint64_t*>(G.cell_fg)[(int64_t)gp * (NCELL / 4) + NCELL / 4 - 1];
  auto cell_fg = [fga, fgb](int o) { return static_cast<int>((o >= 4 ? fgb : fga) >> (16 * (o & 3))) & 0xffff; };
  int fg[NCW], cut[NCW];
  T am[ALL ? NCW : 1][C::NRT][NKS];
#pragma unroll
  for (int i = 0; i < NCW; ++i) {
    fg[i] = cell_fg(i * NW + wave);
    cut[i] = G.cell_cut[(int64_t)gp * NCELL + i * NW + wave];
  }
#pragma unroll
  for (int i = 0; i < (ALL ? NCW : 1); ++i)
    if (fg[i] & 1) {
#pragma unroll
      for (int rt = 0; rt < C::NRT; ++rt) load_rows(rt, fg[i], cut[i], am[i][rt], i * NW + wave);
    }
  {
    // closure of every column; nodes outside the lattice are zero
    constexpr int NIT = (NC * kMaxCols + TH - 1) / TH;
    constexpr int UB = NIT < 16 ? NIT : 16;
    for (int u0 = 0; u0 < NIT; u0 += UB) {
      if (u0 * TH >= NC * ncol) break;
      T v[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int e = tid + TH * (u0 + u);
        v[u] = 0;
        if (e < NC * ncol) {
          const int c = e / NC, q = e % NC;
          const int q0 = q % W1, q1 = (q / W1) % W1, q2 = q / (W1 * W1);
          const int I0 = K * (V[0] - 1) + q0, I1 = K * (V[1] - 1) + q1, I2 = D == 3 ? K * (V[2] - 1) + q2 : 0;
          const bool in = I0 >= 0 && I0 < nn && I1 >= 0 && I1 < nn && (D == 2 || (I2 >= 0 && I2 < nn));
          if (in) v[u] = x[c * L.n_nodes + cbase + q0 + nn * q1 + (D == 3 ? nn2 * q2 : 0)];
        }
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int e = tid + TH * (u0 + u);
        if (e < NC * kMaxCols) (&sm.xs[0][0])[e] = v[u];
      }
    }
    for (int e = NC * ncol + tid; e < NC * kMaxCols; e += TH) (&sm.xs[0][0])[e] = 0;
  }
  // level tables: mass, jump weights j_m(s) and gc_m j_m(s)
  for (int t = tid; t < N1 * N1; t += TH) (&sm.mh[0][0])[t] = L.tables_t<T>()[S::T_MHAT + t];
  for (int t = tid; t < K * W1; t += TH) {
    (&sm.jm[0][0])[t] = L.tables_t<T>()[S::T_JM + t];
    (&sm.gj[0][0])[t] = L.tables_t<T>()[S::T_GJ + t];
  }
  // (node, column) task of the thread: row ti, columns tc + CPI u
  const int ti = tid % C::NPT, tc = tid / C::NPT;
  int pi[3] = {0, 0, 0};
  T bv[C::NRD];
  if (ti < nj) {
    const int ps = G.pos[off + ti];
    pi[0] = ps % W1;
    pi[1] = (ps / W1) % W1;
    pi[2] = D == 3 ? ps / (W1 * W1) : 0;
    const int node = static_cast<int>(cbase + pi[0] + nn * pi[1] + (D == 3 ? nn2 * pi[2] : 0));
#pragma unroll
    for (int u = 0; u < C::NRD; ++u) {
      const int c = tc + C::CPI * u;
      bv[u] = c < ncol ? b[c * L.n_nodes + node] : (T)0;
    }
    if (tc == 0) {
      sm.node[ti] = node;
      sm.pos[ti] = static_cast<int16_t>(ps);
    }
  }
  __syncthreads();
  // cell rows
#pragma unroll
  for (int i = 0; i < NCW; ++i) {
    const int o = i * NW + wave;
    if (fg[i] & 1) {
      if (!ALL && i > 0) {
#pragma unroll
        for (int rt = 0; rt < C::NRT; ++rt) load_rows(rt, fg[i], cut[i], am[0][rt], o);
      }
#pragma unroll
      for (int rt = 0; rt < C::NRT; ++rt) mul_rows(o, rt, am[ALL ? i : 0][rt]);
    } else {
      for (int e = lane; e < KD * kMaxCols; e += 64) {
        int iloc, pair;
        row_of(o, e % KD, iloc, pair);
        sm.parts[e / KD][pair] = 0;
      }
    }
  }
  // the first row block of the inverse: its loads do not depend on the residual
  const int nrb = (nj + 15) / 16, nkb = (nj + 3) / 4;
  constexpr int NKB = (S::NP + 3) / 4;
  auto load_inv = [&](int rb, T* a) {
    if constexpr (sizeof(T) == 4) {
      const float* t = G.inv_tiles + G.tile_off[gp] + (int64_t)rb * nkb * 64 + lane;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) a[kb] = kb < nkb ? t[kb * 64] : 0.f;
    } else {
      // rows of the symmetric inverse as columns: 16 consecutive entries
      const int i = rb * 16 + lr;
      const double* inv = G.inv_t<double>() + G.inv_off[gp] + (i < nj ? i : nj - 1);
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        const int j = 4 * kb + lk;
        a[kb] = j < nj ? inv[(int64_t)j * nj] : 0.0;
      }
    }
  };
  T ai[NKB];
  if (wave < nrb) load_inv(wave, ai);
  // ghost rows; bit dir 2^(D-1) + t of gmask: that (direction, tangential cell) has a face
  constexpr int NTC = 1 << (D - 1);
  uint32_t gmask = 0;
#pragma unroll
  for (int dt = 0; dt < D * NTC; ++dt) {
    const int dir = dt / NTC, t = dt % NTC;
    const int d0 = dir == 0 ? 1 : 0, d1 = dir == 2 ? 1 : 2;  // tangential directions (d1: 3-D only)
    const int o = ((t & 1) << d0) | (D == 3 ? (t >> 1) << d1 : 0);
    const int glo = cell_fg(o) >> 8, ghi = cell_fg(o | 1 << dir) >> 8;
    if ((glo & (3 << (2 * dir))) || (ghi & (2 << (2 * dir)))) gmask |= 1u << dt;
  }
  auto ghost = [&](int dt, int c) {
    const int dir = dt / NTC, t0 = dt & 1, t1 = D == 3 ? (dt >> 1) & 1 : 0;
    const int d0 = dir == 0 ? 1 : 0, d1 = dir == 2 ? 1 : 2;
    const int o = (t0 << d0) | (D == 3 ? t1 << d1 : 0);
    const int glo = cell_fg(o) >> 8, ghi = cell_fg(o | 1 << dir) >> 8;
    const bool f0 = glo & (1 << (2 * dir)), f1 = glo & (2 << (2 * dir)), f2 = ghi & (2 << (2 * dir));
    const int b0 = lane % 4, b1 = D == 3 ? (lane / 4) % 4 : 0;
    const bool on = ((gmask >> dt) & 1) && c < ncol && b0 < N1 && b1 < N1;
    T y[NP1];
#pragma unroll
    for (int p = 0; p < NP1; ++p) y[p] = 0;
    if (on) {
      const int sd = dir == 0 ? 1 : dir == 1 ? W1 : W1 * W1;
      const int s0 = d0 == 0 ? 1 : W1, s1 = D == 3 ? (d1 == 1 ? W1 : W1 * W1) : 0;
      const T* xl = sm.xs[c] + (K * t0 + b0) * s0 + (K * t1 + b1) * s1;
      const int64_t gd = dir == 0 ? 1 : dir == 1 ? nn : nn2, g0 = d0 == 0 ? 1 : nn, g1 = D == 3 ? (d1 == 1 ? nn : nn2) : 0;
      const T* xg = x + c * L.n_nodes + cbase + (K * t0 + b0) * g0 + (K * t1 + b1) * g1;
      T lo[K], hi[K], xv[2 * K + 1];  // node layers beyond the closure, and in it
#pragma unroll
      for (int q = 0; q < K; ++q) {
        lo[q] = f0 ? xg[(q - K) * gd] : (T)0;
        hi[q] = f2 ? xg[(2 * K + 1 + q) * gd] : (T)0;
      }
#pragma unroll
      for (int q = 0; q <= 2 * K; ++q) xv[q] = xl[q * sd];
#pragma unroll
      for (int m = 0; m < K; ++m) {
        T jm[2 * K + 1], gj[2 * K + 1];
#pragma unroll
        for (int q = 0; q <= 2 * K; ++q) {
          jm[q] = sm.jm[m][q];
          gj[q] = sm.gj[m][q];
        }
        if (f1) {
          T J = 0;
#pragma unroll
          for (int q = 0; q <= 2 * K; ++q) J += jm[q] * xv[q];
#pragma unroll
          for (int p = 1; p < 2 * K; ++p) y[p - 1] += gj[p] * J;
        }
        if (f0) {
          T J = 0;
#pragma unroll
          for (int q = 0; q < K; ++q) J += jm[q] * lo[q];
#pragma unroll
          for (int q = K; q <= 2 * K; ++q) J += jm[q] * xv[q - K];
#pragma unroll
          for (int p = 1; p <= K; ++p) y[p - 1] += gj[p + K] * J;
        }
        if (f2) {
          T J = 0;
#pragma unroll
          for (int q = 0; q <= K; ++q) J += jm[q] * xv[q + K];
#pragma unroll
          for (int q = K + 1; q <= 2 * K; ++q) J += jm[q] * hi[q - K - 1];
#pragma unroll
          for (int p = K; p < 2 * K; ++p) y[p - 1] += gj[p - K] * J;
        }
      }
    }
    // 1-D masses in the tangential directions: row b0 over the lanes of the
    // quad, then row b1 over the quads of the 16 lanes (idle lanes hold zeros)
    T w0[4], w1[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int q1 = (b1 - q) & 3;  // quad that a rotation by 4 q lanes brings here
      w0[q] = b0 < N1 && q < N1 ? sm.mh[b0][q < N1 ? q : 0] : (T)0;
      w1[q] = D == 3 && b1 < N1 && q1 < N1 ? sm.mh[b1][q1] : (T)0;
    }
    const int i0 = b0 - 1 + t0, i1 = b1 - 1 + t1;  // internal rows 0..k-1 of the tangential cell
    const bool put = on && i0 >= 0 && i0 < K && (D == 2 || (i1 >= 0 && i1 < K));
    T* h = sm.H[dir][c < kMaxCols ? c : 0] + (D == 3 ? (t0 * K + i0) * 2 * K + t1 * K + i1 : t0 * K + i0);
#pragma unroll
    for (int p = 0; p < NP1; ++p) {
      T v = w0[0] * lane_dpp<0x00>(y[p]) + w0[1] * lane_dpp<0x55>(y[p]);
      if (N1 > 2) v += w0[2] * lane_dpp<0xaa>(y[p]);
      if (N1 > 3) v += w0[3] * lane_dpp<0xff>(y[p]);
      if (D == 3)
        v = (w1[0] * v + w1[1] * lane_dpp<0x124>(v)) + (w1[2] * lane_dpp<0x128>(v) + w1[3] * lane_dpp<0x12c>(v));
      if (put) h[p * C::HT] = v;
    }
  };
  if (ncol > C::CPW / 2) {
    // a wave per (direction, tangential cell) and CPW columns: the faces are scalar
    for (int wt = wave; wt < D * NTC * C::NGT; wt += NW) {
      const int dt = wt / C::NGT, c0 = (wt % C::NGT) * C::CPW;
      if (((gmask >> dt) & 1) && c0 < ncol) ghost(dt, c0 + lane / C::LPC);
    }
  } else {
    // few columns: several (direction, tangential cell) choices side by side in a wave
    const int ns = D * NTC * ncol;
    for (int wt = wave; wt * C::CPW < ns; wt += NW) {
      const int slot = wt * C::CPW + lane / C::LPC;
      ghost(slot < ns ? slot / ncol : 0, slot < ns ? slot % ncol : kMaxCols);
    }
  }
  __syncthreads();
  // residual rows; rows beyond the patch and columns beyond ncol are zero
  {
    T acc[C::NRD];
#pragma unroll
    for (int u = 0; u < C::NRD; ++u) acc[u] = 0;
    if (ti < nj && tc < ncol) {
      // the node's pairs: per direction index j = p - 1 (layer 0, p <= k) and
      // j = p (layer 1, p >= k)
      int jlo[3] = {0, 0, 0}, jn[3] = {1, 1, 1};
#pragma unroll
      for (int a = 0; a < D; ++a) {
        jlo[a] = pi[a] <= K ? pi[a] - 1 : pi[a];
        jn[a] = pi[a] == K ? 2 : 1;
      }
      // every choice of layers is read, so that the reads are in flight together;
      // those that the node does not have (and unwritten ghost rows) are dropped
#pragma unroll
      for (int e = 0; e < NCELL; ++e) {
        int t = 0, st = 1;
        bool has = true;
#pragma unroll
        for (int a = 0; a < D; ++a) {
          const int ea = (e >> a) & 1;
          has = has && ea < jn[a];
          t += (jlo[a] + (ea & (jn[a] - 1))) * st;
          st *= 2 * K;
        }
#pragma unroll
        for (int u = 0; u < C::NRD; ++u) {
          const T v = sm.parts[C::col(tc, u)][t];
          acc[u] += has ? v : (T)0;
        }
      }
#pragma unroll
      for (int dir = 0; dir < D; ++dir) {
        constexpr int D1[3] = {2, 2, 1};
        const int d0 = dir == 0 ? 1 : 0, d1 = D1[dir];
#pragma unroll
        for (int e = 0; e < NTC; ++e) {
          const int e0 = e & 1, e1 = e >> 1;
          const int j0 = jlo[d0] + (e0 & (jn[d0] - 1)), j1 = D == 3 ? jlo[d1] + (e1 & (jn[d1] - 1)) : 0;
          const int t = (j0 >= K ? 1 : 0) | (j1 >= K ? 2 : 0);
          const bool has = e0 < jn[d0] && (D == 2 || e1 < jn[d1]) && ((gmask >> (dir * NTC + t)) & 1);
          const int at = (pi[dir] - 1) * C::HT + (D == 3 ? j0 * 2 * K + j1 : j0);
#pragma unroll
          for (int u = 0; u < C::NRD; ++u) {
            const T v = sm.H[dir][C::col(tc, u)][at];
            acc[u] += has ? v : (T)0;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < C::NRD; ++u) {
      const int c = tc + C::CPI * u;
      if (c < kMaxCols && ti < C::NPP) sm.rs[c][ti] = ti < nj && c < ncol ? bv[u] - acc[u] : (T)0;
    }
  }
  if constexpr (C::NPT < C::NPP) {
    for (int e = tid; e < kMaxCols * (C::NPP - C::NPT); e += TH)
      sm.rs[e / (C::NPP - C::NPT)][C::NPT + e % (C::NPP - C::NPT)] = 0;
  }
  __syncthreads();
  for (int rb = wave; rb < nrb; rb += NW) {  // wave-uniform: every lane takes part in the products
    if (rb != wave) load_inv(rb, ai);
    Acc d = {0, 0, 0, 0};
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
      if (kb < nkb) d = mfma16(ai[kb], sm.rs[lr % kMaxCols][4 * kb + lk], d);
    if (lr < ncol) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = rb * 16 + Mfma<T>::row(lane, v);
        if (i >= nj) continue;
        if (xb)
          xb[lr * L.n_nodes + sm.node[i]] = sm.xs[lr][sm.pos[i]] + d[v];
        else
          dbuf[lr * G.n_nodes + off + i] = d[v];
      }
    }
  }
}

template <int D, int K, typename T, int NW>
__global__ __launch_bounds__(64 * NW) void k_cut_cols(KLevel L, CutGroupDev G, const T* __restrict__ x,
                                                      const T* __restrict__ b, T* __restrict__ dbuf,
                                                      T* __restrict__ xb, CopyJob cj, int ncol) {
  cut_cols_body<D, K, T, NW>(L, G, x, b, dbuf, xb, cj, ncol);
}

// argument record of k_cut_cols for grouped launches (k_grouped)
template <int D, int K, typename T, int NW>
struct CutColsArgs {
  KLevel L;
  CutGroupDev G;
  const T* x;
  const T* b;
  T* dbuf;
  T* xb;
  CopyJob cj;
  int ncol;
  __device__ void run() const { cut_cols_body<D, K, T, NW>(L, G, x, b, dbuf, xb, cj, ncol); }
};

// dst = src on a node list (the cut region before a run of two-buffer cut steps).
template <typename T>
__device__ __forceinline__ void copy_nodes_body(const int32_t* __restrict__ nodes, int64_t n,
                                                const T* __restrict__ src, T* __restrict__ dst, int64_t ld) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < n) {
    const int64_t o = blockIdx.y * ld + nodes[e];
    dst[o] = src[o];
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_copy_nodes(const int32_t* __restrict__ nodes, int64_t n,
                                                    const T* __restrict__ src, T* __restrict__ dst, int64_t ld) {
  copy_nodes_body<T>(nodes, n, src, dst, ld);
}

// argument record of k_copy_nodes for grouped launches (k_grouped)
template <typename T>
struct CopyNodesArgs {
  const int32_t* nodes;
  int64_t n;
  const T* src;
  T* dst;
  int64_t ld;
  __device__ void run() const { copy_nodes_body<T>(nodes, n, src, dst, ld); }
};

// Cut patches, phase 2: x[I_j] += d_j for all patches of the colour.
template <typename T>
__device__ __forceinline__ void cut_update_body(const int32_t* __restrict__ nodes, int64_t n,
                                                const T* __restrict__ dbuf, T* __restrict__ x, int64_t ldx) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e < n) x[blockIdx.y * ldx + nodes[e]] += dbuf[blockIdx.y * n + e];
}

template <typename T>
__global__ __launch_bounds__(256) void k_cut_update(const int32_t* __restrict__ nodes, int64_t n,
                                                    const T* __restrict__ dbuf, T* __restrict__ x, int64_t ldx) {
  cut_update_body<T>(nodes, n, dbuf, x, ldx);
}

// argument record of k_cut_update for grouped launches (k_grouped)
template <typename T>
struct CutUpdateArgs {
  const int32_t* nodes;
  int64_t n;
  const T* dbuf;
  T* x;
  int64_t ldx;
  __device__ void run() const { cut_update_body<T>(nodes, n, dbuf, x, ldx); }
};

// x_f[I] += sum_J P(I, J) x_c[J] for every active fine node (embedding).
template <int D, int K, typename T>
__device__ __forceinline__ void prolong_add_body(KLevel Lc, KLevel Lf, const T* __restrict__ xc, T* __restrict__ xf) {
  using S = Shape<D, K>;
  constexpr int N1 = S::N1;
  __shared__ double p1d[S::NC1 * N1];
  for (int t = threadIdx.x; t < S::NC1 * N1; t += blockDim.x) p1d[t] = Lf.tables[S::T_P1D + t];
  __syncthreads();
  xc += blockIdx.y * Lc.n_nodes;  // column blockIdx.y
  xf += blockIdx.y * Lf.n_nodes;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= Lf.n_dofs) return;
  const int32_t node = Lf.dof_node[i];
  int J0[3], nq[3];
  double w[3][N1];
  int r = node;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    const int I = r % Lf.nn;
    r /= Lf.nn;
    const int q = I % (2 * K);
    if (q == 0) { J0[a] = I / 2; nq[a] = 1; w[a][0] = 1.0; }
    else {
      J0[a] = K * (I / (2 * K));
      nq[a] = N1;
#pragma unroll
      for (int bb = 0; bb < N1; ++bb) w[a][bb] = p1d[q * N1 + bb];
    }
  }
  // all (k+1)^d coarse values at once (predicated), then the weighted sum in
  // the order of the contributing combinations
  constexpr int NQ = Pow<N1, D>::v;
  T v[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int s0 = q % N1, s1 = (q / N1) % N1, s2 = D == 3 ? q / (N1 * N1) : 0;
    const bool use = s0 < nq[0] && s1 < nq[1] && (D == 2 || s2 < nq[2]);
    int J[3] = {J0[0] + s0, J0[1] + s1, D == 3 ? J0[2] + s2 : 0};
    v[q] = use ? xc[lat(D, Lc.nn, J)] : (T)0;
  }
  T acc = 0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int s0 = q % N1, s1 = (q / N1) % N1, s2 = D == 3 ? q / (N1 * N1) : 0;
    if (s0 < nq[0] && s1 < nq[1] && (D == 2 || s2 < nq[2])) {
      double wt = w[0][s0] * w[1][s1];
      if (D == 3) wt *= w[2][s2];
      acc += (T)wt * v[q];
    }
  }
  xf[node] += acc;
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_prolong_add(KLevel Lc, KLevel Lf, const T* __restrict__ xc,
                                                     T* __restrict__ xf) {
  prolong_add_body<D, K, T>(Lc, Lf, xc, xf);
}

// argument record of k_prolong_add for grouped launches (k_grouped)
template <int D, int K, typename T>
struct ProlongAddArgs {
  KLevel Lc;
  KLevel Lf;
  const T* xc;
  T* xf;
  __device__ void run() const { prolong_add_body<D, K, T>(Lc, Lf, xc, xf); }
};

// Coarse cells per direction of one restriction block.
template <int D, int K>
struct RestrictShape {
  using S = Shape<D, K>;
  static constexpr int TB = ApplyShape<D, K>::B;                  // cells of an operator tile (whose lists are used)
  static constexpr int RB = D == 3 && K > 1 ? 2 : TB;             // cells of a block
  static constexpr int SUB = TB / RB;                             // blocks per tile and direction
  static constexpr int NSUB = Pow<SUB, D>::v;
  static constexpr int O1 = RB * K + 1;                           // owned coarse nodes (last tile: + 1)
  static constexpr int S1 = 2 * K * RB + 2 * K;                   // staged fine nodes
  static constexpr int NT = 4 * K - 1;                            // fine nodes below a coarse vertex node
};

// b_c[J] = sum_I P(I, J) r_f[I] on the coarse nodes of a block of RB^d coarse
// cells (transpose of the embedding), by one 1-D pass per direction in LDS: P is
// a tensor product, and in every direction the fine nodes with a non-zero weight
// form one range, [2J-2k+1, 2J+2k-1] around a coarse vertex node and [2kC+1,
// 2kC+2k-1] inside a coarse cell C.  The blocks are the coarse level's operator
// tiles (those owning active nodes) cut into RB^d cells; fine nodes beyond the
// box count as zero, and coarse nodes that are not active receive the sum of
// the zeros around them.  A block stages its fine nodes with all loads in
// flight; a wave works on rows of one coarse node, so it is bound by a short
// chain where one thread per node made (4k-1)^d steps.  128^3 ball, Q2, FP64: 77.8
// -> 38.6 us on the finest level, 24.6 -> 9.8 us at 32^3 cells; Q3 union at 32^3 94.5
// -> 15.1 us; circle, Q3, 1024^2, 76.1 -> 31.5 us.
template <int D, int K, typename T>
__device__ __forceinline__ void restrict_body(const KLevel& Lc, const KLevel& Lf, const T* __restrict__ rf,
                                              T* __restrict__ bc) {
  using S = Shape<D, K>;
  using R = RestrictShape<D, K>;
  constexpr int N1 = S::N1, S1 = R::S1, O1 = R::O1, NT = R::NT;
  constexpr int NF = Pow<S1, D>::v;       // fine nodes
  constexpr int P1 = S1 | 1;              // line stride in LDS, odd
  constexpr int NL0 = NF / S1;            // lines along direction 0
  constexpr int NG = D == 3 ? S1 * P1 : P1;  // first-pass values per coarse node
  constexpr int NA = NG * O1, NB = D == 3 ? P1 * O1 * O1 : 1;
  __shared__ T f[NL0 * P1 > NB ? NL0 * P1 : NB];  // fine nodes; in 3-D then the second pass
  __shared__ T g[NA];                 // first pass
  __shared__ T w[K][NT];              // weights: 0 the vertex node, i the i-th node inside a cell
  const int ntile = Lc.n_tiles + Lc.n_tiles_sf;
  const int ti = blockIdx.x / R::NSUB;
  if (ti >= ntile) return;  // grouped launches: a block beyond this problem's tiles
  rf += blockIdx.y * Lf.n_nodes;  // column blockIdx.y
  bc += blockIdx.y * Lc.n_nodes;
  for (int t = threadIdx.x; t < K * NT; t += 256) {
    const int i = t / NT, e = t % NT;
    int at = -1;  // entry of the 1-D prolongation table
    if (i == 0) at = e < 2 * K - 1 ? (e + 1) * N1 + K : e > 2 * K - 1 ? (e - (2 * K - 1)) * N1 : -1;
    else if (e < 2 * K - 1) at = (e + 1) * N1 + i;
    w[i][e] = at >= 0 ? (T)Lf.tables[S::T_P1D + at] : i == 0 ? (T)1 : (T)0;
  }
  int c0[3] = {0, 0, 0};  // first coarse node of the block
  {
    const int NTd = (Lc.N + R::TB - 1) / R::TB;
    int r = ti < Lc.n_tiles ? Lc.tiles[ti] : Lc.tiles_sf[ti - Lc.n_tiles], q = blockIdx.x % R::NSUB;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      c0[a] = K * (R::TB * (r % NTd) + R::RB * (q % R::SUB));
      r /= NTd;
      q /= R::SUB;
    }
  }
  const int nf = Lf.nn;
  {
    constexpr int NIT = (NF + 255) / 256, UB = NIT < 12 ? NIT : 12;
    for (int u0 = 0; u0 < NIT; u0 += UB) {
      T v[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int e = threadIdx.x + 256 * (u0 + u);
        int I[3], r = e;
        bool in = e < NF;
#pragma unroll
        for (int a = 0; a < D; ++a) {
          I[a] = 2 * c0[a] - (2 * K - 1) + r % S1;
          r /= S1;
          in = in && I[a] >= 0 && I[a] < nf;
        }
        v[u] = in ? rf[lat(D, nf, I)] : (T)0;
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int e = threadIdx.x + 256 * (u0 + u);
        if (e < NF) f[(e / S1) * P1 + e % S1] = v[u];
      }
    }
  }
  __syncthreads();
  // sum over the fine range of coarse node q on one line; the range of the last
  // node ends with the box (or the node belongs to the next block)
  auto line = [&](const T* s, int q) {
    T acc = 0;
    if (q % K == 0) {
#pragma unroll
      for (int e = 0; e < NT; ++e)
        if (e < 2 * K || q < R::RB * K) acc += w[0][e] * s[2 * q + e];
    } else {
#pragma unroll
      for (int e = 0; e < 2 * K - 1; ++e) acc += w[q % K][e] * s[2 * K * (q / K) + 2 * K + e];
    }
    return acc;
  };
  // direction 0: g[q0][direction 2][direction 1]
  for (int t = threadIdx.x; t < NL0 * O1; t += 256) {
    const int q0 = t / NL0, r = t % NL0;
    g[q0 * NG + (D == 3 ? (r / S1) * P1 + r % S1 : r)] = line(f + r * P1, q0);
  }
  __syncthreads();
  if constexpr (D == 3) {
    // direction 1: f[q1][q0][direction 2]
    for (int t = threadIdx.x; t < S1 * O1 * O1; t += 256) {
      const int s2 = t % S1, q0 = (t / S1) % O1, q1 = t / (S1 * O1);
      f[(q1 * O1 + q0) * P1 + s2] = line(g + q0 * NG + s2 * P1, q1);
    }
    __syncthreads();
  }
  // last direction, at every owned coarse node
  constexpr int NO = Pow<O1, D>::v;
  for (int t = threadIdx.x; t < NO; t += 256) {
    int q[3], J[3], r = t;
    bool own = true;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      q[a] = r % O1;
      r /= O1;
      J[a] = c0[a] + q[a];
      // the last layer belongs to the next block unless the box ends here
      own = own && J[a] < Lc.nn && (q[a] < R::RB * K || J[a] == Lc.nn - 1);
    }
    if (!own) continue;
    bc[lat(D, Lc.nn, J)] = D == 3 ? line(f + (q[1] * O1 + q[0]) * P1, q[2]) : line(g + q[0] * NG, q[1]);
  }
}

template <int D, int K, typename T>
__global__ __launch_bounds__(256) void k_restrict(KLevel Lc, KLevel Lf, const T* __restrict__ rf,
                                                  T* __restrict__ bc) {
  restrict_body<D, K, T>(Lc, Lf, rf, bc);
}

// argument record of k_restrict for grouped launches (k_grouped)
template <int D, int K, typename T>
struct RestrictArgs {
  KLevel Lc;
  KLevel Lf;
  const T* rf;
  T* bc;
  __device__ void run() const { restrict_body<D, K, T>(Lc, Lf, rf, bc); }
};

// x = M b on one level, M dense n x n (row-major): the exact coarse solve, or
// the dense V-cycle of the smallest levels.  One wavefront per row, the active
// entries of up to NCOL columns of b staged in LDS run by run, so that a matrix
// entry is read once for all of them; lane l sums the columns l, l + 64, ... of M
// in increasing order whatever NCOL is.  Bound by the reads of M once n is
// large (1,701 rows, FP64, 23 MB: 11 us).
template <typename T, int NCOL>
__device__ __forceinline__ void coarse_body(const T* __restrict__ inv, const int32_t* __restrict__ dof_node, int n,
                                            const T* __restrict__ b, T* __restrict__ x, int64_t ld, int ncol) {
  constexpr int RUN = NCOL == 1 ? 2048 : 512;
  __shared__ T bs[NCOL][RUN];
  const int row = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  const int lane = threadIdx.x % 64;
  const int c0 = blockIdx.y * NCOL;  // column group
  b += c0 * ld;
  x += c0 * ld;
  ncol = ncol - c0 < NCOL ? ncol - c0 : NCOL;
  const T* m = inv + (int64_t)(row < n ? row : 0) * n;
  T s[NCOL];
#pragma unroll
  for (int c = 0; c < NCOL; ++c) s[c] = 0;
  for (int j0 = 0; j0 < n; j0 += RUN) {
    const int nr = n - j0 < RUN ? n - j0 : RUN;
    if (j0 > 0) __syncthreads();
    for (int j = threadIdx.x; j < nr; j += blockDim.x) {
      const int64_t nd = dof_node[j0 + j];
#pragma unroll
      for (int c = 0; c < NCOL; ++c) bs[c][j] = c < ncol ? b[c * ld + nd] : (T)0;
    }
    __syncthreads();
    if (row < n) {
#pragma unroll 8
      for (int j = lane; j < nr; j += 64) {
        const T e = m[j0 + j];
#pragma unroll
        for (int c = 0; c < NCOL; ++c) s[c] += e * bs[c][j];
      }
    }
  }
  if (row >= n) return;
#pragma unroll
  for (int c = 0; c < NCOL; ++c)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s[c] += __shfl_down(s[c], o, 64);
  if (lane == 0) {
    const int64_t nd = dof_node[row];
#pragma unroll
    for (int c = 0; c < NCOL; ++c)
      if (c < ncol) x[c * ld + nd] = s[c];
  }
}

template <typename T, int NCOL>
__global__ __launch_bounds__(256) void k_coarse(const T* __restrict__ inv, const int32_t* __restrict__ dof_node,
                                                int n, const T* __restrict__ b, T* __restrict__ x, int64_t ld,
                                                int ncol) {
  coarse_body<T, NCOL>(inv, dof_node, n, b, x, ld, ncol);
}

// argument record of k_coarse for grouped launches (k_grouped)
template <typename T, int NCOL>
struct CoarseArgs {
  const T* inv;
  const int32_t* dof_node;
  int n;
  const T* b;
  T* x;
  int64_t ld;
  int ncol;
  __device__ void run() const { coarse_body<T, NCOL>(inv, dof_node, n, b, x, ld, ncol); }
};

// Columns c0 .. c0 + ncol - 1 of the identity on the active nodes of a level.
__global__ __launch_bounds__(256) void k_units(const int32_t* __restrict__ dof_node, int64_t n, int64_t c0,
                                               double* __restrict__ b, int64_t ld) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) b[blockIdx.y * ld + dof_node[i]] = i == c0 + blockIdx.y ? 1.0 : 0.0;
}

// The columns c0 .. of a dense n x n matrix (row-major) from lattice vectors.
__global__ __launch_bounds__(256) void k_put_columns(const int32_t* __restrict__ dof_node, int64_t n, int64_t c0,
                                                     int ncol, const double* __restrict__ x, int64_t ld,
                                                     double* __restrict__ m) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= n * ncol) return;
  const int64_t i = e / ncol, c = e % ncol;
  m[i * n + c0 + c] = x[c * ld + dof_node[i]];
}

__global__ __launch_bounds__(256) void k_round(int64_t n, const double* __restrict__ x, float* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = static_cast<float>(x[i]);
}

template <typename T>
__device__ __forceinline__ void zero_active_body(const int32_t* __restrict__ dof_node, int64_t n, T* __restrict__ x,
                                                 int64_t ld) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) x[blockIdx.y * ld + dof_node[i]] = 0;
}

template <typename T>
__global__ __launch_bounds__(256) void k_zero_active(const int32_t* __restrict__ dof_node, int64_t n,
                                                     T* __restrict__ x, int64_t ld) {
  zero_active_body<T>(dof_node, n, x, ld);
}

// argument record of k_zero_active for grouped launches (k_grouped)
template <typename T>
struct ZeroActiveArgs {
  const int32_t* dof_node;
  int64_t n;
  T* x;
  int64_t ld;
  __device__ void run() const { zero_active_body<T>(dof_node, n, x, ld); }
};

template <typename TS, typename TD>
__global__ __launch_bounds__(256) void k_scatter(const int32_t* __restrict__ dof_node, int64_t n,
                                                 const TS* __restrict__ src, TD* __restrict__ lat_dst, int64_t ld) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) lat_dst[blockIdx.y * ld + dof_node[i]] = (TD)src[blockIdx.y * n + i];
}

template <typename TS, typename TD>
__global__ __launch_bounds__(256) void k_gather(const int32_t* __restrict__ dof_node, int64_t n,
                                                const TS* __restrict__ lat_src, TD* __restrict__ dst, int64_t ld) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) dst[blockIdx.y * n + i] = (TD)lat_src[blockIdx.y * ld + dof_node[i]];
}

}  // namespace dev

// ---------------------------------------------------------------------------
// Host launchers: dispatch on (dimension, degree).
namespace {

inline unsigned blocks(int64_t n, int b = 256) { return static_cast<unsigned>((n + b - 1) / b); }

// Launch recorder of the calling thread (see set_launch_recorder).
thread_local std::vector<LaunchRecord>* t_rec = nullptr;
thread_local int t_segment = 0;

// While recording: append the grouped form of a launch and return true.
template <int LB, typename A>
bool record(dim3 g, dim3 b, const A& a) {
  if (!t_rec) return false;
  LaunchRecord r;
  r.fn = reinterpret_cast<const void*>(&dev::k_grouped<LB, A>);
  r.segment = t_segment;
  r.grid[0] = g.x;
  r.grid[1] = g.y;
  r.block = b.x;
  r.args.assign(reinterpret_cast<const unsigned char*>(&a), reinterpret_cast<const unsigned char*>(&a) + sizeof(A));
  t_rec->push_back(std::move(r));
  return true;
}

// While recording, a launch without a grouped form leaves an empty record
// (the group that recorded it cannot be formed).
bool record_none() {
  if (!t_rec) return false;
  t_rec->push_back(LaunchRecord{});
  t_rec->back().segment = t_segment;
  return true;
}

// The defaults of LaunchPolicy: a grid cap of 256 CUs x 8 resident 256-thread
// blocks for the grid-stride kernels that stage level tables in LDS (every
// block loads the tables once), and larger blocks for cut-patch launches of
// fewer than 1536 patches (the coarse levels).

template <typename F>
hipError_t dispatch(int d, int k, F&& f) {
  if (d == 2 && k == 1) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 1>{});
  if (d == 2 && k == 2) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{});
  if (d == 2 && k == 3) return f(std::integral_constant<int, 2>{}, std::integral_constant<int, 3>{});
  if (d == 3 && k == 1) return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
  if (d == 3 && k == 2) return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{});
  if (d == 3 && k == 3) return f(std::integral_constant<int, 3>{}, std::integral_constant<int, 3>{});
  return hipErrorInvalidValue;
}

}  // namespace

void set_launch_recorder(std::vector<LaunchRecord>* rec) {
  t_rec = rec;
  t_segment = 0;
}
void set_launch_segment(int segment) { t_segment = segment; }
bool launch_recording() { return t_rec != nullptr; }

int tables_size(int d, int k) {
  int n = -1;
  (void)dispatch(d, k, [&](auto D, auto K) {
    n = dev::Shape<D.value, K.value>::T_SIZE;
    return hipSuccess;
  });
  return n;
}

template <typename T>
hipError_t launch_apply(int d, int k, const KLevel& L, const T* x, const T* b, T* y, T* W, T* C, hipStream_t s,
                        int ncol, const LaunchPolicy& lp) {
  if (L.n_dofs == 0) return hipSuccess;
  return dispatch(d, k, [&](auto D, auto K) {
    // while recording, the pre-passes are recorded also where they have no
    // work, so that the launch sequence does not depend on the geometry
    if (L.n_faces > 0 || t_rec) {
      const dim3 g(std::max(1u, blocks(L.n_faces)), ncol);
      if (!record<256>(g, dim3(256), dev::FaceWArgs<D.value, K.value, T>{L, x, W})) {
        hipLaunchKernelGGL((dev::k_face_w<D.value, K.value, T>), g, dim3(256), 0, s, L, x, W);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    }
    if (L.n_spec > 0 || t_rec) {
      using One = dev::CellShape<D.value, K.value, 1>;
      using Many = dev::CellShape<D.value, K.value, kMaxCols>;
      constexpr int CPB = One::CPB;
      const dim3 g(std::max(1u, static_cast<unsigned>((L.n_spec + CPB - 1) / CPB)),
                   ncol == 1 ? 1 : (ncol + kMaxCols - 1) / kMaxCols);
      if (ncol == 1) {
        if (!record<One::TH>(g, dim3(One::TH), dev::CellAxArgs<D.value, K.value, T, 1>{L, x, W, C, 1}))
          hipLaunchKernelGGL((dev::k_cell_ax<D.value, K.value, T, 1>), g, dim3(One::TH), 0, s, L, x, W, C, 1);
      } else if (!record<Many::TH>(g, dim3(Many::TH), dev::CellAxArgs<D.value, K.value, T, kMaxCols>{L, x, W, C, ncol})) {
        hipLaunchKernelGGL((dev::k_cell_ax<D.value, K.value, T, kMaxCols>), g, dim3(Many::TH), 0, s, L, x, W, C, ncol);
      }
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    // the two tile kernels write disjoint owned nodes
    if (L.n_tiles > 0 || t_rec) {
      const unsigned nb = std::max(1u, std::min<unsigned>(static_cast<unsigned>(L.n_tiles), lp.max_blocks / ncol + 1));
      if (!record<256>(dim3(nb, ncol), dim3(256), dev::ApplyArgs<D.value, K.value, T>{L, x, b, y, C})) {
        hipLaunchKernelGGL((dev::k_apply<D.value, K.value, T>), dim3(nb, ncol), dim3(256), 0, s, L, x, b, y, C);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
    }
    if (L.n_tiles_sf > 0 || t_rec) {
      const unsigned nb =
          std::max(1u, std::min<unsigned>(static_cast<unsigned>(L.n_tiles_sf), lp.max_blocks / ncol + 1));
      if (!record<256>(dim3(nb, ncol), dim3(256), dev::ApplySfArgs<D.value, K.value, T>{L, x, b, y})) {
        hipLaunchKernelGGL((dev::k_apply_sf<D.value, K.value, T>), dim3(nb, ncol), dim3(256), 0, s, L, x, b, y);
        return hipGetLastError();
      }
    }
    return hipSuccess;
  });
}

template <typename T>
hipError_t launch_interior_step(int d, int k, const KLevel& L, const int32_t* verts, int nv, T* x, const T* b,
                                hipStream_t s, int ncol, const LaunchPolicy& lp) {
  if (nv == 0 && !t_rec) return hipSuccess;  // recorded also without work (see launch_apply)
  return dispatch(d, k, [&](auto D, auto K) {
    constexpr int PPB = dev::Shape<D.value, K.value>::PPB;
    const unsigned nb = std::max(1u, std::min<unsigned>(blocks(nv, PPB), lp.max_blocks / ncol + 1));
    if (record<256>(dim3(nb, ncol), dim3(256), dev::InteriorStepArgs<D.value, K.value, T>{L, verts, nv, x, b}))
      return hipSuccess;
    hipLaunchKernelGGL((dev::k_interior_step<D.value, K.value, T>), dim3(nb, ncol), dim3(256), 0, s, L, verts, nv,
                       x, b);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t launch_cut_solve(int d, int k, const KLevel& L, const CutGroupDev& G, const T* x, const T* b, T* dbuf,
                            hipStream_t s, int ncol, T* xb, const CopyJob& cj, const LaunchPolicy& lp) {
  if (G.n_patch == 0) return hipSuccess;
  if (record_none()) return hipSuccess;
  return dispatch(d, k, [&](auto D, auto K) {
    if (xb == nullptr && cj.n != 0) return hipErrorInvalidValue;  // a copy job needs the second buffer
    // small launches (the coarse levels) are bound by the latency of one patch
    // block: more threads per patch shorten its serial passes; large ones keep
    // the smaller blocks for occupancy
    auto go = [&](auto th) {
      constexpr int TH = decltype(th)::value;
      using C = dev::CutShape<D.value, K.value, T, TH>;
      CopyJob c2 = cj;
      c2.nblk = static_cast<int>((cj.n + TH * C::COPY - 1) / (TH * C::COPY));
      hipLaunchKernelGGL((dev::k_cut_solve<D.value, K.value, T, TH>), dim3(c2.nblk + G.n_patch, ncol), dim3(TH), 0,
                         s, L, G, x, b, dbuf, xb, c2);
      return hipGetLastError();
    };
    constexpr int TL = dev::CutThreads<D.value, K.value>::v;
    // small launches: Q1 patches (one node) have nothing to split; a 512-thread
    // block takes most of a CU's registers, so Q3 turns to it later
    constexpr int TS = K.value == 1 ? TL : D.value == 2 ? 128 : K.value == 3 ? 512 : 256;
    if (G.n_patch * (TS == 512 ? int64_t{4} : int64_t{1}) < lp.small_cut_launch)
      return go(std::integral_constant<int, TS>{});
    return go(std::integral_constant<int, TL>{});
  });
}

CopyJob cut_copy_job(int d, int k, const CutGroupDev& Gp, int mask) {
  CopyJob cj;
  if (Gp.n_nodes == 0) return cj;
  cj.nodes = Gp.nodes;
  cj.skip = Gp.nxt;
  cj.mask = mask;
  cj.n = Gp.n_nodes;
  (void)d;
  (void)k;
  return cj;  // the launcher sizes the copy blocks for its block size
}

template <typename T>
hipError_t launch_copy_nodes(const int32_t* nodes, int64_t n, const T* src, T* dst, int64_t ld, hipStream_t s,
                             int ncol) {
  if (n == 0) return hipSuccess;
  if (record<256>(dim3(blocks(n), ncol), dim3(256), dev::CopyNodesArgs<T>{nodes, n, src, dst, ld})) return hipSuccess;
  hipLaunchKernelGGL((dev::k_copy_nodes<T>), dim3(blocks(n), ncol), dim3(256), 0, s, nodes, n, src, dst, ld);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_cut_cols(int d, int k, const KLevel& L, const CutGroupDev& G, const T* x, const T* b, T* dbuf,
                           int ncol, hipStream_t s, T* xb, const CopyJob& cj, const LaunchPolicy& lp) {
  if (G.n_patch == 0) return hipSuccess;
  if (ncol < 1 || (xb == nullptr && cj.n != 0)) return hipErrorInvalidValue;
  if (std::is_same<T, float>::value && (!G.inv_tiles || !G.tile_off)) return hipErrorInvalidValue;
  return dispatch(d, k, [&](auto D, auto K) {
    auto go = [&](auto nw) {
      constexpr int NW = decltype(nw)::value;
      using C = dev::ColsShape<D.value, K.value, T, NW>;
      CopyJob c2 = cj;
      c2.nblk = static_cast<int>((cj.n + C::TH * C::COPY - 1) / (C::TH * C::COPY));
      const dim3 g(c2.nblk + G.n_patch, (ncol + kMaxCols - 1) / kMaxCols);
      if (record<C::TH>(g, dim3(C::TH), dev::CutColsArgs<D.value, K.value, T, NW>{L, G, x, b, dbuf, xb, c2, ncol}))
        return hipSuccess;
      hipLaunchKernelGGL((dev::k_cut_cols<D.value, K.value, T, NW>), g, dim3(C::TH), 0, s, L, G, x, b, dbuf, xb, c2,
                         ncol);
      return hipGetLastError();
    };
    // Q1 patches have one internal node.  Else 4 waves (one per cell in 2-D,
    // two cells each in 3-D); in 3-D launches that leave CUs idle take 8, which
    // shortens a patch's serial chain (Q2 in FP64, 5 columns, 13..24 patches:
    // 14.4 -> 11.2 us; at 3,372 Q3 patches 8 waves cost 8%).  Grouped launches
    // must not depend on a member's patch count and carry several members'
    // patches: 4 waves (8 cost 27% on eight Q2 problems at 32^3 cells).  The
    // arithmetic is the same.
    if constexpr (K.value == 1) {
      return go(std::integral_constant<int, 1>{});
    } else {
      if (D.value == 3 && !t_rec && 3 * (int64_t)G.n_patch * ((ncol + kMaxCols - 1) / kMaxCols) < lp.small_cut_launch)
        return go(std::integral_constant<int, D.value == 3 ? 8 : 4>{});
      return go(std::integral_constant<int, 4>{});
    }
  });
}

template <typename T>
hipError_t launch_cut_update(const CutGroupDev& G, const T* dbuf, T* x, int64_t ldx, hipStream_t s, int ncol) {
  if (G.n_nodes == 0) return hipSuccess;
  if (record<256>(dim3(blocks(G.n_nodes), ncol), dim3(256), dev::CutUpdateArgs<T>{G.nodes, G.n_nodes, dbuf, x, ldx}))
    return hipSuccess;
  hipLaunchKernelGGL((dev::k_cut_update<T>), dim3(blocks(G.n_nodes), ncol), dim3(256), 0, s, G.nodes, G.n_nodes, dbuf,
                     x, ldx);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_prolong_add(int d, int k, const KLevel& Lc, const KLevel& Lf, const T* xc, T* xf, hipStream_t s,
                              int ncol) {
  return dispatch(d, k, [&](auto D, auto K) {
    if (record<256>(dim3(blocks(Lf.n_dofs), ncol), dim3(256), dev::ProlongAddArgs<D.value, K.value, T>{Lc, Lf, xc, xf}))
      return hipSuccess;
    hipLaunchKernelGGL((dev::k_prolong_add<D.value, K.value, T>), dim3(blocks(Lf.n_dofs), ncol), dim3(256), 0, s, Lc,
                       Lf, xc, xf);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t launch_restrict(int d, int k, const KLevel& Lc, const KLevel& Lf, const T* rf, T* bc, hipStream_t s,
                           int ncol) {
  return dispatch(d, k, [&](auto D, auto K) {
    const dim3 g(std::max(1, Lc.n_tiles + Lc.n_tiles_sf) * dev::RestrictShape<D.value, K.value>::NSUB, ncol);
    if (record<256>(g, dim3(256), dev::RestrictArgs<D.value, K.value, T>{Lc, Lf, rf, bc})) return hipSuccess;
    hipLaunchKernelGGL((dev::k_restrict<D.value, K.value, T>), g, dim3(256), 0, s, Lc, Lf, rf, bc);
    return hipGetLastError();
  });
}

template <typename T>
hipError_t launch_coarse(const T* inv, const int32_t* dof_node, int n, const T* b, T* x, int64_t ld, hipStream_t s,
                         int ncol) {
  auto go = [&](auto nc) {
    constexpr int NCOL = decltype(nc)::value;
    const dim3 g(blocks(n, 4), (ncol + NCOL - 1) / NCOL);
    if (record<256>(g, dim3(256), dev::CoarseArgs<T, NCOL>{inv, dof_node, n, b, x, ld, ncol})) return hipSuccess;
    hipLaunchKernelGGL((dev::k_coarse<T, NCOL>), g, dim3(256), 0, s, inv, dof_node, n, b, x, ld, ncol);
    return hipGetLastError();
  };
  if (ncol == 1) return go(std::integral_constant<int, 1>{});
  return go(std::integral_constant<int, kMaxCols>{});
}

hipError_t launch_units(const int32_t* dof_node, int64_t n, int64_t c0, int ncol, double* b, int64_t ld,
                        hipStream_t s) {
  hipLaunchKernelGGL(dev::k_units, dim3(blocks(n), ncol), dim3(256), 0, s, dof_node, n, c0, b, ld);
  return hipGetLastError();
}

hipError_t launch_put_columns(const int32_t* dof_node, int64_t n, int64_t c0, int ncol, const double* x, int64_t ld,
                              double* m, hipStream_t s) {
  hipLaunchKernelGGL(dev::k_put_columns, dim3(blocks(n * ncol)), dim3(256), 0, s, dof_node, n, c0, ncol, x, ld, m);
  return hipGetLastError();
}

hipError_t launch_round(int64_t n, const double* x, float* y, hipStream_t s) {
  hipLaunchKernelGGL(dev::k_round, dim3(blocks(n)), dim3(256), 0, s, n, x, y);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_zero_active(const int32_t* dof_node, int64_t n, T* x, int64_t ld, hipStream_t s, int ncol) {
  if (n == 0 && !t_rec) return hipSuccess;
  if (record<256>(dim3(std::max(1u, blocks(n)), ncol), dim3(256), dev::ZeroActiveArgs<T>{dof_node, n, x, ld}))
    return hipSuccess;
  hipLaunchKernelGGL((dev::k_zero_active<T>), dim3(blocks(n), ncol), dim3(256), 0, s, dof_node, n, x, ld);
  return hipGetLastError();
}

template <typename TS, typename TD>
hipError_t launch_scatter(const int32_t* dof_node, int64_t n, const TS* src, TD* lat, int64_t ld, hipStream_t s,
                          int ncol) {
  if (n == 0) return hipSuccess;
  if (record_none()) return hipSuccess;
  hipLaunchKernelGGL((dev::k_scatter<TS, TD>), dim3(blocks(n), ncol), dim3(256), 0, s, dof_node, n, src, lat, ld);
  return hipGetLastError();
}

template <typename TS, typename TD>
hipError_t launch_gather(const int32_t* dof_node, int64_t n, const TS* lat, TD* dst, int64_t ld, hipStream_t s,
                         int ncol) {
  if (n == 0) return hipSuccess;
  if (record_none()) return hipSuccess;
  hipLaunchKernelGGL((dev::k_gather<TS, TD>), dim3(blocks(n), ncol), dim3(256), 0, s, dof_node, n, lat, dst, ld);
  return hipGetLastError();
}

#define CMG_INSTANTIATE(T)                                                                                      \
  template hipError_t launch_apply<T>(int, int, const KLevel&, const T*, const T*, T*, T*, T*, hipStream_t, int, \
                                      const LaunchPolicy&);                                                        \
  template hipError_t launch_interior_step<T>(int, int, const KLevel&, const int32_t*, int, T*, const T*,         \
                                              hipStream_t, int, const LaunchPolicy&);                              \
  template hipError_t launch_cut_solve<T>(int, int, const KLevel&, const CutGroupDev&, const T*, const T*, T*,    \
                                          hipStream_t, int, T*, const CopyJob&, const LaunchPolicy&);              \
  template hipError_t launch_cut_cols<T>(int, int, const KLevel&, const CutGroupDev&, const T*, const T*, T*, int, \
                                         hipStream_t, T*, const CopyJob&, const LaunchPolicy&);                     \
  template hipError_t launch_copy_nodes<T>(const int32_t*, int64_t, const T*, T*, int64_t, hipStream_t, int);      \
  template hipError_t launch_cut_update<T>(const CutGroupDev&, const T*, T*, int64_t, hipStream_t, int);          \
  template hipError_t launch_prolong_add<T>(int, int, const KLevel&, const KLevel&, const T*, T*, hipStream_t,     \
                                            int);                                                                  \
  template hipError_t launch_restrict<T>(int, int, const KLevel&, const KLevel&, const T*, T*, hipStream_t, int); \
  template hipError_t launch_coarse<T>(const T*, const int32_t*, int, const T*, T*, int64_t, hipStream_t, int);  \
  template hipError_t launch_zero_active<T>(const int32_t*, int64_t, T*, int64_t, hipStream_t, int);
CMG_INSTANTIATE(double)
CMG_INSTANTIATE(float)
template hipError_t launch_scatter<double, double>(const int32_t*, int64_t, const double*, double*, int64_t,
                                                   hipStream_t, int);
template hipError_t launch_gather<double, double>(const int32_t*, int64_t, const double*, double*, int64_t,
                                                  hipStream_t, int);
template hipError_t launch_scatter<double, float>(const int32_t*, int64_t, const double*, float*, int64_t,
                                                  hipStream_t, int);
template hipError_t launch_gather<float, double>(const int32_t*, int64_t, const float*, double*, int64_t,
                                                 hipStream_t, int);

}  // namespace cmg

// ---------------------------------------------------------------------------
// Vector kernels of the Krylov solver on compact vectors.
namespace cmg {
namespace dev {

// Per-block partial sums of x . y (fixed order, so repeat runs are bitwise equal).
__global__ __launch_bounds__(256) void k_dot_partial(const double* __restrict__ x, const double* __restrict__ y,
                                                     int64_t n, double* __restrict__ part) {
  __shared__ double red[4];
  x += blockIdx.y * n;  // column blockIdx.y
  y += blockIdx.y * n;
  part += blockIdx.y * gridDim.x;
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    s += x[i] * y[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_axpy(int64_t n, double a, const double* __restrict__ x,
                                              double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] += a * x[i];
}

__global__ __launch_bounds__(256) void k_xpay(int64_t n, double a, const double* __restrict__ x,
                                              double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i] + a * y[i];
}

// part[j * gridDim.x + blockIdx.x]: partial sums of V_j . w for the rows j =
// blockIdx.y of V (rows of n entries), against one vector w.
__global__ __launch_bounds__(256) void k_rows_dot_partial(const double* __restrict__ V, const double* __restrict__ w,
                                                          int64_t n, double* __restrict__ part) {
  __shared__ double red[4];
  V += blockIdx.y * n;
  double s = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    s += V[i] * w[i];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
  if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// y += sum_{j < m} c.v[j] V_j (rows of n entries), in increasing j.
__global__ __launch_bounds__(256) void k_rows_combine(int64_t n, int m, RowCoef c, const double* __restrict__ V,
                                                      double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = y[i];
  for (int j = 0; j < m; ++j) acc += c.v[j] * V[j * n + i];
  y[i] = acc;
}

__global__ __launch_bounds__(256) void k_scale(int64_t n, double a, const double* __restrict__ x,
                                               double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = a * x[i];
}

// Column-wise forms: column c = blockIdx.y of n entries, coefficient a.v[c].
__global__ __launch_bounds__(256) void k_axpy_cols(int64_t n, ColCoef a, const double* __restrict__ x,
                                                   double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t o = blockIdx.y * n;
  if (i < n) y[o + i] += a.v[blockIdx.y] * x[o + i];
}

__global__ __launch_bounds__(256) void k_xpay_cols(int64_t n, ColCoef a, const double* __restrict__ x,
                                                   double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t o = blockIdx.y * n;
  if (i < n) y[o + i] = x[o + i] + a.v[blockIdx.y] * y[o + i];
}

}  // namespace dev

hipError_t launch_dot_partial(const double* x, const double* y, int64_t n, double* part, int nblk, hipStream_t s,
                              int ncol) {
  hipLaunchKernelGGL(dev::k_dot_partial, dim3(nblk, ncol), dim3(256), 0, s, x, y, n, part);
  return hipGetLastError();
}

hipError_t launch_rows_dot_partial(const double* V, const double* w, int64_t n, int m, double* part, int nblk,
                                   hipStream_t s) {
  hipLaunchKernelGGL(dev::k_rows_dot_partial, dim3(nblk, m), dim3(256), 0, s, V, w, n, part);
  return hipGetLastError();
}

hipError_t launch_rows_combine(int64_t n, int m, const RowCoef& c, const double* V, double* y, hipStream_t s) {
  if (n == 0 || m == 0) return hipSuccess;
  if (m > kMaxRows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(dev::k_rows_combine, dim3((n + 255) / 256), dim3(256), 0, s, n, m, c, V, y);
  return hipGetLastError();
}

hipError_t launch_scale(int64_t n, double a, const double* x, double* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_scale, dim3((n + 255) / 256), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

hipError_t launch_axpy_cols(int64_t n, const ColCoef& a, const double* x, double* y, int ncol, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_axpy_cols, dim3((n + 255) / 256, ncol), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

hipError_t launch_xpay_cols(int64_t n, const ColCoef& a, const double* x, double* y, int ncol, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_xpay_cols, dim3((n + 255) / 256, ncol), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

hipError_t launch_axpy(int64_t n, double a, const double* x, double* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_axpy, dim3((n + 255) / 256), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

hipError_t launch_xpay(int64_t n, double a, const double* x, double* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_xpay, dim3((n + 255) / 256), dim3(256), 0, s, n, a, x, y);
  return hipGetLastError();
}

}  // namespace cmg

namespace cmg {
namespace dev {

__global__ __launch_bounds__(256) void k_fill(int64_t n, double v, double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = v;
}

__global__ __launch_bounds__(256) void k_copy(int64_t n, const double* __restrict__ x, double* __restrict__ y) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) y[i] = x[i];
}

}  // namespace dev

// The array behind cmg_apply_noalloc.  In host code its name is a host-side
// stand-in, not a device address: the address is taken per device with
// hipGetSymbolAddress and only that address is passed to kernels or copies.
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t noalloc_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device) return hipErrorInvalidDevice;  // the address is per device: take it with that device current
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = ptr;
  return hipSuccess;
}

void* noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

hipError_t launch_fill(int64_t n, double v, double* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_fill, dim3((n + 255) / 256), dim3(256), 0, s, n, v, y);
  return hipGetLastError();
}

hipError_t launch_copy(int64_t n, const double* x, double* y, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(dev::k_copy, dim3((n + 255) / 256), dim3(256), 0, s, n, x, y);
  return hipGetLastError();
}

}  // namespace cmg

// ---- load vector of Fourier data on the device -----------------------------
namespace cmg {
namespace dev {

template <int K>
__device__ __forceinline__ void rhs_basis(const RhsPlanDev& R, double t, double* psi) {
#pragma unroll
  for (int a = 0; a <= K; ++a) {
    double v = R.coef[a][K];
#pragma unroll
    for (int m = K - 1; m >= 0; --m) v = v * t + R.coef[a][m];
    psi[a] = v;
  }
}

// Cell vectors of the uncut active cells: tensor Gauss rule with k+3 points
// per direction.  On a cell with corner lo every mode is a product,
//   cos(pi kappa . x + phase) = Re e^{i(phase + pi kappa . lo)} prod_j e^{i pi kappa_j h t_j},
// so the rule factorises: its sum against psi_a is one phase per cell and mode
// times a complex tensor T_q[a] = prod_j sum_g h w_g psi_{a_j}(g) e^{i pi kappa_j h g} that
// no cell enters.  Every block forms T_q in LDS; a thread then takes one cell,
// one sincospi per mode and 2 (k+1)^d multiply-adds instead of (k+3)^d cosines.
// Union of two balls, Q2, 64^3 cells, 16 modes, 15,382 uncut cells: 504 -> 25 us.
template <int D, int K>
__global__ __launch_bounds__(256) void k_rhs_uncut(RhsPlanDev R, RhsModes M) {
  constexpr int N1 = K + 1, NL = Pow<N1, D>::v, NG = K + 3;
  __shared__ double G[kMaxModes][D][N1][2];
  __shared__ double T[kMaxModes][NL][2];
  for (int t = threadIdx.x; t < M.n * D * N1; t += blockDim.x) {
    const int a = t % N1, j = (t / N1) % D, q = t / (N1 * D);
    double re = 0.0, im = 0.0;
    for (int g = 0; g < NG; ++g) {
      double psi[N1], s, c, pa = 0.0;
      rhs_basis<K>(R, R.gx[g], psi);
#pragma unroll
      for (int m = 0; m < N1; ++m) pa = m == a ? psi[m] : pa;
      sincospi(M.kappa[q][j] * (R.h * R.gx[g]), &s, &c);
      pa *= R.h * R.gw[g];
      re += pa * c;
      im += pa * s;
    }
    G[q][j][a][0] = re;
    G[q][j][a][1] = im;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < M.n * NL; t += blockDim.x) {
    const int q = t / NL;
    int ra = t % NL;
    double re = M.amp[q], im = 0.0;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const double gr = G[q][j][ra % N1][0], gi = G[q][j][ra % N1][1], r0 = re;
      ra /= N1;
      re = r0 * gr - im * gi;
      im = r0 * gi + im * gr;
    }
    T[q][t % NL][0] = re;
    T[q][t % NL][1] = im;
  }
  __syncthreads();
  const int64_t u = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (u >= R.n_uncut) return;
  const int c = R.uncut[u];
  double lo[3];
  {
    int r = c;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      lo[j] = R.lo + (r % R.N) * R.h;
      r /= R.N;
    }
  }
  double acc[NL];
#pragma unroll
  for (int a = 0; a < NL; ++a) acc[a] = 0.0;
  for (int q = 0; q < M.n; ++q) {
    double th = M.phase[q], sn, cs;
#pragma unroll
    for (int j = 0; j < D; ++j) th += M.kappa[q][j] * lo[j];
    sincospi(th, &sn, &cs);
#pragma unroll
    for (int a = 0; a < NL; ++a) acc[a] += cs * T[q][a][0] - sn * T[q][a][1];
  }
  double* out = R.loc + (int64_t)R.act_id[c] * NL;
#pragma unroll
  for (int a = 0; a < NL; ++a) out[a] = acc[a];
}

// Partial cell vectors of the cut cells: one block per chunk of at most
// kRhsChunk quadrature columns of one cell, one column per thread.  A kinked
// cell of a union has up to hundreds of times the columns of a smooth one, so
// a block per cell (the former split) ran as long as its longest cell's serial
// loop: 22,459 -> 858 us on the union of two balls, Q2, 64^3 cells, 16 modes (6.6
// million columns, 26,167 chunks; now bound by FP64 arithmetic, about 2,000
// operations a column).
// Along a column only direction e varies, so f there is sum_m C_m cos(pi m t)
// - S_m sin(pi m t) over the distinct m = kappa_e, with (C_m, S_m) summed over
// the modes of that m at the column's base point.  The modes come sorted by
// kappa_e (M.ord), and e^{i pi m t} moves from one m to the next by complex
// multiplication with e^{i pi t} (started again from sincospi after kRhsPow
// products, so at most that many roundings add up).  Each column leaves its
// 1-D factors in LDS (psi_a of the base point, along e the weighted sum of f
// psi_a), and the block then sums their products over the columns for every
// cell node, in a fixed order.
template <int D, int K, int NQ>
__global__ __launch_bounds__(256) void k_rhs_cut(RhsPlanDev R, RhsModes M) {
  constexpr int N1 = K + 1, NL = Pow<N1, D>::v, NG = kRhsChunk / NL;
  static_assert(NG >= 1, "a thread per cell node at least");
  __shared__ double F[D][N1][kRhsChunk + 1];
  __shared__ double gs[NG][NL];
  __shared__ double mk[D][kMaxModes][D], ma[D][kMaxModes], mp[D][kMaxModes];
  __shared__ int me[D][kMaxModes];
  for (int t = threadIdx.x; t < D * M.n; t += blockDim.x) {
    const int e = t / M.n, i = t % M.n, q = M.ord[e][i];
#pragma unroll
    for (int j = 0; j < D; ++j) mk[e][i][j] = j == e ? 0.0 : (double)M.kappa[q][j];
    ma[e][i] = M.amp[q];
    mp[e][i] = M.phase[q];
    me[e][i] = M.kappa[q][e];
  }
  const int ch = blockIdx.x;
  const int ci = R.chunk_cell[ch];
  const int64_t c0 = R.col_off[ci] + (int64_t)kRhsChunk * (ch - R.chunk_off[ci]);
  const int64_t left = R.col_off[ci + 1] - c0;
  const int n = left < kRhsChunk ? (int)left : kRhsChunk;
  __syncthreads();
  const int tid = threadIdx.x;
  if (tid < n) {
    const int64_t col = c0 + tid;
    double lo[D], x[D];
    {
      int r = R.cut[ci];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        lo[j] = R.lo + (r % R.N) * R.h;
        r /= R.N;
      }
    }
    const int e = R.ce[col];
#pragma unroll
    for (int j = 0; j < D; ++j) x[j] = R.cx[j * R.n_col + col];
    const double w = R.cw[col], t0 = R.ct0[col], len = R.ct1[col] - t0;
    double f[NQ], zr[NQ], zi[NQ], pr[NQ], pi[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      f[t] = 0.0;
      sincospi(t0 + len * R.tx[t], &zi[t], &zr[t]);
      pr[t] = 1.0;
      pi[t] = 0.0;
    }
    int cur = 0, used = 0;  // e^{i pi cur t} is held; products since it was last formed
    for (int i = 0; i < M.n;) {
      const int m = me[e][i];
      double C = 0.0, S = 0.0;
      do {
        double th = mp[e][i], sn, cs;
#pragma unroll
        for (int j = 0; j < D; ++j) th += j == e ? 0.0 : mk[e][i][j] * x[j];
        sincospi(th, &sn, &cs);
        C += ma[e][i] * cs;
        S += ma[e][i] * sn;
        ++i;
      } while (i < M.n && me[e][i] == m);
      if (m < cur || (unsigned)m - (unsigned)cur > (unsigned)(kRhsPow - used)) {
#pragma unroll
        for (int t = 0; t < NQ; ++t) sincospi(m * (t0 + len * R.tx[t]), &pi[t], &pr[t]);
        used = 0;
      } else {
        for (int s = cur; s < m; ++s) {
#pragma unroll
          for (int t = 0; t < NQ; ++t) {
            const double r0 = pr[t];
            pr[t] = r0 * zr[t] - pi[t] * zi[t];
            pi[t] = r0 * zi[t] + pi[t] * zr[t];
          }
        }
        used += m - cur;
      }
      cur = m;
#pragma unroll
      for (int t = 0; t < NQ; ++t) f[t] += C * pr[t] - S * pi[t];
    }
    double loe = lo[0];
#pragma unroll
    for (int j = 1; j < D; ++j) loe = j == e ? lo[j] : loe;
    double ae[N1];
#pragma unroll
    for (int a = 0; a < N1; ++a) ae[a] = 0.0;
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
      double pe[N1];
      rhs_basis<K>(R, (t0 + len * R.tx[t] - loe) / R.h, pe);
      const double fv = f[t] * w * len * R.tw[t];
#pragma unroll
      for (int a = 0; a < N1; ++a) ae[a] += fv * pe[a];
    }
#pragma unroll
    for (int j = 0; j < D; ++j) {
      double psi[N1];
      rhs_basis<K>(R, (x[j] - lo[j]) / R.h, psi);
#pragma unroll
      for (int a = 0; a < N1; ++a) F[j][a][tid] = j == e ? ae[a] : psi[a];
    }
  }
  __syncthreads();
  const int g = tid / NL, a = tid % NL;
  constexpr int RUN = (kRhsChunk + NG - 1) / NG;  // columns of one group of NL threads
  if (g < NG) {
    const double* fa[D];
    int ra = a;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      fa[j] = F[j][ra % N1];
      ra /= N1;
    }
    double s = 0.0;
    const int hi = (g + 1) * RUN < n ? (g + 1) * RUN : n;
    for (int q = g * RUN; q < hi; ++q) {
      double v = fa[0][q];
#pragma unroll
      for (int j = 1; j < D; ++j) v *= fa[j][q];
      s += v;
    }
    gs[g][a] = s;
  }
  __syncthreads();
  if (tid < NL) {
    double s = gs[0][tid];
#pragma unroll 1
    for (int q = 1; q < NG; ++q) s += gs[q][tid];
    R.part[(int64_t)ch * NL + tid] = s;
  }
}

// Cell vectors of the cut cells: the partial vectors of a cell's chunks summed
// in a fixed order (groups of NL threads take every NG-th chunk, then the
// groups in order); zero for a cell without columns.
template <int D, int K>
__global__ __launch_bounds__(256) void k_rhs_cut_sum(RhsPlanDev R) {
  constexpr int NL = Pow<K + 1, D>::v, NG = 256 / NL;
  __shared__ double gs[NG][NL];
  const int ci = blockIdx.x, g = threadIdx.x / NL, a = threadIdx.x % NL;
  const int lo = R.chunk_off[ci], hi = R.chunk_off[ci + 1];
  if (g < NG) {
    double s = 0.0;
#pragma unroll 8
    for (int q = lo + g; q < hi; q += NG) s += R.part[(int64_t)q * NL + a];
    gs[g][a] = s;
  }
  __syncthreads();
  if (threadIdx.x < NL) {
    double s = gs[0][a];
    for (int q = 1; q < NG && q < hi - lo; ++q) s += gs[q][a];
    R.loc[(int64_t)R.act_id[R.cut[ci]] * NL + a] = s;
  }
}

// b at every DoF: the cell vectors of the (up to 2^d) active cells that
// contain its node, in a fixed order.
template <int D, int K>
__global__ __launch_bounds__(256) void k_rhs_gather(RhsPlanDev R, const int32_t* __restrict__ dof_node,
                                                    int64_t n, double* __restrict__ b) {
  constexpr int N1 = K + 1;
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  int I[3];
  {
    int r = dof_node[i];
#pragma unroll
    for (int j = 0; j < D; ++j) {
      I[j] = r % R.nn;
      r /= R.nn;
    }
  }
  double v = 0.0;
#pragma unroll
  for (int comb = 0; comb < (1 << D); ++comb) {
    int cell = 0, loc = 0, sc = 1, sl = 1;
    bool ok = true;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      const int sel = (comb >> j) & 1;  // 0: the cell below the node (or the one holding it), 1: above
      int cj, lj;
      if (I[j] % K == 0) {
        cj = I[j] / K - 1 + sel;
        lj = sel ? 0 : K;
      } else {
        ok = ok && sel == 0;
        cj = I[j] / K;
        lj = I[j] % K;
      }
      ok = ok && cj >= 0 && cj < R.N;
      cell += cj * sc;
      loc += lj * sl;
      sc *= R.N;
      sl *= N1;
    }
    if (!ok) continue;
    const int a = R.act_id[cell];
    if (a >= 0) v += R.loc[(int64_t)a * Pow<N1, D>::v + loc];
  }
  b[i] = v;
}

}  // namespace dev

hipError_t launch_rhs_fourier(int d, int k, const RhsPlanDev& R, const RhsModes& M, const int32_t* dof_node,
                              int64_t n_dofs, double* b, hipStream_t s) {
  return dispatch(d, k, [&](auto D, auto K) {
    if (R.n_uncut > 0)
      hipLaunchKernelGGL((dev::k_rhs_uncut<D.value, K.value>), dim3(static_cast<unsigned>((R.n_uncut + 255) / 256)),
                         dim3(256), 0, s, R, M);
    if (R.n_chunk > 0) {
      const dim3 g(static_cast<unsigned>(R.n_chunk)), t(kRhsChunk);
      // quad_n points in registers; the default rule has 14, any other is padded to 16 with zero weights
      if (R.nq == 14)
        hipLaunchKernelGGL((dev::k_rhs_cut<D.value, K.value, 14>), g, t, 0, s, R, M);
      else
        hipLaunchKernelGGL((dev::k_rhs_cut<D.value, K.value, 16>), g, t, 0, s, R, M);
    }
    if (R.n_cut > 0)
      hipLaunchKernelGGL((dev::k_rhs_cut_sum<D.value, K.value>), dim3(static_cast<unsigned>(R.n_cut)), dim3(256), 0,
                         s, R);
    if (n_dofs > 0)
      hipLaunchKernelGGL((dev::k_rhs_gather<D.value, K.value>), dim3(static_cast<unsigned>((n_dofs + 255) / 256)),
                         dim3(256), 0, s, R, dof_node, n_dofs, b);
    return hipGetLastError();
  });
}

}  // namespace cmg
