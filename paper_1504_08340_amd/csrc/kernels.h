// HIP kernels of the hot path (CDNA4 / gfx950).
//
//   element_kernel (element.h): the element operators of a stage and the
//                             gradient terms.
//   nodal_rk_kernel         : nodal PML terms, M^{-1}, classical RK4 stage
//                             combination of (6), source injection.
//
// Register layout (per source, type R): U part 6 x n_nodes
//   [x1 u_x, u_y, u_z | x2 u_x, u_y, u_z] on the full grid, then P part
//   21 x n_pml [x0 u (3) | x0 S (6) | x1 S (6) | x2 S (6)] on the PML shell.
//   Stress order (xx, yy, zz, yz, xz, xy).
//
// Element work is done per tile of bricks.  Scatter without atomics: a node
// lies on the upper face (local index 2*count) of at most one tile per axis, so
// the set c of axes on which it is an upper-face node differs for every tile
// containing it.  A tile stores its partial sum for a box node with a plain
// store into partial
// array c; the nodal kernel adds the arrays c that can be non-zero for the
// node.  Array 0 uses the register index spaces (full grid for u-rows, PML
// shell for S-rows); arrays c != 0 use the full grid with the axes in c
// compressed to the upper-face positions.  Entries nobody writes stay zero
// from the initial clear.
//
// Tiles are handed to the XCDs in contiguous runs: workgroup b of a grid
// whose size is a multiple of 8 runs on XCD b mod 8 and takes tile
// (b mod 8) * (grid/8) + b / 8, so neighbouring tiles share an L2.
#pragma once
#include "geometry.h"

// Element tiles (bricks per axis).  5x4x2 cuts the 5-brick PML and the
// 40x40x20-brick interior without ragged tiles along x and y.
#ifndef PMLFWI_TX
#define PMLFWI_TX 5
#define PMLFWI_TY 4
#define PMLFWI_TZ 2
#endif
// Threads that hold one node each of a tile's node box: 512 fits the
// 11 x 9 x 5 node box of a 5x4x2 tile.
#ifndef PMLFWI_ETHREADS
#define PMLFWI_ETHREADS 512
#endif
// Threads per nodal workgroup (128 measured a little faster than 256, 512 slower).
#ifndef PMLFWI_NODAL_THREADS
#define PMLFWI_NODAL_THREADS 128
#endif

namespace pmlfwi {

enum { P_X0U = 0, P_X0S = 3, P_X1S = 9, P_X2S = 15, P_NCOMP = 21, U_NCOMP = 6 };

// State register of one source.  Node part: x1 u as [sn][3], then x2 u as
// [sn][3]; PML part (from entry 6 sn): x0 u as [sp][3], then x0 S, x1 S and
// x2 S as [sp][6] each.  A field's components at a node are contiguous, so a
// kernel loads or stores them as one vector.
// Entry of u-component d (0..2: x1 u, 3..5: x2 u) of node `node`:
__host__ __device__ __forceinline__ size_t u_at(size_t nn, int d, size_t node) {
  return d < 3 ? 3 * node + d : 3 * nn + 3 * node + (d - 3);
}
// Entry of PML component q (P_X0U .. P_NCOMP-1) of PML node p, relative to
// the PML part:
__host__ __device__ __forceinline__ size_t p_at(size_t np, int q, size_t p) {
  if (q < P_X0S) return 3 * p + q;
  const int b = q < P_X1S ? P_X0S : (q < P_X2S ? P_X1S : P_X2S);
  return (size_t)b * np + 6 * p + (q - b);
}

// Voigt slot of the symmetric pair (i, k).
__host__ __device__ constexpr int vidx(int i, int k) { return i == k ? i : 6 - i - k; }

// Derivative of 1D basis a at LGL point q: D[q][a] (nodes -1, 0, 1).
__device__ __forceinline__ float dlgl(int q, int a) {
  // rows q = 0: (-3/2, 2, -1/2); q = 1: (-1/2, 0, 1/2); q = 2: (1/2, -2, 3/2)
  const float r0 = a == 0 ? -1.5f : (a == 1 ? 2.0f : -0.5f);
  const float r1 = a == 0 ? -0.5f : (a == 1 ? 0.0f : 0.5f);
  const float r2 = a == 0 ? 0.5f : (a == 1 ? -2.0f : 1.5f);
  return q == 0 ? r0 : (q == 1 ? r1 : r2);
}
__device__ __forceinline__ double wlgl(int a) { return a == 1 ? 4.0 / 3.0 : 1.0 / 3.0; }

struct Tile {  // bricks [x, x+cx) x [y, y+cy) x [z, z+cz)
  int x, y, z, c;  // c = cx | cy << 8 | cz << 16
};

struct Part {             // partial residual arrays of one source
  long long off[8];       // element offset of array c (array 0 at 0)
  long long size[8];      // nodes of array c (c != 0: compressed box)
  int nx[8], ny[8];       // x / y extents of array c
  long long per_src;      // elements per source
};

__device__ __forceinline__ int face_mask(const Geo& g, int i, int j, int k) {
  return (g.fo[i] >= 0) | ((g.fo[ax_y(g) + j] >= 0) << 1) | ((g.fo[ax_z(g) + k] >= 0) << 2);
}

__device__ __forceinline__ size_t part_node(const Geo& g, const Part& P, int c, int i, int j, int k) {
  const int ii = (c & 1) ? g.fo[i] : i;
  const int jj = (c & 2) ? g.fo[ax_y(g) + j] : j;
  const int kk = (c & 4) ? g.fo[ax_z(g) + k] : k;
  return (size_t)ii + (size_t)P.nx[c] * ((size_t)jj + (size_t)P.ny[c] * kk);
}

// Offsets of a node's rows in partial array c (within one source).  A node's
// rows are contiguous, so they are stored and gathered as short vectors: array
// 0 holds the three u-rows of every node ([sn][3]) followed by the six S-rows
// of every PML node ([sp][6]); array c != 0 holds [size_c][3] u-rows followed
// by [size_c][6] S-rows, indexed by the node's place in the compressed box.
// u-row d sits at u + d, S-row v at s + v.  Computed once per node before its
// stores, so the lane-varying lookups of the array constants and face
// ordinals are waited for once rather than once per row.
struct RowAddr {
  size_t u, s;
};

__device__ __forceinline__ RowAddr row_addr(const Geo& g, const Part& P, int c, int i, int j, int k,
                                            size_t node, size_t p) {
  RowAddr a;
  if (c == 0) {
    a.u = 3 * node;
    a.s = 3 * (size_t)g.sn + 6 * p;
    return a;
  }
  const size_t n = part_node(g, P, c, i, j, k);
  a.u = (size_t)P.off[c] + 3 * n;
  a.s = (size_t)P.off[c] + 3 * (size_t)P.size[c] + 6 * n;
  return a;
}

__device__ __forceinline__ int xcd_tile() {
  const int per = gridDim.x >> 3;
  const int b = blockIdx.x;
  return (b & 7) * per + (b >> 3);
}

// Per-dimension list of the bricks of a tile that contain local node l:
// (brick offset, position of the node in that brick).  At most two.
__device__ __forceinline__ int node_bricks(int l, int cnt, int* e, int* p) {
  if (l & 1) {
    e[0] = (l - 1) >> 1;
    p[0] = 1;
    e[1] = e[0];
    p[1] = 1;
    return 1;
  }
  int n = 0;
  if (l >= 2) {
    e[n] = (l >> 1) - 1;
    p[n] = 2;
    ++n;
  }
  if ((l >> 1) < cnt) {
    e[n] = l >> 1;
    p[n] = 0;
    ++n;
  }
  if (n == 1) {
    e[1] = e[0];
    p[1] = p[0];
  }
  return n;
}

// The two candidate bricks of a tile along one axis for local node l
// (0 <= l <= 2 cnt): the brick below (l odd: the only one) and the brick above
// (l even), as offsets se * brick + sp * (position of the node in the brick)
// into brick-local arrays, each with a flag telling whether it holds the node.
__device__ __forceinline__ void axis_bricks(int l, int cnt, int se, int sp, int o[2], bool v[2]) {
  const int e0 = (l - 1) >> 1, e1 = l >> 1;
  o[0] = se * e0 + sp * (l - 2 * e0);
  o[1] = se * e1 + sp * (l - 2 * e1);
  v[0] = l >= 1;
  v[1] = !(l & 1) && e1 < cnt;
}

template <typename R>
__device__ __forceinline__ void atomic_add(R* p, R v) {
  unsafeAtomicAdd(p, v);
}

// ---------------------------------------------------------------------------
// PML bricks.  Forward (ADJ = false), for the input register (x0, x1, x2):
//   u-rows:  r_u += int grad w~ : (S' Le + S Lp + Sbar Lw)
//   S-rows:  r_S -= int T~ : (mu (H + H^T) + lam tr(H) I),
//            H_ik = d/dx_k (Le_kk u'_i + Lp_kk u_i + Lw_kk ubar_i)
// Transposed (ADJ = true): the same blocks transposed, applied to the adjoint
// register (y0, y1, y2) in the slots of (x0, x1, x2):
//   u-rows:  r_u += int grad w~ : T',  T'_ik = -(mu (1+d_ik) Z_k,ik + lam d_ik tr Z_i),
//            Z_k = Le_kk T2 + Lp_kk T1 + Lw_kk T0 (symmetric stress-like fields)
//   S-rows:  r_S += int T~_ab (H_ab + H_ba)  (a != b),  H_aa  (a = b).
//
// The S-rows depend on the displacements only (through W and Q) and the
// u-rows on the stresses only (through T), so the operator splits into two
// independent parts.
enum { PML_SROWS = 1, PML_UROWS = 2 };

template <typename R>
struct PmlNode {          // register values of one box node for one source
  R u1[3], u2[3], u0[3], s0[6], s1[6], s2[6];
};

template <typename R, bool U, bool S>
__device__ __forceinline__ void pml_load_node(const R* __restrict__ Y, size_t nn, size_t np, size_t gnode,
                                              size_t gp, bool hist, PmlNode<R>& v) {
  const R* P = Y + 6 * nn;
  if constexpr (U) {
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      v.u1[d] = Y[u_at(nn, d, gnode)];
      v.u2[d] = Y[u_at(nn, 3 + d, gnode)];
      v.u0[d] = hist ? P[p_at(np, P_X0U + d, gp)] : R(0);
    }
  }
  if constexpr (S) {
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      v.s1[c] = P[p_at(np, P_X1S + c, gp)];
      v.s2[c] = P[p_at(np, P_X2S + c, gp)];
      v.s0[c] = hist ? P[p_at(np, P_X0S + c, gp)] : R(0);
    }
  }
}

// Phase 1 for one node: W (U) from the displacements.
template <typename R, int NB>
__device__ __forceinline__ void pml_node_w(const PmlNode<R>& v, const R Le[3], const R Lp[3], const R Lw[3], int n,
                                           R (&sW)[9][NB]) {
#pragma unroll
  for (int kk = 0; kk < 3; ++kk)
#pragma unroll
    for (int ii = 0; ii < 3; ++ii) sW[3 * kk + ii][n] = Le[kk] * v.u2[ii] + Lp[kk] * v.u1[ii] + Lw[kk] * v.u0[ii];
}

// Phase 1 for one node: T from the stresses.
template <typename R, bool ADJ, int NB>
__device__ __forceinline__ void pml_node_t(const PmlNode<R>& v, const R Le[3], const R Lp[3], const R Lw[3], R la,
                                           R m, int n, R (&sT)[9][NB]) {
  if constexpr (!ADJ) {
#pragma unroll
    for (int ii = 0; ii < 3; ++ii)
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        const int c = vidx(ii, kk);
        sT[3 * ii + kk][n] = Le[kk] * v.s2[c] + Lp[kk] * v.s1[c] + Lw[kk] * v.s0[c];
      }
  } else {
    const R t2 = v.s2[0] + v.s2[1] + v.s2[2], t1 = v.s1[0] + v.s1[1] + v.s1[2], t0 = v.s0[0] + v.s0[1] + v.s0[2];
#pragma unroll
    for (int ii = 0; ii < 3; ++ii)
#pragma unroll
      for (int kk = 0; kk < 3; ++kk) {
        const int c = vidx(ii, kk);
        const R z = Le[kk] * v.s2[c] + Lp[kk] * v.s1[c] + Lw[kk] * v.s0[c];
        R val = (ii == kk ? R(2) : R(1)) * m * z;
        if (ii == kk) val += la * (Le[ii] * t2 + Lp[ii] * t1 + Lw[ii] * t0);
        sT[3 * ii + kk][n] = -val;
      }
  }
}

// Phase 3, S-rows of box node (lx, ly, lz): the sum of the point values of
// every tile brick containing the node.
template <typename R, int TX, int TY, int TZ>
__device__ __forceinline__ void pml_s_rows(int cx, int cy, int cz, int lx, int ly, int lz,
                                           const R* __restrict__ sQ, R q6[6]) {
  constexpr int NP = 27 * TX * TY * TZ;
  int ox[2], oy[2], oz[2];
  bool vx[2], vy[2], vz[2];
  axis_bricks(lx, cx, 27, 1, ox, vx);
  axis_bricks(ly, cy, 27 * TX, 3, oy, vy);
  axis_bricks(lz, cz, 27 * TX * TY, 9, oz, vz);
#pragma unroll
  for (int v = 0; v < 6; ++v) q6[v] = 0;
#pragma unroll
  for (int a3 = 0; a3 < 2; ++a3)
#pragma unroll
    for (int a2 = 0; a2 < 2; ++a2)
#pragma unroll
      for (int a1 = 0; a1 < 2; ++a1) {
        if (!(vx[a1] && vy[a2] && vz[a3])) continue;
        const int qn = ox[a1] + oy[a2] + oz[a3];
#pragma unroll
        for (int v = 0; v < 6; ++v) q6[v] += sQ[v * NP + qn];
      }
}

// Per-node constants of phase 1: PML coefficients, history flag, indices.
template <typename R>
__device__ __forceinline__ void pml_node_setup(const Geo& g, int gi, int gj, int gk, R Le[3], R Lp[3], R Lw[3],
                                               bool& hist, size_t& gnode, size_t& gp) {
  gnode = (size_t)gi + (size_t)g.NX * (gj + (size_t)g.NY * gk);
  gp = (size_t)pml_index(g, gi, gj, gk);
  // products of the 1D stretching factors in the state precision
  const int nt = ax_n(g);
  const double* A = g.tab;
  const double* B = g.tab + nt;
  const R ax = R(A[gi]), ay = R(A[ax_y(g) + gj]), az = R(A[ax_z(g) + gk]);
  const R bx = R(B[gi]), by = R(B[ax_y(g) + gj]), bz = R(B[ax_z(g) + gk]);
  hist = (B[gi] > 0.0) + (B[ax_y(g) + gj] > 0.0) + (B[ax_z(g) + gk] > 0.0) >= 2;   // as the layout decides
  Le[0] = ay * az; Lp[0] = ay * bz + by * az; Lw[0] = by * bz;
  Le[1] = ax * az; Lp[1] = ax * bz + bx * az; Lw[1] = bx * bz;
  Le[2] = ax * ay; Lp[2] = ax * by + bx * ay; Lw[2] = bx * by;
}

// Nodal part of one RK4 stage.  With r the element residual of the stage input
// Y, the rates are K = (x1|PML, x2, M^{-1}(f - r - nodal PML terms)) and the
// stages keep their own registers, Y1 = Xn, Y2, Y3, Y4:
//   modes 0, 1:  Yout = Xn + cY K   (mode 0: the stage input is Xn)
//   mode 2:      Xn += h/6 (K1 + 2 K2 + 2 K3 + K4), from what the registers hold:
//                x0, x1 rows: K_s is the x1, x2 row of Y_s, so they sum rates;
//                x2 rows:     h/2 K1 = Y2 - Xn, h/2 K2 = Y3 - Xn, h K3 = Y4 - Xn
//                (differences of near values, exact or nearly so), K4 at hand.
// Bound by HBM: FP32 moves its counted bytes at 5.1-5.5 TB/s, FP64 at 4.6-4.9,
// where a plain stream of 3 reads and 2 writes of the same sizes reaches 6.4.
// Kept registers cost less than an accumulator: per step an x1 row is read and
// written 8 times and an x2 row 13 times, against 16 times each with acc += c K
// in every stage.  The x0 S and x1 rows take one rounding of the sum instead of
// one per stage; the x2 rows, and the stage 1 term of the x0 u rows, carry the
// roundings of the stages' registers as an accumulator would.  Measured (62,500
// bricks, 4 sources, mean per stage): FP32 99 -> 76 us, FP64 232 -> 174 us;
// error of FP32 traces after 400 steps of 864 bricks against FP64 4.0e-7 ->
// 2.1e-7.
template <typename R>
struct NodalArgs {
  const R* Yin;
  R* Yout;
  R* Xn;
  const R* Y2;                // mode 2: the inputs of stages 2 and 3
  const R* Y3;
  const R* res;               // partial arrays of source 0
  Part part;
  const R* invMu;
  long long reg;
  R cY;                       // modes 0, 1: dt/2 or dt; mode 2: dt/6
  const int* src_node;        // nullptr: no load
  const double* src_dir;      // (nsrc, 3)
  const double* wav;          // (nsrc, wav_len)
  int wav_len, wav_idx;
  R* store;                   // x1 displacement ([si][3]) of the produced register on the
  long long store_stride;     // interior closure (per source stride), or nullptr
  R* pstore;                  // PML displacement fields of the produced register
  long long pstore_stride;    // [x1 u | x2 u | x0 u] x sp per source, or nullptr
  long long rows;             // rows of this launch: [0, sn) node rows, then PML rows
  unsigned rot;               // workgroup b takes rows of block (b + rot) mod the grid
};

// Where a node's contributions sit in the partial arrays: array 0 always, and
// array c != 0 when every axis of c is an upper-face axis of the node.
struct PartSlots {
  int mask;
  size_t nc[8];   // node index inside array c (c != 0: compressed box)
};

__device__ __forceinline__ PartSlots part_slots(const Geo& g, const Part& P, int i, int j, int k) {
  PartSlots S;
  const int fx = g.fo[i], fy = g.fo[ax_y(g) + j], fz = g.fo[ax_z(g) + k];
  S.mask = (fx >= 0) | ((fy >= 0) << 1) | ((fz >= 0) << 2);
#pragma unroll
  for (int c = 1; c < 8; ++c) {
    const int ii = (c & 1) ? fx : i, jj = (c & 2) ? fy : j, kk = (c & 4) ? fz : k;
    S.nc[c] = (size_t)ii + (size_t)P.nx[c] * ((size_t)jj + (size_t)P.ny[c] * kk);
  }
  return S;
}

// Sum over the partial arrays of a node's NR = 3 u-rows (SROWS false; base0 =
// 3 node) or NR = 6 S-rows (SROWS true; base0 = 3 sn + 6 p), each array's rows
// read as one contiguous vector.  The single-axis arrays (c = 1, 2, 4) are read
// unconditionally, at their first node when the node is not on that face, and
// the values are discarded by a select: the loads then issue together with the
// others instead of one branch at a time.  Nodes on two or three faces (1/32
// of the nodes or fewer per array) take a branch.
template <typename R, int NR, bool SROWS>
__device__ __forceinline__ void gather_rows(const Part& P, const PartSlots& S, const R* res, size_t base0,
                                            R out[NR]) {
  auto first = [&](int c, size_t n) {
    return (size_t)P.off[c] + (SROWS ? 3 * (size_t)P.size[c] + 6 * n : 3 * n);
  };
  R t[3][NR];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const int c = 1 << b;
    const bool on = (S.mask & c) != 0;
    const size_t o = first(c, on ? S.nc[c] : 0);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const R v = res[o + r];
      t[b][r] = on ? v : R(0);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) out[r] = __builtin_nontemporal_load(&res[base0 + r]) + t[0][r] + t[1][r] + t[2][r];
  if (S.mask == 3 || S.mask == 5 || S.mask == 6 || S.mask == 7) {
#pragma unroll
    for (int c = 3; c < 8; ++c)
      if (c != 4 && (S.mask & c) == c) {
        const size_t o = first(c, S.nc[c]);
#pragma unroll
        for (int r = 0; r < NR; ++r) out[r] += res[o + r];
      }
  }
}

// Nodal part of one stage for node rows and PML rows; MODE as described above,
// STORE >= 1 writes the produced x1 displacement on the interior closure,
// STORE = 2 also the PML displacement fields (full gradient).
// Threads [0, sn) take the displacement rows of node gid (none past n_nodes),
// threads [sn, sn + n_pml) the PML rows; every load of a thread is issued
// before its first store, first those that need no table, then the tables, then
// what these tell, so that few waits follow one another (62,500 bricks, 4
// sources, stages 1, 2 and 4: FP32 60.5, 76.5, 98 -> 59.0, 75.7, 93.5 us; FP64
// 141, 170, 227 -> 140, 166, 222 us).  With the history rows also before the
// gather, the registers for them cost FP32 a wave and stage 4 98 us.  The kept stage displacement is written, and Xn, the
// stage inputs and the residual partials are read, with non-temporal hints:
// none of them is touched again before the next stage's nodal pass (the kept
// displacement not before the adjoint), so they should not displace the stage
// output that the next element launch reads.
template <typename R, int MODE, int STORE>
__global__ void __launch_bounds__(PMLFWI_NODAL_THREADS) nodal_rk_kernel(Geo g, NodalArgs<R> A) {
  const int src = blockIdx.y;
  const unsigned turned = blockIdx.x + A.rot, blk = turned < gridDim.x ? turned : turned - gridDim.x;
  const long long gid = (long long)blk * blockDim.x + threadIdx.x;
  if (gid >= A.rows) return;
  const size_t nn = (size_t)g.sn, np = (size_t)g.sp;
  const size_t so = (size_t)src * A.reg;
  const R* Y = A.Yin + so;
  R* X = A.Xn + so;
  R* D = MODE == 2 ? X : A.Yout + so;      // the produced register
  const R* Y2 = MODE == 2 ? A.Y2 + so : nullptr;
  const R* Y3 = MODE == 2 ? A.Y3 + so : nullptr;
  const R* __restrict__ res = A.res + (size_t)src * A.part.per_src;
  const R cY = A.cY, third = R(1.0 / 3.0);
  // NV values of a field at entry o of a register
  auto fetch = [](const R* p, size_t o, auto& v) {
    constexpr int n = sizeof(v) / sizeof(R);
#pragma unroll
    for (int q = 0; q < n; ++q) v[q] = __builtin_nontemporal_load(&p[o + q]);
  };
  auto put = [](R* p, size_t o, const auto& v) {
    constexpr int n = sizeof(v) / sizeof(R);
#pragma unroll
    for (int q = 0; q < n; ++q) p[o + q] = v[q];
  };
  // the produced value of an x0 or x1 row (rates r1 .. r4: the next row of the
  // four stage inputs; modes 0 and 1: r4 the input's) and of an x2 row (y2 ..
  // y4: that row of the inputs, k its rate)
  auto advance = [&](R x, R r1, R r2, R r3, R r4) {
    if (MODE == 2) return x + cY * (r1 + r4 + 2 * (r2 + r3));
    return x + cY * r4;
  };
  auto advance2 = [&](R x, R y2, R y3, R y4, R k) {
    if (MODE == 2) return x + third * ((y2 - x) + 2 * (y3 - x) + (y4 - x) + 3 * cY * k);
    return x + cY * k;
  };

  if (gid < (long long)nn) {
    if (gid >= g.n_nodes) return;
    const int node = (int)gid;
    const int k = node / g.plane;
    const int r_ = node - k * g.plane;
    const int j = r_ / g.NX, i = r_ - j * g.NX;
    if (is_dirichlet(g, i, j, k)) return;
    const bool pml = in_pml(g, i, j, k);
    // what needs no table goes out first, then the tables, then what they tell
    R u2[3], rr[3], x1[3], x2[3], y2[3] = {0, 0, 0}, y3[3] = {0, 0, 0};
    const size_t o1 = u_at(nn, 0, node), o2 = u_at(nn, 3, node);   // x1 u, x2 u of the node
    fetch(X, o1, x1);
    fetch(X, o2, x2);
    if (MODE == 0) {          // the first stage's input is Xn itself
#pragma unroll
      for (int d = 0; d < 3; ++d) u2[d] = x2[d];
    } else {
      fetch(Y, o2, u2);
    }
    if (MODE == 2) {
      fetch(Y2, o2, y2);
      fetch(Y3, o2, y3);
    }
    const R im = A.invMu[node];
    const PartSlots PS = part_slots(g, A.part, i, j, k);
    R kap = 0, cb = 0, cc = 0, cd = 0, h1[3] = {0, 0, 0}, h0[3] = {0, 0, 0};
    if (pml) {
      double mrd, mp;
      lumped_masses_tab(g, i, j, k, mrd, mp);
      const PmlCoef c = pml_coef_tab(g, i, j, k);
      kap = R(mp) / (R(mrd) + R(c.a) * R(mp));
      cb = R(c.b);
      if (c.nbeta >= 2) {     // c and d vanish elsewhere
        cc = R(c.c);
        cd = R(c.d);
        const R* P = Y + 6 * nn + p_at(np, P_X0U, (size_t)pml_index(g, i, j, k));
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          h1[d] = MODE == 0 ? x1[d] : Y[o1 + d];
          h0[d] = P[d];
        }
      }
    }
    gather_rows<R, 3, false>(A.part, PS, res, 3 * (size_t)node, rr);
    R a2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) a2[d] = -im * rr[d];
    if (A.src_node && A.src_node[src] == node) {
      const double s = A.wav[(size_t)src * A.wav_len + A.wav_idx];
#pragma unroll
      for (int d = 0; d < 3; ++d) a2[d] += im * R(A.src_dir[3 * src + d] * s);
    }
    if (pml) {
#pragma unroll
      for (int d = 0; d < 3; ++d) a2[d] -= kap * (cb * u2[d] + (cc * h1[d] + cd * h0[d]));
    }
    R out1[3], out2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      out1[d] = advance(x1[d], x2[d], y2[d], y3[d], u2[d]);
      out2[d] = advance2(x2[d], y2[d], y3[d], u2[d], a2[d]);
    }
    put(D, o1, out1);
    put(D, o2, out2);
    if (STORE == 2 && pml) {
      R* PS_ = A.pstore + (size_t)src * A.pstore_stride;
      const size_t p = (size_t)pml_index(g, i, j, k);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        PS_[(size_t)d * np + p] = out1[d];
        PS_[(size_t)(3 + d) * np + p] = out2[d];
      }
    }
    if (STORE) {
      const int mi = interior_index(g, i, j, k);
      if (mi >= 0) {
        R* S = A.store + (size_t)src * A.store_stride;
#pragma unroll
        for (int d = 0; d < 3; ++d) __builtin_nontemporal_store(out1[d], &S[3 * (size_t)mi + d]);
      }
    }
    return;
  }
  const long long pp = gid - (long long)nn;
  if (pp >= (long long)g.n_pml) return;
  const size_t p = (size_t)pp;
  int i, j, k;
  pml_coords(g, (int)p, i, j, k);
  const size_t P0 = 6 * nn;                 // the registers' PML part
  // x0 u: 3 components, on history nodes off the Dirichlet boundary; x0 S: 6,
  // on history nodes; x1 S, x2 S: 6 each.  A field's components move with one
  // vector load or store.
  const size_t b0u = P0 + p_at(np, P_X0U, p), b0s = P0 + p_at(np, P_X0S, p);
  const size_t b1s = P0 + p_at(np, P_X1S, p), b2s = P0 + p_at(np, P_X2S, p);
  R rv[6], s2[6], x1[6], x2[6], y2[6] = {0, 0, 0, 0, 0, 0}, y3[6] = {0, 0, 0, 0, 0, 0}, t[6];
  fetch(X, b1s, x1);
  fetch(X, b2s, x2);
  if (MODE == 0) {
#pragma unroll
    for (int v = 0; v < 6; ++v) s2[v] = x2[v];
  } else {
    fetch(Y, b2s, s2);
  }
  if (MODE == 2) {
    fetch(Y2, b2s, y2);
    fetch(Y3, b2s, y3);
  }
  const PartSlots PS = part_slots(g, A.part, i, j, k);
  const PmlCoef c = pml_coef_tab(g, i, j, k);
  double mrd, mp;
  lumped_masses_tab(g, i, j, k, mrd, mp);
  const bool hist = c.nbeta >= 2;
  const bool hu = hist && !is_dirichlet(g, i, j, k);
  const R ia = R(1) / R(c.a), iam = R(1) / (R(c.a) * R(mp));
  const R cb = R(c.b), cc = R(c.c), cd = R(c.d);
  gather_rows<R, 6, true>(A.part, PS, res, 3 * nn + 6 * p, rv);
#pragma unroll
  for (int v = 0; v < 6; ++v) t[v] = cb * s2[v];
  R x0s[6];
  if (hist) {
    R s0[6], s1[6], r1[6], r2[6] = {0, 0, 0, 0, 0, 0}, r3[6] = {0, 0, 0, 0, 0, 0};
    if (MODE == 0) {
#pragma unroll
      for (int v = 0; v < 6; ++v) s1[v] = r1[v] = x1[v];
      fetch(X, b0s, x0s);
#pragma unroll
      for (int v = 0; v < 6; ++v) s0[v] = x0s[v];
    } else {
      fetch(Y, b1s, s1);
      fetch(Y, b0s, s0);
      fetch(X, b0s, x0s);
#pragma unroll
      for (int v = 0; v < 6; ++v) r1[v] = x1[v];
    }
    if (MODE == 2) {
      fetch(Y2, b1s, r2);
      fetch(Y3, b1s, r3);
    }
#pragma unroll
    for (int v = 0; v < 6; ++v) {
      t[v] += cc * s1[v] + cd * s0[v];
      x0s[v] = advance(x0s[v], r1[v], r2[v], r3[v], s1[v]);
    }
  }
  R x0u[3];
  if (hu) {
    const size_t o1 = u_at(nn, 0, (size_t)i + (size_t)g.NX * (j + (size_t)g.NY * k));
    R q4[3];
    fetch(X, b0u, x0u);
#pragma unroll
    for (int d = 0; d < 3; ++d) q4[d] = Y[o1 + d];
    if (MODE == 2) {
      // the node rows of this launch overwrite Xn's x1 u, so stage 1's rate comes
      // from the x0 rows: h/2 K1 = Y2 - Xn
      R q2[3], q3[3], z2[3];
      fetch(Y2, o1, q2);
      fetch(Y3, o1, q3);
      fetch(Y2, b0u, z2);
#pragma unroll
      for (int d = 0; d < 3; ++d)
        x0u[d] += third * ((z2[d] - x0u[d]) + 3 * cY * (2 * (q2[d] + q3[d]) + q4[d]));
    } else {
#pragma unroll
      for (int d = 0; d < 3; ++d) x0u[d] += cY * q4[d];
    }
  }
  R o2s[6];
#pragma unroll
  for (int v = 0; v < 6; ++v) {
    const R r = -rv[v] * iam - ia * t[v];
    o2s[v] = advance2(x2[v], y2[v], y3[v], s2[v], r);
    x1[v] = advance(x1[v], x2[v], y2[v], y3[v], s2[v]);
  }
  if (hu) {
    put(D, b0u, x0u);
    if (STORE == 2) {   // x0 u of a history node
#pragma unroll
      for (int d = 0; d < 3; ++d) A.pstore[(size_t)src * A.pstore_stride + (size_t)(6 + d) * np + p] = x0u[d];
    }
  }
  if (hist) put(D, b0s, x0s);
  put(D, b1s, x1);
  put(D, b2s, o2s);
}

// 1/M_uu at every node (0 on Dirichlet nodes): rho (m_rd + a m_p).
template <typename R>
__global__ void inv_mass_kernel(Geo g, const double* __restrict__ rho, R* __restrict__ invMu) {
  const int node = blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= g.n_nodes) return;
  const int k = node / g.plane, r_ = node - k * g.plane;
  const int j = r_ / g.NX, i = r_ - j * g.NX;
  if (is_dirichlet(g, i, j, k)) {
    invMu[node] = R(0);
    return;
  }
  double mrd, mp;
  lumped_masses_tab(g, i, j, k, mrd, mp);
  const PmlCoef c = pml_coef_tab(g, i, j, k);
  invMu[node] = R(1.0 / (rho[material_index(g, i, j, k)] * (mrd + c.a * mp)));
}

}  // namespace pmlfwi
