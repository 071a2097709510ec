// Element operators of one RK4 stage: the interior stiffness (first term of
// (3a)), the PML u-rows and S-rows of (3a)-(3b), forward or transposed, and
// the Lame-gradient terms (C.1f)-(C.1g), as ONE launch.
//
// A workgroup takes one part of one tile of bricks (and one source; the
// gradient part takes a group of the tile's sources in turn, whose terms it
// sums):
//   gradient   products of the adjoint's and the stored forward's strains
//   interior   K_RD u
//   S-rows     from the displacements
//   u-rows     from the stresses
// The parts write disjoint rows, so they need no order among them.
//
// What bounds it and why it is split this way.  All parts together need
// 148 MB a stage (62,500 bricks, 4 sources, FP32) and move 209 MB (counters; the
// tiles' halo planes and upper faces), 33 us at the 6.3 TB/s of a 1 GiB copy; with a
// thread per point the launches were bound by VALU issue (75 us of it a
// stage, two thirds of that index arithmetic, coefficient selects and
// divergent gathers), so here
//  * a thread keeps a column of box nodes (all z of one x, y): the node index,
//    the x and y coefficients, the row addresses are formed once per column,
//    and the stencil along z runs in registers;
//  * the PML parts have no brick-local stage at all.  Points and nodes
//    coincide (LGL), and the material of a point is its node's, so the sum of
//    a node's point terms over its bricks factors into a weighted 5-point
//    stencil along each axis times the 1D weights of the two others; the
//    material is applied once per node;
//  * the interior part, whose stress mixes derivatives of all axes at a point,
//    takes one thread per (brick, plane of 9 points): derivatives in x and y
//    and their transposes run in registers with compile-time coefficients,
//    the plane exchanges one value per point and component along z through LDS.
// Measured (62,500 bricks, 4 sources, mean per stage): three launches of a
// thread per point 117 us (FP32, forward) and 135 us (with gradient), this
// launch 57 us and 75 us; FP64 128 us and 165 us.  One launch instead of three
// on two streams also halves a small problem's pass: at 864 bricks a stage
// waited 45 us for the host and the streams' events, now 15 us.  Two things in
// it count beyond the instructions: the loads of a column are all on their way
// before the first is used (with the z profile read node by node between them
// each node waited in turn: FP32 61 and 81 us, FP64 133 and 181 us), and a
// plane's own values stay in registers for the derivatives along z, which takes
// a quarter off the interior's LDS reads (FP64 131 and 177 us without).
#pragma once
#include "kernels.h"

namespace pmlfwi {

template <int TX, int TY, int TZ>
struct TileDims {
  static constexpr int BX = 2 * TX + 1, BY = 2 * TY + 1, BZ = 2 * TZ + 1;
  static constexpr int NC = BX * BY, NB = NC * BZ;       // node columns, box nodes
  static constexpr int NE = TX * TY, NIT = 3 * NE * TZ;  // (brick, plane of points) items
  static constexpr int THREADS = ((NC > NIT ? NC : NIT) + 63) / 64 * 64;
  // LDS entries: two materials and the exchange buffer of the interior part
  // (the node fields, then one value per point and component), or six nodal
  // fields of a PML part
  static constexpr int XBUF = 27 * NIT > 6 * NB ? 27 * NIT : 6 * NB;
  static constexpr int LDS = 2 * NB + XBUF;
};

template <typename R>
struct ElementArgs {
  const Tile* tiles_int;
  const Tile* tiles_pml;
  int nint, npml, nsrc;   // tiles and sources
  // workgroups per part and source (the gradient part: per group of sources):
  // its tiles rounded up to a multiple of 8, or 0 for a part that is not asked
  // for; the gradient's groups (group q: sources q, q + ggrp, ..)
  int gint, gpml, ggint, ggrp;
  const R* Y;
  long long ystride;
  const R* lam;
  const R* mu;
  R* res;
  Part PT;
  // gradient (GRAD): stored forward stage, its weight, FP64 accumulators of
  // every group
  const R* fwd;
  long long fstride;
  const R* pfwd;
  long long pfstride;
  double gw;
  double* gacc;           // [ggrp][PG.per_src]
  Part PG;
  // receivers (forward, FP64 and FP32): workgroups from brec on, grec a source,
  // write the x1 displacement of Y there as the traces of a step
  unsigned brec;
  int grec, nrec, step, nsteps;
  const int* rec;
  double* traces;
};

// Entry i of a table that no kernel writes (tile lists, axis profiles), i the
// same in all lanes: one scalar load, in the constant address space because the
// compiler cannot see that the table is constant.
template <typename T>
__device__ __forceinline__ T uniform_entry(const T* table, int i) {
  return ((const __attribute__((address_space(4))) T*)table)[__builtin_amdgcn_readfirstlane(i)];
}

__device__ __forceinline__ Tile uniform_tile(const Tile* tiles, int i) {
  const int* t = (const int*)(tiles + __builtin_amdgcn_readfirstlane(i));
  return Tile{uniform_entry(t, 0), uniform_entry(t, 1), uniform_entry(t, 2), uniform_entry(t, 3)};
}

// A thread's column of box nodes: node (lx, ly, 0) and what its nodes share.
struct Column {
  bool live;
  int lx, ly, gi, gj, gk0;   // box and grid position of the column's lowest node
  int cxy;                   // its upper-face axes among x, y
};

template <typename D>
__device__ __forceinline__ Column tile_column(const Tile& t, int cx, int cy) {
  Column c;
  const int n = threadIdx.x;
  c.lx = n % D::BX;
  c.ly = n / D::BX;
  c.live = n < D::NC && c.lx <= 2 * cx && c.ly <= 2 * cy;
  c.gi = 2 * t.x + c.lx;
  c.gj = 2 * t.y + c.ly;
  c.gk0 = 2 * t.z;
  c.cxy = (c.lx == 2 * cx) | ((c.ly == 2 * cy) << 1);
  return c;
}

// Row addresses of a column's nodes in the partial arrays (see row_addr): all
// nodes but the top one lie in array cxy, at a constant distance; the top one
// lies in array cxy | 4.
struct ColumnRows {
  size_t u, s, utop, stop_;
  size_t du, ds;
};

__device__ __forceinline__ ColumnRows column_rows(const Geo& g, const Part& P, const Column& c, int cz) {
  ColumnRows r;
  const RowAddr t = row_addr(g, P, c.cxy | 4, c.gi, c.gj, c.gk0 + 2 * cz, 0, 0);
  r.utop = t.u;
  r.stop_ = t.s;
  if (c.cxy == 0) {
    r.u = 3 * ((size_t)c.gi + (size_t)g.NX * (c.gj + (size_t)g.NY * c.gk0));
    r.du = 3 * (size_t)g.plane;
    r.s = r.ds = 0;          // by the node's place in the shell
  } else {
    const RowAddr a = row_addr(g, P, c.cxy, c.gi, c.gj, c.gk0, 0, 0);
    const size_t stride = (size_t)P.nx[c.cxy] * P.ny[c.cxy];
    r.u = a.u;
    r.s = a.s;
    r.du = 3 * stride;
    r.ds = 6 * stride;
  }
  return r;
}

// Weighted 5-point stencils along one axis of a tile, at local node l of cnt
// bricks, over the bricks of the tile that contain l.  With w the LGL weight
// and D the derivative of the 1D basis:
//   T = false   sum_e w(q) sum_a D[q][a] f(a), q the node:  derivative at the node
//                 l odd (0, -2/3, 0, 2/3, 0); brick below (1/6, -2/3, 1/2, 0, 0),
//                 brick above (0, 0, -1/2, 2/3, -1/6)
//   T = true    sum_e sum_q w(q) D[q][a] f(q), a the node:  its transpose, i.e.
//                 the same with the off-centre signs reversed
// S is the sum of the weights at l.  Offsets are clamped to the box (the
// clamped reads have coefficient 0).
template <typename R, bool T>
__device__ __forceinline__ void line_stencil(int l, int cnt, R c[5], int o[5], R& S) {
  const bool odd = l & 1, lo = l >= 1, hi = !odd && (l >> 1) < cnt;
  const R sg = T ? R(-1) : R(1);
  const R third = R(1.0 / 3.0), sixth = R(1.0 / 6.0), two3 = R(2.0 / 3.0);
  c[0] = (!odd && lo) ? sg * sixth : R(0);
  c[1] = lo ? -sg * two3 : R(0);
  c[2] = odd ? R(0) : R(lo ? 0.5 : 0.0) - R(hi ? 0.5 : 0.0);
  c[3] = (odd || hi) ? sg * two3 : R(0);
  c[4] = hi ? -sg * sixth : R(0);
  S = odd ? R(4.0 / 3.0) : R(lo ? third : R(0)) + R(hi ? third : R(0));
#pragma unroll
  for (int k = 0; k < 5; ++k) o[k] = min(max(l - 2 + k, 0), 2 * cnt);
}

// The same along z for a whole column in registers (f = 0 above 2 cz).
template <typename R, bool T, int BZ>
__device__ __forceinline__ void column_stencil(int cz, const R (&f)[BZ][3], R (&e)[BZ][3]) {
  const R sixth = T ? R(-1.0 / 6.0) : R(1.0 / 6.0), two3 = T ? R(-2.0 / 3.0) : R(2.0 / 3.0);
#pragma unroll
  for (int l = 0; l < BZ; ++l)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      R v = 0;
      if (l & 1) {
        v = two3 * (f[l + 1][i] - f[l - 1][i]);
      } else {
        if (l > 0) v += sixth * f[l - 2][i] - two3 * f[l - 1][i] + R(0.5) * f[l][i];
        if (l + 2 < BZ && l < 2 * cz) v += R(-0.5) * f[l][i] + two3 * f[l + 1][i] - sixth * f[l + 2][i];
      }
      e[l][i] = v;
    }
}

// Sum of the 1D weights at local z node l (compile time but for the top).
template <typename R, int BZ>
__device__ __forceinline__ R z_weight(int l, int cz) {
  if (l & 1) return R(4.0 / 3.0);
  return (l > 0 ? R(1.0 / 3.0) : R(0)) + ((l + 2 < BZ && l < 2 * cz) ? R(1.0 / 3.0) : R(0));
}

// PML profile of a column and its nodes' places in the shell.
template <typename R, int BZ>
struct PmlColumn {
  R ax, ay, bx, by;
  int nbeta;                // of the two axes
  R az[BZ], bz[BZ];         // z profile (the same for the whole workgroup)
  size_t node, ring0;       // node id of the lowest node; shell index on the first frame plane
};

template <typename R, int BZ>
__device__ __forceinline__ PmlColumn<R, BZ> pml_column(const Geo& g, const Column& c, int cz) {
  PmlColumn<R, BZ> p;
  const double* A = g.tab;
  const double* B = g.tab + ax_n(g);
  const double bx = B[c.gi], by = B[ax_y(g) + c.gj];
  p.ax = R(A[c.gi]);
  p.ay = R(A[ax_y(g) + c.gj]);
  p.bx = R(bx);
  p.by = R(by);
  p.nbeta = (bx > 0.0) + (by > 0.0);
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    const int k = ax_z(g) + c.gk0 + min(l, 2 * cz);
    p.az[l] = R(uniform_entry(A, k));
    p.bz[l] = R(uniform_entry(B, k));
  }
  p.node = (size_t)c.gi + (size_t)g.NX * (c.gj + (size_t)g.NY * c.gk0);
  p.ring0 = (size_t)pml_index(g, c.gi, c.gj, g.zb + 1);
  return p;
}

// Shell index of a column's node at plane k = gk0 + l.
template <typename R, int BZ>
__device__ __forceinline__ size_t shell_index(const Geo& g, const PmlColumn<R, BZ>& p, int gk0, int l) {
  const int k = gk0 + l;
  return k <= g.zb ? p.node + (size_t)l * g.plane : p.ring0 + (size_t)(k - g.zb - 1) * g.ring;
}

// Stretch factors of one node from its column's and its z profile.
template <typename R>
struct Stretch {
  R Le[3], Lp[3], Lw[3];
};

template <typename R, int BZ>
__device__ __forceinline__ Stretch<R> stretch_at(const PmlColumn<R, BZ>& p, int l) {
  Stretch<R> s;
  const R az = p.az[l], bz = p.bz[l];
  s.Le[0] = p.ay * az; s.Lp[0] = p.ay * bz + p.by * az; s.Lw[0] = p.by * bz;
  s.Le[1] = p.ax * az; s.Lp[1] = p.ax * bz + p.bx * az; s.Lw[1] = p.bx * bz;
  s.Le[2] = p.ax * p.ay; s.Lp[2] = p.ax * p.by + p.bx * p.ay; s.Lw[2] = p.bx * p.by;
  return s;
}

// e_ik at every node of the column: the sum over the node's bricks of w d_k
// W_k,i, from the fields W_x,i and W_y,i in LDS and the column's z terms.
template <typename R, typename D>
__device__ __forceinline__ void node_gradients(const Column& c, int cx, int cy, int cz, R f, const R* sF, int l,
                                               const R (&ez)[3], const R cX[5], const int oX[5], R Sx,
                                               const R cY[5], const int oY[5], R Sy, R ex_[3], R ey_[3], R ez_[3]) {
  R dx[3] = {0, 0, 0}, dy[3] = {0, 0, 0};
  const int row = D::BX * c.ly + D::NC * l, colm = c.lx + D::NC * l;
#pragma unroll
  for (int k = 0; k < 5; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      dx[i] += cX[k] * sF[i * D::NB + row + oX[k]];
      dy[i] += cY[k] * sF[(3 + i) * D::NB + colm + D::BX * oY[k]];
    }
  const R Sz = z_weight<R, D::BZ>(l, cz);
  const R fx = f * Sy * Sz, fy = f * Sx * Sz, fz = f * Sx * Sy;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    ex_[i] = fx * dx[i];
    ey_[i] = fy * dy[i];
    ez_[i] = fz * ez[i];
  }
}

// S-rows of one PML tile and source: W_k = Le_kk u' + Lp_kk u + Lw_kk ubar at
// the nodes, H_ik = d_k W_k,i summed over the node's bricks with the weights,
// then -(mu (H + H^T) + lam tr(H) I) (forward) or H_ab + H_ba, H_aa
// (transposed) with the node's material.
template <typename R, typename D, bool ADJ>
__device__ __forceinline__ void pml_s_part(const Geo& g, const ElementArgs<R>& A, const Tile& t, int src, R* smem) {
  constexpr int BZ = D::BZ;
  const int cx = t.c & 255, cy = (t.c >> 8) & 255, cz = (t.c >> 16) & 255;
  const Column c = tile_column<D>(t, cx, cy);
  const size_t nn = (size_t)g.sn, np = (size_t)g.sp;
  R ez[BZ][3], la[BZ], m[BZ];
  PmlColumn<R, BZ> pc{};
  if (c.live) {
    pc = pml_column<R, BZ>(g, c, cz);
    const R* Y = A.Y + (size_t)src * A.ystride;
    const R* P = Y + 6 * nn;
    R wz[BZ][3], u1[BZ][3], u2[BZ][3], u0[BZ][3];
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
      if (l <= 2 * cz) {
        const size_t n3 = 3 * (pc.node + (size_t)l * g.plane);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          u1[l][d] = Y[n3 + d];
          u2[l][d] = Y[3 * nn + n3 + d];
        }
        if constexpr (!ADJ) {
          const int mi = material_index(g, c.gi, c.gj, c.gk0 + l);
          la[l] = A.lam[mi];
          m[l] = A.mu[mi];
        }
      }
    }
    // after the loads above, as these wait for the x and y profile
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
#pragma unroll
      for (int d = 0; d < 3; ++d) u0[l][d] = R(0);
      if (l <= 2 * cz && pc.nbeta + (pc.bz[l] > 0) >= 2) {
        const size_t p = shell_index(g, pc, c.gk0, l);
#pragma unroll
        for (int d = 0; d < 3; ++d) u0[l][d] = P[p_at(np, P_X0U, p) + d];
      }
    }
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
      if (l <= 2 * cz) {
        const Stretch<R> s = stretch_at(pc, l);
        const int n = threadIdx.x + D::NC * l;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          smem[i * D::NB + n] = s.Le[0] * u2[l][i] + s.Lp[0] * u1[l][i] + s.Lw[0] * u0[l][i];
          smem[(3 + i) * D::NB + n] = s.Le[1] * u2[l][i] + s.Lp[1] * u1[l][i] + s.Lw[1] * u0[l][i];
          wz[l][i] = s.Le[2] * u2[l][i] + s.Lp[2] * u1[l][i] + s.Lw[2] * u0[l][i];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) wz[l][i] = R(0);
      }
    }
    column_stencil<R, false, BZ>(cz, wz, ez);
  }
  __syncthreads();
  if (!c.live) return;
  R cX[5], cY[5], Sx, Sy;
  int oX[5], oY[5];
  line_stencil<R, false>(c.lx, cx, cX, oX, Sx);
  line_stencil<R, false>(c.ly, cy, cY, oY, Sy);
  const R f = R(0.25 * g.h * g.h);   // (h/2)^3 times 2/h
  const ColumnRows rows = column_rows(g, A.PT, c, cz);
  R* res = A.res + (size_t)src * A.PT.per_src;
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    if (l > 2 * cz) break;
    R ex_[3], ey_[3], ez_[3], q[6];
    node_gradients<R, D>(c, cx, cy, cz, f, smem, l, ez[l], cX, oX, Sx, cY, oY, Sy, ex_, ey_, ez_);
    q[0] = ex_[0];
    q[1] = ey_[1];
    q[2] = ez_[2];
    q[3] = ez_[1] + ey_[2];
    q[4] = ez_[0] + ex_[2];
    q[5] = ey_[0] + ex_[1];
    if constexpr (!ADJ) {
      const R lt = la[l] * (q[0] + q[1] + q[2]), m2 = 2 * m[l];
#pragma unroll
      for (int v = 0; v < 3; ++v) q[v] = -(lt + m2 * q[v]);
#pragma unroll
      for (int v = 3; v < 6; ++v) q[v] = -m[l] * q[v];
    }
    const size_t o = l == 2 * cz ? rows.stop_
                                 : (c.cxy ? rows.s + (size_t)l * rows.ds
                                          : 3 * nn + 6 * shell_index(g, pc, c.gk0, l));
#pragma unroll
    for (int v = 0; v < 6; ++v) res[o + v] = q[v];
  }
}

// u-rows of one PML tile and source from the nodal tensor
//   forward      T_ik = Le_kk S'_ik + Lp_kk S_ik + Lw_kk Sbar_ik
//   transposed   T_ik = -(mu (1 + d_ik) Z_k,ik + lam d_ik tr Z_i), Z_k the same
//                combination of the adjoint stresses.
template <typename R, typename D, bool ADJ>
__device__ __forceinline__ void pml_u_part(const Geo& g, const ElementArgs<R>& A, const Tile& t, int src, R* smem) {
  constexpr int BZ = D::BZ;
  const int cx = t.c & 255, cy = (t.c >> 8) & 255, cz = (t.c >> 16) & 255;
  const Column c = tile_column<D>(t, cx, cy);
  const size_t nn = (size_t)g.sn, np = (size_t)g.sp;
  R ez[BZ][3];
  if (c.live) {
    const PmlColumn<R, BZ> pc = pml_column<R, BZ>(g, c, cz);
    const R* P = A.Y + (size_t)src * A.ystride + 6 * nn;
    R tz[BZ][3];
    R f0[BZ][6], f1[BZ][6], f2[BZ][6];
    // the stresses of node l, loaded AHEAD nodes before they are used (as the
    // registers allow; five ahead in FP32 or two in FP64 measured no faster)
    constexpr int AHEAD = sizeof(R) == 4 ? 3 : 1;
    auto load = [&](int l) {
      if (l > 2 * cz) return;
      const size_t p = shell_index(g, pc, c.gk0, l);
#pragma unroll
      for (int v = 0; v < 6; ++v) f1[l][v] = P[p_at(np, P_X1S, p) + v];
#pragma unroll
      for (int v = 0; v < 6; ++v) f2[l][v] = P[p_at(np, P_X2S, p) + v];
#pragma unroll
      for (int v = 0; v < 6; ++v) f0[l][v] = R(0);
      if (pc.nbeta + (pc.bz[l] > 0) >= 2) {
#pragma unroll
        for (int v = 0; v < 6; ++v) f0[l][v] = P[p_at(np, P_X0S, p) + v];
      }
    };
#pragma unroll
    for (int l = 0; l < AHEAD && l < BZ; ++l) load(l);
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
      if (l + AHEAD < BZ) load(l + AHEAD);
      if (l <= 2 * cz) {
        const R(&s0)[6] = f0[l];
        const R(&s1)[6] = f1[l];
        const R(&s2)[6] = f2[l];
        const Stretch<R> s = stretch_at(pc, l);
        const int n = threadIdx.x + D::NC * l;
        R T[3][3];
        if constexpr (!ADJ) {
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const int v = vidx(i, k);
              T[i][k] = s.Le[k] * s2[v] + s.Lp[k] * s1[v] + s.Lw[k] * s0[v];
            }
        } else {
          const int mi = material_index(g, c.gi, c.gj, c.gk0 + l);
          const R la = A.lam[mi], m = A.mu[mi];
          const R t2 = s2[0] + s2[1] + s2[2], t1 = s1[0] + s1[1] + s1[2], t0 = s0[0] + s0[1] + s0[2];
#pragma unroll
          for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              const int v = vidx(i, k);
              const R z = s.Le[k] * s2[v] + s.Lp[k] * s1[v] + s.Lw[k] * s0[v];
              R val = (i == k ? R(2) : R(1)) * m * z;
              if (i == k) val += la * (s.Le[i] * t2 + s.Lp[i] * t1 + s.Lw[i] * t0);
              T[i][k] = -val;
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          smem[i * D::NB + n] = T[i][0];
          smem[(3 + i) * D::NB + n] = T[i][1];
          tz[l][i] = T[i][2];
        }
      } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) tz[l][i] = R(0);
      }
    }
    column_stencil<R, true, BZ>(cz, tz, ez);
  }
  __syncthreads();
  if (!c.live || c.gi == 0 || c.gi == g.NX - 1 || c.gj == 0 || c.gj == g.NY - 1) return;   // Dirichlet columns
  R cX[5], cY[5], Sx, Sy;
  int oX[5], oY[5];
  line_stencil<R, true>(c.lx, cx, cX, oX, Sx);
  line_stencil<R, true>(c.ly, cy, cY, oY, Sy);
  const R f = R(0.25 * g.h * g.h);
  const ColumnRows rows = column_rows(g, A.PT, c, cz);
  R* res = A.res + (size_t)src * A.PT.per_src;
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    if (l > 2 * cz) break;
    if (c.gk0 + l == 0) continue;   // Dirichlet plane
    R ex_[3], ey_[3], ez_[3];
    node_gradients<R, D>(c, cx, cy, cz, f, smem, l, ez[l], cX, oX, Sx, cY, oY, Sy, ex_, ey_, ez_);
    const size_t o = l == 2 * cz ? rows.utop : rows.u + (size_t)l * rows.du;
#pragma unroll
    for (int i = 0; i < 3; ++i) res[o + i] = ex_[i] + ey_[i] + ez_[i];
  }
}

// Adds a tile's gradient terms to the accumulators (column sums gl, gm).  All
// loads of the column stand before its first store: node by node, where the
// compiler has to keep their order, the ten round trips to memory took longer
// than the rest of a tile of one source.
template <int BZ>
__device__ __forceinline__ void add_gradient(const Geo& g, const Part& PG, const Column& c, int cz, double gw,
                                             const double (&gl)[BZ], const double (&gm)[BZ], double* gacc) {
  const int ct = c.cxy | 4;
  double* low = gacc + PG.off[c.cxy] + part_node(g, PG, c.cxy, c.gi, c.gj, c.gk0);
  double* top = gacc + PG.off[ct] + part_node(g, PG, ct, c.gi, c.gj, c.gk0 + 2 * cz);
  const size_t d = (size_t)PG.nx[c.cxy] * PG.ny[c.cxy];
  const long long slow = PG.size[c.cxy], stop_ = PG.size[ct];
  double vl[BZ], vm[BZ];
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    const double* p = l >= 2 * cz ? top : low + (size_t)l * d;   // above the top: its value again
    vl[l] = p[0];
    vm[l] = p[l >= 2 * cz ? stop_ : slow];
  }
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    if (l > 2 * cz) break;
    double* p = l == 2 * cz ? top : low + (size_t)l * d;
    p[0] = vl[l] + gw * gl[l];
    p[l == 2 * cz ? stop_ : slow] = vm[l] + gw * gm[l];
  }
}

// Sum over a node column's bricks of brick-local values in LDS: value v of
// local node (pa, pb, pc) of brick (ex, ey, ez) at
// [(9 v + 3 pb + pa) NIT + ex + TX ey + NE (3 ez + pc)].
template <typename R, typename D, int TX, int NV>
__device__ __forceinline__ void column_gather(const Column& c, int cx, int cy, int cz, const R* X, R (&acc)[D::BZ][NV]) {
#pragma unroll
  for (int l = 0; l < D::BZ; ++l)
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[l][v] = 0;
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      // brick below (a = 0; odd nodes have only this one) and above (a = 1)
      const int ex = a ? c.lx >> 1 : (c.lx - 1) >> 1, ey = b ? c.ly >> 1 : (c.ly - 1) >> 1;
      const bool vx = a ? !(c.lx & 1) && ex < cx : c.lx >= 1, vy = b ? !(c.ly & 1) && ey < cy : c.ly >= 1;
      if (!(vx && vy)) continue;
      const R* x = X + (3 * (c.ly - 2 * ey) + (c.lx - 2 * ex)) * D::NIT + ex + TX * ey;
#pragma unroll
      for (int l = 0; l < D::BZ; ++l) {
        if (l > 2 * cz) break;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          if (l & 1) {
            acc[l][v] += x[9 * v * D::NIT + D::NE * (3 * (l >> 1) + 1)];
          } else {
            if (l > 0) acc[l][v] += x[9 * v * D::NIT + D::NE * (3 * (l / 2 - 1) + 2)];
            if (l + 2 < D::BZ && l < 2 * cz) acc[l][v] += x[9 * v * D::NIT + D::NE * (3 * (l / 2))];
          }
        }
      }
    }
}

// Derivative of a brick line's three values at its point q, and the transpose
// (row of node a from the three point values); q and a known at compile time.
template <typename R>
__device__ __forceinline__ R line_diff(int q, R f0, R f1, R f2) {
  if (q == 1) return R(0.5) * (f2 - f0);
  return q == 0 ? R(-1.5) * f0 + R(2) * f1 - R(0.5) * f2 : R(0.5) * f0 - R(2) * f1 + R(1.5) * f2;
}
template <typename R>
__device__ __forceinline__ R line_diff_t(int a, R s0, R s1, R s2) {
  if (a == 1) return R(2) * (s0 - s2);
  return a == 0 ? R(-1.5) * s0 - R(0.5) * s1 + R(0.5) * s2 : R(-0.5) * s0 + R(0.5) * s1 + R(1.5) * s2;
}

// The displacement at the nodes of a brick's plane [d][b][a] (x: the plane's
// first node in the box fields).
template <typename R, typename D>
__device__ __forceinline__ void plane_nodes(const R* x, R (&u)[3][3][3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d)
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a) u[d][b][a] = x[d * D::NB + a + D::BX * b];
}

// This thread's (brick, plane) item of an interior tile, and the weights
// w_q (h/2)^3 (2/h)^2 of its points by their place in the plane.
template <typename R>
struct PlaneItem {
  bool live;
  int q, n0;                 // item; the plane's first box node
  R wc, we, wm;              // weight of the plane's corners, edges, centre
  // The brick's two other planes (distance in box nodes and in items) and,
  // with D the derivative of the 1D basis, what this one, the next (1) and the
  // one after (2) weigh in the derivative along z at this plane's points, and
  // in its transpose at this plane's nodes.  A thread so takes its own plane's
  // values from registers.
  int n1, n2, q1, q2;
  R d0, d1, d2, t1, t2;      // d0 is its own transpose
  __device__ __forceinline__ R weight(int a, int b) const {
    return (a == 1) + (b == 1) == 0 ? wc : ((a == 1) + (b == 1) == 1 ? we : wm);
  }
};

// Strain (xx, yy, zz, 2 yz, 2 xz, 2 xy, times h/2) at point (a, b) of an item's
// plane; x0: the plane's first node in the box fields.
template <typename R, typename D>
__device__ __forceinline__ void point_strain(const R* x0, const R (&u)[3][3][3], const PlaneItem<R>& it, int a, int b,
                                             R (&e)[6]) {
  R gx[3], gy[3], gz[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const R* x = x0 + d * D::NB + a + D::BX * b;
    gx[d] = line_diff<R>(a, u[d][b][0], u[d][b][1], u[d][b][2]);
    gy[d] = line_diff<R>(b, u[d][0][a], u[d][1][a], u[d][2][a]);
    gz[d] = it.d0 * u[d][b][a] + it.d1 * x[it.n1] + it.d2 * x[it.n2];
  }
  e[0] = gx[0];
  e[1] = gy[1];
  e[2] = gz[2];
  e[3] = gz[1] + gy[2];
  e[4] = gz[0] + gx[2];
  e[5] = gy[0] + gx[1];
}

// The same with the plane's values read from LDS.
template <typename R, typename D>
__device__ __forceinline__ void row_strain(const R* x0, const PlaneItem<R>& it, int a, int b, R (&e)[6]) {
  R gx[3], gy[3], gz[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const R* x = x0 + d * D::NB + a + D::BX * b;
    const R* r = x0 + d * D::NB + D::BX * b;
    const R* t = x0 + d * D::NB + a;
    gx[d] = line_diff<R>(a, r[0], r[1], r[2]);
    gy[d] = line_diff<R>(b, t[0], t[D::BX], t[2 * D::BX]);
    gz[d] = it.d0 * x[0] + it.d1 * x[it.n1] + it.d2 * x[it.n2];
  }
  e[0] = gx[0];
  e[1] = gy[1];
  e[2] = gz[2];
  e[3] = gz[1] + gy[2];
  e[4] = gz[0] + gx[2];
  e[5] = gy[0] + gx[1];
}

template <typename R, int TX, int TY, int TZ>
__device__ __forceinline__ PlaneItem<R> plane_item(const Geo& g, int cx, int cy, int cz) {
  using D = TileDims<TX, TY, TZ>;
  PlaneItem<R> it;
  it.q = threadIdx.x;
  const int ex = it.q % TX, ey = (it.q / TX) % TY, zz = it.q / D::NE, ez = zz / 3;
  const int qc = zz - 3 * ez;   // place of the plane in its brick
  it.live = it.q < D::NIT && ex < cx && ey < cy && ez < cz;
  it.n0 = 2 * ex + D::BX * (2 * ey) + D::NC * (2 * ez + qc);
  const int s1 = qc == 2 ? -2 : 1, s2 = qc == 0 ? 2 : -1;
  it.n1 = s1 * D::NC;
  it.n2 = s2 * D::NC;
  it.q1 = s1 * D::NE;
  it.q2 = s2 * D::NE;
  it.d0 = R(1.5) * R(qc - 1);
  it.d1 = qc == 0 ? R(2) : R(0.5);
  it.d2 = qc == 2 ? R(-2) : R(-0.5);
  it.t1 = qc == 1 ? R(-2) : R(-0.5);
  it.t2 = qc == 1 ? R(2) : R(0.5);
  const R wz = R(0.5 * g.h) * (qc == 1 ? R(4.0 / 3.0) : R(1.0 / 3.0));
  it.wc = wz * R(1.0 / 9.0);
  it.we = wz * R(4.0 / 9.0);
  it.wm = wz * R(16.0 / 9.0);
  return it;
}

// Interior bricks of one tile and source: r_u += K_RD u (u = x1 displacement
// of the input register).
template <typename R, int TX, int TY, int TZ>
__device__ __forceinline__ void interior_part(const Geo& g, const ElementArgs<R>& A, const Tile& t, int src, R* smem) {
  using D = TileDims<TX, TY, TZ>;
  constexpr int BX = D::BX, BZ = D::BZ, NC = D::NC, NB = D::NB, NIT = D::NIT;
  const int cx = t.c & 255, cy = (t.c >> 8) & 255, cz = (t.c >> 16) & 255;
  const Column c = tile_column<D>(t, cx, cy);
  R* sLam = smem;
  R* sMu = smem + NB;
  R* X = smem + 2 * NB;   // node fields, then per-point values
  if (c.live) {
    const size_t nplane = (size_t)g.NIX * g.NIY;
    const size_t node = (size_t)c.gi + (size_t)g.NX * (c.gj + (size_t)g.NY * c.gk0);
    const size_t mi = (size_t)(c.gi - 2 * g.ps) + (size_t)g.NIX * ((c.gj - 2 * g.ps) + (size_t)g.NIY * (c.gk0 - 2 * g.pb));
    const R* Yu = A.Y + (size_t)src * A.ystride + 3 * node;
    R u[BZ][3], la[BZ], m[BZ];
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
      if (l <= 2 * cz) {
#pragma unroll
        for (int d = 0; d < 3; ++d) u[l][d] = Yu[3 * (size_t)l * g.plane + d];
        la[l] = A.lam[mi + l * nplane];
        m[l] = A.mu[mi + l * nplane];
      }
    }
#pragma unroll
    for (int l = 0; l < BZ; ++l) {
      if (l <= 2 * cz) {
        const int n = threadIdx.x + NC * l;
#pragma unroll
        for (int d = 0; d < 3; ++d) X[d * NB + n] = u[l][d];
        sLam[n] = la[l];
        sMu[n] = m[l];
      }
    }
  }
  __syncthreads();
  const PlaneItem<R> it = plane_item<R, TX, TY, TZ>(g, cx, cy, cz);
  R out[3][3][3];   // rows of the plane's nodes [d][b][a]
  R s[9][6];        // strains, then weighted stresses, at the points
  if (it.live) {
    R u[3][3][3];
    plane_nodes<R, D>(X + it.n0, u);
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const int k = 3 * b + a, nq = it.n0 + a + BX * b;
        point_strain<R, D>(X + it.n0, u, it, a, b, s[k]);
        const R w = it.weight(a, b);
        const R m = w * sMu[nq], m2 = 2 * m, lt = w * sLam[nq] * (s[k][0] + s[k][1] + s[k][2]);
#pragma unroll
        for (int v = 0; v < 3; ++v) s[k][v] = lt + m2 * s[k][v];
#pragma unroll
        for (int v = 3; v < 6; ++v) s[k][v] = m * s[k][v];
      }
    // transposed derivatives along x and y inside the plane
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          constexpr int vx[3] = {0, 5, 4}, vy[3] = {5, 1, 3};
          out[d][b][a] = line_diff_t<R>(a, s[3 * b][vx[d]], s[3 * b + 1][vx[d]], s[3 * b + 2][vx[d]]) +
                         line_diff_t<R>(b, s[a][vy[d]], s[3 + a][vy[d]], s[6 + a][vy[d]]);
        }
  }
  __syncthreads();
  if (it.live) {
    constexpr int vz[3] = {4, 3, 2};
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 9; ++k) X[(9 * d + k) * NIT + it.q] = s[k][vz[d]];
  }
  __syncthreads();
  if (it.live) {
    // transposed derivative along z: this plane's nodes gather the z stress of
    // the brick's three planes
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      R z1[9], z2[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const R* x = X + (9 * d + k) * NIT + it.q;
        z1[k] = x[it.q1];
        z2[k] = x[it.q2];
      }
      constexpr int vz[3] = {4, 3, 2};
#pragma unroll
      for (int k = 0; k < 9; ++k)
        out[d][k / 3][k % 3] += it.d0 * s[k][vz[d]] + it.t1 * z1[k] + it.t2 * z2[k];
    }
  }
  __syncthreads();
  if (it.live) {
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int k = 0; k < 9; ++k) X[(9 * d + k) * NIT + it.q] = out[d][k / 3][k % 3];
  }
  __syncthreads();
  if (!c.live) return;
  R acc[BZ][3];
  column_gather<R, D, TX, 3>(c, cx, cy, cz, X, acc);
  const ColumnRows rows = column_rows(g, A.PT, c, cz);
  R* res = A.res + (size_t)src * A.PT.per_src;
#pragma unroll
  for (int l = 0; l < BZ; ++l) {
    if (l > 2 * cz) break;
    const size_t o = l == 2 * cz ? rows.utop : rows.u + (size_t)l * rows.du;
#pragma unroll
    for (int d = 0; d < 3; ++d) res[o + d] = acc[l][d];
  }
}

// Gradient terms of the interior bricks of one tile:
//   g -= b_s * sum_e w|J| (div z div u_f, 2 eps(z):eps(u_f))
// at the LGL nodes, z = the x1 displacement of the input register, u_f = the
// stored forward stage, summed over the sources of group grp and added to its
// FP64 accumulators (gacc: [8][2][n_nodes], slot c indexed like the partial
// arrays).
// A part of its own: with the stiffness in the same workgroup a thread held
// both fields' strains, the stresses and the rows (247 registers in FP32, two
// waves per SIMD for every part of the launch).
template <typename R, int TX, int TY, int TZ>
__device__ __forceinline__ void interior_grad_part(const Geo& g, const ElementArgs<R>& A, const Tile& t, int grp,
                                                   R* X) {
  using D = TileDims<TX, TY, TZ>;
  constexpr int BZ = D::BZ, NC = D::NC, NB = D::NB, NIT = D::NIT;
  const int cx = t.c & 255, cy = (t.c >> 8) & 255, cz = (t.c >> 16) & 255;
  const Column c = tile_column<D>(t, cx, cy);
  const size_t nplane = (size_t)g.NIX * g.NIY;
  const size_t node = (size_t)c.gi + (size_t)g.NX * (c.gj + (size_t)g.NY * c.gk0);
  const size_t mi = (size_t)(c.gi - 2 * g.ps) + (size_t)g.NIX * ((c.gj - 2 * g.ps) + (size_t)g.NIY * (c.gk0 - 2 * g.pb));
  const PlaneItem<R> it = plane_item<R, TX, TY, TZ>(g, cx, cy, cz);
  double gl[BZ], gm[BZ];
#pragma unroll
  for (int l = 0; l < BZ; ++l) gl[l] = gm[l] = 0.0;
#pragma unroll 1
  for (int src = grp; src < A.nsrc; src += A.ggrp) {
    if (c.live) {
      const R* Yu = A.Y + (size_t)src * A.ystride + 3 * node;
      const R* F = A.fwd + (size_t)src * A.fstride + 3 * mi;
      R u[BZ][3], v[BZ][3];
#pragma unroll
      for (int l = 0; l < BZ; ++l) {
        if (l <= 2 * cz) {
#pragma unroll
          for (int d = 0; d < 3; ++d) u[l][d] = Yu[3 * (size_t)l * g.plane + d];
#pragma unroll
          for (int d = 0; d < 3; ++d) v[l][d] = __builtin_nontemporal_load(&F[3 * l * nplane + d]);
        }
      }
#pragma unroll
      for (int l = 0; l < BZ; ++l) {
        if (l <= 2 * cz) {
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            X[d * NB + threadIdx.x + NC * l] = u[l][d];
            X[(3 + d) * NB + threadIdx.x + NC * l] = v[l][d];
          }
        }
      }
    }
    __syncthreads();
    R pl[9], pm[9];   // products at the points in the state precision; summed in FP64 below
    if (it.live) {
      // FP32: both fields' planes in registers.  FP64: a point's values read
      // from LDS as it comes (both planes and the sums are more than the 256
      // registers of two waves; the clobber keeps the reads where they stand).
      // With gradient at 62,500 bricks and 4 sources FP64 196 -> 181 us, while
      // FP32 read so takes 90 us instead of 81.
      constexpr bool ROWS = sizeof(R) == 8;
      R u[3][3][3], v[3][3][3];
      if constexpr (!ROWS) {
        plane_nodes<R, D>(X + it.n0, u);
        plane_nodes<R, D>(X + 3 * NB + it.n0, v);
      }
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          R e[6], f[6];
          if constexpr (ROWS) {
            row_strain<R, D>(X + it.n0, it, a, b, e);
            row_strain<R, D>(X + 3 * NB + it.n0, it, a, b, f);
            asm volatile("" ::: "memory");
          } else {
            point_strain<R, D>(X + it.n0, u, it, a, b, e);
            point_strain<R, D>(X + 3 * NB + it.n0, v, it, a, b, f);
          }
          const R w = it.weight(a, b);
          R ee = 2 * (e[0] * f[0] + e[1] * f[1] + e[2] * f[2]);
          ee += e[3] * f[3] + e[4] * f[4] + e[5] * f[5];
          pl[3 * b + a] = w * (e[0] + e[1] + e[2]) * (f[0] + f[1] + f[2]);
          pm[3 * b + a] = w * ee;
          __builtin_amdgcn_sched_barrier(0);   // one point's strains at a time in registers
        }
    }
    __syncthreads();
    if (it.live) {
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        X[k * NIT + it.q] = pl[k];
        X[(9 + k) * NIT + it.q] = pm[k];
      }
    }
    __syncthreads();
    if (c.live) {
      R acc[BZ][2];
      column_gather<R, D, TX, 2>(c, cx, cy, cz, X, acc);
#pragma unroll
      for (int l = 0; l < BZ; ++l) {
        gl[l] += (double)acc[l][0];
        gm[l] += (double)acc[l][1];
      }
    }
    __syncthreads();
  }
  if (c.live) add_gradient<BZ>(g, A.PG, c, cz, A.gw, gl, gm, A.gacc + (size_t)grp * A.PG.per_src);
}

// Traces of a step: tr (source, step) at receiver r from the displacements U.
template <typename R>
__device__ __forceinline__ void record_traces(const R* U, int sn, const int* rec, int r, double* tr) {
  const int node = rec[r];
  for (int d = 0; d < 3; ++d) tr[3 * (size_t)r + d] = (double)U[u_at(sn, d, node)];
}

// The launch: 1D grid; first the gradient part (with GRAD; it walks the
// sources and runs longest), then the stiffness, S-rows and u-rows.  Every
// part's share is a multiple of 8 workgroups, so workgroup b runs on XCD
// b mod 8 and each XCD walks a contiguous run of tiles.  The first launch of a
// forward step also records the traces of the step before, whose end is its
// input: a launch of their own took 2.4 us of a step's 51 at 256 bricks in FP32.
template <typename R, int TX, int TY, int TZ, bool ADJ, bool GRAD>
__global__ void __launch_bounds__((TileDims<TX, TY, TZ>::THREADS), (GRAD ? (sizeof(R) == 4 ? 3 : 2) : 1))
element_kernel(Geo g, ElementArgs<R> A) {
  using D = TileDims<TX, TY, TZ>;
  __shared__ R smem[D::LDS];
  int b = blockIdx.x;
  auto tile_of = [](int i, int n) { return (i & 7) * (n >> 3) + (i >> 3); };
  if constexpr (GRAD) {
    if (b < A.ggint * A.ggrp) {
      const int grp = b / A.ggint;
      const int ti = tile_of(b - grp * A.ggint, A.ggint);
      if (ti < A.nint) interior_grad_part<R, TX, TY, TZ>(g, A, uniform_tile(A.tiles_int, ti), grp, smem);
      return;
    }
    b -= A.ggint * A.ggrp;
  }
  if constexpr (!ADJ) {
    if (blockIdx.x >= A.brec) {
      b -= (int)A.brec;
      const int src = b / A.grec, r = (b - src * A.grec) * D::THREADS + threadIdx.x;
      if (r < A.nrec)
        record_traces<R>(A.Y + (size_t)src * A.ystride, g.sn, A.rec, r,
                         A.traces + ((size_t)src * (A.nsteps + 1) + A.step) * A.nrec * 3);
      return;
    }
  }
  if (b < A.gint * A.nsrc) {
    const int src = b / A.gint;
    const int ti = tile_of(b - src * A.gint, A.gint);
    if (ti < A.nint) interior_part<R, TX, TY, TZ>(g, A, uniform_tile(A.tiles_int, ti), src, smem);
    return;
  }
  b -= A.gint * A.nsrc;
  const int part = b / (A.gpml * A.nsrc);
  b -= part * A.gpml * A.nsrc;
  const int src = b / A.gpml;
  const int ti = tile_of(b - src * A.gpml, A.gpml);
  if (ti >= A.npml) return;
  const Tile t = uniform_tile(A.tiles_pml, ti);
  if (part == 0) pml_s_part<R, D, ADJ>(g, A, t, src, smem);
  else pml_u_part<R, D, ADJ>(g, A, t, src, smem);
}

// Gradient terms of the PML S-rows under the material extension (the chain
// rule through the interface values a PML node takes).  The S-row of a PML
// node j carries -w_q [mu_j (H + H^T) + lam_j tr(H) I] summed over its bricks,
// H from the forward stage's (u', u, ubar); with z the adjoint stress at j
// (x1 S of the adjoint stage), the gradient gains
// -gw (tr(e) sum_a z_aa, sum_v z_v (e_ab + e_ba)), e the weighted sum of H,
// summed over a group's sources, in its FP64 accumulators indexed like the partial
// arrays.  pfwd: stored forward PML displacements of the stage, per source
// [x1 u (3) | x2 u (3) | x0 u (3)] x sp on the PML shell.
// A launch of its own (full gradient only): in the stage launch its registers
// would cost every part occupancy.
template <typename R, int TX, int TY, int TZ>
__global__ void __launch_bounds__((TileDims<TX, TY, TZ>::THREADS)) pml_gradient_kernel(Geo g, ElementArgs<R> A) {
  using D = TileDims<TX, TY, TZ>;
  constexpr int BZ = D::BZ;
  __shared__ R smem[6 * D::NB];
  // The sums of the two terms over sources: in FP64 a thread's own entries in
  // LDS, which brings it from 420 registers to 234 (62,500 bricks, 4 sources:
  // 110 -> 69 us); in FP32 they fit the registers (55 us, in LDS 60 us).
  constexpr bool SUM_LDS = sizeof(R) == 8;
  __shared__ double sum[SUM_LDS ? 2 * D::NB : 1];
  double gl[BZ], gm[BZ];
#pragma unroll
  for (int l = 0; l < BZ; ++l) gl[l] = gm[l] = 0.0;
  const int ti = xcd_tile(), grp = blockIdx.y;
  if (ti >= A.npml) return;
  const Tile t = uniform_tile(A.tiles_pml, ti);
  const int cx = t.c & 255, cy = (t.c >> 8) & 255, cz = (t.c >> 16) & 255;
  const Column c = tile_column<D>(t, cx, cy);
  const size_t nn = (size_t)g.sn, np = (size_t)g.sp;
  const R f = R(0.25 * g.h * g.h);
  R cX[5], cY[5], Sx, Sy;
  int oX[5], oY[5];
  line_stencil<R, false>(c.lx, cx, cX, oX, Sx);
  line_stencil<R, false>(c.ly, cy, cY, oY, Sy);
  const bool side = c.gi == 0 || c.gi == g.NX - 1 || c.gj == 0 || c.gj == g.NY - 1;
  if (SUM_LDS && c.live)
    for (int l = 0; l < BZ; ++l) sum[threadIdx.x + D::NC * l] = sum[D::NB + threadIdx.x + D::NC * l] = 0.0;
#pragma unroll 1
  for (int src = grp; src < A.nsrc; src += A.ggrp) {
    // the column's profile is formed anew for every source: kept, it and the
    // addresses and stretch factors of all its nodes take 200 registers
    Column cs = c;
    asm volatile("" : "+v"(cs.gi), "+v"(cs.gj), "+v"(cs.gk0));
    PmlColumn<R, BZ> pc{};
    if (c.live) pc = pml_column<R, BZ>(g, cs, cz);
    R ez[BZ][3];
    if (c.live) {
      const R* F = A.pfwd + (size_t)src * A.pfstride;
      R wz[BZ][3];
#pragma unroll
      for (int l = 0; l < BZ; ++l) {
        if (l <= 2 * cz) {
          const size_t p = shell_index(g, pc, cs.gk0, l);
          const bool on = !side && c.gk0 + l > 0, hist = on && pc.nbeta + (pc.bz[l] > 0) >= 2;
          const Stretch<R> s = stretch_at(pc, l);
          const int n = threadIdx.x + D::NC * l;
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            const R u1 = on ? F[i * np + p] : R(0), u2 = on ? F[(3 + i) * np + p] : R(0);
            const R u0 = hist ? F[(6 + i) * np + p] : R(0);
            smem[i * D::NB + n] = s.Le[0] * u2 + s.Lp[0] * u1 + s.Lw[0] * u0;
            smem[(3 + i) * D::NB + n] = s.Le[1] * u2 + s.Lp[1] * u1 + s.Lw[1] * u0;
            wz[l][i] = s.Le[2] * u2 + s.Lp[2] * u1 + s.Lw[2] * u0;
          }
        } else {
#pragma unroll
          for (int i = 0; i < 3; ++i) wz[l][i] = R(0);
        }
      }
      column_stencil<R, false, BZ>(cz, wz, ez);
    }
    __syncthreads();
    if (c.live) {
      const R* P = A.Y + (size_t)src * A.ystride + 6 * nn;
#pragma unroll
      for (int l = 0; l < BZ; ++l) {
        if (l > 2 * cz) break;
        R ex_[3], ey_[3], ez_[3], z[6];
        node_gradients<R, D>(c, cx, cy, cz, f, smem, l, ez[l], cX, oX, Sx, cY, oY, Sy, ex_, ey_, ez_);
        const size_t p = shell_index(g, pc, cs.gk0, l);
#pragma unroll
        for (int v = 0; v < 6; ++v) z[v] = P[p_at(np, P_X1S, p) + v];
        R em = 2 * (z[0] * ex_[0] + z[1] * ey_[1] + z[2] * ez_[2]);
        em += z[3] * (ez_[1] + ey_[2]) + z[4] * (ez_[0] + ex_[2]) + z[5] * (ey_[0] + ex_[1]);
        double* pl = SUM_LDS ? &sum[threadIdx.x + D::NC * l] : &gl[l];
        double* pm = SUM_LDS ? &sum[D::NB + threadIdx.x + D::NC * l] : &gm[l];
        *pl -= (double)((ex_[0] + ey_[1] + ez_[2]) * (z[0] + z[1] + z[2]));
        *pm -= (double)em;
      }
    }
    __syncthreads();
  }
  if (!c.live) return;
#pragma unroll
  for (int l = 0; SUM_LDS && l < BZ; ++l) {
    gl[l] = sum[threadIdx.x + D::NC * l];
    gm[l] = sum[D::NB + threadIdx.x + D::NC * l];
  }
  add_gradient<BZ>(g, A.PG, c, cz, A.gw, gl, gm, A.gacc + (size_t)grp * A.PG.per_src);
}

}  // namespace pmlfwi
