// Control-problem terms on the closed interior (Sec. 3.1.3 and App. C), FP64.
//
//   Tikhonov (8):        R_TN(f) = 1/2 int |grad f|^2,        gradient (C.1b-c)
//   total variation (9): R_TV(f) = int (|grad f|^2 + eps)^1/2, gradient (C.1d-e)
//   M~ (C.1a):           lumped (LGL) mass of the closed interior, diagonal
//   (18):                g = M~^{-1} (g_mis + R g_reg)
//
// f is a nodal field on the closed-interior grid (id jx + NIX*(jy + NIY*jz)),
// integrals use the 3x3x3 LGL rule of every interior brick.  The TV
// denominator is evaluated pointwise at the LGL points, and the functional
// carries R rather than R/2 so that its derivative is the TV form of (17).
#pragma once
#include "geometry.h"
#include "reduce.h"

namespace pmlfwi {

__device__ __forceinline__ double dlgl64(int q, int a) {
  // derivative of 1D basis a at LGL point q (nodes -1, 0, 1)
  const double r0 = a == 0 ? -1.5 : (a == 1 ? 2.0 : -0.5);
  const double r1 = a == 0 ? -0.5 : (a == 1 ? 0.0 : 0.5);
  const double r2 = a == 0 ? 0.5 : (a == 1 ? -2.0 : 1.5);
  return q == 0 ? r0 : (q == 1 ? r1 : r2);
}
__device__ __forceinline__ double wlgl64(int a) { return a == 1 ? 4.0 / 3.0 : 1.0 / 3.0; }

enum { REG_TN = 0, REG_TV = 1 };

// grad f at LGL point q of a brick; base: the point's entry in f, whose rows lie
// sy and planes sz apart.
__device__ __forceinline__ void point_grad(const Geo& g, const double* f, int base, int sy, int sz, int qx, int qy,
                                           int qz, double G[3]) {
  const int sx = 1;
  double gx = 0, gy = 0, gz = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    gx += dlgl64(qx, a) * f[base + (a - qx) * sx];
    gy += dlgl64(qy, a) * f[base + (a - qy) * sy];
    gz += dlgl64(qz, a) * f[base + (a - qz) * sz];
  }
  const double s = 2.0 / g.h;
  G[0] = s * gx;
  G[1] = s * gy;
  G[2] = s * gz;
}

// Quadrature term of the functional and the flux coefficient at one point.
__device__ __forceinline__ void point_terms(int kind, double eps, const double G[3], double w, double* val,
                                            double* coef) {
  const double s2 = G[0] * G[0] + G[1] * G[1] + G[2] * G[2];
  if (kind == REG_TN) {
    *val = 0.5 * w * s2;
    *coef = w;
  } else {
    const double r = sqrt(s2 + eps);
    *val = w * r;
    *coef = w / r;
  }
}

// Bricks of one axis, of those in [lo, hi), that contain interior-closure index
// l: (brick - lo, local position).
__device__ __forceinline__ int axis_bricks(int l, int lo, int hi, int* b, int* p) {
  if (l & 1) {
    b[0] = (l >> 1) - lo;
    p[0] = 1;
    return 1;
  }
  int n = 0;
  if ((l >> 1) > lo) {
    b[n] = (l >> 1) - 1 - lo;
    p[n] = 2;
    ++n;
  }
  if ((l >> 1) < hi) {
    b[n] = (l >> 1) - lo;
    p[n] = 0;
    ++n;
  }
  return n;
}

// grad[j] = d R(f) / d f_j, gathered per node over the bricks that contain it
// (deterministic: no atomics).
// A workgroup takes the nodes of 4 x 4 x 2 bricks (and the closing planes of the
// last ones): it forms the flux once at every point of those bricks and of one
// layer below them, in LDS, and each node adds what its three lines hold.  Bound
// by the flux's roots and divisions; a node that formed the fluxes it needs (9 in
// each of its bricks, so every flux seven times) took 61 us at 139,425 nodes, this 15 us.
constexpr int REG_X = 4, REG_Y = 4, REG_Z = 2, REG_THREADS = 256;

inline unsigned reg_tiles(const Geo& g) {
  return (unsigned)((g.ex + REG_X - 1) / REG_X) * ((g.ey + REG_Y - 1) / REG_Y) * ((g.ez + REG_Z - 1) / REG_Z);
}

__global__ void __launch_bounds__(REG_THREADS) reg_gradient_kernel(Geo g, int kind, double eps,
                                                                   const double* __restrict__ f,
                                                                   double* __restrict__ grad) {
  constexpr int NF = (2 * REG_X + 3) * (2 * REG_Y + 3) * (2 * REG_Z + 3);
  constexpr int NQ = 27 * (REG_X + 1) * (REG_Y + 1) * (REG_Z + 1);
  __shared__ double sF[NF], sQ[3][NQ];
  const int tx = (g.ex + REG_X - 1) / REG_X, ty = (g.ey + REG_Y - 1) / REG_Y;
  const int X0 = REG_X * (blockIdx.x % tx), Y0 = REG_Y * (blockIdx.x / tx % ty), Z0 = REG_Z * (blockIdx.x / (tx * ty));
  // bricks [lo, hi) of each axis, their nodes [2 lo, 2 hi]
  const int xl = max(X0 - 1, 0), xh = min(X0 + REG_X, g.ex), yl = max(Y0 - 1, 0), yh = min(Y0 + REG_Y, g.ey);
  const int zl = max(Z0 - 1, 0), zh = min(Z0 + REG_Z, g.ez);
  const int bx = xh - xl, by = yh - yl, bz = zh - zl, mx = 2 * bx + 1, my = 2 * by + 1, mz = 2 * bz + 1;
  for (int i = threadIdx.x; i < mx * my * mz; i += REG_THREADS) {
    const int x = i % mx, r = i / mx, y = r % my, z = r / my;
    sF[i] = f[(2 * xl + x) + (size_t)g.NIX * ((2 * yl + y) + (size_t)g.NIY * (2 * zl + z))];
  }
  __syncthreads();
  const double vol = 0.125 * g.h * g.h * g.h, s = 2.0 / g.h;
  for (int i = threadIdx.x; i < 27 * bx * by * bz; i += REG_THREADS) {
    const int e = i / 27, q = i - 27 * e, qx = q % 3, qy = q / 3 % 3, qz = q / 9;
    const int x = e % bx, r = e / bx, y = r % by, z = r / by;
    double G[3], val, coef;
    point_grad(g, sF, (2 * x + qx) + mx * ((2 * y + qy) + my * (2 * z + qz)), mx, mx * my, qx, qy, qz, G);
    point_terms(kind, eps, G, vol * wlgl64(qx) * wlgl64(qy) * wlgl64(qz), &val, &coef);
#pragma unroll
    for (int d = 0; d < 3; ++d) sQ[d][i] = coef * G[d] * s;
  }
  __syncthreads();
  // the tile's nodes: up to its upper planes, which the next tile holds
  const int nx = 2 * (xh - X0) + (xh == g.ex), ny = 2 * (yh - Y0) + (yh == g.ey), nz = 2 * (zh - Z0) + (zh == g.ez);
  for (int i = threadIdx.x; i < nx * ny * nz; i += REG_THREADS) {
    const int jx = 2 * X0 + i % nx, r = i / nx, jy = 2 * Y0 + r % ny, jz = 2 * Z0 + r / ny;
    int ex[2], px[2], ey[2], py[2], ez[2], pz[2];
    const int kx = axis_bricks(jx, xl, xh, ex, px), ky = axis_bricks(jy, yl, yh, ey, py),
              kz = axis_bricks(jz, zl, zh, ez, pz);
    double acc = 0.0;
    for (int c = 0; c < kz; ++c)
      for (int b = 0; b < ky; ++b)
        for (int a = 0; a < kx; ++a) {
          const int p[3] = {px[a], py[b], pz[c]}, m[3] = {1, 3, 9};
          const int q0 = 27 * (ex[a] + bx * (ey[b] + by * ez[c])) + p[0] + 3 * p[1] + 9 * p[2];
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int q = 0; q < 3; ++q) acc += sQ[d][q0 + (q - p[d]) * m[d]] * dlgl64(q, p[d]);
        }
    grad[jx + (size_t)g.NIX * (jy + (size_t)g.NIY * jz)] = acc;
  }
}

// value[0] = R(f) (parts and slot as in reduce.h: deterministic).
__global__ void __launch_bounds__(RED_ONE) reg_value_kernel(Geo g, int kind, double eps,
                                                            const double* __restrict__ f,
                                                            double* __restrict__ value, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  const long long npts = 27LL * g.ex * g.ey * g.ez, span = red_span(npts, nb);
  const double vol = 0.125 * g.h * g.h * g.h;
  double r;
  auto one = [&](int part, int th) {
    double acc = 0.0;
    for (long long t = part * span + th; t < min(npts, (part + 1) * span); t += RED_THREADS) {
      const int q = (int)(t % 27);
      const unsigned e = (unsigned)(t / 27), er = e / (unsigned)g.ex;   // fewer bricks than nodes
      const int ex = (int)(e - er * g.ex), ez = (int)(er / (unsigned)g.ey), ey = (int)(er - ez * g.ey);
      const int qx = q % 3, qy = (q / 3) % 3, qz = q / 9;
      double G[3], val, coef;
      point_grad(g, f, (2 * ex + qx) + g.NIX * ((2 * ey + qy) + g.NIY * (2 * ez + qz)), g.NIX, g.NIX * g.NIY, qx, qy,
                 qz, G);
      point_terms(kind, eps, G, vol * wlgl64(qx) * wlgl64(qy) * wlgl64(qz), &val, &coef);
      acc += val;
    }
    return acc;
  };
  if (reduce_parts<RedSum>(nb, slot, sh, r, one) && threadIdx.x == 0) value[0] = r;
}

// M~ diagonal (C.1a): interior lumped mass of every closed-interior node.
__global__ void material_mass_kernel(Geo g, double* __restrict__ m) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= g.n_int) return;
  const int jz = j / (g.NIX * g.NIY), r_ = j - jz * g.NIX * g.NIY, jy = r_ / g.NIX, jx = r_ - jy * g.NIX;
  double mrd, mp;
  lumped_masses_tab(g, jx + 2 * g.ps, jy + 2 * g.ps, jz + 2 * g.pb, mrd, mp);
  m[j] = mrd;
}

// (18): g = M~^{-1} (g_mis + R g_reg); g_reg may be null (R = 0).
__global__ void gradient_finalize_kernel(Geo g, const double* __restrict__ gmis, const double* __restrict__ greg,
                                         double R, double* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= g.n_int) return;
  const int jz = j / (g.NIX * g.NIY), r_ = j - jz * g.NIX * g.NIY, jy = r_ / g.NIX, jx = r_ - jy * g.NIX;
  double mrd, mp;
  lumped_masses_tab(g, jx + 2 * g.ps, jy + 2 * g.ps, jz + 2 * g.pb, mrd, mp);
  const double v = gmis[j] + (greg ? R * greg[j] : 0.0);
  out[j] = v / mrd;
}

// out = alpha x + beta y (y may be null when beta = 0; out may alias x or y):
// the vector updates of the optimizer (L-BFGS two-loop recursion, the model
// update (19), the biased direction (25), y = g1 - g).  FP64, elementwise.
__global__ void axpby_kernel(long long n, double alpha, const double* x, double beta, const double* y,
                             double* out) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = beta == 0.0 ? alpha * x[i] : alpha * x[i] + beta * y[i];
}

}  // namespace pmlfwi
