// Kernels of the learned warm start: a small 3D convolutional network that
// maps surface traces to a coarse (lam, mu) perturbation, trained on traces
// the forward solver produces.  FP32, NCDHW layout (batch, channel, then the
// three spatial axes with the last fastest), cubic kernels of size 1 or 3
// with zero padding K/2, per-axis strides, optional ReLU after the bias.
// Every reduction runs in a fixed order (no atomics), so training is
// reproducible bit for bit.
#pragma once
#include <hip/hip_runtime.h>

#include "mfma.h"
#include "reduce.h"

namespace pmlfwi {

struct ConvShape {
  int N, Ci, D, H, W;      // input
  int Co, K;               // output channels, kernel size (1 or 3)
  int sd, sh, sw;          // strides
  int Do, Ho, Wo;          // output
};

__host__ __device__ inline int conv_out(int n, int K, int s) { return (n + 2 * (K / 2) - K) / s + 1; }

// x / d for 0 <= x < 2^31 and a divisor known to the host.
struct FastDiv {
  unsigned m, s;
};
inline FastDiv fast_div(unsigned d) {
  unsigned s = 0;
  while ((1ull << s) < d) ++s;
  return {(unsigned)((((1ull << s) - d) << 32) / d + 1), s};
}
__device__ __forceinline__ unsigned div_by(unsigned x, FastDiv f) { return (__umulhi(f.m, x) + x) >> f.s; }

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// The convolutions are implicit GEMMs on the matrix cores: no im2col buffer, a
// lane gathers the operand of its own position.  A thread per output (two loads
// and an index chain per product) reached 1-2 TFLOP/s; here one load feeds a
// product with 16 or 32 rows.  FP32 products are FP32 MFMA, never a split.

constexpr int CONV_THREADS = 256;   // 4 waves

// g = dL/d(pre-activation) from dL/dy and, with ReLU, the activated output y.
__device__ __forceinline__ float pre_grad(const float* dy, const float* y, int relu, long long i) {
  return (relu && !(y[i] > 0.0f)) ? 0.0f : dy[i];
}

// Places of a position's taps along one axis: the source index of tap k, or -1.
// Forward: input i = o s + k - p.  Data gradient: output o with o s + k - p = i.
template <int K, bool DATA>
__device__ __forceinline__ void tap_places(int pos, int stride, int n, int (&at)[K]) {
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (DATA) {
      const int a = pos + K / 2 - k;
      at[k] = a >= 0 && a % stride == 0 && a / stride < n ? a / stride : -1;
    } else {
      const int i = pos * stride + k - K / 2;
      at[k] = i >= 0 && i < n ? i : -1;
    }
  }
}

// FP32 forward (y = act(b + w * x)) and data gradient (dx = w^T * g):
//   out[row][p] = b[row] + sum over channels c, taps t of A[row][c, t] src[c][place(p, t)]
// A wave takes 64 positions, one per lane, and R rows on the one-product MFMA
// forms (32x32x1 in two blocks, 16x16x1 in four): a step is one product of every
// row and position, so a result is a chain of single multiply-adds in the order
// (c, kd, kh, kw) from the bias.  That order is kept for the forward pass because
// a pre-activation within rounding of 0 decides a ReLU mask: another order of the
// same sums moved whole weight gradients by 2e-4.  A lane's 27 places are formed
// once; the weights of 8 channels are staged in LDS for the workgroup; a channel's
// gathers are in flight during the products of the one before; taps that no
// position of the wave has (borders, the odd places of a strided data gradient)
// are skipped.
// 16 rows where 32 would leave less than one wave a SIMD.  Of the network's
// training step at batch 8 the five forward launches take 0.33 ms (2.0 ms with a
// thread per output) and the four data gradients 0.41 ms (4.9 ms); the chain of
// 64-cycle products alone is 0.08 ms a pass.
constexpr int CONV_STAGE = 8;   // channels staged together

template <int K, bool DATA, int R>
__global__ void __launch_bounds__(CONV_THREADS, (DATA ? 2 : 3))
conv3d_f32_kernel(ConvShape c, const float* __restrict__ src, const float* __restrict__ act,
                  const float* __restrict__ w, const float* __restrict__ b, int relu, int ptiles,
                  float* __restrict__ out) {
  constexpr int T3 = K * K * K, LR = R + 1, NACC = R == 32 ? 32 : 16;
  typedef float vacc __attribute__((ext_vector_type(NACC)));
  __shared__ float sA[CONV_STAGE * T3 * LR];
  const int C = DATA ? c.Co : c.Ci, M = DATA ? c.Ci : c.Co;
  const int PD = DATA ? c.D : c.Do, PH = DATA ? c.H : c.Ho, PW = DATA ? c.W : c.Wo;
  const int SD = DATA ? c.Do : c.D, SH = DATA ? c.Ho : c.H, SW = DATA ? c.Wo : c.W;
  const int P = PD * PH * PW;
  const size_t svol = (size_t)SD * SH * SW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tile = blockIdx.x * 4 + wave;          // over the batch's position tiles
  const int n = min(tile / ptiles, c.N - 1);
  const int p = tile < c.N * ptiles ? (tile - n * ptiles) * 64 + lane : P;
  const int row0 = blockIdx.y * R;
  long long at[K * K];                              // places of the tap rows, and along w
  int aw[K];
  unsigned here = 0, any = 0;                       // taps this lane, this wave has
  {
    const int q = min(p, P - 1), r = q / PW;
    int ad[K], ah[K];
    tap_places<K, DATA>(r / PH, c.sd, SD, ad);
    tap_places<K, DATA>(r % PH, c.sh, SH, ah);
    tap_places<K, DATA>(q % PW, c.sw, SW, aw);
#pragma unroll
    for (int t = 0; t < T3; ++t) {
      const int a = ad[t / (K * K)], d = ah[(t / K) % K];
      const bool ok = p < P && a >= 0 && d >= 0 && aw[t % K] >= 0;
      if (t % K == 0) at[t / K] = a >= 0 && d >= 0 ? ((long long)a * SH + d) * SW : 0;
      here |= (unsigned)ok << t;
      any |= (unsigned)(__ballot(ok) != 0) << t;
    }
    any = __builtin_amdgcn_readfirstlane(any);
  }
  vacc acc;
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    const int row = row0 + (R == 32 ? 8 * ((i >> 2) & 3) + 4 * (lane >> 5) + (i & 3) : 4 * (lane >> 4) + (i & 3));
    acc[i] = !DATA && b && row < M ? b[row] : 0.0f;
  }
  const float* sn = src + (size_t)n * C * svol;
  const float* an = DATA && relu ? act + (size_t)n * C * svol : nullptr;
  // gathers of one channel; they are issued a channel ahead of their products
  auto gather = [&](int ch, float (&v)[T3], float (&m)[DATA ? T3 : 1]) {
    const float* sc = sn + (size_t)ch * svol;
#pragma unroll
    for (int t = 0; t < T3; ++t) {
      v[t] = 0.0f;
      if constexpr (DATA) m[t] = 1.0f;
      if ((here >> t) & 1) {
        const long long o = at[t / K] + aw[t % K];
        v[t] = sc[o];
        if (DATA && relu) m[t] = an[(size_t)ch * svol + o];
      }
    }
  };
  float v[T3];
  {
    float m[DATA ? T3 : 1];
    gather(0, v, m);
    if constexpr (DATA) {
#pragma unroll
      for (int t = 0; t < T3; ++t) v[t] = m[t] > 0.0f ? v[t] : 0.0f;
    }
  }
#pragma unroll 1
  for (int ch = 0; ch < C; ++ch) {
    const int ci = ch % CONV_STAGE;
    if (ci == 0) {
      const int cn = min(CONV_STAGE, C - ch);
      __syncthreads();
      for (int i = threadIdx.x; i < cn * T3 * R; i += CONV_THREADS) {
        // forward: a row's channels and taps are contiguous; data: a channel's rows and taps
        const int row = DATA ? (i / T3) % R : i / (cn * T3), k = DATA ? (i / (R * T3)) * T3 + i % T3 : i - row * (cn * T3);
        const size_t o = DATA ? ((size_t)(ch + k / T3) * c.Ci + row0 + row) * T3 + k % T3
                              : ((size_t)(row0 + row) * c.Ci + ch) * T3 + k;
        sA[k * LR + row] = row0 + row < M ? w[o] : 0.0f;
      }
      __syncthreads();
    }
    float vn[T3], mn[DATA ? T3 : 1];
    gather(min(ch + 1, C - 1), vn, mn);
    const float* a = sA + ci * T3 * LR + (lane & (R - 1));
#pragma unroll
    for (int t = 0; t < T3; ++t) {
      if (!((any >> t) & 1)) continue;
      if constexpr (R == 32) acc = __builtin_amdgcn_mfma_f32_32x32x1f32(a[t * LR], v[t], acc, 0, 0, 0);
      else acc = __builtin_amdgcn_mfma_f32_16x16x1f32(a[t * LR], v[t], acc, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < T3; ++t) v[t] = DATA && !(mn[DATA ? t : 0] > 0.0f) ? 0.0f : vn[t];
  }
  // accumulator i of a lane: 32 rows: block i / 16 of 32 positions; 16: block i / 4 of 16
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    const int row = row0 + (R == 32 ? 8 * ((i >> 2) & 3) + 4 * (lane >> 5) + (i & 3) : 4 * (lane >> 4) + (i & 3));
    const int pos = p - lane + (R == 32 ? 32 * (i >> 4) + (lane & 31) : 16 * (i >> 2) + (lane & 15));
    if (row >= M || pos >= P || tile >= c.N * ptiles) continue;
    float v = acc[i];
    if (!DATA && relu && v < 0.0f) v = 0.0f;
    out[((size_t)n * M + row) * P + pos] = v;
  }
}

// dw[co][ci][tap] = sum over batch and outputs of g * x, and db[co] = sum of g.
// A workgroup of 4 waves takes one tile (taps (kd, kh) with all kw, 16 output
// channels, 16 input channels) on v_mfma_f32_16x16x4f32 and one of nsplit shares
// of the outputs; the waves take 16 outputs at a time in turn and their sums are
// added in LDS in a fixed order.  The shares' sums meet in the stream's slot: the
// last share of a tile to arrive adds them in order (a launch without a slot
// takes the shares of a tile in turn in one workgroup: the same bits).  A lane
// holds four neighbouring outputs of one channel (lane group q the outputs 4 q ..
// 4 q + 3), so the g it loads serve 4 K products, and with SW = 1 or 2 (the w
// stride; extents and pointers allow vector loads) so does one strip of x: the
// K shifted operands come from two or three loads.  SW = 0: any shape, element
// by element.  The workgroups of taps (0, 0) and input channel 0 also sum g.
// Of the network's training step at batch 8 this takes 0.77 ms; one workgroup
// per weight walking all outputs took 13.0 ms with the bias sums.
constexpr int WGRAD_THREADS = 256, WGRAD_WAVES = WGRAD_THREADS / 64;
constexpr int WGRAD_SLOTS = 4;              // streams that may hold a slot (per device)
constexpr int WGRAD_TILES = 1024;           // most tiles of a split launch
constexpr int WGRAD_ENTRY = 3 * 256 + 16;   // a tile's sums of one share, and its channels' sums of g
constexpr int WGRAD_ENTRIES = 1280;         // tiles x shares of a split launch
struct WgradSlot {
  float part[WGRAD_ENTRIES][WGRAD_ENTRY];
  unsigned count[WGRAD_TILES];
};
static __device__ WgradSlot wgrad_slots[WGRAD_SLOTS];   // counts start at 0

template <int K, int SW>
__global__ void __launch_bounds__(WGRAD_THREADS)
conv3d_wgrad_kernel(ConvShape c, const float* __restrict__ dy, const float* __restrict__ y, int relu,
                    const float* __restrict__ x, float* __restrict__ dw, float* __restrict__ db, FastDiv dWo,
                    FastDiv dHo, int pchunks, int ntiles, int nsplit, int slot) {
  constexpr int T2 = K * K, pad = K / 2;
  __shared__ float sAcc[WGRAD_WAVES][K * 256];
  __shared__ float sB[WGRAD_WAVES][64];
  __shared__ bool last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const int tile = blockIdx.x % ntiles;
  const int tap = tile % T2, kd = tap / K, kh = tap % K;
  const int ci_tiles = (c.Ci + 15) / 16, ct = tile / T2;
  const int co = (ct / ci_tiles) * 16 + r, ci = (ct % ci_tiles) * 16 + r;
  const bool von = co < c.Co, xon = ci < c.Ci;
  const int P = c.Do * c.Ho * c.Wo;
  const size_t vol = (size_t)c.D * c.H * c.W;
  const bool bias = db && tap == 0 && ct % ci_tiles == 0;
  // operands of one chunk: g (per tap: zero where the output lacks it), x, and
  // the sum of g over the lane's outputs
  auto load = [&](int n, int pc, float (&g)[K][4], float (&v)[K][4], float& gs) {
    const int p = pc * 16 + 4 * q;
    const unsigned pp = (unsigned)min(p, P - 1), row = div_by(pp, dWo);
    int ow = (int)(pp - row * c.Wo);
    const unsigned od_ = div_by(row, dHo);
    int od = (int)od_, oh = (int)(row - od_ * c.Ho);
    const float* gn = dy + ((size_t)n * c.Co + co) * P;
    const float* yn = y + ((size_t)n * c.Co + co) * P;
    const float* xn = x + ((size_t)n * c.Ci + ci) * vol;
    if constexpr (SW == 0) {
      gs = 0.0f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int id = od * c.sd + kd - pad, ih = oh * c.sh + kh - pad;
        const bool row_in = p + j < P && id >= 0 && id < c.D && ih >= 0 && ih < c.H;
        const float e = von && p + j < P ? pre_grad(gn, yn, relu, p + j) : 0.0f;
        gs += e;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          const int iw = ow * c.sw + k - pad;
          const bool in = row_in && iw >= 0 && iw < c.W;
          g[k][j] = in ? e : 0.0f;
          v[k][j] = in && xon ? xn[((size_t)id * c.H + ih) * c.W + iw] : 0.0f;
        }
        if (++ow == c.Wo) {
          ow = 0;
          if (++oh == c.Ho) {
            oh = 0;
            ++od;
          }
        }
      }
    } else {
      // Wo a multiple of 4: the four outputs share a row; their strip of x is
      // [SW ow - 1, SW ow + 4 SW], all inside the row but for the ends below
      const int id = od * c.sd + kd - pad, ih = oh * c.sh + kh - pad;
      const bool in = p < P && id >= 0 && id < c.D && ih >= 0 && ih < c.H;
      v4f t = {0, 0, 0, 0}, m = {1, 1, 1, 1}, x0 = {0, 0, 0, 0}, x1 = {0, 0, 0, 0};
      float el = 0.0f, er = 0.0f;
      const bool hl = pad && ow > 0, hr = pad && SW == 1 && ow + 4 < c.W;   // neighbours of the strip
      if (von && p < P) {
        t = *(const v4f*)(gn + p);
        if (relu) m = *(const v4f*)(yn + p);
      }
      if (in && xon) {
        const float* s = xn + ((size_t)id * c.H + ih) * c.W + SW * ow;
        x0 = *(const v4f*)s;
        if (SW == 2) x1 = *(const v4f*)(s + 4);
        if (hl) el = s[-1];
        if (hr) er = s[4];
      }
      float e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = m[j] > 0.0f ? t[j] : 0.0f;
      gs = (e[0] + e[1]) + (e[2] + e[3]);
      const float strip[10] = {el, x0[0], x0[1], x0[2], x0[3], SW == 2 ? x1[0] : er, x1[1], x1[2], x1[3], 0.0f};
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[k][j] = strip[SW * j + k + 1 - pad];
          const bool lost = (k < pad && j == 0 && !hl) || (SW == 1 && k > pad && j == 3 && !hr);
          g[k][j] = in && !lost ? e[j] : 0.0f;
        }
    }
  };
  constexpr int U = K == 1 ? 4 : 2;          // chunks in flight
  const int t = threadIdx.x;
  const long long chunks = (long long)c.N * pchunks;
  WgradSlot* const S = slot < 0 ? nullptr : &wgrad_slots[slot];
  float dsum[K], gsum = 0.0f;                // this thread's entries of the tile, of db
#pragma unroll
  for (int k = 0; k < K; ++k) dsum[k] = 0.0f;
  const int s0 = S ? (int)(blockIdx.x / ntiles) : 0, s1 = S ? s0 + 1 : nsplit;
  for (int sp = s0; sp < s1; ++sp) {
    v4f acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = {0.0f, 0.0f, 0.0f, 0.0f};
    float bsum = 0.0f;
    const long long end = chunks * (sp + 1) / nsplit;
    long long ch = chunks * sp / nsplit + wave;
    int n = (int)(ch / pchunks), pc = (int)(ch - (long long)n * pchunks);
    while (ch < end) {
      float g[U][K][4], v[U][K][4], gs[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (ch < end) {
          load(n, pc, g[u], v[u], gs[u]);
          ch += WGRAD_WAVES;
          pc += WGRAD_WAVES;
          while (pc >= pchunks) {
            pc -= pchunks;
            ++n;
          }
        } else {
          gs[u] = 0.0f;
#pragma unroll
          for (int k = 0; k < K; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) g[u][k][j] = v[u][k][j] = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (bias) bsum += gs[u];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int k = 0; k < K; ++k)
            acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(g[u][k][j], v[u][k][j], acc[k], 0, 0, 0);
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) sAcc[wave][256 * k + (4 * q + i) * 16 + r] = acc[k][i];
    sB[wave][lane] = bsum;
    __syncthreads();
    float d[K], e = 0.0f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      d[k] = 0.0f;
#pragma unroll
      for (int wv = 0; wv < WGRAD_WAVES; ++wv) d[k] += sAcc[wv][256 * k + t];
    }
    if (t < 16)
      for (int wv = 0; wv < WGRAD_WAVES; ++wv)
        for (int j = 0; j < 4; ++j) e += sB[wv][16 * j + t];
    if (S) {   // agent scope: the shares cross the caches of the XCDs
      float* const part = S->part[(size_t)tile * nsplit + sp];
#pragma unroll
      for (int k = 0; k < K; ++k)
        __hip_atomic_store(&part[256 * k + t], d[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < 16) __hip_atomic_store(&part[256 * K + t], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
#pragma unroll
      for (int k = 0; k < K; ++k) dsum[k] += d[k];
      gsum += e;
    }
    __syncthreads();
  }
  if (S) {
    __threadfence();
    __syncthreads();
    if (t == 0)
      last = __hip_atomic_fetch_add(&S->count[tile], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nsplit - 1;
    __syncthreads();
    if (!last) return;
#pragma unroll 4
    for (int sp = 0; sp < nsplit; ++sp) {
      const float* const part = S->part[(size_t)tile * nsplit + sp];
#pragma unroll
      for (int k = 0; k < K; ++k)
        dsum[k] += __hip_atomic_load(&part[256 * k + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (t < 16) gsum += __hip_atomic_load(&part[256 * K + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (t == 0) __hip_atomic_store(&S->count[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const int o = (ct / ci_tiles) * 16 + t / 16, i = (ct % ci_tiles) * 16 + t % 16;
  if (o < c.Co && i < c.Ci) {
#pragma unroll
    for (int k = 0; k < K; ++k) dw[(((size_t)o * c.Ci + i) * T2 + tap) * K + k] = dsum[k];
  }
  if (bias && t < 16 && (ct / ci_tiles) * 16 + t < c.Co) db[(ct / ci_tiles) * 16 + t] = gsum;
}

// ---- BF16 inference on the matrix cores -----------------------------------
__global__ void to_bf16_kernel(long long n, const float* __restrict__ in, unsigned short* __restrict__ out) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = bf16_bits(in[i]);
}

// The same GEMM on v_mfma_f32_32x32x16_bf16 with FP32 accumulation, 32
// positions and 32 rows a workgroup: lanes 0-31 hold channels 0-7, lanes 32-63
// channels 8-15 of a group of 16 at their positions.  All taps' weights (27 x 32
// rows x 32 channels, 69 KB) are staged once per 32 input channels (16 bytes a
// load where rows allow), and the four waves share the positions, each taking
// every fourth (tap, channel group), four of them in flight: the inference of
// one set of traces has at most 256 tiles a layer, so it is the length of a
// wave's chain that counts.  Bias and ReLU in FP32, output rounded to BF16
// (hidden layers) or kept FP32 (the head).  32 x 64 x 16 x 16 to 32 channels at
// stride (2, 1, 1): 12.7 us (139 us with one wave per 16 positions, no staging and
// no gathers in flight).
typedef unsigned short v8us __attribute__((ext_vector_type(8)));

template <int K>
__global__ void __launch_bounds__(CONV_THREADS)
conv3d_bf16_mfma_kernel(ConvShape c, const unsigned short* __restrict__ x, const unsigned short* __restrict__ w,
                        const float* __restrict__ b, int relu, int out_fp32, int wvec, void* __restrict__ y) {
  constexpr int T3 = K * K * K, ROWS = 32, LC = 40;   // LDS row of 32 channels, padded to spread the banks
  constexpr int NA = T3 * ROWS * LC, NS = 2 * 4 * 16 * 64;
  __shared__ __align__(16) unsigned short sA[NA > NS ? NA : NS];
  const int P = c.Do * c.Ho * c.Wo;
  const size_t vol = (size_t)c.D * c.H * c.W;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
  const int n = blockIdx.y, p = blockIdx.x * 32 + col, row0 = blockIdx.z * ROWS;
  const int pq = min(p, P - 1), pr = pq / c.Wo;
  const int d0 = (pr / c.Ho) * c.sd - K / 2, h0 = (pr % c.Ho) * c.sh - K / 2, w0 = (pq % c.Wo) * c.sw - K / 2;
  v16f acc = {};
  for (int c0 = 0; c0 < c.Ci; c0 += 32) {
    const int cn = min(32, c.Ci - c0), groups = (cn + 15) / 16, rows = min(ROWS, c.Co - row0);
    const unsigned short* wc = w + ((size_t)row0 * c.Ci + c0) * T3;
    if (c0) __syncthreads();
    if (wvec && cn == 16 * groups && rows == ROWS) {
      const int per_row = cn * T3 / 8;     // 16-byte pieces
#pragma unroll 7
      for (int i = threadIdx.x; i < ROWS * per_row; i += CONV_THREADS) {
        const int row = i / per_row, e = 8 * (i - row * per_row);
        const v8us v = *(const v8us*)(wc + (size_t)row * c.Ci * T3 + e);
        int ci = e / T3, t = e - ci * T3;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          sA[(t * ROWS + row) * LC + ci] = v[k];
          if (++t == T3) {
            t = 0;
            ++ci;
          }
        }
      }
    } else {
      const int per_row = 16 * groups * T3;
#pragma unroll 8
      for (int i = threadIdx.x; i < ROWS * per_row; i += CONV_THREADS) {
        const int row = i / per_row, e = i - row * per_row, ci = e / T3, t = e - ci * T3;
        sA[(t * ROWS + row) * LC + ci] = ci < cn && row < rows ? wc[(size_t)row * c.Ci * T3 + e] : (unsigned short)0;
      }
    }
    const unsigned short* xn = x + ((size_t)n * c.Ci + c0 + 8 * h) * vol;
    constexpr int U = 4;
    const int steps = T3 * groups;
    bool staged = false;
    for (int s0 = wave; s0 < steps; s0 += 4 * U) {
      v8us bx[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = s0 + 4 * u, t = groups == 1 ? s : s >> 1, g = groups == 1 ? 0 : s & 1;
        const int id = d0 + t / (K * K), ih = h0 + (t / K) % K, iw = w0 + t % K;
        const bool ok = s < steps && p < P && id >= 0 && id < c.D && ih >= 0 && ih < c.H && iw >= 0 && iw < c.W;
        const unsigned short* xp = xn + (size_t)(16 * g) * vol + (ok ? ((size_t)id * c.H + ih) * c.W + iw : 0);
#pragma unroll
        for (int j = 0; j < 8; ++j) bx[u][j] = ok && 16 * g + 8 * h + j < cn ? xp[j * vol] : (unsigned short)0;
      }
      if (!staged) {       // the first gathers fly while the weights are staged
        __syncthreads();
        staged = true;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = s0 + 4 * u;
        if (s >= steps) break;
        const int t = groups == 1 ? s : s >> 1, g = groups == 1 ? 0 : s & 1;
        const v8us a = *(const v8us*)&sA[(t * ROWS + col) * LC + 16 * g + 8 * h];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, bx[u]), acc,
                                                      0, 0, 0);
      }
    }
    if (!staged) __syncthreads();   // a wave without steps
  }
  float* sR = (float*)sA;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) sR[(wave * 16 + r) * 64 + lane] = acc[r];
  __syncthreads();
  // each wave finishes four of the sixteen rows of a lane
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * wave + i, co = row0 + 8 * (r >> 2) + 4 * h + (r & 3);
    if (p >= P || co >= c.Co) continue;
    float v = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) v += sR[(k * 16 + r) * 64 + lane];
    v += b ? b[co] : 0.0f;
    if (relu && v < 0.0f) v = 0.0f;
    const size_t o = ((size_t)n * c.Co + co) * P + p;
    if (out_fp32) ((float*)y)[o] = v;
    else ((unsigned short*)y)[o] = bf16_bits(v);
  }
}

// L = 1/(2n) sum (y - t)^2 over n entries; grad = (y - t)/n (parts and slot as
// in reduce.h).
__global__ void __launch_bounds__(RED_THREADS) mse_kernel(long long n, const float* __restrict__ y,
                                                          const float* __restrict__ t, float* __restrict__ loss,
                                                          float* __restrict__ grad, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  const float inv = 1.0f / (float)n;
  const long long step = (long long)nb * RED_THREADS;
  double s;
  if (reduce_parts<RedSum>(nb, red_slot(slot), sh, s, [&](int part) {
        double acc = 0.0;
        for (long long i = (long long)part * RED_THREADS + threadIdx.x; i < n; i += step) {
          const float r = y[i] - t[i];
          acc += (double)r * (double)r;
          if (grad) grad[i] = r * inv;
        }
        return acc;
      }) && threadIdx.x == 0 && loss)
    loss[0] = (float)(0.5 * s / (double)n);
}

// Adam (Kingma and Ba, 2015) with bias correction; step t counts from 1.
__global__ void adam_kernel(long long n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                            float* __restrict__ v, float lr, float b1, float b2, float eps, int t) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float mi = b1 * m[i] + (1.0f - b1) * g[i];
  const float vi = b2 * v[i] + (1.0f - b2) * g[i] * g[i];
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / (1.0f - powf(b1, (float)t));
  const float vh = vi / (1.0f - powf(b2, (float)t));
  p[i] -= lr * mh / (sqrtf(vh) + eps);
}

// Network input from FP64 traces [nsrc][nsteps+1][nrec][3]: component comp at
// the receivers rec_idx[H*W] and steps t0 + t*tstride, t < T, times scale;
// out [nsrc][T][H][W] (one sample of the batch).
__global__ void trace_features_kernel(const double* __restrict__ traces, int nsrc, int nsteps, int nrec,
                                      const int* __restrict__ rec_idx, int HW, int T, int t0, int tstride,
                                      int comp, float scale, float* __restrict__ out) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long long)nsrc * T * HW) return;
  const int r = (int)(i % HW);
  const int t = (int)((i / HW) % T);
  const int s = (int)(i / ((long long)HW * T));
  const long long step = (long long)t0 + (long long)t * tstride;
  out[i] = step <= nsteps
               ? scale * (float)traces[(((long long)s * (nsteps + 1) + step) * nrec + rec_idx[r]) * 3 + comp]
               : 0.0f;
}

// Coarse cell-centred field c[Dz][Gy][Gx] (cells of a regular grid over the
// closed interior box, z index 0 at the top) -> nodes of the closed interior:
// out = base * (1 + trilinear(c)), clamped to the cell centres at the edges.
__global__ void grid_to_nodes_kernel(const float* __restrict__ c, int Gx, int Gy, int Gz, int NIX, int NIY,
                                     int NIZ, const double* __restrict__ base, double* __restrict__ out) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= NIX * NIY * NIZ) return;
  const int jz = j / (NIX * NIY), r = j - jz * NIX * NIY, jy = r / NIX, jx = r - jy * NIX;
  // node position in cell units: cell k spans [k, k+1), centre k + 1/2
  auto coord = [](int jn, int nn, int G, int& k0, float& f) {
    float u = (float)jn / (float)(nn - 1) * (float)G - 0.5f;
    u = fminf(fmaxf(u, 0.0f), (float)(G - 1));
    k0 = min((int)u, G - 2 >= 0 ? G - 2 : 0);
    f = G > 1 ? u - (float)k0 : 0.0f;
  };
  int cx0, cy0, cz0;
  float fx, fy, fz;
  coord(jx, NIX, Gx, cx0, fx);
  coord(jy, NIY, Gy, cy0, fy);
  coord(NIZ - 1 - jz, NIZ, Gz, cz0, fz);          // depth index from the top
  const int cx1 = min(cx0 + 1, Gx - 1), cy1 = min(cy0 + 1, Gy - 1), cz1 = min(cz0 + 1, Gz - 1);
  auto at = [&](int z, int y, int x) { return c[((long long)z * Gy + y) * Gx + x]; };
  const float v = (1 - fz) * ((1 - fy) * ((1 - fx) * at(cz0, cy0, cx0) + fx * at(cz0, cy0, cx1)) +
                              fy * ((1 - fx) * at(cz0, cy1, cx0) + fx * at(cz0, cy1, cx1))) +
                  fz * ((1 - fy) * ((1 - fx) * at(cz1, cy0, cx0) + fx * at(cz1, cy0, cx1)) +
                        fy * ((1 - fx) * at(cz1, cy1, cx0) + fx * at(cz1, cy1, cx1)));
  out[j] = base[j] * (1.0 + (double)v);
}

}  // namespace pmlfwi
