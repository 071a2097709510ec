// Kernels of the learned warm start: a small 3D convolutional network that
// maps surface traces to a coarse (lam, mu) perturbation, trained on traces
// the forward solver produces.  FP32, NCDHW layout (batch, channel, then the
// three spatial axes with the last fastest), cubic kernels of size 1 or 3
// with zero padding K/2, per-axis strides, optional ReLU after the bias.
// Every reduction runs in a fixed order (no atomics), so training is
// reproducible bit for bit.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

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

// x / d for 0 <= x < 2^31 and a divisor known to the host: the round-up
// multiplier of Granlund and Montgomery (1994).
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

// Most workgroups of a launch: the threads of an axis are counted in 32 bits, and of
// more only what is left past a multiple of 2^32 runs, without an error.
constexpr long long CONV_GRID = (1LL << 32) / CONV_THREADS - 1;

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

// Place of position q among P = . x PH x PW; divisions in 64 bits only where needed.
__device__ __forceinline__ void split_position(long long q, long long P, int PH, int PW, int& d, int& h, int& w) {
  if (P <= 0x7fffffff) {
    const unsigned r = (unsigned)q / PW;
    d = r / PH;
    h = r % PH;
    w = (unsigned)q % PW;
  } else {
    const long long r = q / PW;
    d = (int)(r / PH);
    h = (int)(r % PH);
    w = (int)(q % PW);
  }
}

// One result of the forward pass or the data gradient: acc plus the products of the
// taps it has, multiply-adds in the order (c, kd, kh, kw).  row: its channel, (pd, ph,
// pw) its place in sample n.
template <bool DATA>
__device__ __forceinline__ float conv_one(const ConvShape& c, const float* __restrict__ src,
                                          const float* __restrict__ act, const float* __restrict__ w, int relu,
                                          int n, int row, int pd, int ph, int pw, float acc) {
  const int C = DATA ? c.Co : c.Ci, SD = DATA ? c.Do : c.D, SH = DATA ? c.Ho : c.H, SW = DATA ? c.Wo : c.W;
  const int K = c.K, T3 = K * K * K;
  auto at = [&](int pos, int k, int stride, int size) {   // as tap_places
    const int a = DATA ? pos + K / 2 - k : pos * stride + k - K / 2;
    if (DATA) return a >= 0 && a % stride == 0 && a / stride < size ? a / stride : -1;
    return a >= 0 && a < size ? a : -1;
  };
  for (int ch = 0; ch < C; ++ch) {
    const long long base = ((long long)n * C + ch) * SD * SH * SW;
    const float* wc = w + (DATA ? (long long)ch * c.Ci + row : (long long)row * c.Ci + ch) * T3;
    for (int kd = 0; kd < K; ++kd) {
      const int d = at(pd, kd, c.sd, SD);
      if (d < 0) continue;
      for (int kh = 0; kh < K; ++kh) {
        const int h = at(ph, kh, c.sh, SH);
        if (h < 0) continue;
        for (int kw = 0; kw < K; ++kw) {
          const int x = at(pw, kw, c.sw, SW);
          if (x < 0) continue;
          const long long o = base + ((long long)d * SH + h) * SW + x;
          acc = fmaf(wc[(kd * K + kh) * K + kw], DATA ? pre_grad(src, act, relu, o) : src[o], acc);
        }
      }
    }
  }
  return acc;
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
// are skipped.  A tap that some positions have and others not (a border) is a product
// with zero for these, which an infinite or undefined weight turns into NaN: a wave
// with a result that is not finite forms its results again, each from the taps it has.
// 16 rows where 32 would leave less than one wave a SIMD.  Of the network's
// training step at batch 8 the five forward launches take 0.34 ms (2.0 ms with a
// thread per output) and the four data gradients 0.35 ms (4.9 ms); the chain of
// 64-cycle products alone is 0.08 ms a pass.
constexpr int CONV_STAGE = 8;   // channels staged together

struct ConvArgs {
  ConvShape c;
  const float *src, *act, *w, *b;   // act: activated outputs (data gradient with ReLU); b: bias or null
  float* out;
  int relu, ptiles, first;          // ptiles: tiles of 64 positions a sample; first: tile of this launch
};

// A wave's results one by one: a lane those of its position.
template <bool DATA, int R>
__device__ __forceinline__ void conv_wave(const ConvArgs& A) {
  const ConvShape& c = A.c;
  const int M = DATA ? c.Ci : c.Co, PD = DATA ? c.D : c.Do, PH = DATA ? c.H : c.Ho, PW = DATA ? c.W : c.Wo;
  const long long P = (long long)PD * PH * PW;
  const int tile = A.first + blockIdx.x * 4 + (threadIdx.x >> 6), n = tile / A.ptiles;
  const long long p = (tile - n * A.ptiles) * 64LL + (threadIdx.x & 63);
  if (n >= c.N || p >= P) return;
  int pd, ph, pw;
  split_position(p, P, PH, PW, pd, ph, pw);
  const int row0 = blockIdx.y * R;
#pragma unroll 1
  for (int row = row0; row < min(row0 + R, M); ++row) {
    const float v = conv_one<DATA>(c, A.src, A.act, A.w, A.relu, n, row, pd, ph, pw, !DATA && A.b ? A.b[row] : 0.0f);
    A.out[((size_t)n * M + row) * P + p] = !DATA && A.relu && v < 0.0f ? 0.0f : v;
  }
}

template <int K, bool DATA, int R>
__global__ void __launch_bounds__(CONV_THREADS, (DATA ? 2 : 3)) conv3d_f32_kernel(ConvArgs A) {
  const ConvShape& c = A.c;
  const float* __restrict__ const src = A.src;
  const float* __restrict__ const act = A.act;
  const float* __restrict__ const w = A.w;
  const float* __restrict__ const b = A.b;
  float* __restrict__ const out = A.out;
  const int relu = A.relu, ptiles = A.ptiles;
  constexpr int T3 = K * K * K, LR = R + 1, NACC = R == 32 ? 32 : 16;
  typedef float vacc __attribute__((ext_vector_type(NACC)));
  __shared__ float sA[CONV_STAGE * T3 * LR];
  const int C = DATA ? c.Co : c.Ci, M = DATA ? c.Ci : c.Co;
  const int PD = DATA ? c.D : c.Do, PH = DATA ? c.H : c.Ho, PW = DATA ? c.W : c.Wo;
  const int SD = DATA ? c.Do : c.D, SH = DATA ? c.Ho : c.H, SW = DATA ? c.Wo : c.W;
  const long long P = (long long)PD * PH * PW;   // may pass 2^31
  const size_t svol = (size_t)SD * SH * SW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tile = A.first + blockIdx.x * 4 + wave;   // over the batch's position tiles
  const int n = min(tile / ptiles, c.N - 1);
  const long long p = tile < c.N * ptiles ? (tile - n * ptiles) * 64LL + lane : P;
  const int row0 = blockIdx.y * R;
  long long at[K * K];                              // places of the tap rows, and along w
  int aw[K];
  unsigned here = 0, any = 0;                       // taps this lane, this wave has
  {
    const long long q = min(p, P - 1);
    int qd, qh, qw;
    split_position(q, P, PH, PW, qd, qh, qw);
    int ad[K], ah[K];
    tap_places<K, DATA>(qd, c.sd, SD, ad);
    tap_places<K, DATA>(qh, c.sh, SH, ah);
    tap_places<K, DATA>(qw, c.sw, SW, aw);
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
  float zero = 0.0f;
#pragma unroll
  for (int i = 0; i < NACC; ++i) zero = fmaf(acc[i], 0.0f, zero);
  if (__ballot(zero != 0.0f)) {
    // The arguments are read again: held until here for this rare pass, they do not
    // fit the scalar registers beside the taps' masks (180 us in place of 167 at 64 x
    // 64 channels and 32,768 positions).
    const ConvArgs* args = (const ConvArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    conv_wave<DATA, R>(*args);
    return;
  }
  // accumulator i of a lane: 32 rows: block i / 16 of 32 positions; 16: block i / 4 of 16
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    const int row = row0 + (R == 32 ? 8 * ((i >> 2) & 3) + 4 * (lane >> 5) + (i & 3) : 4 * (lane >> 4) + (i & 3));
    const long long pos = p - lane + (R == 32 ? 32 * (i >> 4) + (lane & 31) : 16 * (i >> 2) + (lane & 15));
    if (row >= M || pos >= P || tile >= c.N * ptiles) continue;
    float v = acc[i];
    if (!DATA && relu && v < 0.0f) v = 0.0f;
    out[((size_t)n * M + row) * P + pos] = v;
  }
}

// The same results a thread each: layers of so few channels that a wave's rows are
// mostly padding.
template <bool DATA>
__global__ void __launch_bounds__(CONV_THREADS) conv3d_direct_kernel(ConvArgs A) {
  const ConvShape& c = A.c;
  const int M = DATA ? c.Ci : c.Co, PD = DATA ? c.D : c.Do, PH = DATA ? c.H : c.Ho, PW = DATA ? c.W : c.Wo;
  const long long P = (long long)PD * PH * PW, i = (long long)blockIdx.x * CONV_THREADS + threadIdx.x;
  if (i >= (long long)c.N * M * P) return;
  const long long nr = i / P;
  const int n = (int)(nr / M), row = (int)(nr % M);
  int pd, ph, pw;
  split_position(i - nr * P, P, PH, PW, pd, ph, pw);
  const float v = conv_one<DATA>(c, A.src, A.act, A.w, A.relu, n, row, pd, ph, pw, !DATA && A.b ? A.b[row] : 0.0f);
  A.out[i] = !DATA && A.relu && v < 0.0f ? 0.0f : v;
}

// dw[co][ci][tap] = sum over batch and outputs of g * x, and db[co] = sum of g.
// Order of the sums: the outputs, numbered through the batch, are dealt to 256
// chains (output T to chain T mod 256), each chain adds its products one by one,
// and the chains are joined in a tree (chain t and t + 128, then t + 64, ..).  As
// in the forward pass the order is part of the result: an update that differs in
// the last bit of a few weights can turn a ReLU mask of the next step.
// A workgroup takes the K taps of one row (kd, kh) of 4 T output and 4 T input
// channels and all 256 chains, a wave 64 of them, on the one-product MFMA form
// 4x4x1 in 16 blocks: lane 4 b + i holds channel i of four for block b, and each of
// a step's four products is one output of 64 chains.  With SW = 1 or 2 (the w stride;
// extents and pointers allow vector loads) a lane's four outputs are neighbours,
// one vector of dL/dy, and their strip of x serves all K taps; SW = 0: any shape,
// the outputs 64 apart, element by element.  Where the places lie is worked out once
// for the four lanes of a quad and four steps (SW = 0: one step).  Neither the waves
// nor the workgroups wait for one another before the tree, which is joined in LDS,
// so a launch needs no memory but its operands and runs alike on every stream and
// in a captured graph.
// Bound by the loads: an operand serves 4 T rows, and channels a power of two apart
// fall on the same channel of the L2 (products alone: 12 us of 109 at 32 x 32
// channels and 8 x 16 x 16 x 16 outputs).  The network's training step at batch 8
// takes 0.65 ms here; one workgroup per weight walking all outputs, in the same
// order, took 12.9 ms.  16 x 16 channels and all chains of one tap in a workgroup of
// 16 waves, operands shared through LDS: 98 us, but 497 us where 9 x 32 channels
// leave 54 workgroups (here 240).
// The workgroups of the first row and input channel 0 also sum g.
constexpr int WGRAD_THREADS = 256;

// WIDE: offsets in 64 bits (32 while both tensors have at most 2^30 entries).
template <int K, int T, int SW, bool WIDE, bool RELU>
__global__ void __launch_bounds__(WGRAD_THREADS, T == 1 ? 3 : 1)
conv3d_wgrad_kernel(ConvShape c, const float* __restrict__ dy, const float* __restrict__ y,
                    const float* __restrict__ x, float* __restrict__ dw, float* __restrict__ db, FastDiv dWo,
                    FastDiv dHo, FastDiv dP) {
  using I = std::conditional_t<WIDE, long long, int>;
  using O = std::conditional_t<WIDE, unsigned long long, unsigned>;
  constexpr int T3 = K * K * K, pad = K / 2, AHEAD = SW ? 4 : 2;   // steps in flight
  __shared__ float sh[4][16][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = lane >> 2, i = lane & 3;
  const int co_tiles = (c.Co + 4 * T - 1) / (4 * T), ci_tiles = (c.Ci + 4 * T - 1) / (4 * T);
  const int co0 = 4 * T * (blockIdx.x % co_tiles), rest = blockIdx.x / co_tiles;
  const int ci0 = 4 * T * (rest % ci_tiles), kd = rest / ci_tiles / K, kh = rest / ci_tiles % K;
  const I P = (I)c.Do * c.Ho * c.Wo, vol = (I)c.D * c.H * c.W;
  // rows past the last repeat it and are not stored
  O lo[T], li[T];
#pragma unroll
  for (int h = 0; h < T; ++h) {
    lo[h] = 4 * (O)(min(co0 + 4 * h + i, c.Co - 1) * P);
    li[h] = 4 * (O)(min(ci0 + 4 * h + i, c.Ci - 1) * vol);
  }
  const bool bias = db && kd == 0 && kh == 0 && ci0 == 0;
  const long long total = (long long)c.N * P, steps = (total + 255) / 256;
  // byte offsets of an output in dL/dy and of its place in x at the middle tap, both
  // from channel 0, and flags: the output exists, the row of taps does; the places
  // left and right of it (of its strip) do
  enum : unsigned { ON = 1, IN = 2, LEFT = 1, RIGHT = 2 };
  struct Place {
    O o, i;
  };
  auto place = [&](long long t) {
    const bool on = t < total;
    const I at = on ? (I)t : 0;
    auto over = [](I v, FastDiv f, I d) { return WIDE ? v / d : (I)div_by((unsigned)v, f); };
    const I n = over(at, dP, P), p = at - n * P, row = over(p, dWo, c.Wo), od = over(row, dHo, c.Ho);
    const I id = od * c.sd + kd - pad, ih = (row - od * c.Ho) * c.sh + kh - pad, iw = (p - row * c.Wo) * c.sw;
    const bool in = on && id >= 0 && id < c.D && ih >= 0 && ih < c.H;
    Place s;
    s.o = (on ? 4 * (O)(n * c.Co * P + p) | ON : 0) | (in ? IN : 0);
    s.i = in ? 4 * (O)(n * c.Ci * vol + (id * c.H + ih) * c.W + iw) | (iw > 0 ? LEFT : 0) |
                   (iw + (SW ? 4 * SW : 1) < c.W ? RIGHT : 0)
             : 0;
    return s;
  };
  auto of_quad = [](O v, auto k) {   // lane 4 b + k's value
    constexpr int q = decltype(k)::value * 0x55;
    O r = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, q, 0xf, 0xf, true);
    if constexpr (WIDE) r |= (O)(unsigned)__builtin_amdgcn_update_dpp(0, (int)(v >> 32), q, 0xf, 0xf, true) << 32;
    return r;
  };
  auto at = [](const float* base, O o) { return (const float*)((const char*)base + o); };
  struct Chunk {             // four outputs of a lane: dL/dy, activated output, x at their taps, flags
    v4f t[T], m[T];
    v4f x0[T], x1[T];        // SW: the strip; SW = 0: the middle taps,
    v4f l[T], r[T];          // left and right of it (SW: l[0], r[0])
    unsigned f[SW ? 1 : 4];
  };
  // a step's loads: every one always, from a place that exists (behind a branch
  // the number in flight is unknown to the compiler, and each step waits for all)
  auto load = [&](Place s, auto k_) {
    Chunk k;
    if constexpr (SW != 0) {   // places of four steps, a quad's lanes one each
      const O so = of_quad(s.o, k_), si = of_quad(s.i, k_);
      k.f[0] = (unsigned)(so & 3) | (unsigned)(si & 3) << 2;
#pragma unroll
      for (int h = 0; h < T; ++h) {
        const O o = (so & ~(O)3) + lo[h], p = (si & ~(O)3) + li[h];
        k.t[h] = *(const v4f*)at(dy, o);
        if (RELU) k.m[h] = *(const v4f*)at(y, o);
        k.x0[h] = *(const v4f*)at(x, p);
        if (SW == 2) k.x1[h] = *(const v4f*)at(x, p + 16);
        if (K > 1) k.l[h][0] = *at(x, p - (si & LEFT ? 4 : 0));
        if (K > 1 && SW == 1) k.r[h][0] = *at(x, p + (si & RIGHT ? 16 : 0));
      }
    } else {                   // places of one step, a quad's lanes one output each
      auto one = [&](auto j_) {
        constexpr int j = decltype(j_)::value;
        const O so = of_quad(s.o, j_), si = of_quad(s.i, j_);
        k.f[j] = (unsigned)(so & 3) | (unsigned)(si & 3) << 2;
#pragma unroll
        for (int h = 0; h < T; ++h) {
          const O o = (so & ~(O)3) + lo[h], p = (si & ~(O)3) + li[h];
          k.t[h][j] = *at(dy, o);
          if (RELU) k.m[h][j] = *at(y, o);
          k.x0[h][j] = *at(x, p);
          if (K > 1) k.l[h][j] = *at(x, p - (si & LEFT ? 4 : 0));
          if (K > 1) k.r[h][j] = *at(x, p + (si & RIGHT ? 4 : 0));
        }
      };
      one(std::integral_constant<int, 0>{});
      one(std::integral_constant<int, 1>{});
      one(std::integral_constant<int, 2>{});
      one(std::integral_constant<int, 3>{});
    }
    __builtin_amdgcn_sched_barrier(0);   // the loads in this order: a step waits for its own only
    return k;
  };
  float bsum[T][4] = {};
  v4f acc[K][T][T][4] = {};
  auto run = [&](auto bias_) {
    // a step's products, zeros where the output or its tap is absent (what was
    // loaded instead may be no number)
    auto multiply = [&](const Chunk& k) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const unsigned f = k.f[SW ? 0 : j];
        const bool in = f & IN, left = in && (f & LEFT << 2), right = in && (f & RIGHT << 2);
        bool live[T];
#pragma unroll
        for (int h = 0; h < T; ++h) {
          live[h] = !RELU || k.m[h][j] > 0.0f;
          if constexpr (decltype(bias_)::value) bsum[h][j] += (f & ON) && live[h] ? k.t[h][j] : 0.0f;
        }
#pragma unroll
        for (int w = 0; w < K; ++w) {
          const bool has = w < pad && (SW == 0 || j == 0) ? left
                           : (w > pad && (SW == 0 || (SW == 1 && j == 3)) ? right : in);
          float g[T], v[T];
#pragma unroll
          for (int h = 0; h < T; ++h) {
            const float strip[10] = {k.l[h][0], k.x0[h][0], k.x0[h][1], k.x0[h][2], k.x0[h][3],
                                     SW == 2 ? k.x1[h][0] : k.r[h][0], k.x1[h][1], k.x1[h][2], k.x1[h][3], 0.0f};
            const float e = SW ? strip[SW * j + w - pad + 1] : (w < pad ? k.l[h][j] : (w > pad ? k.r[h][j] : k.x0[h][j]));
            g[h] = has && live[h] ? k.t[h][j] : 0.0f;
            v[h] = has ? e : 0.0f;
          }
#pragma unroll
          for (int o = 0; o < T; ++o)
#pragma unroll
            for (int h = 0; h < T; ++h)
              acc[w][o][h][j] = __builtin_amdgcn_mfma_f32_4x4x1f32(g[o], v[h], acc[w][o][h][j], 0, 0, 0);
        }
      }
    };
    // a lane's place: SW: of its step of the four of group g, SW = 0: of its output of step g
    auto place_of = [&](long long g) {
      return place(SW ? 1024 * g + 256 * i + 64 * wave + 4 * b : 256 * g + 64 * i + 16 * wave + b);
    };
    Chunk buf[AHEAD];
    Place s{};
    auto fetch = [&](long long first, auto k_) {   // step first + k
      constexpr int k = decltype(k_)::value;
      if (SW == 0) s = place_of(first + k);
      buf[k] = load(s, k_);
    };
    auto each = [](auto&& f) {
      f(std::integral_constant<int, 0>{});
      f(std::integral_constant<int, 1>{});
      if constexpr (AHEAD == 4) {
        f(std::integral_constant<int, 2>{});
        f(std::integral_constant<int, 3>{});
      }
    };
    if (SW) s = place_of(0);
    each([&](auto k) { fetch(0, k); });
#pragma unroll 1
    for (long long first = 0; first < steps; first += AHEAD) {   // steps past the last hold zeros
      if (SW) s = place_of(first / AHEAD + 1);
      each([&](auto k) {
        multiply(buf[decltype(k)::value]);
        fetch(first + AHEAD, k);
      });
    }
  };
  if (bias) run(std::true_type{});
  else run(std::false_type{});
  // The tree: thread (w, s) joins the chains s + 16 k of weight w (levels 128 .. 16),
  // 16 neighbours the rest.  Chain 64 wave + 4 b + j, or (SW = 0) 64 j + 16 wave + b.
  const int w = threadIdx.x >> 4, s16 = threadIdx.x & 15;
  auto join = [&](int row, int col) {
    float v[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int ch = s16 + 16 * k;
      v[k] = SW ? sh[ch >> 6][4 * row + (ch & 3)][4 * ((ch >> 2) & 15) + col]
                : sh[(ch >> 4) & 3][4 * row + (ch >> 6)][4 * (ch & 15) + col];
    }
#pragma unroll
    for (int h = 8; h > 0; h >>= 1)
#pragma unroll
      for (int k = 0; k < h; ++k) v[k] += v[k + h];
#pragma unroll
    for (int h = 8; h > 0; h >>= 1) v[0] += __shfl_down(v[0], h);
    return v[0];
  };
#pragma unroll
  for (int k = 0; k < K * T * T; ++k) {
    const int o = k / T % T, h = k % T, tap = k / (T * T);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int row = 0; row < 4; ++row) sh[wave][4 * row + j][lane] = acc[tap][o][h][j][row];
    __syncthreads();
    const float v = join(w >> 2, w & 3);
    const int row = co0 + 4 * o + (w >> 2), col = ci0 + 4 * h + (w & 3);
    if (s16 == 0 && row < c.Co && col < c.Ci) dw[((size_t)row * c.Ci + col) * T3 + (kd * K + kh) * K + tap] = v;
    __syncthreads();
  }
  if (bias) {
#pragma unroll
    for (int h = 0; h < T; ++h)
#pragma unroll
      for (int j = 0; j < 4; ++j) sh[wave][4 * h + j][lane] = bsum[h][j];
    __syncthreads();
    if (w < 4 * T) {
      const float v = join(w >> 2, w & 3);
      if (s16 == 0 && co0 + w < c.Co) db[co0 + w] = v;
    }
  }
}

// ---- BF16 inference on the matrix cores -----------------------------------
__global__ void to_bf16_kernel(long long n, const float* __restrict__ in, unsigned short* __restrict__ out) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    out[i] = bf16_bits(in[i]);
}

// The convolution as an implicit GEMM: C[co][p] = sum_k W[co][k] X[k][p], bias and ReLU
// in FP32, output rounded to BF16 (hidden layers) or kept FP32 (the head).
//
// Few input channels: k = (ci, kd, kh, kw) as it comes, so that 16 k's are up to 16
// taps of one channel.  One wave per 16 output positions and every 16-row tile of
// output channels, v_mfma 16x16x16 BF16 with FP32 accumulation.  Bound by its index
// arithmetic, 1.4 us a step of 16 k's and 16 rows where the positions are few.
__global__ void __launch_bounds__(CONV_THREADS)
conv3d_bf16_narrow_kernel(ConvShape c, const unsigned short* __restrict__ x, const unsigned short* __restrict__ w,
                          const float* __restrict__ b, int relu, int out_fp32, unsigned first, void* __restrict__ y) {
  const unsigned P = (unsigned)c.Do * c.Ho * c.Wo;   // below 2^32
  const int KK = c.K * c.K * c.K, Kdim = c.Ci * KK, pad = c.K / 2;
  const int n = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const unsigned p = (first + blockIdx.x) * 64 + wave * 16 + i;   // this lane's output position (B column)
  const bool pin = p < P;
  const unsigned pr = pin ? p / c.Wo : 0;
  const int ow = pin ? p % c.Wo : 0, oh = pr % c.Ho, od = pr / c.Ho;
  const unsigned short* xn = x + (size_t)n * c.Ci * c.D * c.H * c.W;
  const int nrt = (c.Co + 15) / 16;
  for (int rt = 0; rt < nrt; ++rt) {
    const int row = rt * 16 + i;                 // this lane's A row (output channel)
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < Kdim; k0 += 16) {
      v4s a, bb;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = k0 + 4 * g + j;
        a[j] = (row < c.Co && k < Kdim) ? (short)w[(size_t)row * Kdim + k] : (short)0;
        short v = 0;
        if (pin && k < Kdim) {
          const int ci = k / KK, r = k - ci * KK;
          const int kd = r / (c.K * c.K), kh = (r / c.K) % c.K, kw = r % c.K;
          const int id = od * c.sd + kd - pad, ih = oh * c.sh + kh - pad, iw = ow * c.sw + kw - pad;
          if (id >= 0 && id < c.D && ih >= 0 && ih < c.H && iw >= 0 && iw < c.W)
            v = (short)xn[(((size_t)ci * c.D + id) * c.H + ih) * c.W + iw];
        }
        bb[j] = v;
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, bb, acc, 0, 0, 0);
    }
    // lane holds C[rt*16 + 4 g + r][p], r = 0..3
    if (pin) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int co = rt * 16 + 4 * g + r;
        if (co >= c.Co) continue;
        float v = acc[r] + (b ? b[co] : 0.0f);
        if (relu && v < 0.0f) v = 0.0f;
        const size_t o = ((size_t)n * c.Co + co) * P + p;
        if (out_fp32) ((float*)y)[o] = v;
        else ((unsigned short*)y)[o] = bf16_bits(v);
      }
    }
  }
}

// Otherwise v_mfma_f32_32x32x16_bf16 with FP32 accumulation, 32
// positions and 32 rows a workgroup: lanes 0-31 hold channels 0-7, lanes 32-63
// channels 8-15 of a group of 16 at their positions.  All taps' weights (27 x 32
// rows x 32 channels, 69 KB) are staged once per 32 input channels (16 bytes a
// load where rows allow), and the four waves share the positions, each taking
// every fourth (tap, channel group), four of them in flight: the inference of
// one set of traces has at most 256 tiles a layer, so it is the length of a
// wave's chain that counts.  32 x 64 x 16 x 16 to 32 channels at stride (2, 1, 1):
// 12.7 us (139 us with one wave per 16 positions, no staging and no gathers in
// flight).
typedef unsigned short v8us __attribute__((ext_vector_type(8)));

template <int K>
__global__ void __launch_bounds__(CONV_THREADS)
conv3d_bf16_mfma_kernel(ConvShape c, const unsigned short* __restrict__ x, const unsigned short* __restrict__ w,
                        const float* __restrict__ b, int relu, int out_fp32, int wvec, unsigned first, void* __restrict__ y) {
  constexpr int T3 = K * K * K, ROWS = 32, LC = 40;   // LDS row of 32 channels, padded to spread the banks
  // K = 1: one step a channel group, so the waves take 32 positions each instead
  // (24 x 18 x 26 x 32 to 7 channels: 7.9 us a call sharing them, 7.6 us)
  constexpr bool OWN = K == 1;
  constexpr int WS = OWN ? 1 : 4;                     // distance of a wave's steps
  constexpr int NA = T3 * ROWS * LC, NS = 2 * 4 * 16 * 64;
  __shared__ __align__(16) unsigned short sA[NA > NS ? NA : NS];
  const unsigned P = (unsigned)c.Do * c.Ho * c.Wo;   // below 2^32
  const size_t vol = (size_t)c.D * c.H * c.W;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
  const int n = blockIdx.y, row0 = blockIdx.z * ROWS;
  const unsigned p = (OWN ? (first + blockIdx.x) * 4 + wave : first + blockIdx.x) * 32 + col;
  const unsigned pq = min(p, P - 1), pr = pq / c.Wo;
  const int d0 = (int)(pr / c.Ho) * c.sd - K / 2, h0 = (int)(pr % c.Ho) * c.sh - K / 2, w0 = (int)(pq % c.Wo) * c.sw - K / 2;
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
      // rows past the last stay as they are: nothing of them is stored (32 rows of 16
      // channels cost a narrow layer more than its products)
#pragma unroll 8
      for (int i = threadIdx.x; i < rows * per_row; i += CONV_THREADS) {
        const int row = i / per_row, e = i - row * per_row, ci = e / T3, t = e - ci * T3;
        sA[(t * ROWS + row) * LC + ci] = ci < cn ? wc[(size_t)row * c.Ci * T3 + e] : (unsigned short)0;
      }
    }
    const unsigned short* xn = x + ((size_t)n * c.Ci + c0 + 8 * h) * vol;
    constexpr int U = 4;
    const int steps = T3 * groups;
    bool staged = false;
    for (int s0 = OWN ? 0 : wave; s0 < steps; s0 += WS * U) {
      v8us bx[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = s0 + WS * u, t = groups == 1 ? s : s >> 1, g = groups == 1 ? 0 : s & 1;
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
        const int s = s0 + WS * u;
        if (s >= steps) break;
        const int t = groups == 1 ? s : s >> 1, g = groups == 1 ? 0 : s & 1;
        const v8us a = *(const v8us*)&sA[(t * ROWS + col) * LC + 16 * g + 8 * h];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, bx[u]), acc,
                                                      0, 0, 0);
      }
    }
  }
  auto store = [&](int r, float v) {
    const int co = row0 + 8 * (r >> 2) + 4 * h + (r & 3);
    if (p >= P || co >= c.Co) return;
    v += b ? b[co] : 0.0f;
    if (relu && v < 0.0f) v = 0.0f;
    const size_t o = ((size_t)n * c.Co + co) * P + p;
    if (out_fp32) ((float*)y)[o] = v;
    else ((unsigned short*)y)[o] = bf16_bits(v);
  };
  if constexpr (OWN) {
#pragma unroll
    for (int r = 0; r < 16; ++r) store(r, acc[r]);
    return;
  }
  float* sR = (float*)sA;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) sR[(wave * 16 + r) * 64 + lane] = acc[r];
  __syncthreads();
  // each wave finishes four of the sixteen rows of a lane
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * wave + i;
    float v = 0.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) v += sR[(k * 16 + r) * 64 + lane];
    store(r, v);
  }
}

// L = 1/(2n) sum (y - t)^2 over n entries; grad = (y - t)/n (parts and slot as
// in reduce.h).
__global__ void __launch_bounds__(RED_ONE) mse_kernel(long long n, const float* __restrict__ y,
                                                      const float* __restrict__ t, float* __restrict__ loss,
                                                      float* __restrict__ grad, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  const float inv = 1.0f / (float)n;
  double s;
  auto one = [&](int part, int th) {
    double acc = 0.0;
    red_entries(part, th, nb, n, [&](long long i) { return y[i] - t[i]; }, [&](float r, long long i) {
      acc = fma((double)r, (double)r, acc);
      if (grad) grad[i] = r * inv;
    });
    return acc;
  };
  if (reduce_parts<RedSum>(nb, slot, sh, s, one) && threadIdx.x == 0 && loss)
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
