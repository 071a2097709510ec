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
// Order of the sums: the outputs, numbered through the batch, are dealt to 256
// chains (output T to chain T mod 256), each chain adds its products one by one,
// and the chains are joined in a tree (chain t and t + 128, then t + 64, ..).  As
// in the forward pass the order is part of the result: an update that differs in
// the last bit of a few weights can turn a ReLU mask of the next step.
// A workgroup of 4 waves takes a tile (taps (kd, kh) with all kw, 16 output and 16
// input channels) and a quarter of the chains, a wave 16 of them, on the one-product MFMA form
// 16x16x1 in four blocks: block q and the step's product j hold chain
// 16 cg + 4 q + j.  So a lane loads four neighbouring outputs of its channel at
// once, which serve 4 K products, and with SW = 1 or 2 (the w stride; extents and
// pointers allow vector loads) so does one strip of x; SW = 0: any shape, element
// by element.  The
// next WGRAD_AHEAD chunks of 16 outputs are in flight during the products of the
// ones before.  The first two levels of the tree join the waves, in LDS; the
// quarters meet in the stream's slot, where the last of a tile to arrive joins
// them.  Without a slot, or with more tiles than one holds (then tiles enough to
// fill the chip), one workgroup takes a tile's taps and quarters in turn (SPLIT =
// false): the same bits.
// The workgroups of taps (0, 0) and input channel 0 also sum g.
// Of the network's training step at batch 8 this takes 0.67 ms; one workgroup
// per weight walking all outputs, in the same order, took 13.0 ms with the bias
// sums.  Eight chunks ahead, or the loads by neighbouring lanes and an exchange
// through LDS, measured no faster, one tap instead of three to a wave slower
// (0.86 ms); products of four outputs each (16x16x4, another order) took 0.77 ms.
constexpr int WGRAD_THREADS = 256, WGRAD_WAVES = WGRAD_THREADS / 64, WGRAD_AHEAD = 4;
constexpr int WGRAD_SLOTS = 4;              // streams that may hold a slot (per device)
constexpr int WGRAD_TILES = 48;             // most tiles of a split launch
constexpr int WGRAD_ENTRY = 3 * 256 + 16;   // sums of one chain: a tile's weights, its channels' g
struct WgradSlot {
  float part[WGRAD_TILES][4][16][WGRAD_ENTRY];
  unsigned count[WGRAD_TILES];
};
static __device__ WgradSlot wgrad_slots[WGRAD_SLOTS];   // counts start at 0

// One chunk of a lane: four outputs of channel co, and their strip of x or (SW =
// 0) their places in x for each tap.
template <int SW, int KT>
struct WgradChunk {
  v4f t, m;                 // dL/dy, and the activated output (ReLU) or 1
  v4f x0, x1;               // strip of x
  float el, er;             // its neighbours
  bool on, in, hl, hr;      // the outputs exist; the taps' row does; the neighbours do
};
template <int KT>
struct WgradChunk<0, KT> {
  v4f e, g[KT], v[KT];      // g, g where the output has the tap, x there
};

template <int K, int SW, bool SPLIT>
__global__ void __launch_bounds__(WGRAD_THREADS, 1)
conv3d_wgrad_kernel(ConvShape c, const float* __restrict__ dy, const float* __restrict__ y, int relu,
                    const float* __restrict__ x, float* __restrict__ dw, float* __restrict__ db, FastDiv dWo,
                    FastDiv dHo, FastDiv dP, int ntiles, int slot) {
  constexpr int T2 = K * K, pad = K / 2;
  constexpr int KT = SPLIT ? K : 1;          // taps along w at a time
  __shared__ float sAcc[2][64][64 + 1];      // two waves' accumulators, a lane's 64 to a row
  __shared__ float sB[WGRAD_WAVES][64][4];
  __shared__ bool last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const int tile = blockIdx.x % ntiles;
  const int tap = tile % T2, kd = tap / K, kh = tap % K;
  const int ci_tiles = (c.Ci + 15) / 16, ct = tile / T2;
  const int co0 = (ct / ci_tiles) * 16, ci0 = (ct % ci_tiles) * 16;
  const int co = co0 + r, ci = ci0 + r;
  const bool von = co < c.Co, xon = ci < c.Ci;
  const int P = c.Do * c.Ho * c.Wo;
  const size_t vol = (size_t)c.D * c.H * c.W;
  const int cor = min(co, c.Co - 1), cir = min(ci, c.Ci - 1);   // rows past the last are not stored
  const float* const mask = relu ? y : dy;
  const bool bias = db && tap == 0 && ci0 == 0;
  const long long total = (long long)c.N * P, chunks = (total + 15) / 16;
  auto load = [&](int n, int p, bool on, int kw) {   // on: output p of sample n exists; kw: first tap
    WgradChunk<SW, KT> k;
    const unsigned pp = on ? (unsigned)p : 0u, row = div_by(pp, dWo);
    if (!on) n = 0;
    int ow = (int)(pp - row * c.Wo);
    const unsigned od_ = div_by(row, dHo);
    int od = (int)od_, oh = (int)(row - od_ * c.Ho);
    if constexpr (SW == 0) {
      int pj = (int)pp;
      const long long left = total - ((long long)n * P + pj);   // outputs from here on
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int id = od * c.sd + kd - pad, ih = oh * c.sh + kh - pad;
        const bool here = on && j < left, row_in = here && id >= 0 && id < c.D && ih >= 0 && ih < c.H;
        const size_t o = ((size_t)n * c.Co + co) * P;
        k.e[j] = here && von ? pre_grad(dy + o, y + o, relu, pj) : 0.0f;
#pragma unroll
        for (int i = 0; i < KT; ++i) {
          const int iw = ow * c.sw + kw + i - pad;
          const bool in = row_in && iw >= 0 && iw < c.W;
          k.g[i][j] = in ? k.e[j] : 0.0f;
          k.v[i][j] = in && xon ? x[((size_t)n * c.Ci + ci) * vol + ((size_t)id * c.H + ih) * c.W + iw] : 0.0f;
        }
        ++pj;
        if (++ow == c.Wo) {
          ow = 0;
          if (++oh == c.Ho) {
            oh = 0;
            if (++od == c.Do) {
              od = 0;
              pj = 0;
              n = min(n + 1, c.N - 1);
            }
          }
        }
      }
    } else {
      // Wo a multiple of 4: the four outputs share a row; their strip of x is
      // [SW ow - 1, SW ow + 4 SW], all inside the row but for the ends below
      const int id = od * c.sd + kd - pad, ih = oh * c.sh + kh - pad;
      k.on = on;
      k.in = on && id >= 0 && id < c.D && ih >= 0 && ih < c.H;
      k.hl = pad && k.in && ow > 0;
      k.hr = pad && k.in && SW == 1 && ow + 4 < c.W;
      // every load always, from a place that exists: behind a branch the number
      // in flight is unknown to the compiler, and each chunk waits for them all
      const size_t o = ((size_t)n * c.Co + cor) * P + pp;
      k.t = *(const v4f*)(dy + o);
      k.m = *(const v4f*)(mask + o);
      const float* s = x + ((size_t)n * c.Ci + cir) * vol + (k.in ? ((size_t)id * c.H + ih) * c.W + SW * ow : 0);
      k.x0 = *(const v4f*)s;
      if (SW == 2) k.x1 = *(const v4f*)(s + 4);
      if (pad) k.el = s[k.hl ? -1 : 0];
      if (pad && SW == 1) k.er = s[k.hr ? 4 : 0];
    }
    return k;
  };
  WgradSlot* const S = SPLIT ? &wgrad_slots[slot] : nullptr;
  const int t = threadIdx.x;
  // tap (kw of the pass's first) of an operand pair of a chunk
  auto operands = [&](const WgradChunk<SW, KT>& k, const float (&e)[4], int kw, int i, int j, float& g, float& v) {
    if constexpr (SW == 0) {
      g = k.g[i][j];
      v = k.v[i][j];
    } else {
      const float strip[10] = {k.el, k.x0[0], k.x0[1], k.x0[2], k.x0[3], SW == 2 ? k.x1[0] : k.er,
                               SW == 2 ? k.x1[1] : 0.0f, SW == 2 ? k.x1[2] : 0.0f, SW == 2 ? k.x1[3] : 0.0f, 0.0f};
      const int at = KT == 1 ? kw : i;
      const bool lost = (at < pad && j == 0 && !k.hl) || (SW == 1 && at > pad && j == 3 && !k.hr);
      g = k.in && !lost ? e[j] : 0.0f;
      if (KT == K) v = strip[SW * j + i + 1 - pad];
      else v = at < pad ? strip[SW * j] : (at == pad ? strip[SW * j + 1] : strip[SW * j + 2]);
      if (!k.in || lost) v = 0.0f;   // what was loaded instead may be no number
    }
  };
#pragma unroll 1
  for (int kw = 0; kw < K; kw += KT) {
    // not SPLIT: joined quarters 0 + 2 and 1 + 3 of wave 0
    v16f even[SPLIT ? 1 : 4], odd[SPLIT ? 1 : 4];
    float evenb[4], oddb[4];
#pragma unroll 1
    for (int turn = 0; turn < (SPLIT ? 1 : 4); ++turn) {
      const int quarter = SPLIT ? (int)(blockIdx.x / ntiles) : (turn >> 1 | (turn & 1) << 1);   // 0, 2, 1, 3
      const int cg = quarter + 4 * wave;
      v16f acc[KT][4] = {};
      float bsum[4] = {0, 0, 0, 0};
      // this lane's next output: T = 16 (cg + 16 step) + 4 q
      long long T = 16LL * cg + 4 * q;
      int n = (int)(T / P), p = (int)(T - (long long)n * P);
      const long long steps = (chunks - cg + 15) / 16;
      auto next = [&]() {
        const WgradChunk<SW, KT> k = load(n, p, T < total, kw);
        T += 256;
        p += 256;
        if (p >= P) {
          const unsigned d = div_by((unsigned)p, dP);
          n += (int)d;
          p -= (int)(d * P);
        }
        return k;
      };
      WgradChunk<SW, KT> buf[WGRAD_AHEAD];
#pragma unroll
      for (int u = 0; u < WGRAD_AHEAD; ++u) buf[u] = next();
      for (long long step = 0; step < steps; step += WGRAD_AHEAD) {
#pragma unroll
        for (int u = 0; u < WGRAD_AHEAD; ++u) {   // chunks past the last hold zeros
          const WgradChunk<SW, KT> k = buf[u];
          buf[u] = next();
          float e[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if constexpr (SW == 0) e[j] = k.e[j];
            else e[j] = k.on && (!relu || k.m[j] > 0.0f) ? k.t[j] : 0.0f;
            bsum[j] += e[j];
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < KT; ++i) {
              float g, v;
              operands(k, e, kw, i, j, g, v);
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x1f32(g, v, acc[i][j], 0, 0, 0);
            }
        }
      }
      // the tree's levels 128 and 64: waves 0 + 2 and 1 + 3, then 0 + 1
#pragma unroll
      for (int j = 0; j < 4; ++j) sB[wave][lane][j] = bsum[j];
#pragma unroll
      for (int i = 0; i < KT; ++i)
#pragma unroll
        for (int half = 2; half > 0; half >>= 1) {
          if (wave >= half && wave < 2 * half)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int o = 0; o < 16; ++o) sAcc[wave - half][lane][16 * j + o] = acc[i][j][o];
          __syncthreads();
          if (wave < half)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int o = 0; o < 16; ++o) acc[i][j][o] += sAcc[wave][lane][16 * j + o];
          __syncthreads();
        }
      if (wave == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) bsum[j] = (sB[0][lane][j] + sB[2][lane][j]) + (sB[1][lane][j] + sB[3][lane][j]);
        if constexpr (SPLIT) {   // agent scope: the quarters cross the caches of the XCDs
          float (*const part)[WGRAD_ENTRY] = S->part[tile][quarter];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int i = 0; i < KT; ++i)
#pragma unroll
              for (int o = 0; o < 16; ++o)
                __hip_atomic_store(&part[4 * (o >> 2) + j][256 * i + (4 * q + (o & 3)) * 16 + r], acc[i][j][o],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&part[4 * q + j][256 * K + r], bsum[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (turn == 0) {
              even[j] = acc[0][j];
              evenb[j] = bsum[j];
            } else if (turn == 1) {
              even[j] += acc[0][j];
              evenb[j] += bsum[j];
            } else if (turn == 2) {
              odd[j] = acc[0][j];
              oddb[j] = bsum[j];
            } else {
              even[j] += odd[j] + acc[0][j];
              evenb[j] += oddb[j] + bsum[j];
            }
          }
        }
      }
      __syncthreads();
    }
    if constexpr (!SPLIT) {
      if (wave != 0) continue;
      // a lane's 16 chains (block q', product j) of four weights, then of its channel's g
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        float v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (even[j][o] + even[j][o + 8]) + (even[j][o + 4] + even[j][o + 12]);
        const int row = co0 + 4 * q + o;
        if (row < c.Co && xon) dw[(((size_t)row * c.Ci + ci) * T2 + tap) * K + kw] = (v[0] + v[2]) + (v[1] + v[3]);
      }
      float e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        e[j] = evenb[j] + __shfl_xor(evenb[j], 32);
        e[j] += __shfl_xor(e[j], 16);
      }
      if (bias && kw == 0 && q == 0 && von) db[co] = (e[0] + e[2]) + (e[1] + e[3]);
    }
  }
  if constexpr (SPLIT) {
    __threadfence();
    __syncthreads();
    if (t == 0) last = __hip_atomic_fetch_add(&S->count[tile], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == 3u;
    __syncthreads();
    if (!last) return;
    // entry e of the chains: quarters 0 + 2 and 1 + 3, their sum, then the tree over the 16
    auto join = [&](int e) {
      float v[16], w[4][16];
#pragma unroll
      for (int k = 0; k < 16; ++k)
#pragma unroll
        for (int h = 0; h < 4; ++h)
          w[h][k] = __hip_atomic_load(&S->part[tile][h][k][e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = (w[0][k] + w[2][k]) + (w[1][k] + w[3][k]);
#pragma unroll
      for (int h = 8; h > 0; h >>= 1)
#pragma unroll
        for (int k = 0; k < h; ++k) v[k] += v[k + h];
      return v[0];
    };
    const int o = co0 + t / 16, i = ci0 + t % 16;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const float d = join(256 * k + t);
      if (o < c.Co && i < c.Ci) dw[(((size_t)o * c.Ci + i) * T2 + tap) * K + k] = d;
    }
    if (bias && t < 16) {
      const float e = join(256 * K + t);
      if (co0 + t < c.Co) db[co0 + t] = e;
    }
    if (t == 0) __hip_atomic_store(&S->count[tile], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
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
  // K = 1: one step a channel group, so the waves take 32 positions each instead
  // (24 x 18 x 26 x 32 to 7 channels: 7.9 us a call sharing them, 7.6 us)
  constexpr bool OWN = K == 1;
  constexpr int WS = OWN ? 1 : 4;                     // distance of a wave's steps
  constexpr int NA = T3 * ROWS * LC, NS = 2 * 4 * 16 * 64;
  __shared__ __align__(16) unsigned short sA[NA > NS ? NA : NS];
  const int P = c.Do * c.Ho * c.Wo;
  const size_t vol = (size_t)c.D * c.H * c.W;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 31, h = lane >> 5;
  const int n = blockIdx.y, p = (OWN ? blockIdx.x * 4 + wave : blockIdx.x) * 32 + col, row0 = blockIdx.z * ROWS;
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
    if (!staged) __syncthreads();   // a wave without steps
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
