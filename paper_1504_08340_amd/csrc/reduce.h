// Deterministic reductions over many workgroups in one launch.
//
// A reduction of n entries is cut into nb contiguous parts (a function of n alone);
// a part's threads walk its entries in strides of the workgroup, add in a fixed tree,
// and the nb part values are added in a fixed tree again.  Each workgroup
// leaves its part value in a slot and counts itself in; the last one to arrive
// forms the result and sets the count back, so that the launch needs no second
// kernel and no clear.  One workgroup streams about 0.1 TB/s, which bounded
// every inner product of the optimizer: 278,850 entries with weights took
// 100 us in one workgroup and take 6.9 us in 137 (most of it the launch and
// the two trees); an L-BFGS iteration's optimizer work (60 of them) 7.15 -> 1.6 ms.
//
// Whether nb workgroups or one carry it out does not change a bit of the result.
// A slot belongs to a stream, whose launches do not overlap, until another stream
// needs it and all launches in it have ended; a launch that has none (see
// stream_slot) takes one workgroup of 16 waves, a wave a part: it forms what the
// part's 256 threads would, four a lane, and joins them between its lanes, so that
// no wave waits for another before the last tree.  Of 16 parts or fewer the waves
// take quarters, and meet once more.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace pmlfwi {

constexpr int RED_THREADS = 256;      // threads of a part
constexpr int RED_ONE = 1024;         // threads of a workgroup that walks all parts
constexpr int RED_PARTS = 256;        // most parts of a reduction
constexpr int RED_PER_PART = 2048;    // entries that pay for a workgroup
constexpr int RED_SLOTS = 64;         // streams that may hold a slot (per device)

struct RedSlot {
  double part[RED_PARTS];
  unsigned count;
  unsigned pad[63];
};

static __device__ RedSlot red_slots[RED_SLOTS];   // counts start at 0
static __device__ unsigned red_done[RED_SLOTS];   // launches that have left their slot

__host__ __device__ inline int red_parts(long long n) {
  const long long nb = (n + RED_PER_PART - 1) / RED_PER_PART;
  return nb < 1 ? 1 : (nb > RED_PARTS ? RED_PARTS : (int)nb);
}

struct RedSum {
  static __device__ double init() { return 0.0; }
  static __device__ double join(double a, double b) { return a + b; }
};
struct RedMax {
  static __device__ double init() { return 0.0; }
  static __device__ double join(double a, double b) { return fmax(a, b); }
};
// Tree over the workgroup's values: the upper half onto the lower, and again.
// Down to a wave's 64 values through LDS, below that between its lanes, without
// a barrier a level.  The result is valid in thread 0.
template <typename Op>
__device__ __forceinline__ double red_tree(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = RED_THREADS / 2; s >= 64; s >>= 1) {
    if ((int)threadIdx.x < s) v = sh[threadIdx.x] = Op::join(v, sh[threadIdx.x + s]);
    __syncthreads();
  }
  for (int s = 32; s > 0; s >>= 1) v = Op::join(v, __shfl_down(v, s));
  return v;
}

// The same tree over the 256 values that a wave holds, four a lane: those of threads
// lane + 64 k, or (QUADS) 4 lane + k.  The result is valid in lane 0.
template <typename Op, bool QUADS>
__device__ __forceinline__ double red_wave(double (&v)[4]) {
  auto lanes = [](double r) {
    for (int s = 32; s > 0; s >>= 1) r = Op::join(r, __shfl_down(r, s));
    return r;
  };
  if (QUADS)
    for (int k = 0; k < 4; ++k) v[k] = lanes(v[k]);
  const double r = Op::join(Op::join(v[0], v[2]), Op::join(v[1], v[3]));
  return QUADS ? r : lanes(r);
}

// Entries of a part: those from part * span on, as far as there are any.
__device__ __forceinline__ long long red_span(long long n, int nb) {
  return ((n + nb - 1) / nb + RED_THREADS - 1) / RED_THREADS * RED_THREADS;
}

// add(load(i)) over thread t's entries of part `part` of nb, in order: eight loads are
// in flight together, where one by one each waits for memory (eight waits of an
// average thread).
template <typename L, typename A>
__device__ __forceinline__ void red_entries(int part, int t, int nb, long long n, L&& load, A&& add) {
  constexpr int U = RED_PER_PART / RED_THREADS;
  const long long span = red_span(n, nb), first = part * span + t, end = min(n, (part + 1) * span);
  for (long long i = first; i < end; i += U * RED_THREADS) {
    decltype(load(i)) v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long j = i + u * RED_THREADS;
      v[u] = load(j < end ? j : i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * RED_THREADS < end) add(v[u], i + u * RED_THREADS);
  }
}

// The same for the threads 4 lane + k, k < 4: add(k, entry, its index).
template <typename L, typename A>
__device__ __forceinline__ void red_quads(int part, int lane, int nb, long long n, L&& load, A&& add) {
  constexpr int U = RED_PER_PART / RED_THREADS / 4;
  const long long span = red_span(n, nb), first = part * span + 4 * lane, end = min(n, (part + 1) * span);
  for (long long i = first; i < end; i += U * RED_THREADS) {
    if (i + (U - 1) * RED_THREADS + 3 < end) {
      decltype(load(i)) v[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[u][k] = load(i + u * RED_THREADS + k);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) add(k, v[u][k], i + u * RED_THREADS + k);
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        for (int u = 0; u < U; ++u)
          if (i + u * RED_THREADS + k < end) add(k, load(i + u * RED_THREADS + k), i + u * RED_THREADS + k);
    }
  }
}

// Joins one value per part; launch: nb workgroups of RED_THREADS (with one part no
// slot is needed), or one of RED_ONE.  Returns true in the threads of the workgroup
// or wave whose thread 0 holds the result.
// f(part, t): thread t's share of a part.  quads(part, lane, v), if there is one: those
// of threads 4 lane + k, added to v[k], for entries that are read and no more (loads
// of 8 bytes keep a CU at half the rate of vectors: 10^6 products with weights 380 us
// one by one, 343 so; where each entry is written or gathered for, neighbours in
// neighbouring lanes are faster).
struct RedNone {};
template <typename Op, typename F, typename Q = RedNone>
__device__ __forceinline__ bool reduce_parts(int nb, int slot, double* sh, double& result, F&& f, Q&& quads = {}) {
  constexpr bool QUADS = !std::is_same<std::decay_t<Q>, RedNone>::value;
  if (blockDim.x > RED_THREADS) {
    __shared__ double parts[RED_PARTS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int WAVES = RED_ONE / 64;
    double v[4];
    if (nb <= WAVES) {
      __shared__ double quarter[4 * WAVES][64];
      for (int u = wave; u < 4 * nb; u += WAVES) quarter[u][lane] = f(u >> 2, lane + 64 * (u & 3));
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = wave < nb ? quarter[4 * wave + k][lane] : Op::init();
      const double r = red_wave<Op, false>(v);
      if (lane == 0 && wave < nb) parts[wave] = r;
    } else {
      for (int b = wave; b < nb; b += WAVES) {
        if constexpr (QUADS) {
          v[0] = v[1] = v[2] = v[3] = Op::init();
          quads(b, lane, v);
        } else {
#pragma unroll 1
          for (int k = 0; k < 4; ++k) {
            const double s = f(b, lane + 64 * k);
            v[0] = k == 0 ? s : v[0];
            v[1] = k == 1 ? s : v[1];
            v[2] = k == 2 ? s : v[2];
            v[3] = k == 3 ? s : v[3];
          }
        }
        const double r = red_wave<Op, QUADS>(v);
        if (lane == 0) parts[b] = r;
      }
    }
    __syncthreads();
    if (wave) return false;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = lane + 64 * k < nb ? parts[lane + 64 * k] : Op::init();
    result = red_wave<Op, false>(v);
    return true;
  }
  const double v = red_tree<Op>(f((int)blockIdx.x, (int)threadIdx.x), sh);
  if (nb == 1) {
    result = Op::join(v, Op::init());   // as the tree over the parts would
    return true;
  }
  __shared__ bool last;
  RedSlot* const S = &red_slots[slot];
  if (threadIdx.x == 0) {
    // agent scope: the parts cross the caches of the XCDs
    __hip_atomic_store(&S->part[blockIdx.x], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(&S->count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nb - 1;
  }
  __syncthreads();
  if (!last) return false;
  result = red_tree<Op>((int)threadIdx.x < nb ? __hip_atomic_load(&S->part[threadIdx.x], __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT)
                                              : Op::init(), sh);
  if (threadIdx.x == 0) {
    __hip_atomic_store(&S->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(&red_done[slot], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
  return true;
}

static_assert(RED_PARTS <= RED_THREADS, "one thread per part value");

// out[0] = sum_i a_i b_i (w_i)
__global__ void __launch_bounds__(RED_ONE) dot_kernel(long long n, const double* __restrict__ a,
                                                      const double* __restrict__ b, const double* __restrict__ w,
                                                      double* __restrict__ out, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  double r;
  // multiply-adds written out: left to the compiler, they may differ between the routes
  struct Pair {
    double x, y;
  };
  auto plain = [&](long long i) { return Pair{a[i], b[i]}; };
  auto weighted = [&](long long i) { return Pair{a[i] * b[i], w[i]}; };
  auto one = [&](int part, int t) {
    double acc = 0.0;
    auto add = [&](Pair p, long long) { acc = fma(p.x, p.y, acc); };
    if (w) red_entries(part, t, nb, n, weighted, add);
    else red_entries(part, t, nb, n, plain, add);
    return acc;
  };
  auto quads = [&](int part, int lane, double (&v)[4]) {
    auto add = [&](int k, Pair p, long long) { v[k] = fma(p.x, p.y, v[k]); };
    if (w) red_quads(part, lane, nb, n, weighted, add);
    else red_quads(part, lane, nb, n, plain, add);
  };
  if (reduce_parts<RedSum>(nb, slot, sh, r, one, quads) && threadIdx.x == 0) out[0] = r;
}

// out[0] = max_i |x_i|
__global__ void __launch_bounds__(RED_ONE) absmax_kernel(long long n, const double* __restrict__ x,
                                                         double* __restrict__ out, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  double r;
  auto load = [&](long long i) { return x[i]; };
  auto one = [&](int part, int t) {
    double m = 0.0;
    red_entries(part, t, nb, n, load, [&](double v, long long) { m = fmax(m, fabs(v)); });
    return m;
  };
  auto quads = [&](int part, int lane, double (&v)[4]) {
    red_quads(part, lane, nb, n, load, [&](int k, double e, long long) { v[k] = fmax(v[k], fabs(e)); });
  };
  if (reduce_parts<RedMax>(nb, slot, sh, r, one, quads) && threadIdx.x == 0) out[0] = r;
}

}  // namespace pmlfwi
