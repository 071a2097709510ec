// Deterministic reductions over many workgroups in one launch.
//
// A reduction of n entries is cut into nb parts (a function of n alone); part
// b's threads walk its entries in strides of the workgroup, add in a fixed tree,
// and the nb part values are added in a fixed tree again.  Each workgroup
// leaves its part value in a slot and counts itself in; the last one to arrive
// forms the result and sets the count back, so that the launch needs no second
// kernel and no clear.  One workgroup streams about 0.1 TB/s, which bounded
// every inner product of the optimizer: 278,850 entries with weights took
// 100 us in one workgroup and take 6.9 us in 137 (most of it the launch and
// the two trees); an L-BFGS iteration's optimizer work (60 of them) 7.15 -> 1.6 ms.
//
// Whether nb workgroups or one (walking the parts in turn) carry it out does not
// change a bit of the result.  A slot belongs to a stream, whose launches do
// not overlap; a launch that has none (see stream_slot) takes one workgroup.
#pragma once
#include <hip/hip_runtime.h>

namespace pmlfwi {

constexpr int RED_THREADS = 256;
constexpr int RED_PARTS = 256;        // most parts of a reduction
constexpr int RED_PER_PART = 2048;    // entries that pay for a workgroup
constexpr int RED_SLOTS = 64;         // streams that may hold a slot (per device)

struct RedSlot {
  double part[RED_PARTS];
  unsigned count;
  unsigned pad[63];
};

static __device__ RedSlot red_slots[RED_SLOTS];   // counts start at 0
__device__ __forceinline__ RedSlot* red_slot(int i) { return i < 0 ? nullptr : &red_slots[i]; }

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

// add(load(i)) over this thread's entries of a part, in order: eight loads are in
// flight together, where one by one each waits for memory (eight waits of an
// average thread).
template <typename L, typename A>
__device__ __forceinline__ void red_entries(int part, long long n, long long step, L&& load, A&& add) {
  constexpr int U = RED_PER_PART / RED_THREADS;
  for (long long i = (long long)part * RED_THREADS + threadIdx.x; i < n; i += U * step) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long j = i + u * step;
      v[u] = load(j < n ? j : i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * step < n) add(v[u]);
  }
}

// Joins one value per part; grid: nb workgroups, or one that has left all nb
// part values in LDS.  Returns true in the workgroup that holds the result.
// F: double f(int part) is this thread's share of a part.
template <typename Op, typename F>
__device__ __forceinline__ bool reduce_parts(int nb, RedSlot* slot, double* sh, double& result, F&& f) {
  if (gridDim.x == 1) {
    __shared__ double parts[RED_PARTS];
    for (int b = 0; b < nb; ++b) {
      const double v = red_tree<Op>(f(b), sh);
      if (threadIdx.x == 0) parts[b] = v;
    }
    __syncthreads();
    result = red_tree<Op>((int)threadIdx.x < nb ? parts[threadIdx.x] : Op::init(), sh);
    return true;
  }
  __shared__ bool last;
  const double v = red_tree<Op>(f((int)blockIdx.x), sh);
  if (threadIdx.x == 0) {
    // agent scope: the parts cross the caches of the XCDs
    __hip_atomic_store(&slot->part[blockIdx.x], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(&slot->count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)nb - 1;
  }
  __syncthreads();
  if (!last) return false;
  result = red_tree<Op>((int)threadIdx.x < nb ? __hip_atomic_load(&slot->part[threadIdx.x], __ATOMIC_RELAXED,
                                                                  __HIP_MEMORY_SCOPE_AGENT)
                                              : Op::init(), sh);
  if (threadIdx.x == 0) __hip_atomic_store(&slot->count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

static_assert(RED_PARTS <= RED_THREADS, "one thread per part value");

// out[0] = sum_i a_i b_i (w_i)
__global__ void __launch_bounds__(RED_THREADS) dot_kernel(long long n, const double* __restrict__ a,
                                                          const double* __restrict__ b, const double* __restrict__ w,
                                                          double* __restrict__ out, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  double r;
  const long long step = (long long)nb * RED_THREADS;
  if (reduce_parts<RedSum>(nb, red_slot(slot), sh, r, [&](int part) {
        double acc = 0.0;
        auto add = [&](double v) { acc += v; };
        if (w) red_entries(part, n, step, [&](long long i) { return a[i] * b[i] * w[i]; }, add);
        else red_entries(part, n, step, [&](long long i) { return a[i] * b[i]; }, add);
        return acc;
      }) && threadIdx.x == 0)
    out[0] = r;
}

// out[0] = max_i |x_i|
__global__ void __launch_bounds__(RED_THREADS) absmax_kernel(long long n, const double* __restrict__ x,
                                                             double* __restrict__ out, int nb, int slot) {
  __shared__ double sh[RED_THREADS];
  double r;
  const long long step = (long long)nb * RED_THREADS;
  if (reduce_parts<RedMax>(nb, red_slot(slot), sh, r, [&](int part) {
        double m = 0.0;
        red_entries(part, n, step, [&](long long i) { return x[i]; }, [&](double v) { m = fmax(m, fabs(v)); });
        return m;
      }) && threadIdx.x == 0)
    out[0] = r;
}

}  // namespace pmlfwi
