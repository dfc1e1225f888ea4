// reduce.hpp -- deterministic float64 per-configuration reductions (reduce.hip).
#pragma once

#include <vector>

#include "nbr.hpp"

namespace nepmi {

constexpr int kRedValues = 11;    // energy, 9 virial components, kinetic energy
// Atoms per item, by the atoms of the configuration: a small one is one item; up
// to 65,536 atoms an item is one atom per thread and the items' sums one per
// thread, the shortest chain (an MD step's sums of 3,686 atoms in items of 2,048:
// 11.6 us, of 256: 6.4); more atoms take fewer, longer items (900,000 atoms in
// items of 2,048: 24 us).
constexpr int64_t red_chunk(int64_t atoms) { return atoms <= 512 ? 512 : atoms <= 65536 ? 256 : 2048; }

struct RedItem {
  int cfg;
  int pad;
  int64_t a0, a1;  // caller-order atom range
};

// What the sums read and write; any array of values and any output may be null.
template <class T>
struct SumArgs {
  const RedItem* items = nullptr;
  const int* start = nullptr;  // first item of each configuration (n_cfg + 1)
  int* done = nullptr;         // per configuration, items summed so far: 0 between launches
  double* part = nullptr;      // [n_items][kRedValues]
  int n_items = 0;
  const T* Ei = nullptr;       // [N] caller order
  const T* Wi = nullptr;       // [N][9]
  const T* Ki = nullptr;       // [N]
  double* E = nullptr;         // [n_cfg]
  double* V = nullptr;         // [n_cfg][9]
  double* K = nullptr;         // [n_cfg]
};

struct Reducer {
  int n_cfg = 0, n_items = 0;
  DevBuf items_dev, start_dev, done_dev, part;
  // host copies of the plan, the sources of the upload
  std::vector<RedItem> host_items;
  std::vector<int> host_start, host_done;
  // Plan the sums of a batch and add the plan to `up`.
  int setup(int n_cfg, const int64_t* atom_off, Uploader& up);
  void use_arena(Arena* a) {
    for (DevBuf* b : {&items_dev, &start_dev, &done_dev, &part}) {
      b->release();
      b->arena = a;
    }
  }
  // The arguments of one round of sums, for a launch that takes n_items blocks
  // for them (sum_item), and that launch with nothing beside the sums.
  template <class T>
  SumArgs<T> args(const T* Ei, const T* Wi, const T* Ki, double* E, double* V, double* K) const {
    SumArgs<T> a;
    a.items = items_dev.ptr<RedItem>();
    a.start = start_dev.ptr<int>();
    a.done = done_dev.ptr<int>();
    a.part = part.ptr<double>();
    a.n_items = n_items;
    a.Ei = Ei;
    a.Wi = Wi;
    a.Ki = Ki;
    a.E = E;
    a.V = V;
    a.K = K;
    return a;
  }
  template <class T>
  int run(hipStream_t st, const SumArgs<T>& a) const;
};

// Sum of one item (a chunk of a configuration's caller-order atoms) by a block
// of BS threads; the block that ends a configuration's last item sums its
// items.  Both sums have the shape of a block of kRedThreads threads, whatever
// BS: a thread's atoms in order, a butterfly over the 64 lanes of each
// wavefront, then the wavefronts in order.  none: all of it but the outputs (see
// lists_void).
constexpr int kRedThreads = 256;
struct SumShared {
  double wave[kRedThreads / 64][kRedValues];
  int last;
};

template <int BS, class F>
__device__ __forceinline__ double block_sum(F&& add, SumShared& sh) {
  constexpr int NV = kRedValues;
  for (int t = (int)threadIdx.x; t < kRedThreads; t += BS) {
    double acc[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] = 0.0;
    add(t, acc);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int v = 0; v < NV; ++v) acc[v] += __shfl_xor(acc[v], o, 64);
    if ((t & 63) == 0)
#pragma unroll
      for (int v = 0; v < NV; ++v) sh.wave[t >> 6][v] = acc[v];
  }
  __syncthreads();
  double s = 0.0;
  if ((int)threadIdx.x < NV) {
    s = sh.wave[0][threadIdx.x];
#pragma unroll
    for (int u = 1; u < kRedThreads / 64; ++u) s += sh.wave[u][threadIdx.x];
  }
  return s;
}

template <int BS, class T>
__device__ __forceinline__ void sum_item(int item, const SumArgs<T>& a, SumShared& sh, bool none = false) {
  constexpr int NV = kRedValues;
  const RedItem it = a.items[item];
  double s = block_sum<BS>(
      [&](int t, double(&acc)[NV]) {
        for (int64_t i = it.a0 + t; i < it.a1; i += kRedThreads) {
          if (a.Ei) acc[0] += (double)a.Ei[i];
          if (a.Wi) {
#pragma unroll
            for (int x = 0; x < 9; ++x) acc[1 + x] += (double)a.Wi[i * 9 + x];
          }
          if (a.Ki) acc[10] += (double)a.Ki[i];
        }
      },
      sh);
  const int first = a.start[it.cfg], n = a.start[it.cfg + 1] - first, v = (int)threadIdx.x;
  if (n > 1) {
    // The items' sums are handed over through memory: exchanged into place
    // (the exchange has returned, so it is done, before the item is counted),
    // and read by whoever counts last.  All of it is atomic at the scope of the
    // device; a device-wide fence instead would write back the L2 of the block's
    // XCD (sums of 900,000 atoms: 49 us with fences, 24 without).
    if (v < NV) {
      const long long before = __hip_atomic_exchange(reinterpret_cast<long long*>(&a.part[(int64_t)item * NV + v]),
                                                     __double_as_longlong(s), __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("" ::"v"(before));
    }
    __syncthreads();
    if (v == 0)
      sh.last = __hip_atomic_fetch_add(&a.done[it.cfg], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    __syncthreads();
    if (!sh.last) return;
    s = block_sum<BS>(
        [&](int t, double(&acc)[NV]) {
          for (int w = first + t; w < first + n; w += kRedThreads)
#pragma unroll
            for (int x = 0; x < NV; ++x)
              acc[x] += __hip_atomic_load(&a.part[(int64_t)w * NV + x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        },
        sh);
    if (v == 0) __hip_atomic_store(&a.done[it.cfg], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (none) return;
  if (v == 0 && a.E) a.E[it.cfg] = s;
  if (v >= 1 && v <= 9 && a.V) a.V[(int64_t)it.cfg * 9 + v - 1] = s;
  if (v == 10 && a.K) a.K[it.cfg] = s;
}

}  // namespace nepmi
