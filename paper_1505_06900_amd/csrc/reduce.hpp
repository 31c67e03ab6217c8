// FP64 sums over a grid in a fixed order: wave butterfly (64 lanes) -> LDS across
// waves -> one partial per block -> the sum of the partials, thread t taking blocks
// t, t + 256, ..., then a fixed tree.  Grids of at most kTicketBlocks blocks leave that
// sum to the block that finishes last (the order does not depend on which it is);
// larger ones take a launch for it: a block's ticket costs about 12 ns of a chain
// through one address, so 981 blocks spent 12 us on it where a launch takes 4.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ops.hpp"

namespace lbrr {

constexpr int kTicketBlocks = 256;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sums of v over the block's threads, at out[0 .. NV) written by threads 0 .. NV - 1
// (Shared: with stores that other compute units' caches see).
template <int NV, bool Shared = false>
__device__ __forceinline__ void block_sum_store(double (&v)[NV], double* __restrict__ out) {
  __shared__ double lds[NV][kReduceBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    const double s = wave_sum(v[c]);
    if (lane == 0) lds[c][wid] = s;
  }
  __syncthreads();
  if (threadIdx.x < NV) {
    double s = 0.0;
    for (int w = 0; w < kReduceBlock / 64; ++w) s += lds[threadIdx.x][w];
    if constexpr (Shared) __hip_atomic_store(out + threadIdx.x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else out[threadIdx.x] = s;
  }
}

// Sum of nblocks partials by one block.
template <int NV>
__device__ __forceinline__ void sum_partials(const double* partials, unsigned nblocks, double* __restrict__ out) {
  double acc[NV];
#pragma unroll
  for (int c = 0; c < NV; ++c) acc[c] = 0.0;
  for (unsigned b = threadIdx.x; b < nblocks; b += kReduceBlock) {
#pragma unroll
    for (int c = 0; c < NV; ++c)
      acc[c] += __hip_atomic_load(partials + int64_t(b) * NV + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  block_sum_store<NV>(acc, out);
}

// Adds acc over the whole grid into out[0 .. NV).  partials: NV per block; ticket: 0
// before the launch, and 0 again after it (launches that share it are ordered).
// Without a ticket the partials are left for k_final.
template <int NV>
__device__ __forceinline__ void reduce_blocks(double (&acc)[NV], double* __restrict__ partials,
                                              unsigned* __restrict__ ticket, double* __restrict__ out) {
  __shared__ bool last;
  block_sum_store<NV, true>(acc, partials + int64_t(blockIdx.x) * NV);
  if (!ticket) return;
  if (threadIdx.x < 64) {
    // The wave whose lanes wrote the partials waits for its stores, which bypass the
    // caches that are not shared, before it takes a ticket.  (A device-wide fence
    // in their place writes back the L2 for every block: 60 us more at 2048 blocks.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x;
  }
  __syncthreads();
  if (!last) return;
  sum_partials<NV>(partials, gridDim.x, out);
  if (threadIdx.x == 0) __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int NV>
__global__ void __launch_bounds__(kReduceBlock) k_final(const double* __restrict__ partials, int nblocks,
                                                        double* __restrict__ out) {
  sum_partials<NV>(partials, unsigned(nblocks), out);
}

}  // namespace lbrr
