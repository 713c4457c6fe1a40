// Device helpers shared by the kernel sources: fixed-order block reductions, the block-to-XCD remap and
// scalar-addressed rows.
//
// Wave size is 64.  Every reduction is a fixed tree: per-thread FP64 sums, a wave
// butterfly (__shfl_xor), a fixed-order sum of the waves of a block into one partial
// per block, then a fixed-order strided sum of the partials in a later kernel, so
// results are bitwise reproducible run to run.
#pragma once
#include <hip/hip_runtime.h>

#include <stdint.h>

namespace rmh {

// ------------------------------------------------------------------------------------------
// reductions

// v plus its value in another lane, by data-parallel-primitive moves (CTRL) within rows of 16 lanes
template <int CTRL>
__device__ __forceinline__ double add_dpp(double v) {
  const uint64_t w = __builtin_bit_cast(uint64_t, v);
  const uint32_t l = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)w, CTRL, 0xf, 0xf, false);
  const uint32_t h = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(w >> 32), CTRL, 0xf, 0xf, false);
  return v + __builtin_bit_cast(double, (uint64_t)l | ((uint64_t)h << 32));
}

// Butterfly over lane distances 32, 16, 8, 4, 2, 1, the result in every lane.  Distances 32 and 16 are swaps of
// lane halves and rows; for 8 and 4 a rotation of the row by as much finds the same values (the lanes 8 apart
// are equal by then); 2 and 1 are quad permutations.  Moves through registers: shuffles go through the LDS
// unit, some 90 cycles for each of the six dependent steps.
__device__ __forceinline__ double wave_sum(double v) {
  const auto swap_add = [](double x, auto swap) {
    const uint64_t w = __builtin_bit_cast(uint64_t, x);
    const auto l = swap((uint32_t)w), h = swap((uint32_t)(w >> 32));
    return __builtin_bit_cast(double, (uint64_t)(uint32_t)l[0] | ((uint64_t)(uint32_t)h[0] << 32)) +
           __builtin_bit_cast(double, (uint64_t)(uint32_t)l[1] | ((uint64_t)(uint32_t)h[1] << 32));
  };
  v = swap_add(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
  v = swap_add(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
  v = add_dpp<0x128>(v);   // row_ror:8
  v = add_dpp<0x124>(v);   // row_ror:4
  v = add_dpp<0x4e>(v);    // quad_perm [2, 3, 0, 1]
  return add_dpp<0xb1>(v); // quad_perm [1, 0, 3, 2]
}

// Sum of the waves' values in order; up to four with their reads in flight together (one after the other they
// cost an LDS latency per wave).
__device__ __forceinline__ double waves_sum(const double* w) {
  const int nw = (blockDim.x + 63) >> 6;
  double s = 0.0;
  if (nw <= 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double t = w[i];
      s = i < nw ? s + t : s;
    }
  } else {
    for (int i = 0; i < nw; ++i) s += w[i];
  }
  return s;
}

// Sum over the block (any multiple of 64 threads up to 1024); result valid in thread 0.
template <int NQ>
__device__ __forceinline__ void block_sum(double (&v)[NQ], double (*lds)[16]) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double w = wave_sum(v[q]);
    if (lane == 0) lds[q][wid] = w;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = waves_sum(lds[q]);
  }
  __syncthreads();  // lds may be reused by the caller right away
}

// The same with the result in every thread; the caller does not reuse lds before a barrier.
template <int NQ>
__device__ __forceinline__ void block_sum_all(double (&v)[NQ], double (*lds)[16]) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double w = wave_sum(v[q]);
    if (lane == 0) lds[q][wid] = w;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NQ; ++q) v[q] = waves_sum(lds[q]);
}

// Strided fixed-order sum of n values by a whole block; result in thread 0.
// Fixed-order sum of p[0, n): four independent loads in flight per thread, then the block tree.
__device__ __forceinline__ double block_sum_array(const double* p, int32_t n, double (*lds)[16]) {
  const int32_t B = blockDim.x;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int32_t i = threadIdx.x;
  for (; i + 3 * B < n; i += 4 * B) {
    a0 += p[i];
    a1 += p[i + B];
    a2 += p[i + 2 * B];
    a3 += p[i + 3 * B];
  }
  for (; i < n; i += B) a0 += p[i];
  double v[1] = {(a0 + a1) + (a2 + a3)};
  block_sum<1>(v, lds);
  return v[0];
}

__device__ __forceinline__ int32_t remap_block(int32_t b, int32_t G, int32_t xcd) {
  // Consecutive hardware block ids go round-robin over the 8 XCDs; give each XCD a
  // contiguous range of the lattice so neighbouring sites share its L2.  XCD x runs G / 8 blocks,
  // and one more where x < G % 8.  (Grids that are no multiple of eight are half of all lattices; left
  // unmapped, the FP32 walk at 36x20x20x36 with two fields took 255 us against 149 so, one thread per site and
  // direction pair at 19x15x17x19 with three 87 against 42.)
  if (!xcd) return b;
  const int32_t x = b & 7, r = G & 7;
  return x * (G >> 3) + (x < r ? x : r) + (b >> 3);
}

// The rows (components) of an array at one site per lane: row r at base + r * V, with the base address
// the same for the whole wave, in scalar registers, and an unsigned 32-bit byte offset per lane (at
// most 2^28 sites of 8 bytes) that the load instruction adds by itself.  The empty asm keeps the base
// scalar and stepped from row to row: left alone, the compiler computes every row's address as a
// 64-bit vector add, a quarter of the vector instructions of a hop.  With the 3x3 form's shorter
// arithmetic (mat_hop) this took FP64 at 32^3x64 from 644 to 569 us per application, FP32 at 24^4 (4 fields)
// from 211 to 195 us; the streamed form alone, at equal arithmetic, gains 1-7 %.
template <typename T>
using Global = __attribute__((address_space(1))) T;
template <typename T>
__device__ __forceinline__ uint32_t byte_off(int32_t s) {
  return (uint32_t)s * (uint32_t)sizeof(T);
}
template <typename T>
struct Rows {
  uint64_t b, stride;
  uint32_t o;
  __device__ __forceinline__ Rows(const T* base, int64_t V, uint32_t byte_offset)
      : b((uint64_t)base), stride((uint64_t)V * sizeof(T)), o(byte_offset) {
    asm volatile("" : "+s"(b), "+v"(o));
  }
  __device__ __forceinline__ Global<T>* ptr() const { return (Global<T>*)((Global<char>*)b + o); }
  __device__ __forceinline__ T get() {
    const T x = *ptr();
    next();
    return x;
  }
  __device__ __forceinline__ void next() {
    b += stride;
    asm("" : "+s"(b));
  }
};

}  // namespace rmh
