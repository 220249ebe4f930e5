// Deterministic block reductions shared by the solver's kernels.
#pragma once

#include "kqr_internal.h"

namespace kqr {

// x of one lane in every lane
__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
  return __hiloint2double(hi, lo);
}

// x of another lane by DPP.  0xB1: lane ^ 1; 0x4E: lane ^ 2; 0x141: lane ^ 7
// (row_half_mirror); 0x140: lane ^ 15 (row_mirror); 0x124 / 0x128: the lane 4 /
// 8 further round its row of 16.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_update_dpp(0, int(uint32_t(u)), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, int(uint32_t(u >> 32)), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, (uint64_t(uint32_t(hi)) << 32) | uint32_t(lo));
}

// x + the value of the lane 16 (SWAP16) or 32 lanes away, the same on both lanes
template <bool SWAP16>
__device__ __forceinline__ double swap_sum_f64(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t l = uint32_t(u), h = uint32_t(u >> 32);
  uint32_t l0, l1, h0, h1;
  if constexpr (SWAP16) {
    const auto a = __builtin_amdgcn_permlane16_swap(l, l, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(h, h, false, false);
    l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
  } else {
    const auto a = __builtin_amdgcn_permlane32_swap(l, l, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    l0 = a[0]; l1 = a[1]; h0 = b[0]; h1 = b[1];
  }
  return __builtin_bit_cast(double, (uint64_t(h0) << 32) | l0) + __builtin_bit_cast(double, (uint64_t(h1) << 32) | l1);
}

// Sums over each row of 16 lanes, the same in its lanes: lanes 8, 4, 2, 1 apart
// in turn, or 1, 2, 4, 8 (UP) -- then the mirrors reach the lane 4 and 8 apart,
// the values being equal in groups of four and of eight by that time.
template <bool UP = false>
__device__ __forceinline__ double row16_sum_f64(double x) {
  if (UP) {
    x += dpp_f64<0xB1>(x);
    x += dpp_f64<0x4E>(x);
    x += dpp_f64<0x141>(x);
    return x + dpp_f64<0x140>(x);
  }
  x += dpp_f64<0x128>(x);
  x += dpp_f64<0x124>(x);
  x += dpp_f64<0x4E>(x);
  return x + dpp_f64<0xB1>(x);
}

// Sum of x over the wave, the same in every lane: lanes 32, 16, 8, 4, 2, 1
// apart are added in turn (after the step of 8 the values repeat every 8 lanes,
// so a rotation by 4 reaches the lane 4 apart), the tree and the bits of a
// __shfl_xor loop without its twelve LDS permutes (about 100 cycles each in a
// dependent chain): the 29 sums of a line-search pass at n = 2000 take 10.6
// instead of 19.8 us.
__device__ __forceinline__ double wave_sum_f64(double x) {
  x = swap_sum_f64<false>(x);
  return row16_sum_f64(swap_sum_f64<true>(x));
}

// out[q] = sum over b < nblocks of partials[b nq + q], in a fixed order (one
// 256-thread block).
__device__ __forceinline__ void finish_sums(const double* __restrict__ partials, int nblocks, int nq,
                                            double* __restrict__ out) {
  __shared__ double sh[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int q = 0; q < nq; ++q) {
    double s = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) s += partials[b * nq + q];
    s = wave_sum_f64(s);
    if (lane == 0) sh[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[q] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
    __syncthreads();
  }
}

// Vectors up to this length are reduced by a single workgroup of
// kOneBlockThreads threads (no second pass); longer ones by up to kRedBlocks
// workgroups of kRedThreads whose partials a finishing launch adds.
// Workgroups never wait for one another: on a GPU whose L2 is split over
// several dies, making one workgroup's writes visible to another inside a
// kernel costs an L2 write-back per workgroup.
constexpr int64_t kOneBlockN = 16384;
constexpr int kOneBlockThreads = 1024;

// Block partials (any block size up to 1024); with a single workgroup they
// are the result and go to out directly, otherwise reduce_finalize adds them
// afterwards.  block_sums_at takes the block's index and the grid's size
// explicitly (several grids sharing one launch).
template <int NQ>
__device__ __forceinline__ void block_sums_at(double (&v)[NQ], double* __restrict__ partials,
                                              double* __restrict__ out, int blk, int nblk) {
  __shared__ double sh[NQ][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = int(blockDim.x) >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    double s = v[q];
    s = wave_sum_f64(s);
    if (lane == 0) sh[q][wave] = s;
  }
  __syncthreads();
  if (threadIdx.x < NQ) {
    double s = 0.0;
    for (int w = 0; w < nw; ++w) s += sh[threadIdx.x][w];
    if (nblk == 1) out[threadIdx.x] = s;
    else partials[blk * NQ + threadIdx.x] = s;
  }
}

template <int NQ>
__device__ __forceinline__ void block_sums(double (&v)[NQ], double* __restrict__ partials, double* __restrict__ out) {
  block_sums_at<NQ>(v, partials, out, int(blockIdx.x), int(gridDim.x));
}

// Sum of v over the (single) workgroup in block_sums' order, in every thread.
// Each thread adds the waves' sums itself, so a call has one barrier; calls of
// a kernel alternate SLOT, which keeps a call's sums while the next is formed.
template <int SLOT>
__device__ __forceinline__ double block_sum_all(double v) {
  __shared__ double sh[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = int(blockDim.x) >> 6;
  v = wave_sum_f64(v);
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < nw; ++w) s += sh[w];
  return s;
}

// Single-workgroup PCG kernels keep up to this many vector elements per thread
// in registers (one memory round trip for all of a kernel's loads).
constexpr int kHeld = 4;

// Launch shape of an O(n) reduction: one workgroup of kOneBlockThreads up
// to kOneBlockN elements, else one kRedThreads-thread workgroup per
// kRedThreads elements up to kRedBlocks (grid-stride beyond).
struct RedShape {
  unsigned blocks, threads;
};
inline RedShape red_shape(int64_t n) {
  if (n <= kOneBlockN) return RedShape{1u, unsigned(kOneBlockThreads)};
  const int64_t b = (n + kRedThreads - 1) / kRedThreads;
  return RedShape{unsigned(b < kRedBlocks ? b : kRedBlocks), unsigned(kRedThreads)};
}

}  // namespace kqr
