// Kernel-matrix operators on gfx950: materialisation, the HBM-streamed
// K-apply, the on-the-fly K-apply and single kernel rows.
//
// K_ij = exp(-gamma d_ij) with d the squared Euclidean distance (RBF) or the
// L1 distance (Laplacian) (Section 1).  exp is evaluated as exp2 of
// -gamma log2(e) d on the transcendental unit (kexp2).
#include "kernel_entry.h"
#include "kqr_internal.h"
#include "pstep.h"
#include "reduce.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <mutex>
#include <type_traits>
#include <vector>

namespace kqr {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }
// Round to nearest even (entries are finite).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}

// ================================================================= row norms
// q = the squared norms of the rows of two matrices (nb may be 0), each summed
// in coordinate order.  Eight coordinates are requested at a time: a row's
// loads one after the other took 14.4 us at 100,000 x 30, this 8.6.
__global__ __launch_bounds__(256) void sqnorm_kernel(const float* __restrict__ Xa, int64_t na, float* __restrict__ qa,
                                                     const float* __restrict__ Xb, int64_t nb,
                                                     float* __restrict__ qb, int p) {
  const int64_t i = blockIdx.x * int64_t(256) + threadIdx.x;
  if (i >= na + nb) return;
  const float* x = i < na ? Xa + i * p : Xb + (i - na) * p;
  float s = 0.f;
  int k = 0;
  for (; k + 8 <= p; k += 8) {
    float t[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = x[k + e];
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf(t[e], t[e], s);
  }
  for (; k < p; ++k) s = fmaf(x[k], x[k], s);
  if (i < na) qa[i] = s;
  else qb[i - na] = s;
}

void row_sqnorms2(const float* Xa, int64_t na, float* qa, const float* Xb, int64_t nb, float* qb, int p,
                  hipStream_t st) {
  if (na + nb <= 0) return;
  sqnorm_kernel<<<dim3((unsigned)((na + nb + 255) / 256)), dim3(256), 0, st>>>(Xa, na, qa, Xb, nb, qb, p);
  KQR_LAUNCH_CHECK();
}

void row_sqnorms(const float* X, int64_t n, int p, float* sqn, hipStream_t st) {
  if (n > 0) row_sqnorms2(X, n, sqn, nullptr, 0, nullptr, p, st);
}

// ================================================================= K build
bool kbuild_mfma(const float* X, const float* q, int64_t n, int p, KernelSpec ks, int dtype, void* K, int64_t ldk,
                 int layout, hipStream_t st);  // below, with the matrix-core helpers

// Laplacian, and RBF with p > 32: entries on the VALU.
// Block: 16 rows x 256 columns.  Row tile of X and its norms staged in LDS
// (broadcast reads); each thread keeps its column x_j in registers.
template <int PMAX, bool LAP, bool BF16>
__global__ __launch_bounds__(256) void kbuild_kernel(const float* __restrict__ X,
                                                     const float* __restrict__ q, int64_t n, int p,
                                                     float ng, void* __restrict__ Kout, int64_t ldk) {
  constexpr int TR = 16;
  __shared__ float xs[TR][PMAX];
  __shared__ float qs[TR];
  const int64_t i0 = (int64_t)blockIdx.x * TR;
  const int64_t j = (int64_t)blockIdx.y * 256 + threadIdx.x;
  for (int t = threadIdx.x; t < TR * PMAX; t += 256) {
    const int r = t / PMAX, k = t % PMAX;
    const int64_t i = i0 + r;
    xs[r][k] = (i < n && k < p) ? X[i * p + k] : 0.f;
  }
  if (threadIdx.x < TR) {
    const int64_t i = i0 + threadIdx.x;
    qs[threadIdx.x] = (i < n && !LAP) ? q[i] : 0.f;
  }
  __syncthreads();
  if (j >= ldk) return;
  const bool valid = j < n;
  float xj[PMAX];
#pragma unroll
  for (int k = 0; k < PMAX; ++k) xj[k] = (valid && k < p) ? X[j * p + k] : 0.f;
  const float qj = (valid && !LAP) ? q[j] : 0.f;
  for (int r = 0; r < TR; ++r) {
    const int64_t i = i0 + r;
    if (i >= n) break;
    float val = 0.f;
    if (valid) {
      float d = pair_dist<PMAX, LAP>(xs[r], qs[r], xj, qj);
      if (i == j) d = 0.f;
      val = kexp2(ng * d);
    }
    if (BF16) {
      __builtin_nontemporal_store(f32_to_bf16(val), static_cast<uint16_t*>(Kout) + i * ldk + j);
    } else {
      __builtin_nontemporal_store(val, static_cast<float*>(Kout) + i * ldk + j);
    }
  }
}

template <int PMAX>
static void kbuild_p(const float* X, const float* q, int64_t n, int p, KernelSpec ks, int dtype,
                     void* K, int64_t ldk, hipStream_t st) {
  dim3 grid((unsigned)((n + 15) / 16), (unsigned)((ldk + 255) / 256));
  const float ng = -float(ks.gamma) * kLog2e;
  const bool lap = ks.kind == KQR_LAPLACIAN, bf = dtype == KQR_BF16;
  if (lap && bf) kbuild_kernel<PMAX, true, true><<<grid, 256, 0, st>>>(X, q, n, p, ng, K, ldk);
  else if (lap) kbuild_kernel<PMAX, true, false><<<grid, 256, 0, st>>>(X, q, n, p, ng, K, ldk);
  else if (bf) kbuild_kernel<PMAX, false, true><<<grid, 256, 0, st>>>(X, q, n, p, ng, K, ldk);
  else kbuild_kernel<PMAX, false, false><<<grid, 256, 0, st>>>(X, q, n, p, ng, K, ldk);
  KQR_LAUNCH_CHECK();
}

#define KQR_DISPATCH_P(p, FN, ...)                                   \
  do {                                                               \
    if ((p) <= 8) FN<8>(__VA_ARGS__);                                \
    else if ((p) <= 12) FN<12>(__VA_ARGS__);                         \
    else if ((p) <= 16) FN<16>(__VA_ARGS__);                         \
    else if ((p) <= 20) FN<20>(__VA_ARGS__);                         \
    else if ((p) <= 24) FN<24>(__VA_ARGS__);                         \
    else if ((p) <= 32) FN<32>(__VA_ARGS__);                         \
    else if ((p) <= 48) FN<48>(__VA_ARGS__);                         \
    else if ((p) <= 64) FN<64>(__VA_ARGS__);                         \
    else fail(KQR_EINVAL, "feature dimension p=%d exceeds 64", (p)); \
  } while (0)

void kbuild(const float* X, const float* sqn, int64_t n, int p, KernelSpec ks, int dtype, void* K,
            int64_t ldk, hipStream_t st) {
  if (n <= 0) return;
  if (kbuild_mfma(X, sqn, n, p, ks, dtype, K, ldk, 0, st)) return;  // RBF, p <= 32: Gram on the matrix cores
  KQR_DISPATCH_P(p, kbuild_p, X, sqn, n, p, ks, dtype, K, ldk, st);
}

// ================================================================= materialised K-apply
// One wave streams ROWS whole rows of K with 16-byte non-temporal loads,
// UNROLL chunks per lane per step (ROWS*UNROLL loads in flight per lane); the
// vector chunk it needs is loaded once per step and shared by the ROWS rows.
// Per-lane partial sums are reduced across the wave with shuffles, so every
// output is produced by one wave in a fixed order (deterministic).
//   fast  (EXACT=false): v in FP32, FP32 products summed in FP32 over one step
//                        and then added into FP64 accumulators.
//   exact (EXACT=true) : v in FP64, products and sums in FP64.
// V64 (fast): v comes in FP64 and is rounded to FP32 as it is read, the same
// values as an FP32 copy without the launch and the memory for one.
template <bool BF16>
__device__ __forceinline__ float kelem(const u32x4& w, int e) {
  if (BF16) {
    const uint32_t word = w[e >> 1];
    return (e & 1) ? bf16_hi(word) : bf16_lo(word);
  } else {
    return __uint_as_float(w[e]);
  }
}

// Columns can be split into gridDim.y segments (smaller work items balance the
// tail of the launch); each segment then writes a partial sum per row and
// kapply_seg_reduce adds the segments in order.
template <int ROWS, int UNROLL, bool EXACT, bool BF16, bool V64>
__global__ __launch_bounds__(256) void kapply_rows_kernel(const void* __restrict__ Kp, int64_t ldk,
                                                          int64_t nrows, int64_t ncols,
                                                          const float* __restrict__ v32,
                                                          const double* __restrict__ v64,
                                                          double* __restrict__ u, int64_t ldu,
                                                          int64_t seg_chunks, double* __restrict__ part) {
  constexpr int VEC = BF16 ? 8 : 4;
  constexpr int ESZ = BF16 ? 2 : 4;
  const int lane = threadIdx.x & 63;
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * ROWS;
  if (row0 >= nrows) return;
  const u32x4* rp[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const int64_t rr = (row0 + r < nrows) ? row0 + r : nrows - 1;
    rp[r] = reinterpret_cast<const u32x4*>(static_cast<const char*>(Kp) + rr * ldk * ESZ);
  }
  const int64_t nchunk_all = ncols / VEC;
  const int64_t cbeg = int64_t(blockIdx.y) * seg_chunks;
  const int64_t nchunk = min(nchunk_all, cbeg + seg_chunks);
  const bool last_seg = blockIdx.y == gridDim.y - 1;
  double acc[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) acc[r] = 0.0;

  int64_t c = cbeg + lane;
  for (; c + 64 * (UNROLL - 1) < nchunk; c += 64 * UNROLL) {
    u32x4 kk[ROWS][UNROLL];
#pragma unroll
    for (int s = 0; s < UNROLL; ++s)
#pragma unroll
      for (int r = 0; r < ROWS; ++r) kk[r][s] = __builtin_nontemporal_load(rp[r] + c + 64 * s);
    if (EXACT) {
#pragma unroll
      for (int s = 0; s < UNROLL; ++s) {
        double vv[VEC];
        const double* vp = v64 + (c + 64 * s) * VEC;
#pragma unroll
        for (int e = 0; e < VEC; e += 2) {
          const double2 t = *reinterpret_cast<const double2*>(vp + e);
          vv[e] = t.x;
          vv[e + 1] = t.y;
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[r] = fma(double(kelem<BF16>(kk[r][s], e)), vv[e], acc[r]);
      }
    } else {
      float a32[ROWS];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) a32[r] = 0.f;
#pragma unroll
      for (int s = 0; s < UNROLL; ++s) {
        float vv[VEC];
        if (V64) {
          const double* vp = v64 + (c + 64 * s) * VEC;
#pragma unroll
          for (int e = 0; e < VEC; e += 2) {
            const double2 t = *reinterpret_cast<const double2*>(vp + e);
            vv[e] = float(t.x);
            vv[e + 1] = float(t.y);
          }
        } else {
          const float* vp = v32 + (c + 64 * s) * VEC;
#pragma unroll
          for (int e = 0; e < VEC; e += 4) {
            const float4 t = *reinterpret_cast<const float4*>(vp + e);
            vv[e] = t.x;
            vv[e + 1] = t.y;
            vv[e + 2] = t.z;
            vv[e + 3] = t.w;
          }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
          for (int e = 0; e < VEC; ++e) a32[r] = fmaf(kelem<BF16>(kk[r][s], e), vv[e], a32[r]);
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r) acc[r] += double(a32[r]);
    }
  }
  for (; c < nchunk; c += 64) {
    u32x4 kk[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) kk[r] = __builtin_nontemporal_load(rp[r] + c);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double ve = EXACT ? v64[c * VEC + e] : double(V64 ? float(v64[c * VEC + e]) : v32[c * VEC + e]);
#pragma unroll
      for (int r = 0; r < ROWS; ++r) acc[r] = fma(double(kelem<BF16>(kk[r], e)), ve, acc[r]);
    }
  }
  // trailing columns that do not fill a 16-byte chunk (last segment)
  const int64_t col = nchunk_all * VEC + lane;
  if (last_seg && col < ncols) {
    const double ve = EXACT ? v64[col] : double(V64 ? float(v64[col]) : v32[col]);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const char* base = reinterpret_cast<const char*>(rp[r]);
      const float ke = BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(base)[col])
                            : reinterpret_cast<const float*>(base)[col];
      acc[r] = fma(double(ke), ve, acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < ROWS; ++r) acc[r] = wave_sum_f64(acc[r]);
  if (part) {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (lane == r && row0 + r < nrows) part[int64_t(blockIdx.y) * nrows + row0 + r] = acc[r];
  } else {
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
      if (lane == r && row0 + r < nrows) u[(row0 + r) * ldu] = acc[r];
  }
}

__global__ void kapply_seg_reduce(const double* __restrict__ part, int nseg, int64_t nrows,
                                  double* __restrict__ u, int64_t ldu) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (i >= nrows) return;
  double s = 0.0;
  for (int k = 0; k < nseg; ++k) s += part[int64_t(k) * nrows + i];
  u[i * ldu] = s;
}

// ----------------------------------------------------------------- shapes
namespace {
std::mutex g_shape_mu;
// tuned shapes per [dtype][exact][size bucket]
ApplyShape g_shape[2][2][3];
bool g_shape_set[2][2][3] = {};

int size_bucket(int64_t n) { return n < 8192 ? 0 : (n < 65536 ? 1 : 2); }
}  // namespace

ApplyShape default_apply_shape(int dtype, int exact, int64_t n) {
  std::lock_guard<std::mutex> lk(g_shape_mu);
  const int d = dtype == KQR_BF16, e = exact != 0, b = size_bucket(n);
  if (g_shape_set[d][e][b]) return g_shape[d][e][b];
  ApplyShape s;
  s.unroll = 2;
  s.segs = n >= 16384 ? 4 : 1;  // keeps work items ~n/4 columns long on large matrices
  // Rows per wave (every output's sums are the same for any of them).  Eight
  // read the vector least often but make n / 32 workgroups: CUs idle well below
  // 8192 rows, and from there to about 12,500 a thin second round follows the
  // first.  FP64 products keep two or four rows ahead for longer.  Measured
  // (us; 2 / 4 / 8 rows): FP32 fast n = 2000 5.7 / 6.9 / 10.0, 6000 22 / 25 / 25,
  // 7000 35 / 31 / 32, 8192 49 / 52 / 46, 10,000 58 / 64 / 75, 13,000 106 / 109 / 104;
  // FP32 exact 2000 6.3 / 7.9 / 17.7, 7000 35 / 34 / 57, 13,000 121 / 122 / 139,
  // 16,383 183 / 167 / 181; BF16 fast 2000 4.1 / 5.6 / 8.4, 8192 22 / 31 / 31, 12,000
  // 50 / 46 / 53, 14,000 68 / 67 / 65; BF16 exact 6000 16 / 19 / 18, 7500 28 / 24 / 22,
  // 10,000 52 / 42 / 49, 13,000 95 / 84 / 66.
  const bool thin = n > 8192 && n <= 12500;
  if (n >= 16384) s.rows = 8;
  else if (n <= 6250) s.rows = 2;
  else if (e) s.rows = !d || thin ? 4 : 8;
  else s.rows = thin || (d && n <= 12500) ? 2 : 8;
  return s;
}

void set_apply_shape(int dtype, int exact, int64_t n, ApplyShape s) {
  std::lock_guard<std::mutex> lk(g_shape_mu);
  const int d = dtype == KQR_BF16, e = exact != 0, b = size_bucket(n);
  g_shape[d][e][b] = s;
  g_shape_set[d][e][b] = true;
}

bool apply_shape_supported(const ApplyShape& s) {
  const int key = s.rows * 100 + s.unroll;
  const bool ok = key == 201 || key == 202 || key == 204 || key == 401 || key == 402 || key == 404 ||
                  key == 801 || key == 802 || key == 804;
  return ok && s.segs >= 1 && s.segs <= 64;
}

template <int ROWS, int UNROLL>
static void kapply_rows_launch(const KMat& km, int64_t nrows, int64_t ncols, const float* v32,
                               const double* v64, double* u, int64_t ldu, bool exact, int segs,
                               hipStream_t st, double* scratch, size_t scratch_doubles) {
  const int vec = km.dtype == KQR_BF16 ? 8 : 4;
  const int64_t nchunk = ncols / vec;
  segs = int(std::max<int64_t>(1, std::min<int64_t>(segs, nchunk / 64)));
  int64_t seg_chunks = (nchunk + segs - 1) / segs;
  seg_chunks = (seg_chunks + 63) / 64 * 64;
  if (seg_chunks == 0) seg_chunks = 64;
  segs = int(std::max<int64_t>(1, (nchunk + seg_chunks - 1) / seg_chunks));
  const int64_t waves = (nrows + ROWS - 1) / ROWS;
  const dim3 grid((unsigned)((waves + 3) / 4), (unsigned)segs);
  double* part = nullptr;
  const bool own = segs > 1 && !(scratch && scratch_doubles >= size_t(segs) * size_t(nrows));
  if (segs > 1) part = scratch;
  if (own)
    KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&part), size_t(segs) * nrows * sizeof(double), st));
  const bool bf = km.dtype == KQR_BF16;
#define KQR_ROWS(EX, BF, V)                                                                                       \
  kapply_rows_kernel<ROWS, UNROLL, EX, BF, V><<<grid, 256, 0, st>>>(km.K, km.ld, nrows, ncols, v32, v64, u, ldu, \
                                                                    seg_chunks, part)
  if (exact && bf) KQR_ROWS(true, true, false);
  else if (exact) KQR_ROWS(true, false, false);
  else if (!v32 && bf) KQR_ROWS(false, true, true);
  else if (!v32) KQR_ROWS(false, false, true);
  else if (bf) KQR_ROWS(false, true, false);
  else KQR_ROWS(false, false, false);
#undef KQR_ROWS
  KQR_LAUNCH_CHECK();
  if (part) {
    kapply_seg_reduce<<<dim3((unsigned)((nrows + 255) / 256)), 256, 0, st>>>(part, segs, nrows, u, ldu);
    KQR_LAUNCH_CHECK();
    if (own) KQR_CHECK_HIP(hipFreeAsync(part, st));
  }
}

void kapply_dense(const KMat& km, int64_t nrows, int64_t ncols, const float* v32, const double* v64,
                  double* u, int64_t ldu, bool exact, hipStream_t st, const ApplyShape* shape, double* scratch,
                  size_t scratch_doubles) {
  if (nrows <= 0) return;
  if (km.layout == 1) {  // symmetric upper-triangle tiles (kpacked.hip)
    if (nrows != ncols) fail(KQR_EINVAL, "the packed layout holds square K only");
    const PackedShape ps = default_packed_shape(km.dtype, exact);
    const bool fits = scratch && scratch_doubles >= packed_shape_scratch_doubles(nrows, ps);
    kapply_packed(km, nrows, v32, v64, u, ldu, exact, st, &ps, fits ? scratch : nullptr);
    return;
  }
  const ApplyShape s = shape ? *shape : default_apply_shape(km.dtype, exact, nrows);
  const int key = s.rows * 100 + s.unroll;
  switch (key) {
    case 201: kapply_rows_launch<2, 1>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 202: kapply_rows_launch<2, 2>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 204: kapply_rows_launch<2, 4>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 401: kapply_rows_launch<4, 1>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 402: kapply_rows_launch<4, 2>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 404: kapply_rows_launch<4, 4>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 801: kapply_rows_launch<8, 1>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 802: kapply_rows_launch<8, 2>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    case 804: kapply_rows_launch<8, 4>(km, nrows, ncols, v32, v64, u, ldu, exact, s.segs, st, scratch, scratch_doubles); break;
    default: fail(KQR_EINVAL, "unsupported K-apply shape rows=%d unroll=%d", s.rows, s.unroll);
  }
}

// ================================================================= on-the-fly K-apply
// One thread per output row i keeps x_i (and ||x_i||^2) in registers; the
// block walks a slice of the columns in tiles of 64 staged in LDS (x_j, the
// norms and v_j, read as broadcasts) and forms k(x_i, x_j) in FP32.
//   fast  (EX=false): k * v_j accumulated in FP32 over a tile (v rounded to
//                     FP32), then into an FP64 accumulator;
//   exact (EX=true) : the FP32 entry times the FP64 v_j, FP64 products and
//                     sums (the exact operator of the residuals).
// Columns are split over gridDim.y slices so that small row counts still fill
// the chip; the slices' partial sums are added in a fixed order by a second
// kernel.
constexpr int kOtfTile = 64;

// Column slices of an on-the-fly launch: about 8192 workgroups in all (many
// rounds of the blocks the chip holds at once, so the last round is a small
// tail) unless a target is set, each slice at least 1024 columns.  Every slice
// writes one partial per row, added in a fixed order by otf_reduce_kernel.
std::atomic<int64_t> g_otf_wgs{0};  // target workgroups of a sliced launch (kqr_set_otf_shape); 0: by size

static int64_t otf_slices(int64_t rblk, int64_t nc) {
  const int64_t set = g_otf_wgs.load(), wgs = set > 0 ? set : 8192;
  const int64_t want = (wgs + std::max<int64_t>(rblk, 1) - 1) / std::max<int64_t>(rblk, 1);
  return std::max<int64_t>(1, std::min<int64_t>(want, (nc + 1023) / 1024));
}

template <int PMAX, bool LAP, bool EX>
__global__ __launch_bounds__(256) void kapply_otf_kernel(
    const float* __restrict__ Xr, const float* __restrict__ qr, int64_t nr,
    const float* __restrict__ Xc, const float* __restrict__ qc, int64_t nc, int p, float ng,
    const double* __restrict__ v, int64_t cols_per_slice, double* __restrict__ part) {
  __shared__ float xs[kOtfTile][PMAX];
  __shared__ float qs[kOtfTile];
  __shared__ float vs[kOtfTile];
  __shared__ double vd[kOtfTile];
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const bool row_ok = i < nr;
  float xi[PMAX];
#pragma unroll
  for (int k = 0; k < PMAX; ++k) xi[k] = (row_ok && k < p) ? Xr[i * p + k] : 0.f;
  const float qi = (row_ok && !LAP) ? qr[i] : 0.f;
  const int64_t c0 = int64_t(blockIdx.y) * cols_per_slice;
  const int64_t c1 = min(nc, c0 + cols_per_slice);
  double acc = 0.0;
  for (int64_t jb = c0; jb < c1; jb += kOtfTile) {
    const int cnt = int(min<int64_t>(kOtfTile, c1 - jb));
    __syncthreads();
    for (int t = threadIdx.x; t < kOtfTile * PMAX; t += 256) {
      const int jj = t / PMAX, k = t % PMAX;
      xs[jj][k] = (jj < cnt && k < p) ? Xc[(jb + jj) * p + k] : 0.f;
    }
    if (threadIdx.x < kOtfTile) {
      const int jj = threadIdx.x;
      qs[jj] = (jj < cnt && !LAP) ? qc[jb + jj] : 0.f;
      const double vj = jj < cnt ? v[jb + jj] : 0.0;
      if (EX) vd[jj] = vj;
      else vs[jj] = float(vj);
    }
    __syncthreads();
    if (EX) {
      for (int jj = 0; jj < cnt; ++jj) {
        const float d = pair_dist<PMAX, LAP>(xs[jj], qs[jj], xi, qi);
        acc = fma(double(kexp2(ng * d)), vd[jj], acc);
      }
    } else {
      float a32 = 0.f;
      for (int jj = 0; jj < cnt; ++jj) {
        const float d = pair_dist<PMAX, LAP>(xs[jj], qs[jj], xi, qi);
        a32 = fmaf(kexp2(ng * d), vs[jj], a32);
      }
      acc += double(a32);
    }
  }
  if (row_ok) part[int64_t(blockIdx.y) * nr + i] = acc;
}

// The slices' partial sums of a row: eight threads per row, each taking every
// eighth slice in order.
constexpr int kOtfRed = 8;
__global__ __launch_bounds__(256) void otf_reduce_kernel(const double* __restrict__ part, int nslice, int64_t nr,
                                                         double* __restrict__ u, int64_t ldu, double out_scale,
                                                         double out_shift) {
  __shared__ double sh[kOtfRed][32];
  const int r = threadIdx.x & 31, h = threadIdx.x >> 5;
  const int64_t i = blockIdx.x * int64_t(32) + r;
  const int64_t ic = min(i, nr - 1);
  double s = 0.0;
  for (int k = h; k < nslice; k += kOtfRed) s += part[int64_t(k) * nr + ic];
  sh[h][r] = s;
  __syncthreads();
  if (h == 0 && i < nr) {
#pragma unroll
    for (int k = 1; k < kOtfRed; ++k) s += sh[k][r];
    u[i * ldu] = out_shift + out_scale * s;
  }
}

static void otf_reduce(const double* part, int64_t nslice, int64_t nr, double* u, int64_t ldu, double scale,
                       double shift, hipStream_t st) {
  otf_reduce_kernel<<<dim3((unsigned)((nr + 31) / 32)), 256, 0, st>>>(part, int(nslice), nr, u, ldu, scale, shift);
  KQR_LAUNCH_CHECK();
}

// columns per slice of a launch on the vector unit
static int64_t otf_per(int64_t rblk, int64_t nc) {
  const int64_t nslice = std::min<int64_t>(otf_slices(rblk, nc), 65535);
  const int64_t per = (nc + nslice - 1) / nslice;
  return (per + kOtfTile - 1) / kOtfTile * kOtfTile;
}

template <int PMAX>
static void kapply_otf_p(const float* Xr, const float* qr, int64_t nr, const float* Xc,
                         const float* qc, int64_t nc, int p, KernelSpec ks, const double* v, double* u,
                         int64_t ldu, double scale, double shift, bool exact, hipStream_t st, double* scratch,
                         size_t scratch_doubles) {
  const int64_t rblk = (nr + 255) / 256;
  const int64_t per = otf_per(rblk, nc), nslice = (nc + per - 1) / per;
  const size_t need = size_t(nslice) * size_t(nr);
  const bool own = !scratch || scratch_doubles < need;
  double* part = scratch;
  if (own) KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&part), need * sizeof(double), st));
  const dim3 grid((unsigned)rblk, (unsigned)nslice);
  const float ng = -float(ks.gamma) * kLog2e;
  const bool lap = ks.kind == KQR_LAPLACIAN;
  if (lap && exact) kapply_otf_kernel<PMAX, true, true><<<grid, 256, 0, st>>>(Xr, qr, nr, Xc, qc, nc, p, ng, v, per, part);
  else if (lap) kapply_otf_kernel<PMAX, true, false><<<grid, 256, 0, st>>>(Xr, qr, nr, Xc, qc, nc, p, ng, v, per, part);
  else if (exact) kapply_otf_kernel<PMAX, false, true><<<grid, 256, 0, st>>>(Xr, qr, nr, Xc, qc, nc, p, ng, v, per, part);
  else kapply_otf_kernel<PMAX, false, false><<<grid, 256, 0, st>>>(Xr, qr, nr, Xc, qc, nc, p, ng, v, per, part);
  KQR_LAUNCH_CHECK();
  otf_reduce(part, nslice, nr, u, ldu, scale, shift, st);
  if (own) KQR_CHECK_HIP(hipFreeAsync(part, st));
}

// Laplacian on the fly from fixed-point coordinates.  Column k of X is
// stored as q_ik = round((x_ik - min_k) 2^s) in 32 bits (computed in FP64, so
// the only error is that rounding, at most 2^-(s+1) per coordinate), and the
// L1 distance sum_k |q_ik - q_jk| is an exact integer formed by one
// v_sad_u32 (|a - b| + c) per coordinate, against two FP32 operations per
// coordinate in the float form; s is chosen so that the sum cannot exceed
// 2^32 - 1.  The entry is exp2(-gamma log2(e) 2^-s float(d)), the rest as in
// kapply_otf_kernel.
__device__ __forceinline__ uint32_t sad_u32(uint32_t a, uint32_t b, uint32_t c) {
  return (max(a, b) - min(a, b)) + c;  // one v_sad_u32 (an asm statement here brought an s_nop per four)
}
// a zero the compiler does not know: a sum that starts from a known one costs
// three instructions for its first coordinate
__device__ __forceinline__ uint32_t opaque_zero() {
  uint32_t z = 0;
  asm("" : "+v"(z));
  return z;
}

// Row-streamed form over all n^2 pairs (used when the symmetric form's
// partial sums would exceed the budget below): a workgroup owns 256 R rows and a
// slice of the columns; one partial per slice and row, added by
// otf_reduce_kernel.
template <int PMAX, int R, bool EX>
__global__ __launch_bounds__(256) void kapply_otf_l1q_kernel(const uint32_t* __restrict__ Xq, int64_t n, int p,
                                                             float ngs, const double* __restrict__ v,
                                                             int64_t cols_per_slice, double* __restrict__ part) {
  // a thread owns R rows (256 R per block), so each LDS read of x_j serves R pairs
  static_assert(PMAX % 4 == 0, "coordinates are read from LDS four at a time");
  __shared__ __align__(16) uint32_t xs[kOtfTile][PMAX];
  __shared__ float vs[kOtfTile];
  __shared__ double vd[kOtfTile];
  const int64_t i0 = int64_t(blockIdx.x) * 256 * R + threadIdx.x;
  uint32_t xi[R][PMAX];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + 256 * r;
#pragma unroll
    for (int k = 0; k < PMAX; ++k) xi[r][k] = (i < n && k < p) ? Xq[i * p + k] : 0u;
  }
  const int64_t c0 = int64_t(blockIdx.y) * cols_per_slice;
  const int64_t c1 = min(n, c0 + cols_per_slice);
  const uint32_t zero = opaque_zero();
  double acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0;
  for (int64_t jb = c0; jb < c1; jb += kOtfTile) {
    const int cnt = int(min<int64_t>(kOtfTile, c1 - jb));
    __syncthreads();
    for (int t = threadIdx.x; t < kOtfTile * PMAX; t += 256) {
      const int jj = t / PMAX, k = t % PMAX;
      xs[jj][k] = (jj < cnt && k < p) ? Xq[(jb + jj) * p + k] : 0u;
    }
    if (threadIdx.x < kOtfTile) {
      const int jj = threadIdx.x;
      const double vj = jj < cnt ? v[jb + jj] : 0.0;
      if (EX) vd[jj] = vj;
      else vs[jj] = float(vj);
    }
    __syncthreads();
    float a32[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a32[r] = 0.f;
    for (int jj = 0; jj < cnt; ++jj) {
      uint32_t d[R];
#pragma unroll
      for (int r = 0; r < R; ++r) d[r] = zero;
      const uint4* xr = reinterpret_cast<const uint4*>(xs[jj]);  // broadcast 16-byte LDS reads
#pragma unroll
      for (int k4 = 0; k4 < PMAX / 4; ++k4) {
        const uint4 c = xr[k4];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          d[r] = sad_u32(xi[r][4 * k4], c.x, d[r]);
          d[r] = sad_u32(xi[r][4 * k4 + 1], c.y, d[r]);
          d[r] = sad_u32(xi[r][4 * k4 + 2], c.z, d[r]);
          d[r] = sad_u32(xi[r][4 * k4 + 3], c.w, d[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const float e = kexp2(ngs * float(d[r]));
        if (EX) acc[r] = fma(double(e), vd[jj], acc[r]);
        else a32[r] = fmaf(e, vs[jj], a32[r]);
      }
    }
    if (!EX) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += double(a32[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + 256 * r;
    if (i < n) part[int64_t(blockIdx.y) * n + i] = acc[r];
  }
}

template <int PMAX>
static void kapply_otf_l1q_rows_p(const uint32_t* Xq, int64_t n, int p, float ngs, const double* v, double* u,
                                  int64_t ldu, bool exact, hipStream_t st) {
  // rows per thread: 4 up to 32 coordinates, 2 beyond (registers)
  constexpr int R = PMAX <= 32 ? 4 : 2;
  const int64_t rblk = (n + 256 * R - 1) / (256 * R);
  int64_t nslice = otf_slices(rblk, n);
  nslice = std::min<int64_t>(nslice, 65535);
  int64_t per = (n + nslice - 1) / nslice;
  per = (per + kOtfTile - 1) / kOtfTile * kOtfTile;
  nslice = (n + per - 1) / per;
  double* part = nullptr;
  KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&part), size_t(nslice) * size_t(n) * sizeof(double), st));
  const dim3 grid((unsigned)rblk, (unsigned)nslice);
  if (exact) kapply_otf_l1q_kernel<PMAX, R, true><<<grid, 256, 0, st>>>(Xq, n, p, ngs, v, per, part);
  else kapply_otf_l1q_kernel<PMAX, R, false><<<grid, 256, 0, st>>>(Xq, n, p, ngs, v, per, part);
  KQR_LAUNCH_CHECK();
  otf_reduce(part, nslice, n, u, ldu, 1.0, 0.0, st);
  KQR_CHECK_HIP(hipFreeAsync(part, st));
}


// K is symmetric (Section 1), so each pair is evaluated once: over the
// upper-triangle tiles of kPkT x kPkT entries of the packed geometry.
// Workgroup b takes strip k of tile-row I (pk_strip_coords), the tiles
// J = I + k strip, ... of that row.  Thread t owns the four rows
// I kPkT + t % 32 + 32 r (fixed-point coordinates in registers, v_i) and in
// every tile the sixteen columns t / 32 + 8 c, so the two column groups of a
// wave read adjacent LDS rows (distinct banks) and every 16-byte read of
// x_j serves four pairs.  Per pair: the distance (one v_sad_u32 per
// coordinate), the entry, its product with v_j into the row sum and, off
// the diagonal tile, with v_i into the column sum.  Row sums stay in
// registers over the strip and are added over the eight column groups at its
// end (one partial per strip and row); the column sums of a tile are added
// over the 32 row groups in LDS (one partial per tile and column); a
// diagonal tile feeds its rows only.  packed_reduce adds the partials in a
// fixed order.  Fast: FP32 products and sums within a tile, FP64 beyond;
// exact: FP64 products and sums.  Bound by the vector unit: NC + 10
// instructions per 64 pairs, two waves per SIMD (the rows' coordinates fill
// the registers), so what the lanes do besides counts: NC is p rounded up to
// 2, not the padded PMAX; v is kept in the type it is used in; and the next
// column's first half is read ahead.  30,011 x 30 fast: 700 us with all three
// left out, 605 with them.
template <int PMAX, int NC, bool EX>
__global__ __launch_bounds__(256) void kapply_otf_l1q_sym_kernel(const uint32_t* __restrict__ Xq, int64_t n, int p,
                                                                 float ngs, const double* __restrict__ v, int64_t nt,
                                                                 int strip, int64_t nsx, double* __restrict__ rowpart,
                                                                 double* __restrict__ colpart) {
  static_assert(PMAX % 4 == 0 && NC <= PMAX && NC % 2 == 0, "coordinates are read from LDS four at a time");
  typedef std::conditional_t<EX, double, float> acc_t;
  constexpr int T = kPkT;
  constexpr int R = 4;     // rows per thread
  constexpr int RG = 32;   // row groups: T / R
  constexpr int CPT = 16;  // columns per thread and tile: T / (256 / RG)
  __shared__ __align__(16) uint32_t xs[T][PMAX];
  __shared__ acc_t vs[T];
  __shared__ double red[RG][T + 1];
  const int t = threadIdx.x;
  const int rg = t & (RG - 1), cg = t >> 5;
  int64_t I, k;
  pk_strip_coords(blockIdx.x, nt, strip, I, k);
  const int64_t J0 = I + k * strip, J1 = min(nt, J0 + strip);
  // Rows past n keep the coordinates of row n - 1 and v_i = 0: their row sums
  // are never read and their column contributions vanish.  Every load is
  // issued before any is used (a load whose use is conditional per lane would
  // be moved under the condition and waited for one at a time).
  uint32_t xi[R][NC];
  acc_t vi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t ic = min(I * T + rg + RG * r, n - 1);
#pragma unroll
    for (int kk = 0; kk < NC; ++kk) xi[r][kk] = Xq[ic * p + min(kk, p - 1)];
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = I * T + rg + RG * r;
    const double vv = v[min(i, n - 1)];
    vi[r] = i < n ? acc_t(vv) : acc_t(0);
#pragma unroll
    for (int kk = 0; kk < NC; ++kk) xi[r][kk] = kk < p ? xi[r][kk] : 0u;  // padded coordinates: 0 on both sides
  }
  const uint32_t zero = opaque_zero();
  double acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0;
  // The next tile's columns (coordinates of column n - 1 past n, v_j = 0
  // there) are loaded into registers while the current tile is evaluated.
  uint32_t xc[T * PMAX / 256];
  double vc = 0.0;
  auto load_cols = [&](int64_t J) {
#pragma unroll
    for (int q = 0; q < T * PMAX / 256; ++q) {
      const int e = t + 256 * q;
      const int jj = e / PMAX, kk = e % PMAX;
      xc[q] = Xq[min(J * T + jj, n - 1) * p + min(kk, p - 1)];
    }
    if (t < T) vc = v[min(J * T + t, n - 1)];
  };
  load_cols(J0);
  for (int64_t J = J0; J < J1; ++J) {
    const bool diag = J == I;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < T * PMAX / 256; ++q) {
      const int e = t + 256 * q;
      const int jj = e / PMAX, kk = e % PMAX;
      xs[jj][kk] = kk < p ? xc[q] : 0u;
    }
    if (t < T) vs[t] = J * T + t < n ? acc_t(vc) : acc_t(0);
    __syncthreads();
    if (J + 1 < J1) load_cols(J + 1);
    float a32[R];
#pragma unroll
    for (int r = 0; r < R; ++r) a32[r] = 0.f;
    // the first half of a column's coordinates is requested before the entries
    // of the column before it: with two waves per SIMD nothing else covers it
    // (above 32 coordinates the registers are full)
    constexpr int Q = (NC + 3) / 4, H = PMAX <= 32 ? (Q + 1) / 2 : 0;
    const uint4* xr = reinterpret_cast<const uint4*>(xs[cg]);  // 16-byte LDS reads, two rows per wave
    uint4 head[H > 0 ? H : 1];
#pragma unroll
    for (int q = 0; q < H; ++q) head[q] = xr[q];
#pragma unroll 2
    for (int c = 0; c < CPT; ++c) {
      const int jj = cg + 8 * c;
      uint32_t d[R];
#pragma unroll
      for (int r = 0; r < R; ++r) d[r] = zero;
      auto quad = [&](uint4 x, int k4) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          d[r] = sad_u32(xi[r][4 * k4], x.x, d[r]);
          d[r] = sad_u32(xi[r][4 * k4 + 1], x.y, d[r]);
          if (4 * k4 + 2 < NC) {
            d[r] = sad_u32(xi[r][4 * k4 + 2], x.z, d[r]);
            d[r] = sad_u32(xi[r][4 * k4 + 3], x.w, d[r]);
          }
        }
      };
      if constexpr (H > 0) {
        uint4 tail[Q - H > 0 ? Q - H : 1];
#pragma unroll
        for (int q = H; q < Q; ++q) tail[q - H] = xr[q];
#pragma unroll
        for (int q = 0; q < H; ++q) quad(head[q], q);
        xr = reinterpret_cast<const uint4*>(xs[min(jj + 8, T - 1)]);
#pragma unroll
        for (int q = H; q < Q; ++q) quad(tail[q - H], q);
#pragma unroll
        for (int q = 0; q < H; ++q) head[q] = xr[q];
      } else {
        xr = reinterpret_cast<const uint4*>(xs[jj]);
#pragma unroll
        for (int q = 0; q < Q; ++q) quad(xr[q], q);
      }
      float e[R];
#pragma unroll
      for (int r = 0; r < R; ++r) e[r] = kexp2(ngs * float(d[r]));
      const acc_t vj = vs[jj];
      acc_t cs = acc_t(0);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (EX) {
          acc[r] = fma(double(e[r]), double(vj), acc[r]);
          cs = fma(double(e[r]), double(vi[r]), double(cs));
        } else {
          a32[r] = fmaf(e[r], float(vj), a32[r]);
          cs = fmaf(e[r], float(vi[r]), float(cs));
        }
      }
      // (above 32 coordinates the branch also keeps two columns' registers apart)
      if (PMAX <= 32 || !diag) red[rg][jj] = double(cs);
    }
    if (!EX) {
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += double(a32[r]);
    }
    if (!diag) {  // the same in every thread of the block
      __syncthreads();
      if (t < T) {
        double cs = 0.0;
#pragma unroll 8
        for (int g = 0; g < RG; ++g) cs += red[g][t];
        colpart[size_t(pk_tile_index(I, J, nt)) * T + t] = cs;
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < R; ++r) red[cg][rg + RG * r] = acc[r];
  __syncthreads();
  if (t < T) {
    double rs = 0.0;
#pragma unroll
    for (int g = 0; g < 256 / RG; ++g) rs += red[g][t];
    rowpart[(size_t(I) * nsx + k) * T + t] = rs;
  }
}

// Tiles per workgroup of the symmetric applies, per size class of n (tile
// rows below 64, 256, 1024, and from 1024): installed by kqr_set_otf_shape
// or the on-the-fly autotuner (1..kPkMaxStrip), else by size.
std::atomic<int> g_otf_strip[4] = {{0}, {0}, {0}, {0}};

static int otf_class(int64_t n) {
  const int64_t nt = (n + kPkT - 1) / kPkT;
  return nt >= 1024 ? 3 : (nt >= 256 ? 2 : (nt >= 64 ? 1 : 0));
}

static int otf_sym_strip(int64_t n) {
  const int c = otf_class(n);
  const int s = g_otf_strip[c].load();
  if (s > 0) return s;
  static const int rule[4] = {2, 8, 16, 32};
  return rule[c];
}

void set_otf_shape(int strip, int64_t wgs) {
  for (auto& a : g_otf_strip) a.store(strip);
  g_otf_wgs.store(wgs);
}

void set_otf_strip_for(int64_t n, int strip) { g_otf_strip[otf_class(n)].store(strip); }

int64_t otf_wgs() { return g_otf_wgs.load(); }

void set_otf_wgs(int64_t wgs) { g_otf_wgs.store(wgs); }

int otf_strip_for(int64_t n) { return otf_sym_strip(n); }

// The symmetric applies keep one FP64 partial per tile and column, about
// n^2 / 32 bytes (3 GB at n = 300,000, 31 GB at n = 10^6).  Beyond a
// budget (32 GiB unless set) the row-streamed forms run instead (all n^2
// pairs, O(n) partials).
std::atomic<int64_t> g_otf_sym_budget{int64_t(32) << 30};

void set_otf_sym_budget(int64_t bytes) { g_otf_sym_budget.store(bytes); }

static bool otf_sym_fits(int64_t n) {
  return int64_t(packed_scratch_doubles(n, otf_sym_strip(n)) * sizeof(double)) <= g_otf_sym_budget.load();
}

size_t otf_sym_scratch_doubles(int64_t n) {
  return otf_sym_fits(n) ? packed_scratch_doubles(n, otf_sym_strip(n)) : 0;
}

template <int PMAX>
static void kapply_otf_l1q_p(const uint32_t* Xq, int64_t n, int p, float ngs, const double* v, double* u, int64_t ldu,
                             bool exact, hipStream_t st, double* scratch, size_t scratch_doubles) {
  if (!otf_sym_fits(n)) {
    kapply_otf_l1q_rows_p<PMAX>(Xq, n, p, ngs, v, u, ldu, exact, st);
    return;
  }
  const int64_t nt = (n + kPkT - 1) / kPkT;
  const int strip = otf_sym_strip(n);
  const int64_t nsx = (nt + strip - 1) / strip;
  const size_t need = packed_scratch_doubles(n, strip);
  double* buf = scratch && scratch_doubles >= need ? scratch : nullptr;
  const bool own = buf == nullptr;
  if (own) KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&buf), need * sizeof(double), st));
  double* rowpart = buf;
  double* colpart = buf + size_t(nt) * nsx * kPkT;
  const dim3 grid((unsigned)pk_strips_tail(nt, strip));
  // the coordinates a pair takes: p rounded up to 2 (a padded coordinate adds
  // nothing but costs one operation per pair)
  auto launch = [&](auto nc) {
    constexpr int NC = decltype(nc)::value;
    if (exact)
      kapply_otf_l1q_sym_kernel<PMAX, NC, true><<<grid, 256, 0, st>>>(Xq, n, p, ngs, v, nt, strip, nsx, rowpart, colpart);
    else
      kapply_otf_l1q_sym_kernel<PMAX, NC, false><<<grid, 256, 0, st>>>(Xq, n, p, ngs, v, nt, strip, nsx, rowpart, colpart);
  };
  if constexpr (PMAX == 8 || PMAX == 32) {  // steps of eight
    if (p <= PMAX - 6) launch(std::integral_constant<int, PMAX - 6>{});
    else if (p <= PMAX - 4) launch(std::integral_constant<int, PMAX - 4>{});
    else if (p <= PMAX - 2) launch(std::integral_constant<int, PMAX - 2>{});
    else launch(std::integral_constant<int, PMAX>{});
  } else if constexpr (PMAX < 32) {  // steps of four
    if (p <= PMAX - 2) launch(std::integral_constant<int, PMAX - 2>{});
    else launch(std::integral_constant<int, PMAX>{});
  } else {
    launch(std::integral_constant<int, PMAX>{});
  }
  KQR_LAUNCH_CHECK();
  packed_reduce(rowpart, colpart, n, strip, u, ldu, st);
  if (own) KQR_CHECK_HIP(hipFreeAsync(buf, st));
}

void kapply_otf_l1q(const uint32_t* Xq, int64_t n, int p, double gamma, int shift, const double* v, double* u,
                    int64_t ldu, bool exact, hipStream_t st, double* scratch, size_t scratch_doubles) {
  if (n <= 0) return;
  const float ngs = float(-gamma * double(kLog2e) * std::ldexp(1.0, -shift));
  KQR_DISPATCH_P(p, kapply_otf_l1q_p, Xq, n, p, ngs, v, u, ldu, exact, st, scratch, scratch_doubles);
}

// Per-column minima and maxima of X (FP32 values, exact) over each
// workgroup's rows: part[2 p b + k] and part[2 p b + p + k].  Whole rows are
// read in memory order, 256 / p of them at a time (p <= 64).  30,011 x 30: one
// workgroup per column, every row's line read p times, took 39 us; this 5.
__global__ __launch_bounds__(256) void col_minmax_kernel(const float* __restrict__ X, int64_t n, int p,
                                                         int64_t rows, float* __restrict__ part) {
  __shared__ float sl[256], sh[256];
  const int t = threadIdx.x, step = 256 / p, k = t % p;
  const int64_t r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
  float lo = INFINITY, hi = -INFINITY;
  if (t < step * p) {
#pragma unroll 4
    for (int64_t i = r0 + t / p; i < r1; i += step) {
      const float x = X[i * p + k];
      lo = fminf(lo, x);
      hi = fmaxf(hi, x);
    }
  }
  sl[t] = lo;
  sh[t] = hi;
  __syncthreads();
  if (t < p) {
    for (int e = 1; e < step; ++e) {
      lo = fminf(lo, sl[t + e * p]);
      hi = fmaxf(hi, sh[t + e * p]);
    }
    part[size_t(blockIdx.x) * 2 * p + t] = lo;
    part[size_t(blockIdx.x) * 2 * p + p + t] = hi;
  }
}

struct ColumnMin {
  float v[64];
};

__global__ void quantize_kernel(const float* __restrict__ X, int64_t n, int p, ColumnMin lo, double scale,
                                uint32_t* __restrict__ Xq) {
  const int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (t >= n * p) return;
  Xq[t] = uint32_t(llrint((double(X[t]) - double(lo.v[t % p])) * scale));
}

size_t quantized_words(int64_t n, int p) { return size_t(std::max<int64_t>(n, 2)) * size_t(p); }

int quantize_columns(const float* X, int64_t n, int p, uint32_t* Xq, hipStream_t st) {
  if (n <= 0 || p <= 0) return -1;
  // the partial minima and maxima are kept in Xq (2 p words per workgroup) until the host has them
  const int64_t want = std::min<int64_t>(128, std::max<int64_t>(1, n / 32));
  const int64_t rows = (n + want - 1) / want, blocks = (n + rows - 1) / rows;
  float* part = reinterpret_cast<float*>(Xq);
  col_minmax_kernel<<<dim3((unsigned)blocks), 256, 0, st>>>(X, n, p, rows, part);
  KQR_LAUNCH_CHECK();
  std::vector<float> h(size_t(blocks) * size_t(2 * p));
  KQR_CHECK_HIP(hipMemcpyAsync(h.data(), part, h.size() * sizeof(float), hipMemcpyDeviceToHost, st));
  KQR_CHECK_HIP(hipStreamSynchronize(st));
  double range = 0.0;
  ColumnMin mins = {};
  for (int k = 0; k < p; ++k) {
    float lo = INFINITY, hi = -INFINITY;
    for (int64_t b = 0; b < blocks; ++b) {
      lo = std::fmin(lo, h[size_t(b) * 2 * p + k]);
      hi = std::fmax(hi, h[size_t(b) * 2 * p + p + k]);
    }
    const double r = double(hi) - double(lo);
    if (!std::isfinite(r)) return -1;
    range = std::max(range, r);
    mins.v[k] = lo;
  }
  // largest s <= 23 with p * range * 2^s + p <= 2^32 - 1 (sum of rounded coordinates)
  int s = 23;
  while (s >= 0 && double(p) * (range * std::ldexp(1.0, s) + 1.0) > 4294967295.0) --s;
  if (s >= 0) {
    const int64_t tot = n * p;
    quantize_kernel<<<dim3((unsigned)((tot + 255) / 256)), 256, 0, st>>>(X, n, p, mins, std::ldexp(1.0, s), Xq);
    KQR_LAUNCH_CHECK();
  }
  return s;
}

// RBF on the fly (p <= 32) with the Gram term on the matrix cores.  A
// workgroup is four waves of 32 rows each (two 16-row strips, held as MFMA A
// operands for the whole launch) and walks its columns in stages of 64: four
// 16-column tiles in the operand order of the MFMA, so that a tile's parts
// are read from LDS as consecutive 16-byte (or 4-byte) words of the lanes.
// The lane that holds G[4 g + r][c] forms the entry and accumulates its
// product with v_j (fast: FP32 within a stage or two, then FP64; exact: FP64
// products and sums); the 16 lanes of a row group are reduced at the end.
//
// What bounds it is the vector unit and the matrix cores side by side: per
// 64 pairs an exponential (about 10 cycles of a SIMD), the conversion to FP64
// (5) and the products with v (5 each), against 24 cycles of MFMAs (p > 16),
// which run under other waves' vector work; the clock falls to about 1.8 GHz
// under this load, and a loop of nothing but these instructions on random
// operands takes 85 % of the kernel's time.  So nothing else may take issue
// slots or leave the SIMD waiting: a stage is requested into registers one
// stage ahead and goes to the other LDS buffer after the current one is used
// (one barrier per stage, no wait for memory before it), the next tile's
// MFMAs are issued ahead of this tile's entries, and the MFMA results stay in
// ordinary registers (the second launch bound; without it each is copied from
// the accumulation registers first).  Loading each stage where it was needed,
// a load at a time, against this form, whole calls timed in turn: 100,000 x
// 20,011 at p = 30 exact 755 and 628 us; the square form at 40,000 x 30 exact
// 430 and 346; 20,000 x 5,000 at p = 10 77 and 56.  (The same kernel moves by
// 8 % from run to run with the clock.)
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8_t __attribute__((ext_vector_type(8)));

constexpr int kOtfStage = 64;  // columns per LDS stage

// Gram terms for p <= 16: v_mfma_f32_16x16x4f32 (KP/4 per 16 x 16 block, KP =
// p rounded up to 4; FP32 products and sums), the entry's argument
// -gamma log2(e) (q_i + q_j - 2 G).
template <int KP>
struct GramF32 {
  typedef float col_t;  // the columns: X itself
  static constexpr int kParts = KP / 4;
  static constexpr int kMfmas = 2 * kParts;  // per tile of a wave
  static constexpr int kStageBytes = kOtfStage * KP * 4;
  static constexpr bool kNorms = true;  // the lanes add the squared norms
  static constexpr int kFlush = 1;      // stages per FP32 partial sum (fast mode)
  float a[2][kParts];
  float nx[kParts];

  __device__ __forceinline__ void rows(const float* __restrict__ X, const float* __restrict__, int64_t n, int p,
                                       int64_t r, int s, int lg) {
    const float* x = X + min(r, n - 1) * p;
#pragma unroll
    for (int kb = 0; kb < kParts; ++kb) a[s][kb] = x[min(4 * kb + lg, p - 1)];
#pragma unroll
    for (int kb = 0; kb < kParts; ++kb) a[s][kb] = (r < n && 4 * kb + lg < p) ? a[s][kb] : 0.f;
  }
  // thread t requests coordinate 4 kb + (t / 16) % 4 of column j0 + 16 (t / 64) + t % 16
  __device__ __forceinline__ void fetch(const float* __restrict__ Xc, int64_t nc, int p, int64_t j0, int t) {
    const float* x = Xc + min(j0 + ((t >> 6) << 4) + (t & 15), nc - 1) * p;
#pragma unroll
    for (int kb = 0; kb < kParts; ++kb) nx[kb] = x[min(4 * kb + ((t >> 4) & 3), p - 1)];
  }
  __device__ __forceinline__ void put(char* lds, int p, int t) {
    float* o = reinterpret_cast<float*>(lds) + (t >> 6) * (kParts * 64) + (t & 63);
#pragma unroll
    for (int kb = 0; kb < kParts; ++kb) o[64 * kb] = 4 * kb + ((t >> 4) & 3) < p ? nx[kb] : 0.f;
  }
  __device__ __forceinline__ void gram(const char* lds, int tile, int lane, f32x4_t (&g)[2]) const {
    const float* x = reinterpret_cast<const float*>(lds) + tile * (kParts * 64) + lane;
    g[0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    g[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < kParts; ++kb) {
      const float b = x[64 * kb];
      g[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0][kb], b, g[0], 0, 0, 0);
      g[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1][kb], b, g[1], 0, 0, 0);
    }
  }
  static __device__ __forceinline__ float arg(float g, float qi, float qj, float ng) {
    return ng * (qi + qj - 2.f * g);
  }
};

// Gram terms for 16 < p <= 32 in BF16 on the matrix cores: every FP32
// coordinate is split exactly into three BF16 parts x = h + m + l (round to
// nearest even at each step; 3 x 8 significand bits hold FP32's 24), and
// G = hh + hm + mh + hl + lh + mm (the dropped ml, lm, ll are below 2^-24 of
// |x_i| |x_j| per coordinate) is formed by six v_mfma_f32_16x16x32_bf16 per
// 16 x 16 block (p <= 32, padded to 32), against eight 16x16x4 FP32 MFMAs
// that take 5x the matrix-core time at p = 32.  FP32 sums inside the MFMA.
//
// The column side is split once per launch (kotf_split_cols_kernel) into
// blocks of 16 points, each the h, m and l planes of 32 coordinates in
// operand order, zero filled to a multiple of kB3Pad points.  With p <= 30
// (AUG) the two spare coordinates carry the squared norms and the column side
// the exponent's scale c = -gamma log2(e): row [x_i, 1, q_i] against column
// [-2 c x_j, c q_j, c] (each product rounded once in FP32 before the split),
// so the matrix cores return c d_ij = c (q_i + q_j - 2 x_i . x_j) itself and
// a pair costs the lanes only the clamp at 0, the exponential and the
// product with v_j.  Without AUG the column holds -2 x_j (exact) and the
// lanes add q_i + q_j and scale.
__device__ __forceinline__ void split3_bf16(float x, uint16_t& h, uint16_t& m, uint16_t& l) {
  h = f32_to_bf16(x);
  const float r1 = x - bf16_to_f32(h);  // exact
  m = f32_to_bf16(r1);
  const float r2 = r1 - bf16_to_f32(m);  // exact, at most 8 significant bits
  l = f32_to_bf16(r2);
}

constexpr int kB3Plane = 512;            // halves of a plane of 16 points: 64 lanes x 8
constexpr int kB3Block = 3 * kB3Plane;   // halves per 16 points
constexpr int kB3Pad = 128;

static inline int64_t b3_points(int64_t n) { return (n + kB3Pad - 1) / kB3Pad * kB3Pad; }
static inline size_t b3_bytes(int64_t n) { return size_t(b3_points(n) / 16) * kB3Block * sizeof(uint16_t); }

// halves from the buffer's start to point j's coordinates 8 g .. 8 g + 7 in the h plane
__device__ __forceinline__ int64_t b3_offset(int64_t j, int g) {
  return (j >> 4) * kB3Block + (g * 16 + int(j & 15)) * 8;
}

// Coordinate k of the padded 32-vector of a row (A) or column (B) side, from
// the point's own coordinate x (any value for k >= p) and squared norm q;
// c: the column side's scale (AUG), else 1.
template <bool AUG, bool COL>
__device__ __forceinline__ float b3_coord(float x, float q, int k, int p, float c) {
  if (k < p) return COL ? (-2.f * c) * x : x;
  if (AUG && k == 30) return COL ? c * q : 1.f;
  if (AUG && k == 31) return COL ? c : q;
  return 0.f;
}

// the parts of coordinates 8 g .. 8 g + 7 of point j (zeros unless in)
template <bool AUG, bool COL>
__device__ __forceinline__ void b3_split8(const float* __restrict__ X, const float* __restrict__ qv, int64_t j,
                                          int64_t n, int p, int g, float c, u16x8_t& h, u16x8_t& m, u16x8_t& l) {
  const int64_t jc = min(j, n - 1);
  const float* x = X + jc * p;
  const float q = AUG ? qv[jc] : 0.f;
  float xv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) xv[e] = x[min(8 * g + e, p - 1)];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint16_t hh, mm, ll;
    split3_bf16(j < n ? b3_coord<AUG, COL>(xv[e], q, 8 * g + e, p, c) : 0.f, hh, mm, ll);
    h[e] = hh;
    m[e] = mm;
    l[e] = ll;
  }
}

// One thread per point of the padded set and 8-coordinate group, in buffer
// order, as the column (scaled, COL) or the row side.
template <bool AUG, bool COL = true>
__global__ __launch_bounds__(256) void kotf_split_cols_kernel(const float* __restrict__ Xc,
                                                              const float* __restrict__ qc, int64_t nc, int p,
                                                              float ng, uint16_t* __restrict__ out) {
  const int64_t t = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  const int64_t j = (t >> 6) * 16 + (t & 15);
  if (j >= (nc + kB3Pad - 1) / kB3Pad * kB3Pad) return;
  const int g = int(t >> 4) & 3;
  u16x8_t h, m, l;
  b3_split8<AUG, COL>(Xc, qc, j, nc, p, g, (AUG && COL) ? ng : 1.f, h, m, l);
  uint16_t* o = out + b3_offset(j, g);
  *reinterpret_cast<u16x8_t*>(o) = h;
  *reinterpret_cast<u16x8_t*>(o + kB3Plane) = m;
  *reinterpret_cast<u16x8_t*>(o + 2 * kB3Plane) = l;
}

template <bool AUG>
struct GramB3 {
  typedef uint16_t col_t;  // the columns: their split
  static constexpr int kMfmas = 12;
  static constexpr int kStageBytes = kOtfStage / 16 * kB3Block * 2;
  static constexpr bool kNorms = !AUG;
  static constexpr int kFlush = 2;
  bf16x8_t ah[2], am[2], al[2];
  u16x8_t nx[3];

  __device__ __forceinline__ void rows(const float* __restrict__ X, const float* __restrict__ q, int64_t n, int p,
                                       int64_t r, int s, int lg) {
    u16x8_t h, m, l;
    b3_split8<AUG, false>(X, q, r, n, p, lg, 1.f, h, m, l);
    ah[s] = __builtin_bit_cast(bf16x8_t, h);
    am[s] = __builtin_bit_cast(bf16x8_t, m);
    al[s] = __builtin_bit_cast(bf16x8_t, l);
  }
  // a stage is contiguous: 768 pieces of 16 bytes, three per thread
  __device__ __forceinline__ void fetch(const uint16_t* __restrict__ Bc, int64_t, int, int64_t j0, int t) {
    const u16x8_t* src = reinterpret_cast<const u16x8_t*>(Bc + (j0 >> 4) * kB3Block) + t;
#pragma unroll
    for (int c = 0; c < 3; ++c) nx[c] = src[256 * c];
  }
  __device__ __forceinline__ void put(char* lds, int, int t) {
#pragma unroll
    for (int c = 0; c < 3; ++c) reinterpret_cast<u16x8_t*>(lds)[256 * c + t] = nx[c];
  }
  __device__ __forceinline__ void gram(const char* lds, int tile, int lane, f32x4_t (&g)[2]) const {
    const bf16x8_t* x = reinterpret_cast<const bf16x8_t*>(lds) + tile * (kB3Block / 8) + lane;
    const bf16x8_t bh = x[0], bm = x[64], bl = x[128];
    f32x4_t c0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, c1 = c0;  // smallest products first
    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[0], bm, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[1], bm, c1, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[0], bl, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[1], bl, c1, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[0], bh, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[1], bh, c1, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[0], bm, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[1], bm, c1, 0, 0, 0);
    c0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[0], bh, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am[1], bh, c1, 0, 0, 0);
    g[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[0], bh, c0, 0, 0, 0);
    g[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[1], bh, c1, 0, 0, 0);
  }
  static __device__ __forceinline__ float arg(float g, float qi, float qj, float ng) {
    return AUG ? g : ng * (qi + qj + g);
  }
};

// the entry: ng < 0 and d >= 0, so exp2(ng max(d, 0)) = min(exp2(ng d), 1), the
// clamp to [0, 1] being the exponential's output modifier
__device__ __forceinline__ float otf_entry(float a) { return __builtin_amdgcn_fmed3f(kexp2(a), 0.f, 1.f); }

// The sums are formed here: without this the compiler moves a stage's whole
// vector work behind the next stage's LDS stores (their last use is the next
// iteration), where it no longer overlaps the MFMAs.
template <class T>
__device__ __forceinline__ void otf_pin(T (&acc)[2][4]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) asm volatile("" : "+v"(acc[s][rr]));
}

// u = K(Xr, Xc) v over a slice of the columns (blockIdx.y) for 128 rows
// (blockIdx.x): one partial per slice and row.
template <class G, bool EX>
__global__ __launch_bounds__(256, 4) void kapply_otf_mfma_kernel(
    const float* __restrict__ Xr, const float* __restrict__ qr, int64_t nr,
    const typename G::col_t* __restrict__ Xc, const float* __restrict__ qc, int64_t nc, int p, float ng,
    const double* __restrict__ v, int64_t cols_per_slice, double* __restrict__ part) {
  typedef std::conditional_t<EX, double, float> acc_t;
  __shared__ __align__(16) char xs[2][G::kStageBytes];
  __shared__ acc_t vs[2][kOtfStage];
  __shared__ float qs[2][G::kNorms ? kOtfStage : 1];
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int64_t row0 = int64_t(blockIdx.x) * 128 + wave * 32;
  const int64_t c0 = int64_t(blockIdx.y) * cols_per_slice;
  const int64_t c1 = min(nc, c0 + cols_per_slice);
  G gm;
  double nv;
  float nq = 0.f;
  auto fetch = [&](int64_t jb) {
    gm.fetch(Xc, nc, p, jb, t);
    const int64_t j = min(jb + lane, c1 - 1);
    nv = v[j];
    if (G::kNorms) nq = qc[j];
  };
  auto put = [&](int64_t jb, int b) {
    gm.put(xs[b], p, t);
    if (t < kOtfStage) {  // columns past the slice count with v_j = 0
      vs[b][t] = jb + t < c1 ? acc_t(nv) : acc_t(0);
      if (G::kNorms) qs[b][t] = nq;
    }
  };
  fetch(c0);
  float qi[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    gm.rows(Xr, qr, nr, p, row0 + 16 * s + li, s, lg);
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) qi[s][rr] = G::kNorms ? qr[min(row0 + 16 * s + 4 * lg + rr, nr - 1)] : 0.f;
  }
  put(c0, 0);
  double acc[2][4];
  float a32[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      acc[s][rr] = 0.0;
      a32[s][rr] = 0.f;
    }
  __syncthreads();
  int b = 0;
  for (int64_t jb = c0; jb < c1; jb += kOtfStage, b ^= 1) {
    const bool more = jb + kOtfStage < c1;
    if (more) fetch(jb + kOtfStage);
    f32x4_t g[2][2];
    gm.gram(xs[b], 0, lane, g[0]);
#pragma unroll
    for (int tile = 0; tile < kOtfStage / 16; ++tile) {
      __builtin_amdgcn_s_setprio(1);  // a wave that feeds the matrix cores goes first
      if (tile + 1 < kOtfStage / 16) gm.gram(xs[b], tile + 1, lane, g[(tile + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      const acc_t vj = vs[b][16 * tile + li];
      const float qj = G::kNorms ? qs[b][16 * tile + li] : 0.f;
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const float e = otf_entry(G::arg(g[tile & 1][s][rr], qi[s][rr], qj, ng));
          if (EX) acc[s][rr] = fma(double(e), double(vj), acc[s][rr]);
          else a32[s][rr] = fmaf(e, float(vj), a32[s][rr]);
        }
    }
    if (EX) otf_pin(acc);
    else otf_pin(a32);
    if (!EX && (!more || G::kFlush == 1 || b == 1)) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          acc[s][rr] += double(a32[s][rr]);
          a32[s][rr] = 0.f;
        }
    }
    if (more) put(jb + kOtfStage, b ^ 1);
    __syncthreads();
  }
  // sum over the 16 column lanes of each row group (lane bits 0..3)
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) acc[s][rr] = row16_sum_f64<true>(acc[s][rr]);
  if (li == 0) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int64_t ro = row0 + 16 * s + 4 * lg + rr;
        if (ro < nr) part[int64_t(blockIdx.y) * nr + ro] = acc[s][rr];
      }
  }
}

// Symmetric form for the square K(X, X): each distinct pair once, over the
// upper-triangle 128 x 128 tiles of the packed geometry.  A workgroup takes a
// strip of tiles of tile-row I, two 64-column stages per tile.  Every entry
// feeds the row sum (times v_j) and, off the diagonal tile, the column sum
// (times v_i): of each of the stage's four 16-column tiles a lane adds its
// eight rows, two exchanges add the four lane groups (all four end with the
// sum and store it to the same LDS word), and the four waves are added in LDS.  Row sums are added over the 16 column lanes at the end of
// the strip.  packed_reduce adds the partials in a fixed order.
template <class G, bool EX>
__global__ __launch_bounds__(256, 4) void kapply_otf_mfma_sym_kernel(
    const float* __restrict__ X, const float* __restrict__ q, int64_t n, const typename G::col_t* __restrict__ Xc,
    int p, float ng, const double* __restrict__ v, int64_t nt, int strip, int64_t nsx,
    double* __restrict__ rowpart, double* __restrict__ colpart) {
  typedef std::conditional_t<EX, double, float> acc_t;
  static_assert(2 * kOtfStage == kPkT, "two stages per tile");
  __shared__ __align__(16) char xs[2][G::kStageBytes];
  __shared__ acc_t vs[2][kOtfStage];
  __shared__ float qs[2][G::kNorms ? kOtfStage : 1];
  __shared__ double red[2][4][kOtfStage];
  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int li = lane & 15, lg = lane >> 4;
  int64_t I, kst;
  pk_strip_coords(blockIdx.x, nt, strip, I, kst);
  const int64_t J0 = I + kst * strip, J1 = min(nt, J0 + strip);
  const int64_t row0 = I * kPkT + wave * 32;
  const int64_t c0 = J0 * kPkT, c1 = min(n, J1 * kPkT);
  G gm;
  double nv;
  float nq = 0.f;
  auto fetch = [&](int64_t jb) {
    gm.fetch(Xc, n, p, jb, t);
    const int64_t j = min(jb + lane, n - 1);
    nv = v[j];
    if (G::kNorms) nq = q[j];
  };
  auto put = [&](int64_t jb, int b) {
    gm.put(xs[b], p, t);
    if (t < kOtfStage) {  // columns past n count with v_j = 0 (their own sums are never read)
      vs[b][t] = jb + t < n ? acc_t(nv) : acc_t(0);
      if (G::kNorms) qs[b][t] = nq;
    }
  };
  fetch(c0);
  float qi[2][4];
  acc_t vi[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    gm.rows(X, q, n, p, row0 + 16 * s + li, s, lg);
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int64_t ro = row0 + 16 * s + 4 * lg + rr;
      const int64_t rc = min(ro, n - 1);
      const double vv = v[rc];
      qi[s][rr] = G::kNorms ? q[rc] : 0.f;
      vi[s][rr] = ro < n ? acc_t(vv) : acc_t(0);  // rows past n add nothing to the column sums
    }
  }
  put(c0, 0);
  double acc[2][4];
  float a32[2][4];
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      acc[s][rr] = 0.0;
      a32[s][rr] = 0.f;
    }
  __syncthreads();
  int b = 0;  // the stage's buffers, and its half of the tile (c0 is a multiple of the tile)
  for (int64_t jb = c0; jb < c1; jb += kOtfStage, b ^= 1) {
    const bool more = jb + kOtfStage < c1;
    if (more) fetch(jb + kOtfStage);
    f32x4_t g[2][2];
    gm.gram(xs[b], 0, lane, g[0]);
#pragma unroll
    for (int tile = 0; tile < kOtfStage / 16; ++tile) {
      __builtin_amdgcn_s_setprio(1);  // a wave that feeds the matrix cores goes first
      if (tile + 1 < kOtfStage / 16) gm.gram(xs[b], tile + 1, lane, g[(tile + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(0);
      const acc_t vj = vs[b][16 * tile + li];
      const float qj = G::kNorms ? qs[b][16 * tile + li] : 0.f;
      acc_t c = acc_t(0);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const float e = otf_entry(G::arg(g[tile & 1][s][rr], qi[s][rr], qj, ng));
          if (EX) {
            acc[s][rr] = fma(double(e), double(vj), acc[s][rr]);
            c = fma(double(e), double(vi[s][rr]), double(c));
          } else {
            a32[s][rr] = fmaf(e, float(vj), a32[s][rr]);
            c = fmaf(e, float(vi[s][rr]), float(c));
          }
        }
      const double w = swap_sum_f64<false>(swap_sum_f64<true>(double(c)));
      red[b][wave][16 * tile + li] = w;  // the same value from the four lane groups
    }
    if (EX) otf_pin(acc);
    else otf_pin(a32);
    if (!EX && (!more || b == 1)) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          acc[s][rr] += double(a32[s][rr]);
          a32[s][rr] = 0.f;
        }
    }
    if (more) put(jb + kOtfStage, b ^ 1);
    __syncthreads();
    // the other half of red is written in the next stage, this one only after that stage's barrier
    const int64_t J = jb / kPkT;
    if (t < kOtfStage && J != I)
      colpart[size_t(pk_tile_index(I, J, nt)) * kPkT + b * kOtfStage + t] =
          ((red[b][0][t] + red[b][1][t]) + red[b][2][t]) + red[b][3][t];
  }
  // row sums over the 16 column lanes of each row group (lane bits 0..3)
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) acc[s][rr] = row16_sum_f64<true>(acc[s][rr]);
  if (li == 0) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr)
        rowpart[(size_t(I) * nsx + kst) * kPkT + wave * 32 + 16 * s + 4 * lg + rr] = acc[s][rr];
  }
}

// The column side of a Gram engine: X itself, or its split formed here in buf.
template <class G>
static const typename G::col_t* otf_columns(const float* X, const float* q, int64_t n, int p, float ng, void* buf,
                                            hipStream_t st) {
  if constexpr (std::is_same_v<typename G::col_t, float>) {
    return X;
  } else {
    uint16_t* bc = static_cast<uint16_t*>(buf);
    const dim3 grid((unsigned)(b3_points(n) * 4 / 256));
    kotf_split_cols_kernel<!G::kNorms><<<grid, 256, 0, st>>>(X, q, n, p, ng, bc);
    KQR_LAUNCH_CHECK();
    return bc;
  }
}

template <class G>
static size_t otf_columns_bytes(int64_t n) {
  return std::is_same_v<typename G::col_t, float> ? 0 : b3_bytes(n);
}

// K(X, X) v with each distinct pair once; u = K v.
template <class G>
static void kapply_otf_mfma_sym(const float* X, const float* q, int64_t n, int p, KernelSpec ks, const double* v,
                                double* u, int64_t ldu, bool exact, hipStream_t st, double* scratch,
                                size_t scratch_doubles) {
  const int64_t nt = (n + kPkT - 1) / kPkT;
  const int strip = otf_sym_strip(n);
  const int64_t nsx = (nt + strip - 1) / strip;
  const size_t need = packed_scratch_doubles(n, strip);
  const size_t col_bytes = otf_columns_bytes<G>(n), part_bytes = (need * sizeof(double) + 255) / 256 * 256;
  const size_t have = scratch ? scratch_doubles * sizeof(double) : 0;
  // the sums in the caller's scratch where they fit, the columns too where both do
  const bool sums_in = have >= need * sizeof(double), cols_in = have >= part_bytes + col_bytes;
  const size_t own = (sums_in ? 0 : part_bytes) + (cols_in ? 0 : col_bytes);
  char* buf = nullptr;
  if (own > 0) KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&buf), own, st));
  double* rowpart = sums_in ? scratch : reinterpret_cast<double*>(buf);
  double* colpart = rowpart + size_t(nt) * nsx * kPkT;
  const float ng = -float(ks.gamma) * kLog2e;
  char* col_buf = cols_in ? reinterpret_cast<char*>(scratch) + part_bytes : buf + (sums_in ? 0 : part_bytes);
  const typename G::col_t* cols = otf_columns<G>(X, q, n, p, ng, col_buf, st);
  const dim3 grid((unsigned)pk_strips_tail(nt, strip));
  if (exact)
    kapply_otf_mfma_sym_kernel<G, true><<<grid, 256, 0, st>>>(X, q, n, cols, p, ng, v, nt, strip, nsx, rowpart, colpart);
  else
    kapply_otf_mfma_sym_kernel<G, false><<<grid, 256, 0, st>>>(X, q, n, cols, p, ng, v, nt, strip, nsx, rowpart, colpart);
  KQR_LAUNCH_CHECK();
  packed_reduce(rowpart, colpart, n, strip, u, ldu, st);
  if (buf) KQR_CHECK_HIP(hipFreeAsync(buf, st));
}

// Column slices of a rectangular launch on the matrix cores, in stages of
// `stage` columns: where a target is set, or the launch is more than 32
// workgroups per CU, as otf_slices; below that, so that the workgroups come out in whole rounds of
// the CUs (a CU with one more workgroup than the others is what the launch
// waits for), the time taken as that of the busiest CU, two stages' time for
// a workgroup's start and a half or a fifth more where one or two
// workgroups per CU leave its units waiting.  5,000 x 20,000 at p = 10 takes 48 us in
// 760 workgroups of 17 stages, 52 in 800 of 16.
static int64_t otf_mfma_per(int64_t rblk, int64_t nc, int64_t stage) {
  const int64_t cus = 256, ns = (nc + stage - 1) / stage;
  const int64_t big = std::min<int64_t>(otf_slices(rblk, nc), 65535);
  if (rblk * std::min<int64_t>(ns, big) > 32 * cus || g_otf_wgs.load() > 0)
    return ((nc + big - 1) / big + stage - 1) / stage * stage;
  int64_t best = ns;
  double best_t = 0.0;
  for (int64_t k = 1; k <= 16; ++k) {
    const int64_t slices = std::max<int64_t>(1, std::min(ns, cus * k / rblk));
    const int64_t per = (ns + slices - 1) / slices;
    const int64_t wgs = rblk * ((ns + per - 1) / per);
    const int64_t on_cu = (wgs + cus - 1) / cus;
    const double t = double(on_cu * (per * stage + 128)) * (on_cu == 1 ? 1.5 : on_cu == 2 ? 1.2 : 1.0);
    if (k == 1 || t < best_t) {
      best = per;
      best_t = t;
    }
  }
  return best * stage;
}

template <class G>
static void kapply_otf_mfma_p(const float* Xr, const float* qr, int64_t nr, const float* Xc, const float* qc,
                              int64_t nc, int p, KernelSpec ks, const double* v, double* u, int64_t ldu, double scale,
                              double shift, bool exact, hipStream_t st, double* scratch, size_t scratch_doubles) {
  if (Xr == Xc && qr == qc && nr == nc && scale == 1.0 && shift == 0.0 && otf_sym_fits(nr)) {  // square: symmetric
    kapply_otf_mfma_sym<G>(Xr, qr, nr, p, ks, v, u, ldu, exact, st, scratch, scratch_doubles);
    return;
  }
  const int64_t rblk = (nr + 127) / 128;
  const int64_t per = otf_mfma_per(rblk, nc, int64_t(kOtfStage) * G::kFlush);
  const int64_t nslice = (nc + per - 1) / per;
  const size_t part_bytes = (size_t(nslice) * size_t(nr) * sizeof(double) + 255) / 256 * 256;
  const size_t bytes = part_bytes + otf_columns_bytes<G>(nc);
  const bool own = !scratch || scratch_doubles * sizeof(double) < bytes;
  char* buf = reinterpret_cast<char*>(scratch);
  if (own) KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&buf), bytes, st));
  double* part = reinterpret_cast<double*>(buf);
  const dim3 grid((unsigned)rblk, (unsigned)nslice);
  const float ng = -float(ks.gamma) * kLog2e;
  const typename G::col_t* cols = otf_columns<G>(Xc, qc, nc, p, ng, buf + part_bytes, st);
  if (exact) kapply_otf_mfma_kernel<G, true><<<grid, 256, 0, st>>>(Xr, qr, nr, cols, qc, nc, p, ng, v, per, part);
  else kapply_otf_mfma_kernel<G, false><<<grid, 256, 0, st>>>(Xr, qr, nr, cols, qc, nc, p, ng, v, per, part);
  KQR_LAUNCH_CHECK();
  otf_reduce(part, nslice, nr, u, ldu, scale, shift, st);
  if (own) KQR_CHECK_HIP(hipFreeAsync(buf, st));
}

void kapply_otf(const float* Xr, const float* sqr, int64_t nr, const float* Xc, const float* sqc,
                int64_t nc, int p, KernelSpec ks, const double* v64, double* u, int64_t ldu,
                double out_scale, double out_shift, hipStream_t st, bool exact, double* scratch,
                size_t scratch_doubles) {
  if (nr <= 0) return;
  if (ks.kind == KQR_RBF && p <= 32) {
#define KQR_OTF_MFMA(...) \
  kapply_otf_mfma_p<__VA_ARGS__>(Xr, sqr, nr, Xc, sqc, nc, p, ks, v64, u, ldu, out_scale, out_shift, exact, st, \
                                 scratch, scratch_doubles)
    if (p <= 8) KQR_OTF_MFMA(GramF32<8>);
    else if (p <= 12) KQR_OTF_MFMA(GramF32<12>);
    else if (p <= 16) KQR_OTF_MFMA(GramF32<16>);
    else if (p <= 30) KQR_OTF_MFMA(GramB3<true>);
    else KQR_OTF_MFMA(GramB3<false>);
#undef KQR_OTF_MFMA
    return;
  }
  KQR_DISPATCH_P(p, kapply_otf_p, Xr, sqr, nr, Xc, sqc, nc, p, ks, v64, u, ldu, out_scale, out_shift, exact, st, scratch,
                 scratch_doubles);
}

size_t kapply_otf_scratch_doubles(int64_t nr, int64_t nc, int p, KernelSpec ks, bool square) {
  const bool mfma = ks.kind == KQR_RBF && p <= 32;
  const size_t cols = mfma && p > 16 ? b3_bytes(nc) : 0;
  size_t part = 0;
  if (mfma && square && otf_sym_fits(nr)) {
    part = packed_scratch_doubles(nr, otf_sym_strip(nr));
  } else {
    const int64_t rblk = (nr + (mfma ? 127 : 255)) / (mfma ? 128 : 256);
    const int64_t per = mfma ? otf_mfma_per(rblk, nc, kOtfStage * (p > 16 ? 2 : 1)) : otf_per(rblk, nc);
    part = size_t((nc + per - 1) / per) * size_t(nr);
  }
  return ((part * sizeof(double) + 255) / 256 * 256 + cols) / sizeof(double);
}

// ================================================================= K build on the matrix cores
// RBF with p <= 32: the Gram term of every 16 x 16 block on the matrix cores
// (v_mfma_f32_16x16x32_bf16) from the exact BF16x3 split of both sides (as
// the on-the-fly applies), with the norms and the exponent's scale folded into
// the spare coordinates when p <= 30 (the matrix cores then return
// c d_ij, c = -gamma log2(e)), so an entry costs the lanes a clamp, the
// exponential, the diagonal test and its share of a store.  Both sides are
// split once per build into buffers in operand order (kotf_split_cols_kernel;
// row side [x, 1, q], column side [-2 c x, c q, c]; without the fold [x] and
// [-2 x]).
// FP32 storage takes all six significant products.  BF16 storage takes the
// three leading ones (hi.hi, hi.mid, mid.hi): the dropped ones are at most
// 3 2^-16 sum_k |a_k| |b_k|, and that sum is at most 2 |c| (q_i + q_j)
// (2 |x_i . x_j| <= q_i + q_j), so the entry moves by a relative
// 3 2^-15 gamma (q_i + q_j) at most.  The three products are used only when
// gamma max_i q_i <= 16 / 3, which keeps that below 2^-10, a quarter of
// BF16's unit roundoff 2^-8; inputs far from the origin get the six.
//
// Operand roles: the A operand carries 16 columns j of K and the B operand
// 16 rows i, so the lane that receives C[4 g + r][l] holds K[i0 + l][j0 +
// 4 g + r], r = 0..3.  A workgroup is four waves of 32 rows each (two 16-row
// strips as B operands held in registers); a step covers 64 columns (four
// 16-column blocks, whose column parts each wave loads once from L2, 192
// bytes per column, and uses for both strips).  The step's 32 x 64 entries of
// a wave go through its own LDS slab and leave as whole rows: 16-byte stores,
// 256 contiguous bytes per row (FP32) or 128 (BF16), so every store writes
// full 128-byte lines (the MFMA layout alone would give 64- or 32-byte pieces
// per row and instruction).
//   full layout  : 128 rows x `cols` columns of the n x ldk matrix per workgroup
//                  (columns n..ldk-1 written as 0, rows >= n not written;
//                  ldk and `cols` multiples of 64);
//   packed layout: one 128 x 128 upper-triangle tile per workgroup (entries
//                  beyond n written as 0, as the tile layout requires).
// K_ii is set to exactly 1 (d_ii := 0).
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kBuildStep = 64;               // columns per step
constexpr int kBuildSlab = kBuildStep + 4;   // LDS row of a wave's slab (floats), padded against bank conflicts

template <bool AUG, bool BF, bool PACKED>
__global__ __launch_bounds__(256) void kbuild_b3_kernel(const uint16_t* __restrict__ Pr, const uint16_t* __restrict__ Sc,
                                                        const float* __restrict__ q, int64_t n, float ng,
                                                        void* __restrict__ Kout, int64_t ldk, int64_t nt,
                                                        int64_t cols, const float* __restrict__ qmax, float qlim) {
  // a wave's slab: 32 rows x 64 entries, FP32 or (BF16 storage) the rounded BF16 values
  __shared__ __align__(16) float slab[4][32][kBuildSlab];
  typedef uint16_t bslab_row[2 * kBuildSlab];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: block tests branch on scalars
  const int li = lane & 15, lg = lane >> 4;
  int64_t rbase, cbeg, cend;
  size_t tile_base = 0;
  if (PACKED) {
    const int64_t t = blockIdx.x;
    int64_t lo = 0, hi = nt - 1;  // largest I whose first tile index is <= t
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) / 2;
      if (pk_tile_index(mid, mid, nt) <= t) lo = mid;
      else hi = mid - 1;
    }
    const int64_t J = lo + (t - pk_tile_index(lo, lo, nt));
    rbase = lo * kPkT;
    cbeg = J * kPkT;
    cend = cbeg + kPkT;
    tile_base = size_t(t) * kPkT * kPkT;
  } else {
    rbase = int64_t(blockIdx.x) * 128;
    cbeg = int64_t(blockIdx.y) * cols;
    cend = min(ldk, cbeg + cols);
  }
  const int64_t wrow = rbase + 32 * wave;  // this wave's first row
  // B operands: rows wrow + 16 s + li, coordinates 8 lg .. 8 lg + 7
  bf16x8_t bh[2], bm[2], bl[2];
  float qi[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int64_t ic = min(wrow + 16 * s + li, n - 1);  // rows past n: any valid point (entries not kept)
    const uint16_t* rp = Pr + b3_offset(ic, lg);
    bh[s] = *reinterpret_cast<const bf16x8_t*>(rp);
    bm[s] = *reinterpret_cast<const bf16x8_t*>(rp + kB3Plane);
    bl[s] = *reinterpret_cast<const bf16x8_t*>(rp + 2 * kB3Plane);
    qi[s] = AUG ? 0.f : q[ic];
  }
  const uint32_t col_off = uint32_t(lane) * 8;  // this lane's column part within a plane
  float (*sl)[kBuildSlab] = slab[wave];
  bslab_row* bsl = reinterpret_cast<bslab_row*>(slab[wave]);  // BF16 view: rows of 2 kBuildSlab halves
  // BF16 storage: three products when the largest squared norm allows (see
  // above); one instantiation of the step loop per case, chosen once
  auto steps = [&](auto three_c) {
    constexpr bool three = decltype(three_c)::value;
    for (int64_t jb = cbeg; jb < cend; jb += kBuildStep) {
      // the column parts of the whole step are requested at once: one L2 round
      // trip per step instead of one per 16-column block
      bf16x8_t ahs[kBuildStep / 16], ams[kBuildStep / 16], als[kBuildStep / 16];
      if (jb + kBuildStep <= n) {  // (uniform) whole step inside: a scalar base per block, the lane's offset fixed
#pragma unroll
        for (int blk = 0; blk < kBuildStep / 16; ++blk) {
          const uint16_t* cb = Sc + ((jb >> 4) + blk) * kB3Block;
          ahs[blk] = *reinterpret_cast<const bf16x8_t*>(cb + col_off);
          ams[blk] = *reinterpret_cast<const bf16x8_t*>(cb + col_off + kB3Plane);
          if constexpr (!three) als[blk] = *reinterpret_cast<const bf16x8_t*>(cb + col_off + 2 * kB3Plane);
        }
      } else {
#pragma unroll
        for (int blk = 0; blk < kBuildStep / 16; ++blk) {
          const int64_t jc = min(jb + 16 * blk + li, n - 1);  // columns past n: any valid point (written as 0)
          const uint16_t* cb = Sc + b3_offset(jc, lg);
          ahs[blk] = *reinterpret_cast<const bf16x8_t*>(cb);
          ams[blk] = *reinterpret_cast<const bf16x8_t*>(cb + kB3Plane);
          if constexpr (!three) als[blk] = *reinterpret_cast<const bf16x8_t*>(cb + 2 * kB3Plane);
        }
      }
      // Gram blocks: the two strips' product chains interleaved, and the next
      // block's MFMAs issued before this block's exponentials
      auto gram = [&](int blk, f32x4_t* c) {
        const bf16x8_t ah = ahs[blk], am = ams[blk];
        c[0] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        c[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if constexpr (three) {
          c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh[0], c[0], 0, 0, 0);
          c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh[1], c[1], 0, 0, 0);
          c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm[0], c[0], 0, 0, 0);
          c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm[1], c[1], 0, 0, 0);
          c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[0], c[0], 0, 0, 0);
          c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[1], c[1], 0, 0, 0);
          return;
        }
        // smallest products first
        const bf16x8_t al = als[blk];
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bm[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bm[1], c[1], 0, 0, 0);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh[1], c[1], 0, 0, 0);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl[1], c[1], 0, 0, 0);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(am, bh[1], c[1], 0, 0, 0);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bm[1], c[1], 0, 0, 0);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh[1], c[1], 0, 0, 0);
      };
      f32x4_t cur[2], nxt[2];
      gram(0, cur);
#pragma unroll
      for (int blk = 0; blk < kBuildStep / 16; ++blk) {
        if (blk + 1 < kBuildStep / 16) gram(blk + 1, nxt);
        const int64_t j0 = jb + 16 * blk + 4 * lg;  // this lane's four columns j0 .. j0 + 3
        float qj[4] = {0.f, 0.f, 0.f, 0.f};
        if (!AUG) {
#pragma unroll
          for (int r = 0; r < 4; ++r) qj[r] = q[min(j0 + r, n - 1)];
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const f32x4_t c = cur[s];
          const int64_t iblk = wrow + 16 * s, jblk = jb + 16 * blk;
          f32x4_t e;
          // ng < 0 and d >= 0, so the entry is exp2(min(ng d, 0)) = min(exp2(ng d), 1): the
          // clamp to [0, 1] rides on the exponential as its output modifier
#pragma unroll
          for (int r = 0; r < 4; ++r)
            e[r] = __builtin_amdgcn_fmed3f(kexp2(AUG ? c[r] : ng * (qi[s] + qj[r] + c[r])), 0.f, 1.f);
          if (iblk == jblk || iblk + 16 > n || jblk + 16 > n) {  // (uniform) diagonal or ragged block
            // 32-bit tests against the block's valid extents (both blocks start on multiples of 16)
            const int64_t ri = n - iblk, rj = n - jblk;
            const int ni = ri < 16 ? int(ri) : 16, nj = rj < 16 ? int(rj) : 16;
            const bool diag = iblk == jblk;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int jl = 4 * lg + r;
              e[r] = (jl < nj && li < ni) ? ((diag && jl == li) ? 1.f : e[r]) : 0.f;
            }
          }
          if (BF) {  // round to BF16 here: half the LDS traffic
            u32x2_t w;
            w[0] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{e[0], e[1]}, bf16x2_t));
            w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{e[2], e[3]}, bf16x2_t));
            *reinterpret_cast<u32x2_t*>(&bsl[16 * s + li][16 * blk + 4 * lg]) = w;
          } else {
            *reinterpret_cast<f32x4_t*>(&sl[16 * s + li][16 * blk + 4 * lg]) = e;
          }
        }
        cur[0] = nxt[0];
        cur[1] = nxt[1];
      }
      __syncthreads();  // the slab is complete (each wave reads only its own)
      if (BF) {
        // a row is 64 BF16 = 128 bytes = 8 lanes x 16 bytes; eight rows per store
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int rr = 8 * k + (lane >> 3), cc = 8 * (lane & 7);
          const u32x4_t w = *reinterpret_cast<const u32x4_t*>(&bsl[rr][cc]);
          const int64_t i = wrow + rr;
          if (PACKED) {
            const size_t off = tile_base + size_t(i - rbase) * kPkT + size_t(jb - cbeg + cc);
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(Kout) + off));
          } else if (i < n) {
            const size_t off = size_t(i) * size_t(ldk) + size_t(jb + cc);
            __builtin_nontemporal_store(w, reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(Kout) + off));
          }
        }
      } else {
        // a row is 64 FP32 = 256 bytes = 16 lanes x 16 bytes; four rows per store
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int rr = 4 * k + (lane >> 4), cc = 4 * (lane & 15);
          const f32x4_t x = *reinterpret_cast<const f32x4_t*>(&sl[rr][cc]);
          const int64_t i = wrow + rr;
          if (PACKED) {
            const size_t off = tile_base + size_t(i - rbase) * kPkT + size_t(jb - cbeg + cc);
            __builtin_nontemporal_store(x, reinterpret_cast<f32x4_t*>(static_cast<float*>(Kout) + off));
          } else if (i < n) {
            const size_t off = size_t(i) * size_t(ldk) + size_t(jb + cc);
            __builtin_nontemporal_store(x, reinterpret_cast<f32x4_t*>(static_cast<float*>(Kout) + off));
          }
        }
      }
      __syncthreads();  // the slab is free for the next step
    }
  };
  if (BF && *qmax <= qlim) steps(std::true_type{});
  else steps(std::false_type{});
}

// Columns per workgroup of the full-layout build.
constexpr int64_t kBuildCols = 1024;

// out[0] = max_i q_i (one workgroup of 1024 threads)
__global__ __launch_bounds__(1024) void qmax_kernel(const float* __restrict__ q, int64_t n, float* __restrict__ out) {
  __shared__ float sh[16];
  float m = 0.f;
  for (int64_t i = threadIdx.x; i < n; i += blockDim.x) m = fmaxf(m, q[i]);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) m = fmaxf(m, sh[w]);
    out[0] = fmaxf(m, sh[0]);
  }
}

bool kbuild_mfma(const float* X, const float* q, int64_t n, int p, KernelSpec ks, int dtype, void* K, int64_t ldk,
                 int layout, hipStream_t st) {
  if (ks.kind != KQR_RBF || p > 32 || n <= 0) return false;
  if (layout == 0 && ldk % kBuildStep != 0) return false;  // the stores cover 64-column steps up to ldk
  const bool aug = p <= 30, bf = dtype == KQR_BF16;
  const float ng = -float(ks.gamma) * kLog2e;
  uint16_t* buf = nullptr;
  const size_t half_bytes = b3_bytes(n);
  KQR_CHECK_HIP(hipMallocAsync(reinterpret_cast<void**>(&buf), 2 * half_bytes + 256, st));
  uint16_t* Pr = buf;                      // row side
  uint16_t* Sc = buf + half_bytes / sizeof(uint16_t);  // column side (scaled)
  float* qmax = reinterpret_cast<float*>(buf + 2 * (half_bytes / sizeof(uint16_t)));
  const float qlim = float(16.0 / (3.0 * ks.gamma));  // three products when max q <= qlim
  if (bf) {
    qmax_kernel<<<1, 1024, 0, st>>>(q, n, qmax);
    KQR_LAUNCH_CHECK();
  }
  const dim3 sgrid((unsigned)(b3_points(n) * 4 / 256));
  if (aug) {
    kotf_split_cols_kernel<true, false><<<sgrid, 256, 0, st>>>(X, q, n, p, ng, Pr);
    kotf_split_cols_kernel<true, true><<<sgrid, 256, 0, st>>>(X, q, n, p, ng, Sc);
  } else {
    kotf_split_cols_kernel<false, false><<<sgrid, 256, 0, st>>>(X, q, n, p, ng, Pr);
    kotf_split_cols_kernel<false, true><<<sgrid, 256, 0, st>>>(X, q, n, p, ng, Sc);
  }
  KQR_LAUNCH_CHECK();
  const int64_t nt = (n + kPkT - 1) / kPkT;
  dim3 grid;
  if (layout == 1) grid = dim3((unsigned)packed_tile_count(n));
  else grid = dim3((unsigned)((n + 127) / 128), (unsigned)((ldk + kBuildCols - 1) / kBuildCols));
#define KQR_B3(A, B, P) \
  kbuild_b3_kernel<A, B, P><<<grid, 256, 0, st>>>(Pr, Sc, q, n, ng, K, ldk, nt, kBuildCols, qmax, qlim)
  if (layout == 1) {
    if (aug && bf) KQR_B3(true, true, true);
    else if (aug) KQR_B3(true, false, true);
    else if (bf) KQR_B3(false, true, true);
    else KQR_B3(false, false, true);
  } else {
    if (aug && bf) KQR_B3(true, true, false);
    else if (aug) KQR_B3(true, false, false);
    else if (bf) KQR_B3(false, true, false);
    else KQR_B3(false, false, false);
  }
#undef KQR_B3
  KQR_LAUNCH_CHECK();
  KQR_CHECK_HIP(hipFreeAsync(buf, st));
  return true;
}

// ================================================================= one kernel row
template <bool BF16>
__global__ void krow_from_mat_kernel(const void* __restrict__ K, int64_t ldk, int64_t n, int64_t s,
                                     double* __restrict__ out) {
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  if (BF16) out[j] = bf16_to_f32(static_cast<const uint16_t*>(K)[s * ldk + j]);
  else out[j] = static_cast<const float*>(K)[s * ldk + j];
}

template <int PMAX, bool LAP>
__global__ void krow_from_x_kernel(const float* __restrict__ X, const float* __restrict__ q,
                                   int64_t n, int p, float ng, int64_t s, double* __restrict__ out) {
  __shared__ float xs[PMAX];
  if (threadIdx.x < PMAX) xs[threadIdx.x] = threadIdx.x < p ? X[s * p + threadIdx.x] : 0.f;
  __syncthreads();
  const int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (j >= n) return;
  float xj[PMAX];
#pragma unroll
  for (int k = 0; k < PMAX; ++k) xj[k] = k < p ? X[j * p + k] : 0.f;
  float d = pair_dist<PMAX, LAP>(xs, LAP ? 0.f : q[s], xj, LAP ? 0.f : q[j]);
  if (j == s) d = 0.f;
  out[j] = kexp2(ng * d);
}

template <int PMAX>
static void krow_p(const float* X, const float* q, int64_t n, int p, KernelSpec ks, int64_t s,
                   double* out, hipStream_t st) {
  const dim3 grid((unsigned)((n + 255) / 256));
  const float ng = -float(ks.gamma) * kLog2e;
  if (ks.kind == KQR_LAPLACIAN) krow_from_x_kernel<PMAX, true><<<grid, 256, 0, st>>>(X, q, n, p, ng, s, out);
  else krow_from_x_kernel<PMAX, false><<<grid, 256, 0, st>>>(X, q, n, p, ng, s, out);
  KQR_LAUNCH_CHECK();
}

void kernel_row(const KMat& km, const float* X, const float* sqn, int64_t n, int p, KernelSpec ks,
                int64_t s, double* out, hipStream_t st) {
  if (km.K && km.layout == 1) {
    kernel_row_packed(km, n, s, out, st);
    return;
  }
  if (km.K) {
    const dim3 grid((unsigned)((n + 255) / 256));
    if (km.dtype == KQR_BF16) krow_from_mat_kernel<true><<<grid, 256, 0, st>>>(km.K, km.ld, n, s, out);
    else krow_from_mat_kernel<false><<<grid, 256, 0, st>>>(km.K, km.ld, n, s, out);
    KQR_LAUNCH_CHECK();
    return;
  }
  KQR_DISPATCH_P(p, krow_p, X, sqn, n, p, ks, s, out, st);
}

// ================================================================= skinny mat-vec
// 16 lanes per row (4 rows per wave at a time, 4 such row slots per wave):
// a lane reads 16-byte pieces of its row 64 columns apart, x sits in LDS, and
// a 4-step shuffle reduction inside each 16-lane group finishes 4 rows at once.
// (Workgroup blk of the launch; the body also serves the batched PCG steps.)
__device__ __forceinline__ void gemv_skinny_body(const float* __restrict__ A, int64_t lda, int64_t nrows, int ncols,
                                                 const double* __restrict__ x, double* __restrict__ y, int blk) {
  __shared__ double xs[1024 + 4];
  for (int k = threadIdx.x; k < ncols; k += 256) xs[k] = x[k];
  for (int k = ncols + threadIdx.x; k < ((ncols + 3) & ~3); k += 256) xs[k] = 0.0;
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, t = lane & 15;
  const int64_t wrow0 = (int64_t(blk) * 4 + wave) * 16;
  const int nvec = ncols >> 2;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const float* rows[4];
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) {
    const int64_t r = min(wrow0 + sl * 4 + g, nrows - 1);
    rows[sl] = A + r * lda;
  }
  for (int c = t; c < nvec; c += 16) {
    float4 v[4];
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) v[sl] = reinterpret_cast<const float4*>(rows[sl])[c];
    const double x0 = xs[4 * c], x1 = xs[4 * c + 1], x2 = xs[4 * c + 2], x3 = xs[4 * c + 3];
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      acc[sl] = fma(double(v[sl].x), x0, acc[sl]);
      acc[sl] = fma(double(v[sl].y), x1, acc[sl]);
      acc[sl] = fma(double(v[sl].z), x2, acc[sl]);
      acc[sl] = fma(double(v[sl].w), x3, acc[sl]);
    }
  }
  for (int c = nvec * 4 + t; c < ncols; c += 16) {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) acc[sl] = fma(double(rows[sl][c]), xs[c], acc[sl]);
  }
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) acc[sl] = row16_sum_f64(acc[sl]);
  if (t == 0) {
#pragma unroll
    for (int sl = 0; sl < 4; ++sl) {
      const int64_t r = wrow0 + sl * 4 + g;
      if (r < nrows) y[r] = acc[sl];
    }
  }
}

__global__ __launch_bounds__(256) void gemv_skinny_kernel(const float* __restrict__ A, int64_t lda, int64_t nrows,
                                                          int ncols, const double* __restrict__ x,
                                                          double* __restrict__ y) {
  gemv_skinny_body(A, lda, nrows, ncols, x, y, int(blockIdx.x));
}

// Batched PCG steps: Fs = F s_{1..rank} of every fit with rank > 0, each
// over its range of workgroups (64 rows each).
__global__ __launch_bounds__(256) void wood_fs_steps_kernel(const PcgStepDesc* __restrict__ d,
                                                            const int* __restrict__ first, int nf) {
  const int f = step_of_block(first, nf, int(blockIdx.x));
  const PcgStepDesc& e = d[f];
  gemv_skinny_body(e.F, e.ldf, e.n, e.rank, e.s, e.Fs, int(blockIdx.x) - first[f]);
}

void launch_wood_fs_steps(const PcgStepDesc* d, const int* fs_first, int nf, int total, hipStream_t st) {
  if (nf <= 0 || total <= 0) return;
  wood_fs_steps_kernel<<<total, 256, 0, st>>>(d, fs_first, nf);
  KQR_LAUNCH_CHECK();
}

int pcg_step_fs_blocks(const PcgStepDesc& d) { return d.rank > 0 ? int((d.n + 63) / 64) : 0; }

void gemv_skinny(const float* A, int64_t lda, int64_t nrows, int64_t ncols, const double* x, double* y,
                 hipStream_t st) {
  if (nrows <= 0) return;
  if (ncols > 1024 || (lda & 3)) fail(KQR_EINVAL, "gemv_skinny: ncols <= 1024 and lda % 4 == 0 required");
  gemv_skinny_kernel<<<dim3((unsigned)((nrows + 63) / 64)), 256, 0, st>>>(A, lda, nrows, int(ncols), x, y);
  KQR_LAUNCH_CHECK();
}

// ================================================================= FP64 -> FP32
__global__ void to_f32_kernel(const double* __restrict__ src, int64_t n, int m, int64_t lds,
                              float* __restrict__ dst, int64_t ldd) {
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= n * m) return;
  const int64_t i = t / m;
  const int k = int(t % m);
  dst[i * ldd + k] = float(src[i * lds + k]);
}

void to_f32(const double* src, int64_t n, int m, int64_t lds, float* dst, int64_t ldd, hipStream_t st) {
  if (n <= 0) return;
  const int64_t tot = n * m;
  to_f32_kernel<<<dim3((unsigned)((tot + 255) / 256)), 256, 0, st>>>(src, n, m, lds, dst, ldd);
  KQR_LAUNCH_CHECK();
}

}  // namespace kqr
