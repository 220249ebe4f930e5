// Randomly pivoted Cholesky, F = RPCholesky(K, r), K_hat = F F^T (Section 3,
// preconditioner (3.2)), and the rank heuristic of Section 3.
//
// Step i of RPCholesky:
//   s    = first j with sum_{l<=j} d_l > u_i * sum(d)  (pivot ~ residual diagonal)
//   g    = K[:, s] - F[:, :i] F[s, :i]^T
//   F[:, i] = g / sqrt(g_s),  d <- max(d - F[:, i]^2, 0),  d_s <- 0
// Everything stays on the device, one launch per step: the pivot is found by a
// one-wave scan over block sums that the previous step produced, the
// correction F[:, :i] F[s, :i]^T streams F, and the early stop
// (sum(d) <= 1e-14 tr K) is a device flag, so the host synchronises once at
// the end.
//
// Rank heuristic: r0 = ceil(sqrt n), eigenvalues of F0^T F0, r = smallest index
// with lambda_r <= xi lambda_1.  F0^T F0 is reduced to tridiagonal form by
// Householder reflections in one workgroup (FP64), lambda_1 is found by
// bisection with Sturm counts, and the number of eigenvalues above
// xi lambda_1 by one more Sturm count.
#include "kernel_entry.h"
#include "reduce.h"
#include "vec.h"

#include <cmath>
#include <cstring>
#include <type_traits>

namespace kqr {

namespace {
constexpr int kSelBlocks = 256;
}

__global__ __launch_bounds__(256) void rpc_blocksum_kernel(const double* __restrict__ d, int64_t n, int64_t chunk,
                                                           double* __restrict__ bsum) {
  __shared__ double sh[4];
  const int64_t i0 = int64_t(blockIdx.x) * chunk;
  const int64_t i1 = min(n, i0 + chunk);
  double s = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) s += d[i];
  s = wave_sum_f64(s);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) bsum[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

// The pivot draw, by one wave: first j with sum_{l<=j} d_l > u * sum(d), or -1
// once the residual trace is negligible.  state[0] = tr K (set at step 0),
// state[1] = stopped flag; tr0 and stop return their new values.
__device__ __forceinline__ int64_t rpc_select(const double* __restrict__ d, int64_t n, int64_t chunk,
                                              const double* __restrict__ bsum, int nblk, double u, int step,
                                              const double* __restrict__ state, double& tr0, bool& stop) {
  const int lane = threadIdx.x & 63;
  // prefix sums of the block sums: lane l owns blocks [PER l, PER l + PER)
  constexpr int PER = kSelBlocks / 64;
  double bs[PER];
  double own = 0.0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int b = lane * PER + q;
    const double v = bsum[min(b, nblk - 1)];
    bs[q] = b < nblk ? v : 0.0;
    own += bs[q];
  }
  const double st0 = state[0], st1 = state[1];
  double incl = own;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double t = __shfl_up(incl, off);
    if (lane >= off) incl += t;
  }
  const double total = __shfl(incl, 63);
  stop = step > 0 && st1 != 0.0;
  tr0 = step == 0 ? total : st0;
  if (!(total > 1e-14 * tr0)) stop = true;
  int64_t found = -1;
  if (!stop) {
    const double target = u * total;
    // first block whose running sum passes the target
    int mine = -1;
    double before = 0.0;
    double run_b = incl - own;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const double next = run_b + bs[q];
      if (mine < 0 && next > target && bs[q] > 0.0) {
        mine = lane * PER + q;
        before = run_b;
      }
      run_b = next;
    }
    const unsigned long long hitm = __ballot(mine >= 0);
    int bsel = -1;
    double pref_sel = 0.0;
    if (hitm) {
      const int src = __ffsll((long long)hitm) - 1;
      bsel = __shfl(mine, src);
      pref_sel = __shfl(before, src);
    }
    if (bsel >= 0) {
      // scan from the selected block on (a later block only when the rounding
      // of block sums and running sum disagree next to the target); the
      // entries come four groups of 64 at a time, in one memory round trip
      double run = pref_sel;
      for (int64_t base = int64_t(bsel) * chunk; base < n && found < 0; base += 256) {
        double dv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int64_t i = base + 64 * q + lane;
          const double v = d[min(i, n - 1)];
          dv[q] = i < n ? v : 0.0;
        }
        double inc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) inc[q] = dv[q];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {  // four independent scans, interleaved
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double t = __shfl_up(inc[q], off);
            if (lane >= off) inc[q] += t;
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (found < 0) {
            const bool hit = (run + inc[q] > target) && dv[q] > 0.0;
            const unsigned long long m = __ballot(hit);
            if (m) found = base + 64 * q + __ffsll((long long)m) - 1;
            else run += readlane_f64(inc[q], 63);
          }
        }
      }
    }
    if (found < 0) {  // u*total rounded to the very end: take the last positive entry
      for (int64_t base = ((n - 1) / 64) * 64; base >= 0 && found < 0; base -= 64) {
        const int64_t i = base + lane;
        const unsigned long long m = __ballot(i < n && d[i] > 0.0);
        if (m) found = base + 63 - __clzll((long long)m);
      }
    }
    if (found < 0) stop = true;
  }
  return found;
}

// One step of RPCholesky in one launch (it was four: draw, pivot row, F f_s,
// update).  A workgroup owns one of the kSelBlocks chunks of rows.  Its first
// wave draws the pivot s from the previous step's residual diagonal and block
// sums (every workgroup alike, so nothing is exchanged inside the launch; d,
// the block sums and the state alternate between two buffers), the pivot row
// of F goes to LDS, and then
//   u_j = F[j, :i] . F[s, :i],  g_j = K[s][j] - u_j,  F[j][i] = g_j / sqrt(g_s),
//   d_j <- max(d_j - F[j][i]^2, 0),  d_s <- 0
// with 16 lanes per row (16-byte pieces 64 columns apart, four rows per group
// in flight), and the block sums of the new d.  u_s is formed from the LDS row alongside.
// Per step: the launch, three dependent memory round trips for the draw and
// its row, then F's first i columns (cache-resident for the most part: 50 MB on
// average at n = 50,000, r = 500).  There, 500 steps: 11.1 ms in four launches
// each (12.3 + 5.2 + 3.3 + 1.7 us and their gaps), 7.5 ms now (7 us for an empty step, 23 us for the last).
constexpr int kRpcThreads = 1024;
constexpr int kRpcSlots = 4;                               // rows of a 16-lane group in flight
constexpr int kRpcRows = kRpcThreads / 16 * kRpcSlots;     // rows of a pass

struct RpcStep {
  const double *d, *bsum, *state;  // after the previous step
  double *dn, *bsumn, *staten;     // after this one
  int64_t* piv;
  int64_t chunk;
  double u;  // this step's uniform
};

template <bool STORED>
__global__ __launch_bounds__(kRpcThreads) void rpc_step_kernel(const KMat km, const float* __restrict__ X,
                                                               const float* __restrict__ q, int p, int lap, float ng,
                                                               float* __restrict__ F, int64_t n, int64_t ldf, int i,
                                                               const RpcStep a) {
  static_assert(kRpcRows == 256, "a pass covers the 256 running sums of a block sum");
  __shared__ double xs[1024];
  __shared__ double part[256];
  __shared__ double sh[4];
  __shared__ int64_t pivot;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, t = lane & 15;
  const int64_t i0 = int64_t(blockIdx.x) * a.chunk, i1 = min(n, i0 + a.chunk);
  const int nvec = i >> 2;
  if (wave == 0) {
    double tr0;
    bool stop;
    const int64_t s = rpc_select(a.d, n, a.chunk, a.bsum, kSelBlocks, a.u, i, a.state, tr0, stop);
    if (lane == 0) {
      pivot = stop ? -1 : s;
      if (blockIdx.x == 0) {
        a.piv[i] = stop ? -1 : s;
        a.staten[0] = tr0;
        a.staten[1] = stop ? 1.0 : 0.0;
      }
    }
  }
  __syncthreads();
  const int64_t s = pivot;
  if (s >= 0) {
    for (int k = tid; k < i; k += kRpcThreads) xs[k] = double(F[s * ldf + k]);
  }
  __syncthreads();
  double bs = 0.0;  // of row 64 t + 4 wave + g of every pass, lanes t < kRpcSlots
  for (int64_t base = i0; base < i1; base += kRpcRows) {
    const int64_t j = base + 64 * t + 4 * wave + g;
    const bool mine = t < kRpcSlots && j < i1;
    if (s < 0) {
      if (mine) {
        F[j * ldf + i] = 0.f;
        const double dj = a.d[j];
        a.dn[j] = dj;
        bs += dj;
      }
      continue;
    }
    auto kentry = [&](int64_t jj) -> double {
      if (STORED) {
        const size_t off = km.layout == 1 ? pk_offset(s, jj, km.ld) : size_t(s * km.ld + jj);
        if (km.dtype == KQR_BF16)
          return double(__uint_as_float(uint32_t(static_cast<const uint16_t*>(km.K)[off]) << 16));
        return double(static_cast<const float*>(km.K)[off]);
      }
      float dd = pair_dist_dyn(X + s * p, q ? q[s] : 0.f, X + jj * p, q ? q[jj] : 0.f, p, lap != 0);
      if (jj == s) dd = 0.f;
      return double(kexp2(ng * dd));
    };
    const double ks = STORED ? kentry(s) : 1.0;  // from X: exp2(0)
    double kj = 0.0, dj = 0.0;
    if (mine) {
      kj = kentry(j);
      dj = a.d[j];
    }
    double acc[kRpcSlots] = {0.0, 0.0, 0.0, 0.0}, us = 0.0;
    // slot sl of a group holds row 64 sl + 4 wave + g of the pass, so a short
    // last pass leaves every wave the same share; rows past the chunk repeat its last
    const float* rows[kRpcSlots];
#pragma unroll
    for (int sl = 0; sl < kRpcSlots; ++sl) rows[sl] = F + min(base + 64 * sl + 4 * wave + g, i1 - 1) * ldf;
    // (deeper explicit buffering of these loads was slower every time: past 128
    // registers it spills, and 512 threads leave half the waves for the draw's tail)
#pragma unroll 2
    for (int c = t; c < nvec; c += 16) {
      float4 v[kRpcSlots];
#pragma unroll
      for (int sl = 0; sl < kRpcSlots; ++sl) v[sl] = reinterpret_cast<const float4*>(rows[sl])[c];
      const double x0 = xs[4 * c], x1 = xs[4 * c + 1], x2 = xs[4 * c + 2], x3 = xs[4 * c + 3];
#pragma unroll
      for (int sl = 0; sl < kRpcSlots; ++sl) {
        acc[sl] = fma(double(v[sl].x), x0, acc[sl]);
        acc[sl] = fma(double(v[sl].y), x1, acc[sl]);
        acc[sl] = fma(double(v[sl].z), x2, acc[sl]);
        acc[sl] = fma(double(v[sl].w), x3, acc[sl]);
      }
      us = fma(x0, x0, us);
      us = fma(x1, x1, us);
      us = fma(x2, x2, us);
      us = fma(x3, x3, us);
    }
#pragma unroll 1
    for (int c = nvec * 4 + t; c < i; c += 16) {
#pragma unroll
      for (int sl = 0; sl < kRpcSlots; ++sl) acc[sl] = fma(double(rows[sl][c]), xs[c], acc[sl]);
      us = fma(xs[c], xs[c], us);
    }
    us = row16_sum_f64(us);
#pragma unroll
    for (int sl = 0; sl < kRpcSlots; ++sl) acc[sl] = row16_sum_f64(acc[sl]);
    if (mine) {
      const double gs = ks - us;
      const double inv = gs > 0.0 ? 1.0 / sqrt(gs) : 0.0;
      const double uj = t == 0 ? acc[0] : t == 1 ? acc[1] : t == 2 ? acc[2] : acc[3];
      const double f = (kj - uj) * inv;
      F[j * ldf + i] = float(f);
      const double dnew = j == s ? 0.0 : fmax(dj - f * f, 0.0);
      a.dn[j] = dnew;
      bs += dnew;
    }
  }
  if (t < kRpcSlots) part[64 * t + 4 * wave + g] = bs;
  __syncthreads();
  if (tid < 256) {
    double b = part[tid];
    b = wave_sum_f64(b);
    if ((tid & 63) == 0) sh[tid >> 6] = b;
  }
  __syncthreads();
  if (tid == 0) a.bsumn[blockIdx.x] = ((sh[0] + sh[1]) + sh[2]) + sh[3];
}

__global__ void rpc_diag_kernel(const KMat km, int64_t n, double* __restrict__ d) {
  const int64_t j = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (j >= n) return;
  if (!km.K) { d[j] = 1.0; return; }  // k(x, x) = exp(0) for both kernels
  const size_t off = km.layout == 1 ? pk_offset(j, j, km.ld) : size_t(j * km.ld + j);
  if (km.dtype == KQR_BF16)
    d[j] = __uint_as_float(uint32_t(static_cast<const uint16_t*>(km.K)[off]) << 16);
  else
    d[j] = static_cast<const float*>(km.K)[off];
}

Co<std::vector<int64_t>> rpcholesky(KMat km, const float* X, const float* sqn, int64_t n, int p,
                                    KernelSpec ks, int64_t rank, const double* uniforms, float* F, int64_t ldf,
                                    Exec& ex) {
  const hipStream_t st = ex.st;
  std::vector<int64_t> pivots;
  if (rank <= 0 || n <= 0) co_return pivots;
  rank = std::min<int64_t>(rank, n);
  if (rank > 1024) fail(KQR_EINVAL, "RPCholesky rank %lld exceeds 1024", (long long)rank);
  if (ldf & 3) fail(KQR_EINVAL, "RPCholesky: ldf must be a multiple of 4");
  DevBuf d(size_t(2 * n) * sizeof(double)), bsum(2 * kSelBlocks * sizeof(double)), state(4 * sizeof(double));
  DevBuf piv(size_t(rank) * sizeof(int64_t));
  rpc_diag_kernel<<<dim3((unsigned)((n + 255) / 256)), 256, 0, st>>>(km, n, d.as<double>());
  KQR_LAUNCH_CHECK();
  KQR_CHECK_HIP(hipMemsetAsync(state.ptr, 0, 4 * sizeof(double), st));
  const int64_t chunk = (n + kSelBlocks - 1) / kSelBlocks;
  rpc_blocksum_kernel<<<kSelBlocks, 256, 0, st>>>(d.as<double>(), n, chunk, bsum.as<double>());
  KQR_LAUNCH_CHECK();
  const float ng = -float(ks.gamma) * kLog2e;
  const bool lap = ks.kind == KQR_LAPLACIAN;
  for (int64_t i = 0; i < rank; ++i) {
    const int from = int(i & 1), to = 1 - from;
    RpcStep a;
    a.d = d.as<double>() + from * n;
    a.dn = d.as<double>() + to * n;
    a.bsum = bsum.as<double>() + from * kSelBlocks;
    a.bsumn = bsum.as<double>() + to * kSelBlocks;
    a.state = state.as<double>() + 2 * from;
    a.staten = state.as<double>() + 2 * to;
    a.piv = piv.as<int64_t>();
    a.chunk = chunk;
    a.u = uniforms[i];
    if (km.K)
      rpc_step_kernel<true><<<kSelBlocks, kRpcThreads, 0, st>>>(km, X, nullptr, p, 0, ng, F, n, ldf, int(i), a);
    else
      rpc_step_kernel<false><<<kSelBlocks, kRpcThreads, 0, st>>>(km, X, lap ? nullptr : sqn, p, lap ? 1 : 0, ng, F, n,
                                                                 ldf, int(i), a);
    KQR_LAUNCH_CHECK();
  }
  std::vector<int64_t> h(size_t(rank), -1);
  co_await read_back(ex, piv.ptr, size_t(rank) * sizeof(int64_t), h.data());
  for (int64_t i = 0; i < rank; ++i) {
    if (h[size_t(i)] < 0) break;
    pivots.push_back(h[size_t(i)]);
  }
  co_return pivots;
}

// ================================================================= rank heuristic
// Householder tridiagonalisation of the symmetric m x m matrix whose lower
// triangle is G (ld ldg), in one workgroup; A is m x m scratch.  Writes the
// diagonal dg[m] and the off-diagonal eg[m-1].
__global__ __launch_bounds__(1024) void tridiag_kernel(const double* __restrict__ G, int64_t ldg, int m,
                                                       double* __restrict__ A, double* __restrict__ v,
                                                       double* __restrict__ w, double* __restrict__ dg,
                                                       double* __restrict__ eg) {
  __shared__ double red[32];
  __shared__ double bc[4];
  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63, wid = tid >> 6, nw = nt >> 6;
  auto block_sum = [&](double x) -> double {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    __syncthreads();
    if (lane == 0) red[wid] = x;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < nw; ++k) s += red[k];
    return s;
  };
  for (int64_t e = tid; e < int64_t(m) * m; e += nt) {
    const int i = int(e / m), j = int(e % m);
    A[e] = i >= j ? G[int64_t(i) * ldg + j] : G[int64_t(j) * ldg + i];
  }
  __syncthreads();
  for (int k = 0; k + 2 < m; ++k) {
    const int len = m - k - 1;  // trailing size
    double* col = A + int64_t(k + 1) * m + k;  // A[k+1+i][k], stride m
    double part = 0.0;
    for (int i = tid; i < len; i += nt) {
      const double x = col[int64_t(i) * m];
      part = fma(x, x, part);
    }
    const double xx = block_sum(part);
    const double x0 = col[0];
    if (tid == 0) dg[k] = A[int64_t(k) * m + k];
    if (!(xx > 0.0)) {
      if (tid == 0) eg[k] = 0.0;
      __syncthreads();
      continue;
    }
    const double alpha = x0 >= 0.0 ? -sqrt(xx) : sqrt(xx);
    const double vv = 2.0 * (xx - x0 * alpha);  // ||x - alpha e1||^2
    for (int i = tid; i < len; i += nt) v[i] = col[int64_t(i) * m] - (i == 0 ? alpha : 0.0);
    if (tid == 0) eg[k] = alpha;
    __syncthreads();
    // p = (2 / vv) A22 v  (one wave per row)
    const double* A22 = A + int64_t(k + 1) * m + (k + 1);
    for (int i = wid; i < len; i += nw) {
      const double* row = A22 + int64_t(i) * m;
      double s = 0.0;
      for (int j = lane; j < len; j += 64) s = fma(row[j], v[j], s);
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
      if (lane == 0) w[i] = s * (2.0 / vv);
    }
    __syncthreads();
    part = 0.0;
    for (int i = tid; i < len; i += nt) part = fma(v[i], w[i], part);
    const double Kc = block_sum(part) / vv;
    for (int i = tid; i < len; i += nt) w[i] = w[i] - Kc * v[i];
    __syncthreads();
    // A22 -= v w^T + w v^T
    double* A22w = A + int64_t(k + 1) * m + (k + 1);
    for (int64_t e = tid; e < int64_t(len) * len; e += nt) {
      const int i = int(e / len), j = int(e % len);
      A22w[int64_t(i) * m + j] -= v[i] * w[j] + w[i] * v[j];
    }
    __syncthreads();
  }
  if (tid == 0) {
    if (m >= 2) {
      dg[m - 2] = A[int64_t(m - 2) * m + (m - 2)];
      eg[m - 2] = A[int64_t(m - 1) * m + (m - 2)];
    }
    dg[m - 1] = A[int64_t(m - 1) * m + (m - 1)];
  }
  (void)bc;
}

// The same for m <= kTriRegs with the matrix in registers (kTriRegs^2 doubles
// are 392 of the 512 KB of vector registers of a CU): thread (ti, tj) of a
// 16 x 32 grid holds A[ti + 16 a][tj + 32 b].  Per step, row k goes through LDS
// to every thread, each thread multiplies its block of the trailing matrix by
// its seven entries of v, the row sums are added over the 32 tj lanes by
// halving exchanges (16 of them for 14 rows), and the rank-two update stays in
// registers.  The sums of squares and v . p are formed by every wave alike, so
// a step has two barriers.  The step loop is instantiated per 32-row block of
// the front, which fixes the live register blocks.  Bound by the chain of one
// step (two barriers, one square root, one division, four LDS round trips);
// m = 224: 4443 us with the matrix streamed from L2 in each step (1.2 MB through
// one CU), 476 us here (256 registers, nine of them spilled).  Beyond
// kTriRegs the streamed form takes over at once: 4.4 ms at m = 225.
constexpr int kTriRegs = 224;
constexpr int kTriThreads = 512;

__global__ __launch_bounds__(kTriThreads) void tridiag_regs_kernel(const double* __restrict__ G, int64_t ldg, int m,
                                                                   double* __restrict__ dg, double* __restrict__ eg) {
  constexpr int NA = kTriRegs / 16, NB = kTriRegs / 32;
  __shared__ double col[2][256];  // row k, by the parity of k
  __shared__ double pw[2][256];   // p = (2 / vv) A22 v
  const int tid = threadIdx.x, lane = tid & 63;
  const int ti = tid >> 5, tj = tid & 31;
  double A[NA][NB];
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = ti + 16 * a, j = tj + 32 * b;
      const int ic = min(max(i, j), m - 1), jc = min(min(i, j), m - 1);
      const double g = G[int64_t(ic) * ldg + jc];
      A[a][b] = i < m && j < m ? g : 0.0;
    }
  for (int e = tid; e < 512; e += kTriThreads) {
    col[e >> 8][e & 255] = 0.0;
    pw[e >> 8][e & 255] = 0.0;
  }
  __syncthreads();
  auto front = [&](auto kb_c) {
    constexpr int KB = decltype(kb_c)::value;
    for (int kk = 0; kk < 32; ++kk) {
      const int k = 32 * KB + kk;
      if (k + 2 >= m) return;
      double* c = col[k & 1];
      double* pb = pw[k & 1];
      if (ti == (kk & 15)) {  // row k: register row 2 KB or 2 KB + 1
        if (kk < 16) {
#pragma unroll
          for (int b = KB; b < NB; ++b) c[tj + 32 * b] = A[2 * KB][b];
        } else {
#pragma unroll
          for (int b = KB; b < NB; ++b) c[tj + 32 * b] = A[2 * KB + 1][b];
        }
      }
      __syncthreads();
      // x = row k right of the diagonal (zero past m); every wave forms ||x||^2
      double x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = lane + 64 * q;
        const double t = c[j];
        x[q] = j > k ? t : 0.0;
      }
      const double xx = wave_sum_f64(fma(x[3], x[3], fma(x[2], x[2], fma(x[1], x[1], x[0] * x[0]))));
      const double x0 = c[k + 1];
      if (tid == 0) dg[k] = c[k];
      if (!(xx > 0.0)) {  // the same in every thread
        if (tid == 0) eg[k] = 0.0;
        continue;
      }
      const double alpha = x0 >= 0.0 ? -sqrt(xx) : sqrt(xx);
      const double inv = 1.0 / (2.0 * (xx - x0 * alpha));  // 1 / ||x - alpha e1||^2
      if (tid == 0) eg[k] = alpha;
      auto v_at = [&](int j) {
        const double t = c[j];
        return j <= k ? 0.0 : (j == k + 1 ? t - alpha : t);
      };
      double vc[NB];
#pragma unroll
      for (int b = KB; b < NB; ++b) vc[b] = v_at(tj + 32 * b);
      auto row_part = [&](int a) {  // this thread's part of the product of row ti + 16 a
        double t = 0.0;
        if (a >= 2 * KB && a < NA) {
#pragma unroll
          for (int b = KB; b < NB; ++b) t = fma(A[a][b], vc[b], t);
        }
        return t;
      };
      // sum over tj: each exchange halves the rows a lane carries; the lane ends
      // with row a = 8 bit4 + 4 bit3 + 2 bit2 + bit0 of its lane number
      double s[8];
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const uint64_t u = __builtin_bit_cast(uint64_t, row_part(a)), w = __builtin_bit_cast(uint64_t, row_part(a + 8));
        const auto l = __builtin_amdgcn_permlane16_swap(uint32_t(u), uint32_t(w), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(uint32_t(u >> 32), uint32_t(w >> 32), false, false);
        s[a] = __builtin_bit_cast(double, (uint64_t(h[0]) << 32) | l[0]) +
               __builtin_bit_cast(double, (uint64_t(h[1]) << 32) | l[1]);
      }
      const bool b3 = lane & 8, b2 = lane & 4, b0 = lane & 1;
#pragma unroll
      for (int a = 0; a < 4; ++a) s[a] = (b3 ? s[a + 4] : s[a]) + dpp_f64<0x128>(b3 ? s[a] : s[a + 4]);
#pragma unroll
      for (int a = 0; a < 2; ++a) s[a] = (b2 ? s[a + 2] : s[a]) + dpp_f64<0x141>(b2 ? s[a] : s[a + 2]);
      double p = (b0 ? s[1] : s[0]) + dpp_f64<0xB1>(b0 ? s[0] : s[1]);
      p += dpp_f64<0x4E>(p);
      const int arow = ((lane >> 1) & 8) | ((lane >> 1) & 4) | ((lane >> 1) & 2) | (lane & 1);
      if (!(lane & 2) && arow >= 2 * KB && arow < NA) pb[ti + 16 * arow] = (2.0 * inv) * p;
      __syncthreads();
      // w = p - Kc v with Kc = (v . p) / ||v||^2, formed by every wave
      double dot = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = lane + 64 * q;
        dot = fma(j == k + 1 ? x[q] - alpha : x[q], pb[j], dot);
      }
      const double Kc = wave_sum_f64(dot) * inv;
      double wc[NB];
#pragma unroll
      for (int b = KB; b < NB; ++b) {
        const int j = tj + 32 * b;
        const double t = pb[j];
        wc[b] = j > k ? fma(-Kc, vc[b], t) : 0.0;
      }
      // A22 -= v w^T + w v^T
#pragma unroll
      for (int a = 2 * KB; a < NA; ++a) {
        const int i = ti + 16 * a;
        const double vr = v_at(i);
        const double t = pb[i];
        const double wr = i > k ? fma(-Kc, vr, t) : 0.0;
#pragma unroll
        for (int b = KB; b < NB; ++b) A[a][b] = fma(-vr, wc[b], fma(-wr, vc[b], A[a][b]));
      }
    }
  };
  front(std::integral_constant<int, 0>{});
  front(std::integral_constant<int, 1>{});
  front(std::integral_constant<int, 2>{});
  front(std::integral_constant<int, 3>{});
  front(std::integral_constant<int, 4>{});
  front(std::integral_constant<int, 5>{});
  front(std::integral_constant<int, 6>{});
#pragma unroll
  for (int a = 0; a < NA; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int i = ti + 16 * a, j = tj + 32 * b;
      if (i == j && i < m && i + 2 >= m) dg[i] = A[a][b];
      if (i == m - 1 && j == m - 2) eg[j] = A[a][b];
    }
}

// Number of eigenvalues below x of the symmetric tridiagonal with diagonal d
// and squared off-diagonal e2 (Sturm count), entries of magnitude at most
// about 1.  The quotient is v_rcp_f64 and two Newton steps times e^2, joined
// with the sum in one FMA (|q| >= 1e-18, so nothing overflows): the reciprocal
// is correctly rounded in 99.98 % of 4 million values and off by 0.5000 units in the last
// place at most, and its product is exact inside the FMA, so a quotient is off
// by 0.9993 2^-53 of itself at most (0.37 on average), as a rounded division
// (0.9997 and 0.36).  In this serial chain it takes 99 us at m = 224 where the
// division takes 115.
__device__ __forceinline__ int sturm_below(const double* d, const double* e2, int m, double x) {
  constexpr double tiny = 1e-18;
  double q = d[0] - x;
  int c = q < 0.0;
  for (int i = 1; i < m; ++i) {
    if (fabs(q) < tiny) q = -tiny;
    double y = __builtin_amdgcn_rcp(q);
    y = fma(fma(-q, y, 1.0), y, y);
    y = fma(fma(-q, y, 1.0), y, y);
    q = fma(-e2[i - 1], y, d[i] - x);
    c += q < 0.0;
  }
  return c;
}

// out[0] = r (as double), out[1] = lambda_1.  One workgroup: each of the 256
// threads counts at its own point, so a pass cuts the interval of lambda_1 by
// 257 (seven passes over the recurrence where bisection takes about fifty).
// m = 224: 1065 us by bisection in one thread, 99 us here.
__global__ __launch_bounds__(256) void rank_from_tridiag_kernel(const double* __restrict__ dg,
                                                                const double* __restrict__ eg, int m, double xi,
                                                                double* __restrict__ out) {
  __shared__ double d[1024], e2[1024];
  __shared__ double red[3][256];
  __shared__ int first[4];
  const int t = threadIdx.x;
  // Gershgorin bounds and the largest diagonal entry (lambda_1 is at least that)
  double lo = 0.0, hi = 0.0, top = -INFINITY;
  for (int i = t; i < m; i += 256) {
    const double di = dg[i];
    const double rad = (i > 0 ? fabs(eg[i - 1]) : 0.0) + (i + 1 < m ? fabs(eg[i]) : 0.0);
    lo = fmin(lo, di - rad);
    hi = fmax(hi, di + rad);
    top = fmax(top, di);
  }
  red[0][t] = lo;
  red[1][t] = hi;
  red[2][t] = top;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {
    if (t < off) {
      red[0][t] = fmin(red[0][t], red[0][t + off]);
      red[1][t] = fmax(red[1][t], red[1][t + off]);
      red[2][t] = fmax(red[2][t], red[2][t + off]);
    }
    __syncthreads();
  }
  lo = red[0][0];
  hi = red[1][0];
  top = red[2][0];
  // scaled by a power of two (exact) so that the largest bound is in [1, 2)
  const double big = fmax(fabs(lo), fabs(hi));
  const int ex = big > 0.0 && isfinite(big) ? ilogb(big) : 0;
  for (int i = t; i < m; i += 256) {
    d[i] = ldexp(dg[i], -ex);
    if (i + 1 < m) {
      const double e = ldexp(eg[i], -ex);
      e2[i] = e * e;
    }
  }
  __syncthreads();
  double a = fmax(ldexp(lo, -ex), ldexp(top, -ex)), b = ldexp(hi, -ex);
  for (int it = 0; it < 40 && b - a > 1e-15 * fmax(fabs(a), fabs(b)); ++it) {
    const double h = (b - a) / 257.0;
    const double x = fma(double(t + 1), h, a);
    const unsigned long long hit = __ballot(sturm_below(d, e2, m, x) >= m);  // x at or above lambda_1
    if ((t & 63) == 0) first[t >> 6] = hit ? __ffsll((long long)hit) - 1 : 64;
    __syncthreads();
    int f = 256;
    for (int w = 3; w >= 0; --w)
      if (first[w] < 64) f = 64 * w + first[w];
    const double nb = f < 256 ? fma(double(f + 1), h, a) : b;
    const double na = f > 0 ? fma(double(f), h, a) : a;
    __syncthreads();
    if (na == a && nb == b) break;  // the same in every thread
    a = na;
    b = nb;
  }
  if (t == 0) {
    const int below = sturm_below(d, e2, m, xi * b);  // #{lambda < xi lambda_1}
    out[0] = double(min(m - below + 1, m));           // smallest r with lambda_r <= xi lambda_1
    out[1] = ldexp(b, ex);
  }
}

Co<int64_t> adaptive_rank(const float* F0, int64_t n, int64_t r0, int64_t ldf, double xi, Exec& ex,
                          double* lambda1_out) {
  const hipStream_t st = ex.st;
  if (r0 <= 1) co_return r0;
  Woodbury W(F0, n, r0, ldf);
  const double* G = W.gram(st);  // (r0+1)^2 lower triangle of [F0 1]^T [F0 1]
  const int m = int(r0);
  DevBuf dg(size_t(m) * sizeof(double)), eg(size_t(m) * sizeof(double)), out(2 * sizeof(double));
  DevBuf A, v, w;
  if (m <= kTriRegs) {
    tridiag_regs_kernel<<<1, kTriThreads, 0, st>>>(G, r0 + 1, m, dg.as<double>(), eg.as<double>());
  } else {  // more than the registers hold
    A.alloc(size_t(m) * m * sizeof(double));
    v.alloc(size_t(m) * sizeof(double));
    w.alloc(size_t(m) * sizeof(double));
    tridiag_kernel<<<1, 1024, 0, st>>>(G, r0 + 1, m, A.as<double>(), v.as<double>(), w.as<double>(), dg.as<double>(),
                                       eg.as<double>());
  }
  KQR_LAUNCH_CHECK();
  rank_from_tridiag_kernel<<<1, 256, 0, st>>>(dg.as<double>(), eg.as<double>(), m, xi, out.as<double>());
  KQR_LAUNCH_CHECK();
  double h[2];
  co_await read_back(ex, out.ptr, 2 * sizeof(double), h);
  if (lambda1_out) *lambda1_out = h[1];
  co_return int64_t(h[0]);
}

}  // namespace kqr
