// Active-set update by MaxVol row swaps (the D-optimality / MaxVol basis of the MTP's
// extrapolation grade; the iteration of Goreinov et al. 2010).
//
// One iteration on the device, candidates C [m][n], active set A [n][n], Ainv = A^-1:
//   1. k_best: every workgroup's first entry (row-major) of largest |(c_i Ainv)_k| over its tiles of 16
//      candidate rows, the product on binary64 matrix cores;
//   2. k_select: the first such entry over the workgroups; g = (c_i Ainv)_k, the row r = c_i Ainv - e_k
//      and the column Ainv[:, k]; decides whether the iteration goes on and logs (i, k, g);
//   3. k_update: Ainv is updated by Sherman-Morrison for replacing row k of A by c_i,
//        Ainv' = Ainv - Ainv[:, k] (r - e_k) / g,
//      and rows A[k] and C[i] are exchanged.
// The kernels of an iteration after the last one return at once, so the host enqueues several
// iterations (twice as many each time) before it reads the log.  5000 candidates of 116 columns:
// 152 us per iteration with one wave per 16 rows, the update in one workgroup and a synchronization
// per iteration; 31 us now (k_best 16.5, k_select 8, k_update 3), bound by the latency of three
// dependent kernels that each read what another chiplet's L2 just wrote.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <string>

#include "mtp.h"
#include "mtp_api_internal.h"
#include "mtp_device.h"
#include "mtp_internal.h"

namespace mtp {
namespace {

constexpr int kRowWaves = 4;      // waves of a workgroup of k_best
constexpr int kColTiles = 2;      // column tiles of 16 a wave accumulates at a time
constexpr int kChunk = 128;       // columns of C staged in LDS at a time
constexpr int kMaxParts = 2048;   // workgroups of k_best (more tiles: several per workgroup)
constexpr int kSelThreads = 1024;
constexpr int kSegments = 8;      // partial sums per entry of r

typedef double v4d __attribute__((ext_vector_type(4)));

// device words that steer the iterations of a call
struct Control {
  int done;       // 0: go on, 1: no entry above 1 + tol, 2: the selected entry is not finite
  int swaps;      // swaps done
  int i, k;       // selection of the current iteration
  double g;
};
struct Log {
  double i, k, g;
};

// (value, row-major index) pair kept by the larger value, then the smaller index
__device__ __forceinline__ void keep_max(double& v, long& k, double v2, long k2) {
  if (v2 > v || (v2 == v && k2 < k)) {
    v = v2;
    k = k2;
  }
}
__device__ __forceinline__ void keep_max_across(double& v, long& k, int s) {
  const double v2 = __shfl_xor(v, s, 64);
  const long k2 = __shfl_xor(k, s, 64);
  keep_max(v, k, v2, k2);
}

// V_MFMA_F64_16X16X4F64 layout (wave64): lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16];
// accumulator register r holds D[4 r + l / 16][l % 16].
// A workgroup takes tiles of 16 rows; its waves share the columns, kColTiles tiles each at a time.
// The rows are staged in LDS (padded by two doubles: the 16 rows of an operand read start in
// different banks); Ainv comes from L2.
__global__ __launch_bounds__(64 * kRowWaves) void k_best(const double* __restrict__ C, int m, int n,
                                                         const double* __restrict__ ainv,
                                                         const Control* __restrict__ ctl, double* __restrict__ pv,
                                                         long* __restrict__ pi) {
  if (ctl->done) return;
  __shared__ double rows[16][kChunk + 2];
  __shared__ double sv[kRowWaves];
  __shared__ long si[kRowWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 15, kq = lane >> 4;
  double best = -1.0;
  long at = 0x7FFFFFFFFFFFFFFFL;
  const int tiles = (m + 15) / 16;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int i0 = tile * 16;
    for (int c0 = 0; c0 < n; c0 += 16 * kColTiles * kRowWaves) {
      const int cw = c0 + 16 * kColTiles * wave;  // first column of this wave
      v4d acc[kColTiles];
#pragma unroll
      for (int t = 0; t < kColTiles; ++t) acc[t] = v4d{0.0, 0.0, 0.0, 0.0};
      for (int k0 = 0; k0 < n; k0 += kChunk) {
        const int kc = min(kChunk, n - k0), kr = (kc + 3) & ~3;  // rounded up: zeros
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 16 / kRowWaves; ++q) {
          const int r = wave * (16 / kRowWaves) + q;
#pragma unroll
          for (int h = 0; h < kChunk / 64; ++h) {
            const int c = h * 64 + lane;
            if (c < kr) rows[r][c] = (i0 + r < m && c < kc) ? C[(long)(i0 + r) * n + k0 + c] : 0.0;
          }
        }
        __syncthreads();
        if (cw < n) {
#pragma unroll 8
          for (int k = 0; k < kr; k += 4) {
            const double av = rows[row][k + kq];
            const long kk = min(k0 + k + kq, n - 1);  // past n the operand from C is zero
#pragma unroll
            for (int t = 0; t < kColTiles; ++t) {
              const double bv = ainv[kk * n + min(cw + 16 * t + row, n - 1)];
              // (not a product of zero and a copy of the last row: that one may be infinite)
              acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, k0 + k + kq < n ? bv : 0.0, acc[t], 0, 0, 0);
            }
          }
        }
      }
#pragma unroll
      for (int t = 0; t < kColTiles; ++t) {
        const int col = cw + 16 * t + row;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + 4 * r + kq;
          // a NaN product counts as the largest magnitude, so that it is selected and reported
          const double v = fabs(acc[t][r]);
          if (col < n && i < m) keep_max(best, at, isnan(v) ? INFINITY : v, (long)i * n + col);
        }
      }
    }
  }
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) keep_max_across(best, at, s);
  if (lane == 0) {
    sv[wave] = best;
    si[wave] = at;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kRowWaves; ++w) keep_max(best, at, sv[w], si[w]);
    pv[blockIdx.x] = best;
    pi[blockIdx.x] = at;
  }
}

// One workgroup: the first largest entry over the parts, r = c_i Ainv - e_k (kSegments partial sums per
// entry, added in order), the column Ainv[:, k], and the decision.  The selected index is in range
// (entry (0, 0) always competes); it is still clamped, with g set to NaN, should that ever fail.
__global__ __launch_bounds__(kSelThreads) void k_select(const double* __restrict__ pv, const long* __restrict__ pi,
                                                        int parts, const double* __restrict__ C, int m, int n,
                                                        const double* __restrict__ ainv, double limit,
                                                        Control* __restrict__ ctl, Log* __restrict__ log,
                                                        double* __restrict__ r, double* __restrict__ colk) {
  if (ctl->done) return;
  constexpr int W = kSelThreads / 64, COLS = kSelThreads / kSegments;
  __shared__ double sv[W];
  __shared__ long si[W];
  __shared__ double seg[kSegments][COLS];
  __shared__ double sg;
  double v = -1.0;
  long id = 0x7FFFFFFFFFFFFFFFL;
  for (int t = threadIdx.x; t < parts; t += kSelThreads) keep_max(v, id, pv[t], pi[t]);
#pragma unroll
  for (int s = 32; s > 0; s >>= 1) keep_max_across(v, id, s);
  if ((threadIdx.x & 63) == 0) {
    sv[threadIdx.x >> 6] = v;
    si[threadIdx.x >> 6] = id;
  }
  __syncthreads();
  v = sv[0];
  id = si[0];
  for (int w = 1; w < W; ++w) keep_max(v, id, sv[w], si[w]);
  const bool ok = id >= 0 && id < (long)m * n;
  const int i = ok ? (int)(id / n) : 0, k = ok ? (int)(id % n) : 0;
  const int part = threadIdx.x / COLS, col = threadIdx.x % COLS;
  const int per = (n + kSegments - 1) / kSegments, lo = min(part * per, n), hi = min(lo + per, n);
  for (int j0 = 0; j0 < n; j0 += COLS) {
    const int j = j0 + col;
    double s = 0.0;
    if (j < n) {
#pragma unroll 8
      for (int t = lo; t < hi; ++t) s = fma(C[(long)i * n + t], ainv[(long)t * n + j], s);
    }
    seg[part][col] = s;
    __syncthreads();
    if (part == 0 && j < n) {
      double sum = seg[0][col];
      for (int q = 1; q < kSegments; ++q) sum += seg[q][col];
      if (j == k) sg = sum;
      r[j] = sum - (j == k ? 1.0 : 0.0);
    }
    __syncthreads();
  }
  for (int j = threadIdx.x; j < n; j += kSelThreads) colk[j] = ainv[(long)j * n + k];
  if (threadIdx.x == 0) {
    const double g = ok ? sg : NAN;
    ctl->i = i;
    ctl->k = k;
    ctl->g = g;
    if (!isfinite(g)) {
      ctl->done = 2;
    } else if (!(fabs(g) > limit)) {
      ctl->done = 1;
    } else {
      *log = Log{(double)i, (double)k, g};
      ctl->swaps += 1;
    }
  }
}

// Ainv -= Ainv[:, k] (r - e_k) / g, one workgroup per row; the first one exchanges rows A[k] and C[i].
__global__ __launch_bounds__(128) void k_update(double* __restrict__ C, double* __restrict__ A,
                                                double* __restrict__ ainv, int n, const Control* __restrict__ ctl,
                                                const double* __restrict__ r, const double* __restrict__ colk) {
  if (ctl->done) return;
  const int a = blockIdx.x;
  const double inv_g = 1.0 / ctl->g, f = colk[a];
  for (int b = threadIdx.x; b < n; b += 128) ainv[(long)a * n + b] -= f * (r[b] * inv_g);
  if (a == 0) {
    const int i = ctl->i, k = ctl->k;
    for (int t = threadIdx.x; t < n; t += 128) {
      const double x = A[(long)k * n + t];
      A[(long)k * n + t] = C[(long)i * n + t];
      C[(long)i * n + t] = x;
    }
  }
}

__global__ void k_start(Control* ctl) { *ctl = Control{0, 0, 0, 0, 0.0}; }

}  // namespace
}  // namespace mtp

using namespace mtp;

extern "C" int mtp_maxvol(mtp_model* m, double* cand, int n_cand, int n, double* active, double* ainv, double tol,
                          int max_swaps, int* swaps, double* grades, int* n_swaps, void* stream) {
  if (!m || !n_swaps) return mtp_fail(MTP_ERR_ARG, "null model or swap count");
  *n_swaps = 0;
  if (n < 1 || n > 4096 || n_cand < 0 || max_swaps < 0 || !(tol >= 0.0))
    return mtp_fail(MTP_ERR_ARG, "mtp_maxvol: need 1 <= n <= 4096, n_cand >= 0, max_swaps >= 0, tol >= 0");
  if (!active || !ainv || (n_cand > 0 && !cand)) return mtp_fail(MTP_ERR_ARG, "null matrix");
  if (n_cand == 0 || max_swaps == 0) return MTP_OK;
  hipStream_t s = (hipStream_t)stream;
  const int tiles = (int)(((long)n_cand + 15) / 16), parts = std::min(tiles, kMaxParts);
  constexpr int kMostAhead = 32;  // iterations enqueued between two reads of the log
  int rc;
  if ((rc = m->scratch.reserve((size_t)parts * 16 + (size_t)n * 16 + kMostAhead * sizeof(Log) + sizeof(Control))))
    return rc;
  double* pv = (double*)m->scratch.p;
  long* pi = (long*)(pv + parts);
  double* r = (double*)(pi + parts);
  double* colk = r + n;
  Log* log = (Log*)(colk + n);
  Control* ctl = (Control*)(log + kMostAhead);
  struct {
    Log log[kMostAhead];
    Control ctl;
  } host;  // as laid out on the device
  static_assert(sizeof(host) == kMostAhead * sizeof(Log) + sizeof(Control), "log and control are contiguous");
  hipLaunchKernelGGL(k_start, dim3(1), dim3(1), 0, s, ctl);
  int ahead = 4;
  for (int it = 0; it < max_swaps;) {
    const int batch = std::min(ahead, max_swaps - it);
    for (int q = 0; q < batch; ++q) {
      hipLaunchKernelGGL(k_best, dim3(parts), dim3(64 * kRowWaves), 0, s, cand, n_cand, n, ainv, ctl, pv, pi);
      hipLaunchKernelGGL(k_select, dim3(1), dim3(kSelThreads), 0, s, pv, pi, parts, cand, n_cand, n, ainv, 1.0 + tol,
                         ctl, log + q, r, colk);
      hipLaunchKernelGGL(k_update, dim3(n), dim3(128), 0, s, cand, active, ainv, n, ctl, r, colk);
    }
    if (hipGetLastError() != hipSuccess) return mtp_fail(MTP_ERR_HIP, "mtp_maxvol: launch failed");
    if (hipMemcpyAsync(&host, log, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return mtp_fail(MTP_ERR_HIP, "mtp_maxvol: reading the selection failed");
    for (int q = 0; it + q < host.ctl.swaps; ++q) {
      if (swaps) {
        swaps[2 * (it + q)] = (int)host.log[q].i;
        swaps[2 * (it + q) + 1] = (int)host.log[q].k;
      }
      if (grades) grades[it + q] = host.log[q].g;
    }
    *n_swaps = host.ctl.swaps;
    if (host.ctl.done == 2)
      return mtp_fail(MTP_ERR_ARG, "mtp_maxvol: non-finite grade (candidates or inverse not finite)");
    if (host.ctl.done) break;
    it += batch;
    ahead = std::min(2 * ahead, kMostAhead);
  }
  return MTP_OK;
}
