// Backward of the mined alignment score through the NW DP and the logistic
// scorer (drives the tuning of threshold and penalty, Sec. 5.2).
//
// The NW score of a pair is a maximum of affine path sums
//   sum_{aligned (i,j)} S[i][j] + gap * (number of gap steps),
// so where the optimal path is unique its gradient is the path's DIAG
// indicator P for S and the gap count G = n + m - 2k for gap.  Chained through
// S = sigmoid(z), z = w0 S_raw + w1 rho + b:
//   dL/dz = dL/dS * S (1 - S);  dL/d(w0, w1, b) = sum dL/dz * (S_raw, rho, 1).
//
// k_bwd_dense   the dense chain of grad_S_extra, per row tile in FP32, with
//               grad_S := grad_S_extra; k_bwd_fill where there is no chain:
//               grad_S := grad_S_extra, or 0.
// k_bwd_path    one wave per pair: the path-sparse chain in FP32, grad_S += a_b
//               on the path, per-pair partials (dw0, dw1, db, a_b * G).  Not
//               launched without a score gradient (no path term).  Path cells
//               outside the pair's n x m block are skipped.
// k_bwd_reduce  one block: FP64 sum of all partials in a fixed order.
#include "nwm_internal.h"
#include "libnwmine.h"

namespace nwm {

static __device__ __forceinline__ float wave_sum(float v) {
  // fixed butterfly order: deterministic
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

static __device__ __forceinline__ float rho_of(float ls, float lt) {
  if (ls == 0.0f && lt == 0.0f) return 1.0f;
  return fminf(ls, lt) / fmaxf(ls, lt);
}

// grad_S := E (or 0) over all cells, 16 bytes per access where both start at a
// multiple of 16 bytes (`wide`): 20 M cells zeroed in 40 us by row tiles, 22 so.
__global__ __launch_bounds__(256) void k_bwd_fill(const float *__restrict__ E, float *__restrict__ grad_S,
                                                  int64_t cells, int wide) {
  const int64_t tid = blockIdx.x * (int64_t)256 + threadIdx.x, nthr = (int64_t)gridDim.x * 256;
  int64_t done = 0;
  if (wide) {
    const float4 *from = reinterpret_cast<const float4 *>(E);
    float4 *to = reinterpret_cast<float4 *>(grad_S);
    for (int64_t k = tid; k < cells / 4; k += nthr) to[k] = E ? from[k] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    done = cells / 4 * 4;
  }
  for (int64_t k = done + tid; k < cells; k += nthr) grad_S[k] = E ? E[k] : 0.0f;
}

// The dense chain of E (and grad_S := E) over one row tile.  Bound by memory:
// 12 bytes read and 4 written per cell.  Thread t takes cells t, t + 256, ...
// in order, BWD_CELLS of them in flight at once, and the sentences' lengths come
// from LDS (columns past BWD_LEN: from memory).  One cell at a time with a 64-bit
// division and four offset loads each, a tuning step's 1024 pairs took 193 us,
// 117 so; the sums are the same, in the same order.
constexpr int BWD_CELLS = 8;
constexpr int BWD_LEN = 2048;   // columns whose lengths LDS holds
__global__ __launch_bounds__(256) void k_bwd_dense(PlanDev P, const int64_t *__restrict__ src_off,
                                                   const int64_t *__restrict__ tgt_off,
                                                   const float *__restrict__ E, const float *__restrict__ S,
                                                   const float *__restrict__ S_raw, float *__restrict__ grad_S,
                                                   float *__restrict__ part) {
  __shared__ float red[3][256];
  __shared__ float2 rl[TM], cl[BWD_LEN];   // length and its reciprocal
  const int rt = blockIdx.x;
  const int pair = P.rt_pair[rt];
  const int row0 = P.rt_row0[rt], rows = P.rt_rows[rt];
  const int m = P.m[pair];
  if (m == 0) {   // an empty target side: no cells (and nothing to divide by)
    if (threadIdx.x < 3) part[4 * rt + threadIdx.x] = 0.0f;
    return;
  }
  const int64_t s_first = P.sfirst[pair] + row0;
  const int64_t t_first = P.tfirst[pair];
  const int64_t base = P.s_off[pair] + (int64_t)row0 * m;
  auto length = [](const int64_t *off, int64_t k) {
    const float l = (float)(off[k + 1] - off[k]);
    return make_float2(l, 1.0f / l);
  };
  for (int r = threadIdx.x; r < rows; r += 256) rl[r] = length(src_off, s_first + r);
  for (int j = threadIdx.x; j < min(m, BWD_LEN); j += 256) cl[j] = length(tgt_off, t_first + j);
  __syncthreads();
  float g0 = 0.f, g1 = 0.f, gb = 0.f;
  const int cells = rows * m;
  const int dr = 256 / m, dj = 256 % m;   // from a thread's cell to its next
  int r = (int)threadIdx.x / m, j = (int)threadIdx.x % m;
  for (int c0 = threadIdx.x; c0 < cells; c0 += 256 * BWD_CELLS) {
    float e[BWD_CELLS], s[BWD_CELLS], x[BWD_CELLS];
#pragma unroll
    for (int u = 0; u < BWD_CELLS; ++u) {
      const int c = c0 + 256 * u;
      const bool on = c < cells;
      e[u] = on ? E[base + c] : 0.0f;
      s[u] = on ? S[base + c] : 0.0f;
      x[u] = on ? S_raw[base + c] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < BWD_CELLS; ++u) {
      const int c = c0 + 256 * u;
      if (c < cells) {
        if (grad_S) grad_S[base + c] = e[u];
        const float2 ls = rl[r], lt = j < BWD_LEN ? cl[j] : length(tgt_off, t_first + j);
        // min / max of the lengths: the quotient by the (correctly rounded)
        // reciprocal and one correction of it is the correctly rounded one
        const bool less = ls.x < lt.x;
        const float a = less ? ls.x : lt.x, b = less ? lt.x : ls.x, rb = less ? lt.y : ls.y;
        const float q = a * rb;
        const float rho = b == 0.0f ? 1.0f : fmaf(fmaf(-q, b, a), rb, q);
        const float dz = e[u] * s[u] * (1.0f - s[u]);
        g0 += dz * x[u];
        g1 += dz * rho;
        gb += dz;
      }
      r += dr;
      j += dj;
      if (j >= m) j -= m, ++r;
    }
  }
  red[0][threadIdx.x] = g0;
  red[1][threadIdx.x] = g1;
  red[2][threadIdx.x] = gb;
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if (threadIdx.x < d)
      for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int q = 0; q < 3; ++q) part[4 * rt + q] = red[q][0];
}

__global__ __launch_bounds__(64) void k_bwd_path(PlanDev P, const int64_t *__restrict__ src_off,
                                                 const int64_t *__restrict__ tgt_off,
                                                 const int2 *__restrict__ path, const int32_t *__restrict__ n_diag,
                                                 const float *__restrict__ grad_score, const float *__restrict__ S,
                                                 const float *__restrict__ S_raw, float *__restrict__ grad_S,
                                                 float *__restrict__ part, int want_wb) {
  const int b = blockIdx.x;
  const int n = P.n[b], m = P.m[b];
  const int lane = threadIdx.x;
  const int cap = min(n, m);
  const int k = min(n_diag[b], cap);
  const float a = grad_score[b];
  const int2 *pa = path + P.p_off[b] + (cap - k);
  const int64_t base = P.s_off[b];
  float g0 = 0.f, g1 = 0.f, gb = 0.f;
  // 256 path cells per round, so that a lane's loads are in flight together
  // (1024 pairs of up to 1000 sentences: 14.8 -> 13.9 us, with the chain 21.3 ->
  // 20.7); every lane's cells keep their order
  constexpr int U = 4;
  for (int q0 = 0; q0 < k; q0 += 64 * U) {
    int2 c[U];
    bool ok[U];
    int64_t o[U];
    float s[U], x[U], old[U], ls[U], lt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + 64 * u + lane;
      c[u] = q < k ? pa[q] : make_int2(-1, -1);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      ok[u] = (unsigned)c[u].x < (unsigned)n && (unsigned)c[u].y < (unsigned)m;
      o[u] = base + (int64_t)c[u].x * m + c[u].y;
      s[u] = x[u] = old[u] = ls[u] = lt[u] = 0.0f;
      if (!ok[u]) continue;
      if (grad_S) old[u] = grad_S[o[u]];
      if (want_wb) {
        s[u] = S[o[u]];
        x[u] = S_raw[o[u]];
        ls[u] = (float)(src_off[P.sfirst[b] + c[u].x + 1] - src_off[P.sfirst[b] + c[u].x]);
        lt[u] = (float)(tgt_off[P.tfirst[b] + c[u].y + 1] - tgt_off[P.tfirst[b] + c[u].y]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (!ok[u]) continue;
      if (grad_S) grad_S[o[u]] = old[u] + a;
      if (want_wb) {
        const float dz = a * s[u] * (1.0f - s[u]);
        g0 += dz * x[u];
        g1 += dz * rho_of(ls[u], lt[u]);
        gb += dz;
      }
    }
  }
  g0 = wave_sum(g0);
  g1 = wave_sum(g1);
  gb = wave_sum(gb);
  if (lane == 0) {
    part[4 * b + 0] = g0;
    part[4 * b + 1] = g1;
    part[4 * b + 2] = gb;
    part[4 * b + 3] = a * (float)(n + m - 2 * k);
  }
}

__global__ __launch_bounds__(256) void k_bwd_reduce(int n_path, const float *__restrict__ part_path, int n_dense,
                                                    const float *__restrict__ part_dense,
                                                    double *__restrict__ grad_gap, double *__restrict__ grad_wb) {
  __shared__ double red[4][256];
  double v[4] = {0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < n_path; b += 256)
    for (int q = 0; q < 4; ++q) v[q] += (double)part_path[4 * b + q];
  for (int r = threadIdx.x; r < n_dense; r += 256)
    for (int q = 0; q < 3; ++q) v[q] += (double)part_dense[4 * r + q];
  for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int d = 128; d >= 1; d >>= 1) {
    if (threadIdx.x < d)
      for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + d];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    if (grad_wb) {
      grad_wb[0] = red[0][0];
      grad_wb[1] = red[1][0];
      grad_wb[2] = red[2][0];
    }
    if (grad_gap) grad_gap[0] = red[3][0];
  }
}

hipError_t launch_backward(const PlanDev &P, const int64_t *src_off, const int64_t *tgt_off, const int2 *path,
                           const int32_t *n_diag, const float *grad_score, const float *E, float *grad_S,
                           double *grad_gap, const float *S, const float *S_raw, double *grad_wb,
                           float *part_path, float *part_dense, int64_t cells, hipStream_t st) {
  if (P.B <= 0) return hipSuccess;
  const int want_wb = grad_wb != nullptr;
  const bool chain = E != nullptr && want_wb;
  if (chain && P.n_rt > 0) {
    hipLaunchKernelGGL(k_bwd_dense, dim3(P.n_rt), dim3(256), 0, st, P, src_off, tgt_off, E, S, S_raw, grad_S,
                       part_dense);
  } else if (grad_S && cells > 0) {
    const int wide = (((uintptr_t)E | (uintptr_t)grad_S) & 15) == 0;
    const int64_t blocks = (cells + 1023) / 1024;
    hipLaunchKernelGGL(k_bwd_fill, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(256), 0, st, E, grad_S, cells,
                       wide);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // without a score gradient there is no path term (tb and n_diag unused)
  const int n_path = grad_score ? P.B : 0;
  if (n_path > 0) {
    hipLaunchKernelGGL(k_bwd_path, dim3(P.B), dim3(64), 0, st, P, src_off, tgt_off, path, n_diag, grad_score, S,
                       S_raw, grad_S, part_path, want_wb);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int nd = chain ? P.n_rt : 0;
  hipLaunchKernelGGL(k_bwd_reduce, dim3(1), dim3(256), 0, st, n_path, part_path, nd, part_dense, grad_gap, grad_wb);
  return hipGetLastError();
}

}  // namespace nwm
