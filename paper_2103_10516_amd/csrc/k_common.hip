// Small FP64 kernels of libmlct: Chebyshev coefficients (type-I DCT),
// CSR structure validation, fixed-order reduction of moment partials,
// assembly of the moment table, and the multilevel level combination.
#include <cmath>

#include "device.hpp"

namespace mlct {

namespace {

// Coefficients of the degree-n interpolant at x_k = cos(k pi / n)
// (Section 2.2): c_j = (2/n) sum''_k f~(x_k) cos(pi (j k mod 2n) / n), with
// the end terms of the sum and c_0, c_n halved.  For exp the factor
// exp((a+b)/2) is returned separately as a log-scale.  The angle index
// r = j k mod 2n is folded to [0, n/2] (cos(2 pi - t) = cos t,
// cos(pi - t) = -cos t), so each workgroup evaluates n/2 + 1 cosines once
// into LDS; workgroup w computes c_j for j = 256 w .. 256 w + 255, each as
// one sequential sum over k with the index advanced by additions.
__device__ __forceinline__ void cheb_dct_wg(int kind, double power, double a, double b, int n,
                                            double* __restrict__ c,
                                            double* __restrict__ log_scale, double* lds) {
  double* fk = lds;              // n + 1 samples
  double* cs = lds + (n + 1);    // cos(pi r / n), r = 0 .. n/2
  const double half = 0.5 * (b - a), mid = 0.5 * (a + b);
  const int nh = n / 2;
  for (int k = threadIdx.x; k <= n; k += blockDim.x) {
    const double x = cos(M_PI * (double)k / (double)n);
    fk[k] = (kind == MLCT_EXP) ? exp(half * x) : eval_f(kind, power, half * x + mid);
  }
  for (int r = threadIdx.x; r <= nh; r += blockDim.x) cs[r] = cos(M_PI * (double)r / (double)n);
  __syncthreads();
  const int two_n = 2 * n;
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j <= n) {
    double s = 0.0;
    int jk = 0;  // j k mod 2n, advanced by j each step (j <= n < 2n)
    // (unrolled: the LDS reads of eight terms are in flight at once; n = 256
    // in 34 us one term at a time)
#pragma unroll 8
    for (int k = 0; k <= n; ++k) {
      const int r = jk > n ? two_n - jk : jk;
      jk += j;
      if (jk >= two_n) jk -= two_n;
      const double cr = (r <= nh) ? cs[r] : -cs[n - r];
      const double w = (k == 0 || k == n) ? 0.5 : 1.0;
      s += w * fk[k] * cr;
    }
    s *= 2.0 / (double)n;
    if (j == 0 || j == n) s *= 0.5;
    c[j] = s;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && log_scale) *log_scale = (kind == MLCT_EXP) ? mid : 0.0;
}

__global__ __launch_bounds__(256) void cheb_dct_kernel(int kind, double power, double a,
                                                       double b, int n, double* __restrict__ c,
                                                       double* __restrict__ log_scale) {
  extern __shared__ double lds[];
  cheb_dct_wg(kind, power, a, b, n, c, log_scale, lds);
}

// The items of a batch (blockIdx.y), each with one interpolant.
__global__ __launch_bounds__(256) void cheb_dct_batched_kernel(
    const BatchItemPost* __restrict__ items) {
  extern __shared__ double lds[];
  const BatchItemPost& it = items[blockIdx.y];
  if ((int)blockIdx.x * 256 > it.n) return;
  cheb_dct_wg(it.kind, it.power, it.a, it.b, it.n, it.coef, it.coef + it.n + 1, lds);
}

// flags[0]: bit0 rowptr[0] != 0, bit1 decreasing rowptr, bit2 rowptr[d] != nnz,
// bit3 column out of range.  flags[1]: longest row.
__global__ void csr_validate_kernel(const int32_t* __restrict__ rowptr,
                                    const int32_t* __restrict__ col, int64_t d, int64_t ncols,
                                    int64_t nnz, int32_t* __restrict__ flags) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  int bad = 0, longest = 0;
  for (int64_t i = tid; i < d; i += stride) {
    const int32_t s = rowptr[i], e = rowptr[i + 1];
    if (e < s) bad |= 2;
    else longest = max(longest, e - s);
  }
  if (tid == 0) {
    if (rowptr[0] != 0) bad |= 1;
    if ((int64_t)rowptr[d] != nnz) bad |= 4;
  }
  for (int64_t t = tid; t < nnz; t += stride) {
    const int32_t j = col[t];
    if (j < 0 || (int64_t)j >= ncols) bad |= 8;
  }
  if (bad) atomicOr(&flags[0], bad);
  if (longest) atomicMax(&flags[1], longest);
}

// dots[s][slot][p] = sum_{g = 0..ngroups-1} part[s][slot][g][p].  One
// workgroup per (s, slot) row and chunk of 64 probes; wave w sums the
// groups g = w, w + 4, w + 8, ... with four interleaved accumulators, and
// the partial sums are combined in a fixed order, so the result does not
// depend on timing.
__device__ __forceinline__ void reduce_row(const double* __restrict__ part, int64_t row,
                                           int chunk, int ngroups, int width,
                                           double* __restrict__ dots) {
  __shared__ double sh[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int p = chunk * 64 + lane;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (p < width) {
    const double* src = part + row * ngroups * width + p;
    int g = wave;
    for (; g + 12 < ngroups; g += 16) {
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] += src[(int64_t)(g + 4 * u) * width];
    }
    for (; g < ngroups; g += 4) acc[0] += src[(int64_t)g * width];
  }
  sh[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  __syncthreads();
  if (wave == 0 && p < width)
    dots[row * width + p] = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
}

__global__ __launch_bounds__(256) void reduce_partials_kernel(const double* __restrict__ part,
                                                              int ngroups, int width,
                                                              double* __restrict__ dots) {
  reduce_row(part, blockIdx.x, blockIdx.y, ngroups, width, dots);
}

// The probe blocks of a batch (blockIdx.y), 64 probes each.
__global__ __launch_bounds__(256) void reduce_batched_kernel(
    const BatchBlockPost* __restrict__ blocks) {
  const BatchBlockPost& b = blocks[blockIdx.y];
  if ((int)blockIdx.x < 2 * (b.steps + 1))
    reduce_row(b.part, blockIdx.x, 0, b.ngroups, 64, b.dots);
}

// Moment table rows from the per-step dot products.
// Direct form: mu_0 = z.z, mu_j = z.v_j.
// Symmetric form: mu_1 = v_1.v_0, mu_2 = 2 v_1.v_1 - mu_0,
// mu_{2s-1} = 2 v_s.v_{s-1} - mu_1 and mu_{2s} = 2 v_s.v_s - mu_0 for s >= 2.
// One thread per (probe, step): each has its own two entries (one thread per
// probe and all steps took 26 us at degree 256, the stores of a wave each to
// another row).
__device__ __forceinline__ void assemble_at(const double* __restrict__ dots, int s, int width,
                                            int p, int mode, int n, double* __restrict__ row) {
  auto D = [&](int st, int slot) { return dots[((int64_t)st * 2 + slot) * width + p]; };
  if (s == 0) {
    row[0] = D(0, 0);
  } else if (mode == MLCT_DIRECT) {
    if (s <= n) row[s] = D(s, 0);
  } else if (s == 1) {
    if (n >= 1) row[1] = D(1, 0);
    if (n >= 2) row[2] = 2.0 * D(1, 1) - D(0, 0);
  } else {
    if (2 * s - 1 <= n) row[2 * s - 1] = 2.0 * D(s, 0) - D(1, 0);
    if (2 * s <= n) row[2 * s] = 2.0 * D(s, 1) - D(0, 0);
  }
}

// blockIdx.x: 64 probes; blockIdx.y: four steps.
__global__ __launch_bounds__(256) void assemble_moments_kernel(const double* __restrict__ dots,
                                                               int steps, int width, int active,
                                                               int mode, int n,
                                                               double* __restrict__ mu,
                                                               int64_t ldmu) {
  const int p = blockIdx.x * 64 + (threadIdx.x & 63);
  const int s = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (p < active && s < steps) assemble_at(dots, s, width, p, mode, n, mu + (int64_t)p * ldmu);
}

__global__ __launch_bounds__(256) void assemble_batched_kernel(
    const BatchBlockPost* __restrict__ blocks, int mode) {
  const BatchBlockPost& b = blocks[blockIdx.y];
  const int p = threadIdx.x & 63;
  const int s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (p < b.active && s <= b.steps)
    assemble_at(b.dots, s, 64, p, mode, b.degree, b.mu + (int64_t)p * b.ldmu);
}

constexpr int kCombThreads = 256;

// Sums and maxima over a team of kCombThreads threads (t: the thread's index
// in it); every team of the workgroup takes part.
__device__ double team_sum_fixed(double v, double* sh, int t) {
  sh[t] = v;
  __syncthreads();
  for (int st = kCombThreads / 2; st > 0; st >>= 1) {
    if (t < st) sh[t] += sh[t + st];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__device__ double team_max(double v, double* sh, int t) {
  sh[t] = v;
  __syncthreads();
  for (int st = kCombThreads / 2; st > 0; st >>= 1) {
    if (t < st) sh[t] = fmax(sh[t], sh[t + st]);
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

// Waves of level k in level_values: one per 64 probes, at most kRatios over all
// levels (each leaves one ratio).
constexpr int kRatios = 3 * MLCT_MAX_LEVELS;
__host__ __device__ inline int level_waves(const LevelDesc& lv, int k) {
  const int64_t units = (lv.m[k] + 63) / 64, most = kRatios / lv.L;
  return (int)(units < most ? units : most);
}

// Level variables (eq. def:qlevels), wave w:
//   Q^{(p)} = sum_{j = l_{k-1}+1}^{l_k} c_j mu_j^{(p)}   (truncation), or
//   Q^{(p)} = z^T p_{l_k} z - z^T p_{l_{k-1}} z          (separate interpolants),
// and the largest |mu_j| / mu_0 of its probes into ratio[w].  A lane sums its
// probe's row in degree order; the rows come through LDS in pieces of 32
// degrees, so that the loads are coalesced (a lane walking its own row took
// 150 us for 3,712 probes).
__device__ void level_values(const double* __restrict__ mu, int64_t ldmu,
                             const double* __restrict__ coef, const LevelDesc& lv, int w,
                             double* __restrict__ q, double* __restrict__ ratio) {
  constexpr int kPiece = 32;
  __shared__ double tile[64][kPiece + 1];
  const int lane = threadIdx.x;
  int k = 0, first_w = 0;
  while (k < lv.L && w - first_w >= level_waves(lv, k)) first_w += level_waves(lv, k++);
  if (k >= lv.L) return;
  const int hi = lv.degree[k];
  const int lo = k ? lv.degree[k - 1] : -1;
  const double* ch = lv.interp ? coef + (int64_t)k * lv.coef_stride : coef;
  const double* cl = (lv.interp && k) ? coef + (int64_t)(k - 1) * lv.coef_stride : nullptr;
  const int j0 = lv.interp ? lv.jmin : max(lo + 1, lv.jmin);
  const int nw = level_waves(lv, k);
  double mr = 0.0;
  for (int64_t u = w - first_w; u * 64 < lv.m[k]; u += nw) {
    const int64_t first = lv.off[k] + u * 64;
    const int np = (int)min<int64_t>(64, lv.m[k] - u * 64);
    double qv = 0.0, ql = 0.0, inv0 = 0.0;
    for (int b = 0; b <= hi; b += kPiece) {
      const int c = min(kPiece, hi + 1 - b);
      for (int e = lane; e < np * kPiece; e += 64) {
        const int p = e / kPiece, j = e % kPiece;
        if (j < c) tile[p][j] = mu[(first + p) * ldmu + b + j];
      }
      __syncthreads();
      if (lane < np) {
        if (b == 0) inv0 = 1.0 / tile[lane][0];
        for (int j = 0; j < c; ++j) {
          const double r = tile[lane][j];
          mr = fmax(mr, fabs(r) * inv0);
          if (b + j >= j0) qv += ch[b + j] * r;
          if (cl && b + j >= j0 && b + j <= lo) ql += cl[b + j] * r;
        }
      }
      __syncthreads();
    }
    if (lane < np) q[first + lane] = cl ? qv - ql : qv;
  }
  for (int o = 32; o > 0; o >>= 1) mr = fmax(mr, __shfl_xor(mr, o, 64));
  if (lane == 0) ratio[w] = mr;
}

// Mean and unbiased variance of every level and the largest ratio, four
// levels at a time (a team of 256 threads each), then the multilevel
// estimator (eq. eqn:multiEstimator): Gamma = sum_k mean_k and its variance
// estimate sum_k s_k^2 / m_k, summed over k in order.
constexpr int kTeams = 4;
__device__ void level_finish(const LevelDesc& lv, const double* __restrict__ coef,
                             const double* __restrict__ log_scale, const double* __restrict__ q,
                             const double* __restrict__ ratio, mlct_result* __restrict__ out) {
  __shared__ double sh[kTeams][kCombThreads];
  __shared__ double st[MLCT_MAX_LEVELS][3];
  const int team = threadIdx.x / kCombThreads, t = threadIdx.x % kCombThreads;
  for (int k0 = 0; k0 < lv.L; k0 += kTeams) {
    const int k = k0 + team;
    const int64_t mk = k < lv.L ? lv.m[k] : 0, o = k < lv.L ? lv.off[k] : 0;
    double s = 0.0, mr = 0.0;
    for (int64_t p = t; p < mk; p += kCombThreads) s += q[o + p];
    if (k < lv.L) {
      int w = 0;
      for (int i = 0; i < k; ++i) w += level_waves(lv, i);
      if (t < level_waves(lv, k)) mr = ratio[w + t];
    }
    const double mean = team_sum_fixed(s, sh[team], t) / (double)mk;
    double ss = 0.0;
    for (int64_t p = t; p < mk; p += kCombThreads) {
      const double dlt = q[o + p] - mean;
      ss += dlt * dlt;
    }
    ss = team_sum_fixed(ss, sh[team], t);
    mr = team_max(mr, sh[team], t);
    if (t == 0 && k < lv.L) {
      st[k][0] = mean;
      st[k][1] = mk > 1 ? ss / (double)(mk - 1) : NAN;
      st[k][2] = mr;
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double v = 0.0, var = 0.0, mr = 0.0;
  uint32_t flags = 0;
  // exact low-degree terms with the top interpolant's coefficients
  const int n = lv.degree[lv.L - 1];
  const double* ctop = lv.interp ? coef + (int64_t)(lv.L - 1) * lv.coef_stride : coef;
  for (int j = 0; j < lv.jmin && j <= n; ++j) v += ctop[j] * lv.low_tr[j];
  for (int k = 0; k < lv.L; ++k) {
    v += st[k][0];
    if (lv.m[k] > 1) var += st[k][1] / (double)lv.m[k];
    else flags |= MLCT_FLAG_FEW_SAMPLES;
    mr = fmax(mr, st[k][2]);
    out->level_mean[k] = st[k][0];
    out->level_var[k] = st[k][1];
  }
  for (int k = lv.L; k < MLCT_MAX_LEVELS; ++k) {
    out->level_mean[k] = 0.0;
    out->level_var[k] = 0.0;
  }
  const double ls = *log_scale;
  const double est = v * exp(ls);
  if (!isfinite(est)) flags |= MLCT_FLAG_OVERFLOW;
  if (flags & MLCT_FLAG_FEW_SAMPLES) var = NAN;
  out->value = v;
  out->log_scale = ls;
  out->estimate = est;
  out->est_var = var;
  out->max_moment_ratio = mr;
  out->flags = flags;
}

__global__ __launch_bounds__(64) void level_values_kernel(const double* __restrict__ mu,
                                                          int64_t ldmu,
                                                          const double* __restrict__ coef,
                                                          LevelDesc lv, double* __restrict__ q,
                                                          double* __restrict__ ratio) {
  level_values(mu, ldmu, coef, lv, blockIdx.x, q, ratio);
}

__global__ __launch_bounds__(kTeams* kCombThreads) void level_finish_kernel(
    LevelDesc lv, const double* __restrict__ coef, const double* __restrict__ log_scale,
    const double* __restrict__ q, const double* __restrict__ ratio,
    mlct_result* __restrict__ out) {
  level_finish(lv, coef, log_scale, q, ratio, out);
}

__global__ __launch_bounds__(64) void level_values_batched_kernel(
    const BatchItemPost* __restrict__ items) {
  const BatchItemPost& it = items[blockIdx.y];
  level_values(it.mu, it.n + 1, it.coef, it.lv, blockIdx.x, it.q, it.ratio);
}

__global__ __launch_bounds__(kTeams* kCombThreads) void level_finish_batched_kernel(
    const BatchItemPost* __restrict__ items, mlct_result* __restrict__ out) {
  const BatchItemPost& it = items[blockIdx.x];
  level_finish(it.lv, it.coef, it.coef + (int64_t)(it.lv.interp ? it.lv.L : 1) * (it.n + 1), it.q,
               it.ratio, out + blockIdx.x);
}

int level_waves_all(const LevelDesc& lv) {
  int w = 0;
  for (int k = 0; k < lv.L; ++k) w += level_waves(lv, k);
  return w;
}

}  // namespace

hipError_t launch_cheb_dct(hipStream_t s, int kind, double power, double a, double b, int n,
                           double* c_dev, double* log_scale_dev) {
  const size_t lds = (size_t)(n + 1 + n / 2 + 1) * sizeof(double);
  cheb_dct_kernel<<<(n + 256) / 256, 256, lds, s>>>(kind, power, a, b, n, c_dev, log_scale_dev);
  return hipGetLastError();
}

hipError_t launch_csr_validate(hipStream_t s, const int32_t* rowptr, const int32_t* col,
                               int64_t d, int64_t ncols, int64_t nnz, int32_t* flags_dev) {
  const int64_t work = d > nnz ? d : nnz;
  int64_t blocks = (work + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  csr_validate_kernel<<<(int)blocks, 256, 0, s>>>(rowptr, col, d, ncols, nnz, flags_dev);
  return hipGetLastError();
}

hipError_t launch_reduce_partials(hipStream_t s, const double* part, int steps, int nslots,
                                  int ngroups, int width, double* dots) {
  const dim3 grid(steps * nslots, (width + 63) / 64);
  reduce_partials_kernel<<<grid, 256, 0, s>>>(part, ngroups, width, dots);
  return hipGetLastError();
}

hipError_t launch_assemble_moments(hipStream_t s, const double* dots, int steps, int width,
                                   int active, int mode, int n, double* mu, int64_t ldmu) {
  const dim3 grid((active + 63) / 64, (steps + 3) / 4);
  assemble_moments_kernel<<<grid, 256, 0, s>>>(dots, steps, width, active, mode, n, mu, ldmu);
  return hipGetLastError();
}

hipError_t launch_level_combine(hipStream_t s, const double* mu, int64_t ldmu,
                                const double* coef, const double* log_scale,
                                const LevelDesc& lv, double* q_dev, double* ratio_dev,
                                mlct_result* result_dev) {
  level_values_kernel<<<level_waves_all(lv), 64, 0, s>>>(mu, ldmu, coef, lv, q_dev, ratio_dev);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  level_finish_kernel<<<1, kTeams * kCombThreads, 0, s>>>(lv, coef, log_scale, q_dev, ratio_dev,
                                                          result_dev);
  return hipGetLastError();
}

hipError_t launch_cheb_dct_batched(hipStream_t s, const BatchItemPost* items, int nitems,
                                   int max_n) {
  const size_t lds = (size_t)(max_n + 1 + max_n / 2 + 1) * sizeof(double);
  cheb_dct_batched_kernel<<<dim3((max_n + 256) / 256, nitems), 256, lds, s>>>(items);
  return hipGetLastError();
}

hipError_t launch_batch_moments(hipStream_t s, const BatchBlockPost* blocks, int nblocks,
                                int max_steps, int mode) {
  reduce_batched_kernel<<<dim3(2 * (max_steps + 1), nblocks), 256, 0, s>>>(blocks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  assemble_batched_kernel<<<dim3((max_steps + 4) / 4, nblocks), 256, 0, s>>>(blocks, mode);
  return hipGetLastError();
}

hipError_t launch_batch_levels(hipStream_t s, const BatchItemPost* items, int nitems,
                               mlct_result* out) {
  level_values_batched_kernel<<<dim3(kRatios, nitems), 64, 0, s>>>(items);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  level_finish_batched_kernel<<<nitems, kTeams * kCombThreads, 0, s>>>(items, out);
  return hipGetLastError();
}

namespace {

constexpr int kST = 256;

// Per-workgroup partial sums of diag(A) and of A_ij^2 over rows g, g + G, ...
// of one workgroup per row block (one thread per row, FP64).
__global__ __launch_bounds__(kST) void op_stats_kernel(const int32_t* __restrict__ rowptr,
                                                       const int32_t* __restrict__ col,
                                                       const float* __restrict__ val,
                                                       const void* __restrict__ A, int dtype,
                                                       int64_t lda, int64_t d,
                                                       double* __restrict__ partial) {
  __shared__ double s1[kST], s2[kST];
  double tr = 0.0, fr = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kST + threadIdx.x; i < d;
       i += (int64_t)gridDim.x * kST) {
    if (rowptr) {
      for (int32_t e = rowptr[i]; e < rowptr[i + 1]; ++e) {
        const double a = val ? (double)val[e] : 1.0;
        if (col[e] == i) tr += a;
        fr += a * a;
      }
    } else {
      for (int64_t j = 0; j < d; ++j) {
        const double a = dtype == MLCT_DT_F64 ? static_cast<const double*>(A)[i * lda + j]
                                              : (double)static_cast<const float*>(A)[i * lda + j];
        if (j == i) tr += a;
        fr += a * a;
      }
    }
  }
  s1[threadIdx.x] = tr;
  s2[threadIdx.x] = fr;
  __syncthreads();
  for (int st = kST / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) {
      s1[threadIdx.x] += s1[threadIdx.x + st];
      s2[threadIdx.x] += s2[threadIdx.x + st];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    partial[2 * blockIdx.x] = s1[0];
    partial[2 * blockIdx.x + 1] = s2[0];
  }
}

__global__ void op_stats_reduce_kernel(const double* __restrict__ partial, int g,
                                       double* __restrict__ out) {
  if (threadIdx.x != 0) return;
  double tr = 0.0, fr = 0.0;
  for (int b = 0; b < g; ++b) {
    tr += partial[2 * b];
    fr += partial[2 * b + 1];
  }
  out[0] = tr;
  out[1] = fr;
}

}  // namespace

hipError_t launch_op_stats(hipStream_t s, const mlct_op* op, double* partial, double* out) {
  const int64_t want = (op->d + kST - 1) / kST;
  const int g = (int)(want < kStatsGroups ? want : kStatsGroups);
  const bool csr = op->kind == OP_CSR;
  op_stats_kernel<<<g, kST, 0, s>>>(csr ? op->csr.rowptr : nullptr, csr ? op->csr.col : nullptr,
                                    csr ? op->csr.val : nullptr, csr ? nullptr : op->A, op->dtype,
                                    op->lda, op->d, partial);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  op_stats_reduce_kernel<<<1, 64, 0, s>>>(partial, g, out);
  return hipGetLastError();
}

}  // namespace mlct
