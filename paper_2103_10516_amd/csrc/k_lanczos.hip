// Spectral interval [a, b] for the affine map of Section 2.2 by the Lanczos
// process in FP64 (the paper needs only "a rough estimate" of the extreme
// eigenvalues and gives no procedure; this is the library's choice).
//
// Step j (basis Q = [q_0 .. q_j], q_0 = z / |z| for a Rademacher z):
//   w = A q_j;  h = Q^T w;  w -= Q h;  h' = Q^T w;  w -= Q h'  (classical
//   Gram-Schmidt twice: full reorthogonalisation);
//   alpha_j = h_j + h'_j;  beta_j = |w|;  q_{j+1} = w / beta_j.
// All scalars stay on the device; a step after a breakdown (beta_j tiny) is
// a no-op.  A step reads the basis three times: for h, for the first update
// together with h' (each column's piece is kept in registers between the two),
// and for the second update with the norm.  The extreme eigenvalues of the tridiagonal T_k are found by
// Sturm-sequence bisection and the last entries of their eigenvectors by
// inverse iteration, giving the residual bounds |beta_k s_k|.
#include <cmath>

#include "device.hpp"

namespace mlct {

namespace {

constexpr int kT = 256;

// q_0 = z / |z| with z = Rademacher probe 0 of the seed: |z| = sqrt(d).
__global__ void lz_start_kernel(double* __restrict__ q0, int64_t d, uint64_t seed,
                                LanczosState* st) {
  const uint64_t key = sm_output(seed, 0);
  const double inv = 1.0 / sqrt((double)d);
  for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < d;
       n += (int64_t)gridDim.x * blockDim.x)
    q0[n] = sign_from_word<double>(sm_output(key, (uint64_t)(n >> 6)), n) * inv;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->k = 0;
    st->stopped = 0;
  }
}

// Sums over the chunks of the rows longer than kHubLen (the matrix's hub
// table): one wave per chunk of at most kHubChunk entries, FP64.
__global__ __launch_bounds__(256) void lz_hub_chunk_kernel(const int32_t* __restrict__ col,
                                                           const float* __restrict__ val,
                                                           const int32_t* __restrict__ cs,
                                                           const int32_t* __restrict__ ce,
                                                           int nchunks,
                                                           const double* __restrict__ q,
                                                           double* __restrict__ out,
                                                           const LanczosState* st) {
  if (st->stopped) return;
  const int c = blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (c >= nchunks) return;
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  // (64-bit entries: the last chunk may end at INT32_MAX)
  const int64_t e = ce[c];
  for (int64_t t = (int64_t)cs[c] + lane; t < e; t += 64)
    s += (val ? (double)val[t] : 1.0) * q[col[t]];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) out[c] = s;
}

// w = A q (+ shift * qs when qs is given), CSR, FP64 arithmetic on FP32 or
// implicit-1 values: 8 lanes per row and two rows per 8 lanes, so that a wave
// has up to 64 gathers of 8 entries of q under way (16 lanes on one row left
// it waiting: 171 us a product on the graph of 10^6 vertices).  A row's
// entries are strided over its lanes (coalesced index and value loads) and
// added in a fixed shuffle tree; a row longer than kHubLen adds its chunk sums
// (lz_hub_chunk_kernel) in chunk order.
constexpr int kRowLanes = 8;
constexpr int kRowSets = 2;                          // rows per kRowLanes lanes
constexpr int kWaveRows = 64 / kRowLanes * kRowSets;  // rows per wave
constexpr int kGather = 4;                           // entries per lane in flight and row
__global__ __launch_bounds__(kT) void lz_spmv_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, const double* __restrict__ q,
    double* __restrict__ w, double shift, const double* __restrict__ qs,
    const int32_t* __restrict__ hub_rows, const int32_t* __restrict__ hub_c0, int hub_n,
    const double* __restrict__ hub_part, const LanczosState* st) {
  if (st->stopped) return;
  const int lane = threadIdx.x & 63, sub = lane % kRowLanes;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i0 = wave * kWaveRows; i0 < d; i0 += nw * kWaveRows) {  // uniform over the wave
    // t counts from the row's start: a finished row's goes on by up to
    // kHubLen + 32 while others of the wave have entries, and its start may lie
    // near INT32_MAX
    int64_t i[kRowSets], t0[kRowSets];
    int t[kRowSets], len[kRowSets];
    double s[kRowSets];
    bool hub[kRowSets];
#pragma unroll
    for (int r = 0; r < kRowSets; ++r) {
      i[r] = i0 + r * (64 / kRowLanes) + lane / kRowLanes;
      s[r] = 0.0;
      t0[r] = 0;
      len[r] = 0;
      if (i[r] < d) {
        const int b = rowptr[i[r]];
        t0[r] = b;
        len[r] = rowptr[i[r] + 1] - b;
      }
      hub[r] = hub_n > 0 && len[r] > kHubLen;
      if (hub[r]) len[r] = 0;
      t[r] = sub;
    }
    while (true) {
      bool more = false;
#pragma unroll
      for (int r = 0; r < kRowSets; ++r) more |= t[r] < len[r];
      if (!__any(more)) break;
      int c[kRowSets][kGather];
      double v[kRowSets][kGather];
#pragma unroll
      for (int r = 0; r < kRowSets; ++r)
#pragma unroll
        for (int u = 0; u < kGather; ++u) {
          const int e = t[r] + u * kRowLanes;
          const bool in = e < len[r];
          c[r][u] = in ? col[t0[r] + e] : -1;
          v[r][u] = in && val ? (double)val[t0[r] + e] : 1.0;
        }
#pragma unroll
      for (int r = 0; r < kRowSets; ++r) {
        double x[kGather];
#pragma unroll
        for (int u = 0; u < kGather; ++u) x[u] = c[r][u] >= 0 ? q[c[r][u]] : 0.0;
#pragma unroll
        for (int u = 0; u < kGather; ++u)
          if (c[r][u] >= 0) s[r] += v[r][u] * x[u];
        t[r] += kGather * kRowLanes;
      }
    }
#pragma unroll
    for (int r = 0; r < kRowSets; ++r) {
      for (int o = kRowLanes / 2; o > 0; o >>= 1) s[r] += __shfl_xor(s[r], o, 64);
      if (sub == 0 && i[r] < d) {
        if (hub[r]) {
          int lo = 0, hi = hub_n - 1;  // the row is in the table
          while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (hub_rows[mid] < i[r]) lo = mid + 1; else hi = mid;
          }
          s[r] = 0.0;
          for (int ch = hub_c0[lo]; ch < hub_c0[lo + 1]; ++ch) s[r] += hub_part[ch];
        }
        if (qs) s[r] += shift * qs[i[r]];
        w[i[r]] = s[r];
      }
    }
  }
}

// w = M q (+ shift * qs) for one CSR matrix M, long rows through the chunks.
void lz_csr_product(hipStream_t s, const CsrMat& m, const double* q, double* w, double shift, 
                    const double* qs, double* hub_part, const LanczosState* st) {
  const int64_t rows = kT / 64 * kWaveRows;
  const int grid = (int)((m.nrows + rows - 1) / rows < 4096 ? (m.nrows + rows - 1) / rows : 4096);
  if (m.hub_n > 0)
    lz_hub_chunk_kernel<<<(m.hub_chunks + 3) / 4, 256, 0, s>>>(m.col, m.val, m.hub_cs, m.hub_ce,
                                                               m.hub_chunks, q, hub_part, st);
  lz_spmv_kernel<<<grid, kT, 0, s>>>(m.rowptr, m.col, m.val, m.nrows, q, w, shift, qs,
                                     m.hub_rows, m.hub_c0, m.hub_n, hub_part, st);
}

// w = A q (dense FP64, row-major): one wave per row.
__global__ void lz_gemv_kernel(const double* __restrict__ A, int64_t lda, int64_t d,
                               const double* __restrict__ q, double* __restrict__ w,
                               const LanczosState* st) {
  if (st->stopped) return;
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t nw = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t i = wave; i < d; i += nw) {
    double s = 0.0;
    for (int64_t k = lane; k < d; k += 64) s += A[i * lda + k] * q[k];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if (lane == 0) w[i] = s;
  }
}

// Sum of part[0 .. nb) by one wave in a fixed order: lane l adds entries
// l, l + 64, ..., then a shuffle tree.  Every lane returns the total.
__device__ double wave_sum_fixed(const double* __restrict__ part, int nb) {
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  for (int b = lane; b < nb; b += 64) s += part[b];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  return s;
}

// h[c] = sum_b part[c][b], one wave (workgroup) per column c.  mode 0: first
// pass (alpha_j = h_j); mode 1: second pass (alpha_j += h_j).
__global__ __launch_bounds__(64) void lz_dots_reduce_kernel(const double* __restrict__ part,
                                                            int nb, int ncols,
                                                            double* __restrict__ h, int mode,
                                                            int j, LanczosState* st) {
  if (st->stopped) return;
  const int c = blockIdx.x;
  if (c >= ncols) return;
  const double s = wave_sum_fixed(part + (int64_t)c * nb, nb);
  if (threadIdx.x == 0) {
    h[c] = s;
    if (c == j) st->alpha[j] = (mode == 0) ? s : st->alpha[j] + s;
  }
}

// Lanes swap the halves of 2 M values across lane bit BIT, then of M across the
// next, ...; once one value is left, plain sums over the remaining bits.
template <int M, int BIT, int C>
__device__ __forceinline__ void fold_lanes(double (&v)[C]) {
  if constexpr (BIT >= 1) {
    if constexpr (M >= 1) {
      const bool up = threadIdx.x & BIT;
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const double keep = up ? v[i + M] : v[i], give = up ? v[i] : v[i + M];
        v[i] = keep + __shfl_xor(give, BIT, 64);
      }
    } else {
      v[0] += __shfl_xor(v[0], BIT, 64);
    }
    fold_lanes<M / 2, BIT / 2>(v);
  }
}

// Sums over the wave's lanes of C values per lane (C = 16, 32 or 64, in place),
// fixed tree: the sum of value c ends in the lanes l with l / (64 / C) = c.
// The lanes swap halves of their values, so that C - 1 additions do what C
// trees of 6 would; the two widest exchanges are register swaps.
template <int C>
__device__ __forceinline__ double wave_sums(double (&v)[C]) {
  auto swap_add = [&](double a, double b, auto&& swap) {
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    swap(x.x, y.x);
    swap(x.y, y.y);
    return __builtin_bit_cast(double, x) + __builtin_bit_cast(double, y);
  };
#pragma unroll
  for (int i = 0; i < C / 2; ++i) v[i] = swap_add(v[i], v[i + C / 2], swap32);
#pragma unroll
  for (int i = 0; i < C / 4; ++i) v[i] = swap_add(v[i], v[i + C / 4], swap16);
  fold_lanes<C / 8, 8>(v);
  return v[0];
}

// One pass over the basis, a wave per 64 rows at a time (lane = row), with the
// rows of up to C columns in registers: 64 loads under way per lane.
//   kDots:   part[c][b] = block b's sums of Q[c] . w
//   kUpdate: w -= sum_c h[c] Q[c], then the same sums of the new w
//   kNorm:   w -= sum_c h[c] Q[c], then part[b] = block b's sum of w^2
// More than 64 columns go through in pieces of 64; for kUpdate all but the last
// are then read twice.
enum { kDots = 0, kUpdate = 1, kNorm = 2 };
template <int MODE, int C>
__global__ __launch_bounds__(kT) void lz_pass_kernel(const double* __restrict__ Q, int64_t d,
                                                     int ncols, const double* __restrict__ h,
                                                     double* __restrict__ w,
                                                     double* __restrict__ part,
                                                     const LanczosState* st) {
  constexpr int kWv = kT / 64, kPieces = (kLanczosMaxSteps + 63) / 64;
  constexpr int kSpread = 64 / C;  // lanes that hold one column's sum
  __shared__ double sh[kWv][64];
  if (st->stopped) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int pieces = (ncols + C - 1) / C;
  double acc[C == 64 ? kPieces : 1] = {};
  double nrm = 0.0;
  const int64_t nw = (int64_t)gridDim.x * kWv;
  for (int64_t t = (int64_t)blockIdx.x * kWv + wave; t * 64 < d; t += nw) {
    const int64_t n = t * 64 + lane, nn = n < d ? n : d - 1;
    double s = n < d ? w[n] : 0.0;
    double q[C];
    auto load = [&](int p) {
#pragma unroll
      for (int c0 = 0; c0 < C; c0 += 8) {
        if (p * C + c0 < ncols) {  // uniform
#pragma unroll
          for (int c = c0; c < c0 + 8; ++c)
            q[c] = Q[(int64_t)min(p * C + c, ncols - 1) * d + nn];
        } else {
#pragma unroll
          for (int c = c0; c < c0 + 8; ++c) q[c] = 0.0;
        }
      }
    };
    if constexpr (MODE != kDots) {
      for (int p = 0; p < pieces; ++p) {
        load(p);
#pragma unroll
        for (int c0 = 0; c0 < C; c0 += 8) {
          if (p * C + c0 < ncols) {
#pragma unroll
            for (int c = c0; c < c0 + 8; ++c)
              if (p * C + c < ncols) s -= h[p * C + c] * q[c];
          }
        }
      }
      if (n < d) w[n] = s;
      else s = 0.0;
    }
    if constexpr (MODE == kNorm) {
      nrm += s * s;
    } else {
#pragma unroll
      for (int p = C == 64 ? kPieces - 1 : 0; p >= 0; --p) {
        if (p >= pieces) continue;
        if (MODE == kDots || p != pieces - 1) load(p);
#pragma unroll
        for (int c = 0; c < C; ++c) q[c] *= s;
        acc[p] += wave_sums<C>(q);
      }
    }
  }
  if constexpr (MODE == kNorm) {
    for (int o = 32; o > 0; o >>= 1) nrm += __shfl_xor(nrm, o, 64);
    if (lane == 0) sh[wave][0] = nrm;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (sh[0][0] + sh[1][0]) + (sh[2][0] + sh[3][0]);
  } else {
#pragma unroll
    for (int p = 0; p < (C == 64 ? kPieces : 1); ++p) {
      if (p >= pieces) break;
      __syncthreads();
      sh[wave][lane] = acc[p];
      __syncthreads();
      const int c = p * C + (int)threadIdx.x;
      if ((int)threadIdx.x < C && c < ncols) {
        const int l = threadIdx.x * kSpread;
        part[(int64_t)c * gridDim.x + blockIdx.x] = (sh[0][l] + sh[1][l]) + (sh[2][l] + sh[3][l]);
      }
    }
  }
}

template <int MODE>
void lz_pass(hipStream_t s, int grid, const double* Q, int64_t d, int ncols, const double* h,
             double* w, double* part, const LanczosState* st) {
  if (ncols <= 16) lz_pass_kernel<MODE, 16><<<grid, kT, 0, s>>>(Q, d, ncols, h, w, part, st);
  else if (ncols <= 32) lz_pass_kernel<MODE, 32><<<grid, kT, 0, s>>>(Q, d, ncols, h, w, part, st);
  else lz_pass_kernel<MODE, 64><<<grid, kT, 0, s>>>(Q, d, ncols, h, w, part, st);
}

// beta_j = |w| from the partials of w.w (every wave adds them, in the same
// order); q_{j+1} = w / beta_j, or stop.
__global__ __launch_bounds__(kT) void lz_next_kernel(const double* __restrict__ w, int64_t d,
                                                     const double* __restrict__ part, int nb, int j,
                                                     double* __restrict__ qn, LanczosState* st) {
  if (st->stopped) return;
  const double beta = sqrt(wave_sum_fixed(part, nb));
  const bool stop = !(beta > 1e-12 * fmax(1.0, fabs(st->alpha[j])));
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->beta[j] = beta;
    st->k = j + 1;
    if (stop) st->stopped = 1;
  }
  if (stop) return;
  const double inv = 1.0 / beta;
  for (int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; n < d;
       n += (int64_t)gridDim.x * blockDim.x)
    qn[n] = w[n] * inv;
}

__device__ int sturm_count(const double* al, const double* be, int k, double x) {
  int cnt = 0;
  double dd = 1.0;
  for (int i = 0; i < k; ++i) {
    const double off = i ? be[i - 1] * be[i - 1] / dd : 0.0;
    dd = al[i] - x - off;
    if (dd == 0.0) dd = -1e-300;
    if (dd < 0) ++cnt;
  }
  return cnt;
}

// Eigenvalue number index of T by one wave: each round tries 64 points of the
// interval, so ten rounds do what 60 bisections would, until the ends are
// neighbouring numbers.
__device__ double wave_bisect(const double* al, const double* be, int k, int index) {
  const int lane = threadIdx.x & 63;
  double lo = 1e300, hi = -1e300;
  for (int i = 0; i < k; ++i) {
    const double r = (i ? fabs(be[i - 1]) : 0.0) + (i + 1 < k ? fabs(be[i]) : 0.0);
    lo = fmin(lo, al[i] - r);
    hi = fmax(hi, al[i] + r);
  }
  for (int it = 0; it < 200; ++it) {
    const double mid = 0.5 * (lo + hi);
    if (mid <= lo || mid >= hi) break;
    const double x = lo + (hi - lo) * ((lane + 1) * (1.0 / 65.0));
    // the first point with more than index eigenvalues below it
    const uint64_t above = __ballot(sturm_count(al, be, k, x) > index);
    const int f = above ? __builtin_ctzll(above) : 64;
    const double nlo = f > 0 ? __shfl(x, f - 1, 64) : lo;
    const double nhi = f < 64 ? __shfl(x, f, 64) : hi;
    if (nlo == lo && nhi == hi) break;
    lo = nlo;
    hi = nhi;
  }
  return 0.5 * (lo + hi);
}

// |last entry| of the unit eigenvector of T for eigenvalue theta, by three
// steps of inverse iteration with the tridiagonal (Thomas) solver.
__device__ double last_component(const double* al, const double* be, int k, double theta,
                                 double* x, double* cp, double* dp) {
  const double scale = fmax(fabs(theta), 1e-300);
  for (int i = 0; i < k; ++i) x[i] = 1.0;
  for (int it = 0; it < 3; ++it) {
    // solve (T - theta I) y = x
    for (int i = 0; i < k; ++i) {
      const double sub = i ? be[i - 1] : 0.0;
      double piv = al[i] - theta - (i ? sub * cp[i - 1] : 0.0);
      if (fabs(piv) < 1e-15 * scale) piv = (piv < 0 ? -1e-15 : 1e-15) * scale;
      cp[i] = (i + 1 < k) ? be[i] / piv : 0.0;
      dp[i] = (x[i] - (i ? sub * dp[i - 1] : 0.0)) / piv;
    }
    for (int i = k - 1; i >= 0; --i) x[i] = dp[i] - (i + 1 < k ? cp[i] * x[i + 1] : 0.0);
    double nrm = 0.0;
    for (int i = 0; i < k; ++i) nrm += x[i] * x[i];
    nrm = sqrt(nrm);
    for (int i = 0; i < k; ++i) x[i] /= nrm;
  }
  return fabs(x[k - 1]);
}

// Two waves: the smallest and the largest Ritz value with their residual
// bounds, T and the solver's scratch in LDS (one thread over global memory took
// 910 us for 64 steps).
__global__ __launch_bounds__(128) void lz_interval_kernel(const LanczosState* st, double margin,
                                                          double* out) {
  __shared__ double al[kLanczosMaxSteps], be[kLanczosMaxSteps];
  __shared__ double work[2][3][kLanczosMaxSteps];
  __shared__ double th[2], res[2];
  const int k = st->k;
  for (int i = threadIdx.x; i < k; i += 128) {
    al[i] = st->alpha[i];
    be[i] = st->beta[i];
  }
  __syncthreads();
  const int e = threadIdx.x >> 6;  // 0: smallest, 1: largest
  const double theta = wave_bisect(al, be, k, e ? k - 1 : 0);
  if ((threadIdx.x & 63) == 0) {
    th[e] = theta;
    res[e] = fabs(be[k - 1]) *
             last_component(al, be, k, theta, work[e][0], work[e][1], work[e][2]);
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  const double w = th[1] - th[0];
  out[0] = th[0] - res[0] - margin * w;
  out[1] = th[1] + res[1] + margin * w;
  out[2] = th[0];
  out[3] = th[1];
  out[4] = res[0];
  out[5] = res[1];
  out[6] = (double)k;
}

}  // namespace

hipError_t launch_lanczos(hipStream_t s, const mlct_op* op, const void* a64, int64_t lda,
                          int steps, uint64_t seed, double margin, double* Q, double* w,
                          double* h, double* part, LanczosState* st, double* out, double* tmp,
                          double* hub_part) {
  const int64_t d = op->d;
  // blocks of the passes over the basis: three waves per SIMD
  const int nb = (int)((d + kT - 1) / kT < 768 ? (d + kT - 1) / kT : 768);
  const int grid = (int)((d + kT - 1) / kT < 1024 ? (d + kT - 1) / kT : 1024);
  lz_start_kernel<<<grid, kT, 0, s>>>(Q, d, seed, st);
  for (int j = 0; j < steps; ++j) {
    const double* qj = Q + (int64_t)j * d;
    if (op->kind == OP_CSR) {
      lz_csr_product(s, op->csr, qj, w, 0.0, nullptr, hub_part, st);
    } else if (op->kind == OP_GRAM_CSR) {  // w = X^T (X q) + lambda q
      lz_csr_product(s, op->csrx, qj, tmp, 0.0, nullptr, hub_part, st);
      lz_csr_product(s, op->csr, tmp, w, op->gram_lambda, qj, hub_part, st);
    } else
      lz_gemv_kernel<<<grid, kT, 0, s>>>(static_cast<const double*>(a64), lda, d, qj, w, st);
    lz_pass<kDots>(s, nb, Q, d, j + 1, h, w, part, st);
    lz_dots_reduce_kernel<<<j + 1, 64, 0, s>>>(part, nb, j + 1, h, 0, j, st);
    lz_pass<kUpdate>(s, nb, Q, d, j + 1, h, w, part, st);
    lz_dots_reduce_kernel<<<j + 1, 64, 0, s>>>(part, nb, j + 1, h, 1, j, st);
    lz_pass<kNorm>(s, nb, Q, d, j + 1, h, w, part, st);
    lz_next_kernel<<<grid, kT, 0, s>>>(w, d, part, nb, j, Q + (int64_t)(j + 1) * d, st);
  }
  lz_interval_kernel<<<1, 128, 0, s>>>(st, margin, out);
  return hipGetLastError();
}

}  // namespace mlct
