// Block Chebyshev recurrence over a CSR operator (Section 2.2, eq.
// eqn:recurrence in matrix form) with the per-probe moments fused in.
//
// Layout: a probe block V is row-major d x 64 (probe index fastest), so the
// gather of row j of V is one 256-byte (FP32) or 512-byte (FP64) contiguous
// read by a whole wavefront, lane = probe.  One step computes
//     V_new = ca * (A V_k) + cb * V_k  [- V_prev]
// in place over V_prev (each element is read and then written by the same
// lane), and accumulates per lane, in FP64 with exact FP64 products,
//     ZMODE 0: V_k[i].V_new[i] and V_new[i].V_new[i]   (symmetric form)
//     ZMODE 1: z[i].V_new[i], z regenerated from SplitMix64 (direct form)
//     ZMODE 2: z[i].V_new[i], z read from explicit int8 entries.
// Each workgroup owns a contiguous band of rows and writes one partial sum
// per probe and slot; partials are reduced later in a fixed order, so the
// moments are bitwise reproducible.
//
// Operators whose rows all have at most 8 entries take a wide form of the
// same step (csr_step_wide_kernel, ZMODE 0 and 1): a lane holds 16 bytes of
// probes and a wave instruction moves several rows, with the same row sums,
// update and moment summation order as the lane = probe body.
//
// Longer rows take a form whose lanes also hold 16 bytes of probes, one row
// per group of lanes (long_band); rows past kHubLen, the hubs of power-law
// graphs, would leave one wave walking tens of thousands of gathers, and are
// cut into chunks of kHubChunk that the workgroup of their band shares.
#include <algorithm>
#include <climits>
#include <type_traits>

#include "device.hpp"

namespace mlct {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;

__device__ __forceinline__ void store_partials(double a1, double a2, int g, int ngroups,
                                               double* __restrict__ part,
                                               int probe = lane_id()) {
  __shared__ double sh[2][kWaves][64];
  const int lane = lane_id(), wave = wave_id();
  sh[0][wave][probe] = a1;
  sh[1][wave][probe] = a2;
  __syncthreads();
  if (wave == 0) {
    double s1 = sh[0][0][lane], s2 = sh[1][0][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      s1 += sh[0][w][lane];
      s2 += sh[1][w][lane];
    }
    part[(size_t)g * 64 + lane] = s1;
    part[((size_t)ngroups + g) * 64 + lane] = s2;
  }
}

template <typename T>
__device__ __forceinline__ void probe_init_wg(T* __restrict__ v0, int64_t d, const ProbeSrc& src,
                                              int rows_per_group, int ngroups,
                                              double* __restrict__ part, int bid) {
  const int lane = lane_id(), wave = wave_id();
  const int g = xcd_band(bid, ngroups);
  const int64_t r0 = (int64_t)g * rows_per_group;
  const int64_t r1 = min<int64_t>(r0 + rows_per_group, d);
  const bool act = lane < src.active;
  const uint64_t key = sm_output(src.seed, (uint64_t)(src.first_id + lane));
  int64_t cached = -1;
  uint64_t word = 0;
  double acc = 0.0;
  for (int64_t i = r0 + wave; i < r1; i += kWaves) {
    T z = T(0);
    if (act) {
      if (src.entries) {
        z = (T)src.entries[i * src.ld + src.first_id + lane];
      } else {
        const int64_t c = i >> 6;
        if (c != cached) {
          word = sm_output(key, (uint64_t)c);
          cached = c;
        }
        z = sign_from_word<T>(word, i);
      }
    }
    v0[i * 64 + lane] = z;
    acc += (double)z * (double)z;
  }
  store_partials(acc, 0.0, g, ngroups, part);
}

template <typename T>
__global__ __launch_bounds__(kThreads) void probe_init_kernel(T* __restrict__ v0, int64_t d,
                                                              ProbeSrc src, int rows_per_group,
                                                              int ngroups,
                                                              double* __restrict__ part) {
  probe_init_wg<T>(v0, d, src, rows_per_group, ngroups, part, blockIdx.x);
}

// Per-row epilogue of the recurrence: V_new = ca*acc + cb*V_k[i] (- V_prev[i]),
// written over V_prev (with a non-temporal store unless KEEP: a vector
// gathered again soon is stored normally, to stay in the caches), and the
// lane's moment partials (FP64).  With CLS = 4 (FP32, ZMODE 0 or 1,
// operators whose rows all fit the straight-line path) the partials are kept per row
// class (the row's index in its group, mod 4) and the classes added in
// order at the end: the summation order of the wide step kernel, whose lane
// quads take one class each, so both kernels give the same bits.
template <typename T, int ZMODE, bool HAS_PREV, bool KEEP = false, int CLS = 1>
struct RecEpi {
  static constexpr int kCls = (ZMODE <= 1 && sizeof(T) == 4) ? CLS : 1;
  T ca, cb;
  T* vm;
  ProbeSrc src;
  bool act;
  uint64_t key = 0;
  int64_t cached = -1;
  uint64_t word = 0;
  double a1[kCls] = {}, a2[kCls] = {};
  __device__ RecEpi(T ca_, T cb_, T* vm_, const ProbeSrc& s) : ca(ca_), cb(cb_), vm(vm_), src(s) {
    const int lane = lane_id();
    act = lane < src.active;
    if (ZMODE == 1) key = sm_output(src.seed, (uint64_t)(src.first_id + lane));
  }
  __device__ __forceinline__ T prev(int64_t i) const {
    return HAS_PREV ? __builtin_nontemporal_load(vm + i * 64 + lane_id()) : T(0);
  }
  // r: the row's index in its group (a compile-time constant at every call)
  __device__ __forceinline__ void finish(int64_t i, T acc, T xi, T xp, int r) {
    const int lane = lane_id();
    const int c = r % kCls;
    // one explicit contraction, so every kernel that shares this update
    // (the two-step and wide kernels included) rounds it the same way
    T vn = fma(ca, acc, cb * xi);
    if (HAS_PREV) vn -= xp;
    if (KEEP)
      vm[i * 64 + lane] = vn;
    else
      __builtin_nontemporal_store(vn, vm + i * 64 + lane);
    if (ZMODE == 0) {
      a1[c] += (double)xi * (double)vn;
      a2[c] += (double)vn * (double)vn;
    } else if (ZMODE == 1) {
      const int64_t cw = i >> 6;
      if (cw != cached) {
        word = sm_output(key, (uint64_t)cw);
        cached = cw;
      }
      a1[c] += sign_from_word<double>(word, i) * (double)vn;
    } else {
      const double z = act ? (double)src.entries[i * src.ld + src.first_id + lane] : 0.0;
      a1[c] += z * (double)vn;
    }
  }
  __device__ __forceinline__ double part1() const { return class_sum(a1); }
  __device__ __forceinline__ double part2() const { return class_sum(a2); }
  static __device__ __forceinline__ double class_sum(const double (&a)[kCls]) {
    double s = a[0];
#pragma unroll
    for (int k = 1; k < kCls; ++k) s += a[k];
    return s;
  }
};

// One gathered entry into a row sum: weight w (ignored for patterns) times x,
// or nothing when on is false.
template <typename T, bool PATTERN>
__device__ __forceinline__ T accum(T acc, float w, bool on, T x) {
  const float onf = on ? 1.f : 0.f;
  const float ww = PATTERN ? onf : w * onf;
  return fma((T)ww, x, acc);
}

// Gathers of block rows.  With OFF32 (block under 4 GiB, FP32) they are
// buffer loads: the block base sits in a scalar resource, the row offset
// j * 256 in a scalar register and lane * 4 in one VGPR shared by every
// gather, so a gather costs no address registers.  Out-of-range offsets read
// as 0 (the resource's size is the block's size).
template <typename T, bool OFF32>
struct RowReader {
  const T* base;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t lane_off;
  __device__ __forceinline__ RowReader(const T* b, int64_t d, int lane) : base(b) {
    if (OFF32) {
      rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(b), (short)0,
                                               (int)(uint32_t)(d * 64 * sizeof(T)), 0x00020000);
      lane_off = (uint32_t)lane * sizeof(T);
    }
  }
  __device__ __forceinline__ T operator()(int64_t j, int lane) const {
    if constexpr (OFF32) {
      static_assert(sizeof(T) == 4, "32-bit offsets are for 4-byte elements");
      const uint32_t bits = __builtin_amdgcn_raw_buffer_load_b32(
          rsrc, lane_off, (int)((uint32_t)j * (uint32_t)(64 * sizeof(T))), 0);
      return __uint_as_float(bits);
    } else {
      return base[j * 64 + lane];
    }
  }
};

// Extent of one group of up to ROWS consecutive rows.  The group's rows sit
// in lanes q .. q+ROWS-1 of a batch: rs = start of the row's columns,
// rlen = its length (0 for lanes past the end of the matrix).
template <int ROWS>
struct GroupExt {
  int gs, cnt, nr, maxlen;
  int off[ROWS], len[ROWS];
};

template <int ROWS>
__device__ __forceinline__ GroupExt<ROWS> group_extent(int rs, int rlen, int q, int nr) {
  GroupExt<ROWS> e;
  e.nr = nr;
  e.gs = read_lane(rs, q);
  e.maxlen = 0;
  e.cnt = 0;
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    const bool in = r < nr;
    e.off[r] = in ? read_lane(rs, q + r) - e.gs : 0;
    e.len[r] = in ? read_lane(rlen, q + r) : 0;
    e.maxlen = max(e.maxlen, e.len[r]);
    if (in) e.cnt = e.off[r] + e.len[r];  // static indices only
  }
  return e;
}

// Work split: a workgroup owns a contiguous band of rows (equal row counts,
// or the plan's equal-work bands) cut into groups of ROWS rows; wave w takes
// groups w, w + kWaves, w + 2 kWaves, ..., so the waves of a workgroup sweep
// the band side by side.  A wave fetches the row extents of its next 64/ROWS
// groups in one load (a "batch", prefetched one batch ahead) and the column
// indices and values of a group in one coalesced load, issued while the
// previous group's gathers are in flight.  No row is longer than MAXNZ (and
// ROWS * MAXNZ <= 64), so a group's gathers are straight-line code (unused
// slots gather some valid row with weight 0), all in flight before the first
// is consumed.
template <typename T, bool PATTERN, int MAXNZ, bool OFF32, class Epi>
__device__ __forceinline__ void csr_step_wg(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t nnz, const RowReader<T, OFF32>& rd,
    Epi& epi, const CsrStepPlan& plan, double* __restrict__ part, int bid) {
  constexpr int ROWS = MAXNZ <= 5 ? 8 : 4;
  constexpr int GPB = 64 / ROWS;  // groups per batch
  const int lane = lane_id(), wave = wave_id();
  const int ngroups = plan.ngroups;
  const int g = xcd_band(bid, ngroups);
  const int64_t r0 = plan.band ? (int64_t)plan.band[g] : (int64_t)g * plan.rows_per_group;
  const int64_t r1 = plan.band ? (int64_t)plan.band[g + 1]
                               : min<int64_t>(r0 + plan.rows_per_group, d);

  const int64_t ngrp = r1 > r0 ? (r1 - r0 + ROWS - 1) / ROWS : 0;  // groups in the band
  const int64_t nk = ngrp > wave ? (ngrp - wave + kWaves - 1) / kWaves : 0;  // this wave's
  // first row of this wave's k-th group, and its number of rows
  auto grp_row0 = [&](int64_t k) { return r0 + (k * kWaves + wave) * ROWS; };
  auto grp_rows = [&](int64_t k) { return (int)min<int64_t>(ROWS, r1 - grp_row0(k)); };

  if (nk > 0) {
    auto load_batch = [&](int64_t j, int& rs, int& rlen) {
      const int64_t k = j * GPB + lane / ROWS;
      const int64_t row = grp_row0(k) + lane % ROWS;
      const bool ok = k < nk && row < r1;
      const int64_t rr = ok ? row : r0;
      rs = rowptr[rr];
      rlen = ok ? rowptr[rr + 1] - rs : 0;
    };
    auto load_cols = [&](const GroupExt<ROWS>& e, int& cj, float& av) {
      const int64_t ce = min<int64_t>((int64_t)e.gs + lane, nnz - 1);
      cj = col[ce];
      av = PATTERN ? 1.f : val[ce];
    };
    const int64_t nbatch = (nk + GPB - 1) / GPB;
    int64_t j = 0;
    int rs, rlen, rs_n = 0, rlen_n = 0;
    load_batch(0, rs, rlen);
    if (nbatch > 1) load_batch(1, rs_n, rlen_n);
    int64_t k = 0;
    GroupExt<ROWS> cur = group_extent<ROWS>(rs, rlen, 0, grp_rows(0));
    int cj = 0;
    float av = 0.f;
    // (always so, but without the test the compiler forms the first rows'
    // addresses all at once and spills them: valued FP32 rows of up to 5 entries
    // with explicit probes, d = 10^6, 273 us a step against 255)
    if (nnz > 0) load_cols(cur, cj, av);

    while (true) {
      const int64_t row0 = grp_row0(k);
      T x[ROWS][MAXNZ];
      T xi[ROWS], xp[ROWS];
      // all gathers of the group before anything else is issued
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const int64_t i = row0 + min(r, cur.nr - 1);
#pragma unroll
        for (int t = 0; t < MAXNZ; ++t) x[r][t] = rd(read_lane(cj, min(cur.off[r] + t, 63)), lane);
        xi[r] = rd(i, lane);
        xp[r] = epi.prev(i);
      }
      // next group: extent and column prefetch
      const int64_t kn = k + 1;
      const bool has_next = kn < nk;
      const bool new_batch = has_next && (kn % GPB) == 0;
      GroupExt<ROWS> nxt = cur;
      int cjn = 0;
      float avn = 0.f;
      if (has_next) {
        const int qn = (int)(kn % GPB) * ROWS;
        nxt = new_batch ? group_extent<ROWS>(rs_n, rlen_n, 0, grp_rows(kn))
                        : group_extent<ROWS>(rs, rlen, qn, grp_rows(kn));
        load_cols(nxt, cjn, avn);
      }
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        T acc = T(0);
#pragma unroll
        for (int t = 0; t < MAXNZ; ++t)
          acc = accum<T, PATTERN>(acc, PATTERN ? 1.f : read_lane(av, min(cur.off[r] + t, 63)),
                                  t < cur.len[r], x[r][t]);
        if (r < cur.nr) epi.finish(row0 + r, acc, xi[r], xp[r], r);
      }
      if (!has_next) break;
      if (new_batch) {
        rs = rs_n;
        rlen = rlen_n;
        ++j;
        if (j + 1 < nbatch) load_batch(j + 1, rs_n, rlen_n);
      }
      k = kn;
      cur = nxt;
      cj = cjn;
      av = avn;
    }
  }
  store_partials(epi.part1(), epi.part2(), g, ngroups, part);
}

template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, int MAXNZ, bool OFF32>
__global__ __launch_bounds__(kThreads) void csr_step_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t nnz, const T* __restrict__ vk,
    T* __restrict__ vm, T ca, T cb, ProbeSrc src, CsrStepPlan plan, double* __restrict__ part) {
  RecEpi<T, ZMODE, HAS_PREV, false, 4> epi(ca, cb, vm, src);
  csr_step_wg<T, PATTERN, MAXNZ, OFF32>(rowptr, col, val, d, nnz,
                                        RowReader<T, OFF32>(vk, d, lane_id()), epi, plan, part,
                                        blockIdx.x);
}

// ---- wide form of the step ------------------------------------------------------
// For operators whose rows all fit the straight-line path (no tail) and
// moments of the symmetric form (ZMODE 0) or the direct form with
// regenerated Rademacher probes (ZMODE 1), the same step with a lane
// holding PPL = 16 / sizeof(T) probes (4 in FP32, 2 in FP64): every access
// is 16 bytes, so one wave instruction moves PPL rows (lane group q, of
// 64 / PPL lanes, on the group's rows q, q + PPL, ...) and a step issues
// 1 / PPL of the memory instructions of the lane = probe body.  The work
// split (bands, groups of ROWS rows, wave w on groups w, w + 8, ...), the
// column prefetch, the row sums (entry order, one fma per entry, unused
// slots weighted 0) and the update are those of csr_step_wg with RecEpi; a
// lane's row offset and length are picked from the group's extent by its
// lane group, and its column indices and values come from the group's
// coalesced load by a lane permute.  The moment partials are kept per row
// class (row index in the group mod PPL, one class per lane group) and the
// classes added in order; in FP32 that is the order of RecEpi with CLS = 4,
// so this kernel and the lane = probe body give the same bits.  With SLQ
// the rows are the product of a Lanczos step instead (u = s (A w) stored,
// s = 1 / |w| per probe, partials of (s w) . u, the Jacobi diagonal; FP64, no
// recurrence).
template <typename T>
struct WideVec;
template <>
struct WideVec<float> {
  typedef float V __attribute__((ext_vector_type(4)));
};
template <>
struct WideVec<double> {
  typedef double V __attribute__((ext_vector_type(2)));
};

template <typename T, bool OFF32>
struct WideRows {
  using V = typename WideVec<T>::V;
  const T* base;
  __amdgpu_buffer_rsrc_t rsrc;
  uint32_t lane_off;
  __device__ __forceinline__ WideRows(const T* b, int64_t d, int sub) : base(b) {
    if (OFF32)
      rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(b), (short)0,
                                               (int)(uint32_t)(d * 64 * sizeof(T)), 0x00020000);
    lane_off = (uint32_t)sub * 16;
  }
  // the lane's probes of the block row at byte offset off (past the block: 0)
  __device__ __forceinline__ V at(uint32_t off) const {
    return __builtin_bit_cast(
        V, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + lane_off, 0, 0));
  }
  // the lane's probes of block row j
  __device__ __forceinline__ V operator()(int64_t j) const {
    if constexpr (OFF32)
      return __builtin_bit_cast(
          V, __builtin_amdgcn_raw_buffer_load_b128(
                 rsrc, (uint32_t)j * (uint32_t)(64 * sizeof(T)) + lane_off, 0, 0));
    else
      return *reinterpret_cast<const V*>(base + j * 64 + lane_off / sizeof(T));
  }
};

__device__ __forceinline__ int permute_lane(int v, int src) {
  return __builtin_amdgcn_ds_bpermute(src << 2, v);
}

template <typename T>
using WidePartials = double[2][kWaves][16 / sizeof(T)][64];

// Band g of the wide step: its rows, then its moment partials (sh: the
// workgroup's LDS for the partials).
template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, int MAXNZ, bool OFF32,
          bool SLQ = false>
__device__ __forceinline__ void wide_band(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t nnz, const T* __restrict__ vk,
    T* __restrict__ vm, T ca, T cb, const ProbeSrc& src, const CsrStepPlan& plan,
    double* __restrict__ part, int g, WidePartials<T>& sh, const double* sdev = nullptr) {
  static_assert(ZMODE == 0 || ZMODE == 1, "symmetric or regenerated direct moments");
  static_assert(!SLQ || (ZMODE == 0 && !HAS_PREV), "the Lanczos product has no recurrence");
  using V = typename WideVec<T>::V;
  constexpr int PPL = 16 / (int)sizeof(T);  // probes per lane = rows per wave instruction
  constexpr int LPR = 64 / PPL;             // lanes per row
  constexpr int ROWS = MAXNZ <= 5 ? 8 : 4;
  constexpr int H = ROWS / PPL;   // wave instructions per group
  constexpr int GPB = 64 / ROWS;  // groups per batch of row extents
  static_assert(ROWS * MAXNZ <= 64, "a group's entries fit one coalesced load");
  static_assert(ROWS % PPL == 0, "whole wave instructions per group");
  const int lane = lane_id(), wave = wave_id();
  const int q = lane / LPR, sub = lane % LPR;
  const int ngroups = plan.ngroups;
  const int64_t r0 = plan.band ? (int64_t)plan.band[g] : (int64_t)g * plan.rows_per_group;
  const int64_t r1 = plan.band ? (int64_t)plan.band[g + 1]
                               : min<int64_t>(r0 + plan.rows_per_group, d);
  const int64_t ngrp = r1 > r0 ? (r1 - r0 + ROWS - 1) / ROWS : 0;
  const int64_t nk = ngrp > wave ? (ngrp - wave + kWaves - 1) / kWaves : 0;
  const WideRows<T, OFF32> rd(vk, d, sub);
  T* vm_l = vm + sub * PPL;
  // moment partials of probes PPL sub + e, row class q
  double m1[PPL], m2[PPL];
#pragma unroll
  for (int e = 0; e < PPL; ++e) m1[e] = m2[e] = 0.0;
  // SLQ: the lane's probe scales
  double sc[PPL];
  if constexpr (SLQ) {
#pragma unroll
    for (int e = 0; e < PPL; ++e) sc[e] = sdev[PPL * sub + e];
  }
  // ZMODE 1: the key of probe PPL sub + q and the sign words of the lane's
  // probes for the 64-row chunk `cached` (uniform)
  uint64_t word[PPL], keyq = 0;
  int64_t cached = -1;
  if constexpr (ZMODE == 1) {
#pragma unroll
    for (int e = 0; e < PPL; ++e) word[e] = 0;
    keyq = sm_output(src.seed, (uint64_t)(src.first_id + PPL * sub + q));
  }
  auto grp_row0 = [&](int64_t k) { return r0 + (k * kWaves + wave) * ROWS; };
  auto grp_rows = [&](int64_t k) { return (int)min<int64_t>(ROWS, r1 - grp_row0(k)); };

  if (nk > 0) {
    auto load_batch = [&](int64_t j, int& rs, int& rlen) {
      const int64_t k = j * GPB + lane / ROWS;
      const int64_t row = grp_row0(k) + lane % ROWS;
      const bool ok = k < nk && row < r1;
      const int64_t rr = ok ? row : r0;
      rs = rowptr[rr];
      rlen = ok ? rowptr[rr + 1] - rs : 0;
    };
    auto load_cols = [&](const GroupExt<ROWS>& e, int& cj, float& av) {
      const int64_t ce = min<int64_t>((int64_t)e.gs + lane, nnz - 1);
      cj = col[ce];
      av = PATTERN ? 1.f : val[ce];
    };
    const int64_t nbatch = (nk + GPB - 1) / GPB;
    int64_t j = 0;
    int rs, rlen, rs_n = 0, rlen_n = 0;
    load_batch(0, rs, rlen);
    if (nbatch > 1) load_batch(1, rs_n, rlen_n);
    int64_t k = 0;
    GroupExt<ROWS> cur = group_extent<ROWS>(rs, rlen, 0, grp_rows(0));
    int cj = 0;
    float av = 0.f;
    load_cols(cur, cj, av);

    while (true) {
      const int64_t row0 = grp_row0(k);
      V x[H][MAXNZ], xi[H], xp[H];
      float w[H][MAXNZ];
      int len[H];
      int64_t row[H];
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int rr = PPL * h + q;  // this lane's row in the group
        // its offset and length, selected with static indices (the extent
        // stays in registers)
        int off = cur.off[PPL * h];
        len[h] = cur.len[PPL * h];
#pragma unroll
        for (int r = 1; r < PPL; ++r) {
          off = q == r ? cur.off[PPL * h + r] : off;
          len[h] = q == r ? cur.len[PPL * h + r] : len[h];
        }
        row[h] = row0 + min(rr, cur.nr - 1);
#pragma unroll
        for (int t = 0; t < MAXNZ; ++t) {
          const int src = min(off + t, 63);
          x[h][t] = rd(permute_lane(cj, src));
          w[h][t] = PATTERN ? 1.f : __int_as_float(permute_lane(__float_as_int(av), src));
        }
        xi[h] = rd(row[h]);
        if constexpr (HAS_PREV)
          xp[h] = __builtin_nontemporal_load(reinterpret_cast<const V*>(vm_l + row[h] * 64));
        else
          xp[h] = V{};
      }
      // next group: extent and column prefetch
      const int64_t kn = k + 1;
      const bool has_next = kn < nk;
      const bool new_batch = has_next && (kn % GPB) == 0;
      GroupExt<ROWS> nxt = cur;
      int cjn = 0;
      float avn = 0.f;
      if (has_next) {
        const int qn = (int)(kn % GPB) * ROWS;
        nxt = new_batch ? group_extent<ROWS>(rs_n, rlen_n, 0, grp_rows(kn))
                        : group_extent<ROWS>(rs, rlen, qn, grp_rows(kn));
        load_cols(nxt, cjn, avn);
      }
      // ZMODE 1, a group inside one 64-row chunk: each lane hashes the word
      // of one probe, the lane groups exchange them (one hash per lane per
      // chunk, as in the lane = probe body); a group across two chunks
      // hashes per row below
      bool one_chunk = true;
      if constexpr (ZMODE == 1) {
        const int64_t c0 = row0 >> 6;
        one_chunk = ((row0 + ROWS - 1) >> 6) == c0;
        if (one_chunk && c0 != cached) {
          const uint64_t mine = sm_output(keyq, (uint64_t)c0);
          const int lo = (int)(uint32_t)mine, hi = (int)(uint32_t)(mine >> 32);
#pragma unroll
          for (int e = 0; e < PPL; ++e) {
            const int from = e * LPR + sub;  // lane group e holds probe PPL sub + e
            word[e] = (uint64_t)(uint32_t)permute_lane(lo, from) |
                      ((uint64_t)(uint32_t)permute_lane(hi, from) << 32);
          }
          cached = c0;
        }
      }
#pragma unroll
      for (int h = 0; h < H; ++h) {
        T acc[PPL];
#pragma unroll
        for (int e = 0; e < PPL; ++e) acc[e] = T(0);
#pragma unroll
        for (int t = 0; t < MAXNZ; ++t) {
          const float onf = t < len[h] ? 1.f : 0.f;
          const T ww = (T)(PATTERN ? onf : w[h][t] * onf);
#pragma unroll
          for (int e = 0; e < PPL; ++e) acc[e] = fma(ww, x[h][t][e], acc[e]);
        }
        if (SLQ && PPL * h + q < cur.nr) {
          if constexpr (SLQ) {
            V u;
#pragma unroll
            for (int e = 0; e < PPL; ++e) {
              u[e] = sc[e] * acc[e];
              m1[e] += (sc[e] * xi[h][e]) * u[e];
            }
            __builtin_nontemporal_store(u, reinterpret_cast<V*>(vm_l + row[h] * 64));
          }
        } else if (PPL * h + q < cur.nr) {
          V vn;
#pragma unroll
          for (int e = 0; e < PPL; ++e) {
            T v = fma(ca, acc[e], cb * xi[h][e]);
            if (HAS_PREV) v -= xp[h][e];
            vn[e] = v;
          }
          __builtin_nontemporal_store(vn, reinterpret_cast<V*>(vm_l + row[h] * 64));
          if constexpr (ZMODE == 0) {
#pragma unroll
            for (int e = 0; e < PPL; ++e) {
              m1[e] += (double)xi[h][e] * (double)vn[e];
              m2[e] += (double)vn[e] * (double)vn[e];
            }
          } else {
            // (a group across two chunks: the lane's own keys, rehashed)
            uint64_t wd[PPL];
#pragma unroll
            for (int e = 0; e < PPL; ++e)
              wd[e] = one_chunk ? word[e]
                                : sm_output(sm_output(src.seed, (uint64_t)(src.first_id + PPL * sub + e)),
                                            (uint64_t)(row[h] >> 6));
#pragma unroll
            for (int e = 0; e < PPL; ++e)
              m1[e] += sign_from_word<double>(wd[e], row[h]) * (double)vn[e];
          }
        }
      }
      if (!has_next) break;
      if (new_batch) {
        rs = rs_n;
        rlen = rlen_n;
        ++j;
        if (j + 1 < nbatch) load_batch(j + 1, rs_n, rlen_n);
      }
      k = kn;
      cur = nxt;
      cj = cjn;
      av = avn;
    }
  }
  // per probe: each wave's classes in class order, then the waves in order
#pragma unroll
  for (int e = 0; e < PPL; ++e) {
    sh[0][wave][q][PPL * sub + e] = m1[e];
    sh[1][wave][q][PPL * sub + e] = m2[e];
  }
  __syncthreads();
  if (wave == 0) {
    double s1 = 0.0, s2 = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      double t1 = sh[0][w][0][lane], t2 = sh[1][w][0][lane];
#pragma unroll
      for (int c = 1; c < PPL; ++c) {
        t1 += sh[0][w][c][lane];
        t2 += sh[1][w][c][lane];
      }
      if (w == 0) {
        s1 = t1;
        s2 = t2;
      } else {
        s1 += t1;
        s2 += t2;
      }
    }
    part[(size_t)g * 64 + lane] = s1;
    part[((size_t)ngroups + g) * 64 + lane] = s2;
  }
}

// FP32 direct form with 32-bit gather offsets: at least 4 waves per SIMD
// (128 VGPRs; it otherwise takes 132 and drops to 3: 0.729 against 0.673 ms
// per step on the 2D Laplacian 2048^2; the same bound costs the symmetric
// form 2 % and makes the 64-bit-offset form spill)
template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, int MAXNZ, bool OFF32>
__global__ __launch_bounds__(kThreads, sizeof(T) == 4 && ZMODE == 1 && OFF32 ? 4 : 1) void
csr_step_wide_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t nnz, const T* __restrict__ vk,
    T* __restrict__ vm, T ca, T cb, ProbeSrc src, CsrStepPlan plan, double* __restrict__ part) {
  __shared__ WidePartials<T> sh;
  wide_band<T, PATTERN, ZMODE, HAS_PREV, MAXNZ, OFF32>(rowptr, col, val, d, nnz, vk, vm, ca, cb,
                                                        src, plan, part,
                                                        xcd_band(blockIdx.x, plan.ngroups), sh);
}

// ---- rows of any length ---------------------------------------------------------
// The same step for operators with rows past the straight-line capacity
// (power-law graphs, the two products of a sparse Gram step, Lanczos
// products on such rows).  A lane holds 16 bytes of probes (PPL of them) and
// a group of LPR = 64 / PPL lanes, a slot, walks one row, so a wave sums PPL
// rows at once: a gathered row of V costs 1 / PPL of a load, one lane
// broadcast and one add for its address and PPL fma, about 2 instructions
// against the 10 of one row at a time with lane = probe, which was bound by
// issuing them.  The lanes of a slot load 16 column indices at a time (the
// next 16 while the gathers of the current ones are in flight); entry t is
// spread over the slot by a DPP broadcast within 16 lanes, and a slot past
// its row's end gathers out of range, which costs no memory access.  Each
// row's sum has one fma per entry in entry order, and the moments are summed
// per probe over a wave's rows in order, as with lane = probe.
//
// Rows longer than kHubLen are summed by the whole workgroup of their band:
// chunks of kHubChunk entries, one per slot, each row's chunk sums added in
// order (one row after the other left most slots idle: 1.3 times the step's
// time on a graph of 10^6 vertices).
//
// Bound by the gathers themselves: from one XCD's L2 they run at about 100 G
// rows of 256 bytes per second, from beyond it at 30 G (7.6 TB/s), measured
// with a bare gather loop.  Measured on Chung-Lu graphs (64 probes, FP32, us
// per step, one row at a time with a launch for the long rows' chunks before
// -> now): d = 16,000 71 -> 33, 62,500 77 -> 40, 250,000 179 -> 154, 10^6
// 741 -> 694 (5.9 TB/s of gathered rows); the batch of 64 graphs of 2,048 to
// 65,536 vertices 176 -> 75 ms.
enum { kOpRec = 0, kOpStore = 1, kOpSlq = 2 };

// The slots' PPL x PPL exchange: element e of slot q goes to slot e, element q
// (a lane had PPL probes of its slot's row, and has one probe of PPL rows).
__device__ __forceinline__ void slot_transpose(WideVec<float>::V& v) {
  uint32_t x[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = __float_as_uint(v[e]);
  swap32(x[0], x[2]);
  swap32(x[1], x[3]);
  swap16(x[0], x[1]);
  swap16(x[2], x[3]);
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(x[e]);
}
__device__ __forceinline__ void slot_transpose(WideVec<double>::V& v) {
  uint2 a = __builtin_bit_cast(uint2, (double)v[0]), b = __builtin_bit_cast(uint2, (double)v[1]);
  swap32(a.x, b.x);
  swap32(a.y, b.y);
  v[0] = __builtin_bit_cast(double, a);
  v[1] = __builtin_bit_cast(double, b);
}

// rsh: log2 of the rows of a group (a wave's consecutive rows).
// OP kOpRec: the recurrence over rows 0 .. d - 1 (gathers from vk, own rows
// from vown), kOpStore: the product alone into vm (normal stores: it is
// gathered next), kOpSlq: the product of a Lanczos step.
template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, bool OFF32, int OP = kOpRec>
__device__ __forceinline__ void long_band(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t dv, const T* __restrict__ vk,
    const T* __restrict__ vown, T* __restrict__ vm, T ca, T cb, const ProbeSrc& src,
    const HubRows& hubs, int rsh, const CsrStepPlan& plan, double* __restrict__ part, int g,
    const double* sdev = nullptr) {
  using V = typename WideVec<T>::V;
  constexpr int PPL = 16 / (int)sizeof(T);
  constexpr int LPR = 64 / PPL;
  constexpr int kSlots = kWaves * PPL;
  constexpr uint32_t kRowBytes = 64 * sizeof(T);
  // past every block whose size OFF32 admits, and off + 16 sub cannot wrap
  constexpr uint32_t kOut = 0u - kRowBytes;
  const int lane = lane_id(), wave = wave_id();
  const int q = lane / LPR, sub = lane % LPR, l16 = lane & 15;
  const int64_t r0 = plan.band ? (int64_t)plan.band[g] : (int64_t)g * plan.rows_per_group;
  const int64_t r1 = plan.band ? (int64_t)plan.band[g + 1]
                               : min<int64_t>(r0 + plan.rows_per_group, d);
  const WideRows<T, OFF32> rd(vk, dv, sub);
  T* vm_l = vm + sub * PPL;
  const T* own_l = vown + sub * PPL;
  // moment partials of probe `probe` (rows in order)
  const int probe = PPL * sub + q;
  double m1 = 0.0, m2 = 0.0;
  double sc[PPL];
  if constexpr (OP == kOpSlq) {
#pragma unroll
    for (int e = 0; e < PPL; ++e) sc[e] = sdev[PPL * sub + e];
  }
  uint64_t word = 0, key = 0;
  int64_t cached = -1;
  if constexpr (ZMODE == 1) key = sm_output(src.seed, (uint64_t)(src.first_id + probe));

  // the slot's next 16 entries from `base` of its row (start s, n entries):
  // row offsets (OFF32) or columns, and weights; past the end: out of range,
  // weight 0
  auto load16 = [&](int s, int n, int base, int& o, float& w) {
    const bool in = base + l16 < n;
    int j = 0;
    w = 0.f;
    if (in) {
      j = col[(int64_t)s + base + l16];
      if (!PATTERN) w = val[(int64_t)s + base + l16];
    }
    o = OFF32 ? (in ? (int)((uint32_t)j * kRowBytes) : (int)kOut) : j;
  };
  // N of those entries into acc; `after` issues what the wave needs next
  // behind the gathers
  auto sum_n = [&](auto nc, V& acc, int o, float w, int left, auto&& after) {
    constexpr int N = decltype(nc)::value;
    V x[N];
    static_for<N>([&](auto t) {
      constexpr int I = decltype(t)::value;
      if constexpr (OFF32)
        x[I] = rd.at((uint32_t)bcast16<I>(o));
      else
        x[I] = rd(bcast16<I>(o));
    });
    after();
    // every gather is in flight before the first is used
    __builtin_amdgcn_sched_barrier(0);
    static_for<N>([&](auto t) {
      constexpr int I = decltype(t)::value;
      if constexpr (!OFF32) x[I] = I < left ? x[I] : V{};
      const T wt = PATTERN ? T(1) : (T)__int_as_float(bcast16<I>(__float_as_int(w)));
#pragma unroll
      for (int e = 0; e < PPL; ++e) acc[e] = PATTERN ? acc[e] + x[I][e] : fma(wt, x[I][e], acc[e]);
    });
  };
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  using I16 = std::integral_constant<int, 16>;
  // the slots' sums over their n entries from s (n <= kHubChunk, uniform in a
  // slot), the first 16 already loaded; `last` as `after` of the last part
  auto sum_row = [&](V& acc, int s, int n, int o, float w, auto&& last) {
    int mx = 0;
#pragma unroll
    for (int k = 0; k < PPL; ++k) mx = max(mx, read_lane(n, k * LPR));
    int base = 0;
    while (mx - base > 16) {
      int on = 0;
      float wn = 0.f;
      sum_n(I16(), acc, o, w, n - base, [&] { load16(s, n, base + 16, on, wn); });
      o = on;
      w = wn;
      base += 16;
    }
    if (mx - base > 8) sum_n(I16(), acc, o, w, n - base, last);
    else if (mx - base > 4) sum_n(I8(), acc, o, w, n - base, last);
    else sum_n(I4(), acc, o, w, n - base, last);
  };
  // the slot's new row from its sum
  auto update = [&](int64_t row, const V& acc, const V& xi, const V& xp) {
    V vn;
#pragma unroll
    for (int e = 0; e < PPL; ++e) {
      if constexpr (OP == kOpStore) {
        vn[e] = acc[e];
      } else if constexpr (OP == kOpSlq) {
        vn[e] = sc[e] * acc[e];
      } else {
        T v = fma(ca, acc[e], cb * xi[e]);
        if (HAS_PREV) v -= xp[e];
        vn[e] = v;
      }
    }
    if constexpr (OP == kOpRec)
      __builtin_nontemporal_store(vn, reinterpret_cast<V*>(vm_l + row * 64));
    else
      *reinterpret_cast<V*>(vm_l + row * 64) = vn;
    return vn;
  };
  // moment partials of the wave's PPL rows from row0 on (zeros: no row): the
  // slots exchange their rows so that a lane has one probe of all of them,
  // and adds them in row order
  auto moments = [&](int64_t row0, V xi, V vn) {
    if constexpr (OP == kOpSlq) {
#pragma unroll
      for (int e = 0; e < PPL; ++e) xi[e] = sc[e] * xi[e];
    }
    slot_transpose(vn);
    if constexpr (ZMODE == 0) slot_transpose(xi);
#pragma unroll
    for (int r = 0; r < PPL; ++r) {
      if constexpr (ZMODE == 0) {
        m1 += (double)xi[r] * (double)vn[r];
        if constexpr (OP == kOpRec) m2 += (double)vn[r] * (double)vn[r];
      } else if constexpr (ZMODE == 1) {
        const int64_t c = (row0 + r) >> 6;
        if (c != cached) {
          word = sm_output(key, (uint64_t)c);
          cached = c;
        }
        m1 += sign_from_word<double>(word, row0 + r) * (double)vn[r];
      } else {
        const bool in = probe < src.active && row0 + r < r1;
        const double z = in ? (double)src.entries[(row0 + r) * src.ld + src.first_id + probe] : 0.0;
        m1 += z * (double)vn[r];
      }
    }
  };
  // V_k and V_prev of the slot's row (a hub row: its new row, already there)
  auto load_own = [&](int64_t row, bool hub, V& xi, V& xp) {
    if constexpr (OP != kOpStore) {
      xi = *reinterpret_cast<const V*>(own_l + row * 64);
      if (HAS_PREV || hub)
        xp = __builtin_nontemporal_load(reinterpret_cast<const V*>(vm_l + row * 64));
    }
  };

  if (hubs.n > 0 && r1 > r0) {
    __shared__ V shub[kSlots][LPR], scarry[LPR];
    const int slot = wave * PPL + q;
    int hr = hub_lower(hubs, r0);  // the first row not yet ended
    const int h1 = hub_lower(hubs, r1);
    if (h1 > hr) {
      const int ce = hubs.c0[h1];
      for (int c0 = hubs.c0[hr]; c0 < ce; c0 += kSlots) {
        // one chunk per slot
        const int c = c0 + slot;
        const int cs = c < ce ? hubs.cs[c] : 0;
        const int n = c < ce ? hubs.ce[c] - cs : 0;
        int o;
        float w;
        V acc = V{};
        load16(cs, n, 0, o, w);
        sum_row(acc, cs, n, o, w, [] {});
        shub[slot][sub] = acc;
        __syncthreads();
        // one row per slot: its chunks of this round behind what earlier
        // rounds left; the last row may go on in the next round
        const int h = hr + slot;
        const int b = h < h1 ? hubs.c0[h] : INT_MAX;
        bool ended = false;
        V tot = V{};
        if (b < c0 + kSlots) {
          const int e = hubs.c0[h + 1];
          ended = e <= c0 + kSlots;
          if (b < c0) tot = scarry[sub];
          const int j1 = min(e, c0 + kSlots) - c0;
          for (int j = max(b - c0, 0); j < j1; ++j) tot += shub[j][sub];
          if (ended) {
            const int64_t row = hubs.rows[h];
            V xi = V{}, xp = V{};
            load_own(row, false, xi, xp);
            update(row, tot, xi, xp);
          }
        }
        const int done = __syncthreads_count(ended && sub == 0);
        if (b < c0 + kSlots && !ended) scarry[sub] = tot;
        hr += done;
        // (the next round's first barrier orders the carry before its use)
      }
    }
  }

  // wave w takes the groups w, w + kWaves, ... of 1 << rsh rows, PPL at a time
  const int parts = (1 << rsh) / PPL;
  const int64_t ngrp = r1 > r0 ? (r1 - r0 + (1 << rsh) - 1) >> rsh : 0;
  const int64_t nk = ngrp > wave ? (ngrp - wave + kWaves - 1) / kWaves * parts : 0;
  auto first_row = [&](int64_t k) {
    return r0 + (((k / parts) * kWaves + wave) << rsh) + (k % parts) * PPL;
  };
  if (nk > 0) {
    // row, start and length of the slot's k-th row (length 0: none, or a row
    // that the hub pass took)
    auto extent = [&](int64_t k, int64_t& row, bool& live, bool& hub, int& s, int& n) {
      row = first_row(k) + q;
      live = row < r1;
      row = live ? row : r1 - 1;
      s = rowptr[row];
      n = live ? rowptr[row + 1] - s : 0;
      hub = n > kHubLen;
      if (hub) n = 0;
    };
    int64_t row, row_n = 0;
    bool live, hub, live_n = false, hub_n = false;
    int s, n, s_n = 0, n_n = 0;
    extent(0, row, live, hub, s, n);
    if (nk > 1) extent(1, row_n, live_n, hub_n, s_n, n_n);
    int o, o_n = 0;
    float w, w_n = 0.f;
    load16(s, n, 0, o, w);
    for (int64_t k = 0; k < nk; ++k) {
      V acc = V{}, xi = V{}, xp = V{};
      int64_t row_f = row;
      bool live_f = false, hub_f = false;
      int s_f = 0, n_f = 0;
      sum_row(acc, s, n, o, w, [&] {
        load_own(row, hub, xi, xp);
        load16(s_n, n_n, 0, o_n, w_n);
        if (k + 2 < nk) extent(k + 2, row_f, live_f, hub_f, s_f, n_f);
      });
      V vn = xp;
      if (live && !hub) vn = update(row, acc, xi, xp);
      if constexpr (OP != kOpStore) {
        if (!live) vn = xi = V{};
        moments(first_row(k), xi, vn);
      }
      row = row_n;
      live = live_n;
      hub = hub_n;
      s = s_n;
      n = n_n;
      o = o_n;
      w = w_n;
      row_n = row_f;
      live_n = live_f;
      hub_n = hub_f;
      s_n = s_f;
      n_n = n_f;
    }
  }
  if constexpr (OP != kOpStore)
    store_partials(m1, m2, g, plan.ngroups, part, probe);
}

// (at least 4 waves per SIMD, two workgroups per CU)
template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, bool OFF32>
__global__ __launch_bounds__(kThreads, 4) void csr_step_long_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, const T* __restrict__ vk, T* __restrict__ vm, T ca,
    T cb, ProbeSrc src, HubRows hubs, CsrStepPlan plan, double* __restrict__ part) {
  long_band<T, PATTERN, ZMODE, HAS_PREV, OFF32>(rowptr, col, val, d, d, vk, vk, vm, ca, cb, src,
                                                hubs, 2, plan, part,
                                                xcd_band(blockIdx.x, plan.ngroups));
}

// Gram step, first product: W = X V_k over X's rows (V_k has dv = X's
// column count rows).
template <typename T, bool PATTERN, bool OFF32>
__global__ __launch_bounds__(kThreads, 4) void gram_pass1_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t dv, const T* __restrict__ vk,
    T* __restrict__ W, HubRows hubs, CsrStepPlan plan) {
  long_band<T, PATTERN, 0, false, OFF32, kOpStore>(rowptr, col, val, d, dv, vk, vk, W, T(0), T(0),
                                                   ProbeSrc{}, hubs, 2, plan, nullptr,
                                                   xcd_band(blockIdx.x, plan.ngroups));
}

// Gram step, second product with the recurrence: V_new = ca X^T W + cb V_k
// [- V_prev] over X^T's rows, gathering from W, own rows from V_k.
template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, bool OFF32>
__global__ __launch_bounds__(kThreads, 4) void gram_pass2_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t dv, const T* __restrict__ W,
    const T* __restrict__ vk, T* __restrict__ vm, T ca, T cb, ProbeSrc src, HubRows hubs,
    int rsh, CsrStepPlan plan, double* __restrict__ part) {
  long_band<T, PATTERN, ZMODE, HAS_PREV, OFF32>(rowptr, col, val, d, dv, W, vk, vm, ca, cb, src,
                                                hubs, rsh, plan, part,
                                                xcd_band(blockIdx.x, plan.ngroups));
}

// Lanczos product u = s (A w): rows within the straight-line capacity take
// the wide form, others (MAXNZ 0) the form for rows of any length.
template <bool PATTERN, int MAXNZ, bool OFF32>
__global__ __launch_bounds__(kThreads) void slq_spmm_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    const float* __restrict__ val, int64_t d, int64_t nnz, const double* __restrict__ w,
    double* __restrict__ u, const double* __restrict__ sdev, HubRows hubs, CsrStepPlan plan,
    double* __restrict__ part) {
  const int g = xcd_band(blockIdx.x, plan.ngroups);
  if constexpr (MAXNZ > 0) {
    __shared__ WidePartials<double> sh;
    wide_band<double, PATTERN, 0, false, MAXNZ, false, true>(rowptr, col, val, d, nnz, w, u, 0.0,
                                                             0.0, ProbeSrc{}, plan, part, g, sh,
                                                             sdev);
  } else {
    long_band<double, PATTERN, 0, false, OFF32, kOpSlq>(rowptr, col, val, d, d, w, w, u, 0.0, 0.0,
                                                        ProbeSrc{}, hubs, 2, plan, part, g, sdev);
  }
}

// Equal-work row bands by binary search on rowptr[r] + kBandRowCost * r.
__global__ __launch_bounds__(256) void csr_band_kernel(const int32_t* __restrict__ rowptr,
                                                       int64_t d, int ngroups,
                                                       int32_t* __restrict__ band) {
  const int g = blockIdx.x * 256 + threadIdx.x;
  if (g > ngroups) return;
  const int64_t base = rowptr[0];
  const int64_t work = (int64_t)rowptr[d] - base + kBandRowCost * d;
  const int64_t target = work * g / ngroups;
  int64_t lo = 0, hi = d;  // f(d) = work >= target
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)rowptr[mid] - base + kBandRowCost * mid >= target) hi = mid;
    else lo = mid + 1;
  }
  band[g] = (int32_t)lo;
}

// Rows longer than kHubLen: (row, start, end) triples in any order; the host
// sorts them by row.
__global__ __launch_bounds__(256) void hub_find_kernel(const int32_t* __restrict__ rowptr,
                                                       int64_t d, int32_t* __restrict__ out,
                                                       int32_t* __restrict__ count, int cap) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < d;
       i += (int64_t)gridDim.x * 256) {
    const int32_t s = rowptr[i], e = rowptr[i + 1];
    if (e - s > kHubLen) {
      const int slot = atomicAdd(count, 1);
      if (slot < cap) {
        out[3 * (int64_t)slot] = (int32_t)i;
        out[3 * (int64_t)slot + 1] = s;
        out[3 * (int64_t)slot + 2] = e;
      }
    }
  }
}

// ---- batches of probe blocks over many operators -----------------------------
// One launch covers step s of every block in a table (blocks sorted by their
// number of steps, so the blocks still running at step s are a prefix).  Each
// block's workgroups are a contiguous, 8-aligned range of the grid; a
// workgroup finds its block by binary search over the ranges' starts.
__device__ __forceinline__ int find_block(const BatchBlock* __restrict__ tab, int n, int64_t bid) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tab[mid].group_base <= bid) lo = mid; else hi = mid - 1;
  }
  return lo;
}

template <bool PATTERN, int ZMODE, bool HAS_PREV, int MAXNZ>
__global__ __launch_bounds__(kThreads, MAXNZ == 0 ? 4 : 1) void csr_step_batched_kernel(
    const BatchBlock* __restrict__ tab, const int32_t* __restrict__ xblk,
    const int32_t* __restrict__ xg0, const int64_t* __restrict__ xbase, XcdLaunch xl, int s) {
  const int x = blockIdx.x & 7;
  const int64_t slot = blockIdx.x >> 3;
  if (slot >= xl.slots[x]) return;  // this XCD has no more work in the launch
  int lo = xl.first[x], hi = xl.first[x] + xl.count[x] - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (xbase[mid] <= slot) lo = mid; else hi = mid - 1;
  }
  const int bi = __builtin_amdgcn_readfirstlane(xblk[lo]);
  const BatchBlock& B = tab[bi];
  const int g = xg0[lo] + (int)(slot - xbase[lo]);  // band of the block
  const float* vk = (s - 1) & 1 ? B.v1 : B.v0;
  float* vm = s & 1 ? B.v1 : B.v0;
  const float ca = (float)(HAS_PREV ? 2.0 * B.alpha : B.alpha);
  const float cb = (float)(HAS_PREV ? 2.0 * B.beta : B.beta);
  const CsrStepPlan plan{B.ngroups, B.rows_per_group, B.band};
  double* part = B.part + (size_t)s * 2 * B.ngroups * 64;
  // the single-operator step's forms (same bits)
  if constexpr (MAXNZ > 0) {
    __shared__ WidePartials<float> sh;
    wide_band<float, PATTERN, ZMODE, HAS_PREV, MAXNZ, true>(B.rowptr, B.col, B.val, B.d, B.nnz, vk,
                                                             vm, ca, cb, B.src, plan, part, g, sh);
  } else {
    long_band<float, PATTERN, ZMODE, HAS_PREV, true>(B.rowptr, B.col, B.val, B.d, B.d, vk, vk, vm,
                                                     ca, cb, B.src,
                                                     B.hubs, 2, plan, part, g);
  }
}

// ---- one persistent launch for the steps of a batch ---------------------------
// Step 1 of every block runs as a plain batched launch; steps 2 .. S run in
// one launch whose grid is sized to be resident all at once (cooperative
// launch).  The workgroups of XCD x share that XCD's slot list (the layout
// of the batched launches): at step s, slots 0 .. slots_at[s][x] - 1 belong
// to the blocks still running, and workgroup j of the XCD takes slots j,
// j + P_x, ... .  Before a band of block b starts step s, every band of b
// must have finished step s - 1 (its vector is gathered from all rows); a
// band's arrival is counted in cnt[b] after its writes are released at
// device scope, and the wait acquires them.  A workgroup finishes all its
// step-(s - 1) slots before any step-s slot, so every wait ends once all
// workgroups are resident.  A wait longer than spin_ticks of the 100 MHz
// real-time clock (or a raised abort flag) sets the flag and ends the
// kernel, so no wave can wait forever.
struct PersistLaunch {
  int first[8];            // the XCD's first entry
  int count[8];            // its entries
  int per_xcd;             // workgroups per XCD in the grid
  int steps;               // largest step count
  const int64_t* slots_at; // [steps + 1][8] running slots per XCD and step
  int* cnt;                // [nblocks] band arrivals from step 2 on, zero at launch
  int* abort_flag;         // set on a wait that timed out
  long long spin_ticks;
};

__device__ __forceinline__ bool persist_wait(const PersistLaunch& pl, int blk, int target) {
  __shared__ int ok;
  if (threadIdx.x == 0) {
    const long long t0 = (long long)__builtin_amdgcn_s_memrealtime();
    ok = 1;
    while (__hip_atomic_load(pl.cnt + blk, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target) {
      if (__hip_atomic_load(pl.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
          (long long)__builtin_amdgcn_s_memrealtime() - t0 > pl.spin_ticks) {
        __hip_atomic_store(pl.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ok = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  __syncthreads();
  return ok != 0;
}

// ZMODE: the moment form of steps 2 .. S (0 symmetric, 1 direct).  A
// workgroup's consecutive slots of one block share one wait and one
// release (its arrivals are added together before it waits on another
// block or leaves the step).
template <bool PATTERN, int ZMODE, int MAXNZ>
__global__ __launch_bounds__(kThreads, MAXNZ == 0 ? 4 : 1) void csr_batch_persistent_kernel(
    const BatchBlock* __restrict__ tab, const int32_t* __restrict__ xblk,
    const int32_t* __restrict__ xg0, const int64_t* __restrict__ xbase, PersistLaunch pl) {
  const int x = blockIdx.x & 7;
  const int j = blockIdx.x >> 3;
  auto release = [&](int blk, int n) {
    __syncthreads();  // every wave's rows and partials are written
    if (threadIdx.x == 0)
      __hip_atomic_fetch_add(pl.cnt + blk, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  };
  for (int s = 2; s <= pl.steps; ++s) {
    const int64_t nslots = pl.slots_at[(size_t)s * 8 + x];
    int held = -1, pending = 0;  // block whose barrier this step has passed; arrivals owed
    for (int64_t slot = j; slot < nslots; slot += pl.per_xcd) {
      int lo = pl.first[x], hi = pl.first[x] + pl.count[x] - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (xbase[mid] <= slot) lo = mid; else hi = mid - 1;
      }
      const int bi = __builtin_amdgcn_readfirstlane(xblk[lo]);
      const BatchBlock& B = tab[bi];
      const int g = xg0[lo] + (int)(slot - xbase[lo]);
      if (bi != held) {
        if (pending) release(held, pending);
        pending = 0;
        if (s > 2 && !persist_wait(pl, bi, (s - 2) * B.ngroups)) return;
        held = bi;
      }
      const float* vk = (s - 1) & 1 ? B.v1 : B.v0;
      float* vm = s & 1 ? B.v1 : B.v0;
      const float ca = (float)(2.0 * B.alpha), cb = (float)(2.0 * B.beta);
      const CsrStepPlan plan{B.ngroups, B.rows_per_group, B.band};
      double* part = B.part + (size_t)s * 2 * B.ngroups * 64;
      if constexpr (MAXNZ > 0) {
        __shared__ WidePartials<float> sh;
        wide_band<float, PATTERN, ZMODE, true, MAXNZ, true>(B.rowptr, B.col, B.val, B.d, B.nnz, vk,
                                                             vm, ca, cb, B.src, plan, part, g, sh);
      } else {
        long_band<float, PATTERN, ZMODE, true, true>(B.rowptr, B.col, B.val, B.d, B.d, vk, vk, vm,
                                                     ca, cb, B.src,
                                                     B.hubs, 2, plan, part, g);
      }
      __syncthreads();  // the step body's shared partial buffer is reused
      ++pending;
    }
    if (pending) release(held, pending);
  }
}

__global__ void fill_zero_i32_kernel(int* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

__global__ __launch_bounds__(kThreads) void probe_init_batched_kernel(
    const BatchBlock* __restrict__ tab, int nblocks) {
  const int bi = __builtin_amdgcn_readfirstlane(find_block(tab, nblocks, blockIdx.x));
  const BatchBlock& B = tab[bi];
  const int bid = (int)(blockIdx.x - B.group_base);
  probe_init_wg<float>(B.v0, B.d, B.src, B.rows_per_group, B.ngroups, B.part, bid);
}

// Whether gathers from a block of dv rows can use 32-bit offsets (block under
// 4 GiB).
template <typename T>
bool block_off32(int64_t dv) {
  return (uint64_t)dv * 64 * sizeof(T) <= 0xFFFFFFFFull;
}

// Row capacity of the straight-line path: the smallest of {4, 5, 8} that
// holds the longest row, or 0 (rows of any length).  The straight-line path
// in FP64 (a verification precision) uses one general instantiation; else
// blocks under 4 GiB use 32-bit gather offsets.  F(MAXNZ, OFF32) launches one
// instantiation.
template <typename T, class F>
hipError_t dispatch_shape(const CsrMat& m, int64_t dv, F&& f) {
  using I0 = std::integral_constant<int, 0>;
  using I4 = std::integral_constant<int, 4>;
  using I5 = std::integral_constant<int, 5>;
  using I8 = std::integral_constant<int, 8>;
  using Yes = std::true_type;
  using No = std::false_type;
  if (m.nnz < 1 || m.max_row_nnz > 8)
    return block_off32<T>(dv) ? f(I0(), Yes()) : f(I0(), No());
  if constexpr (sizeof(T) == 4) {
    if (block_off32<T>(dv)) {
      if (m.max_row_nnz <= 4) return f(I4(), Yes());
      if (m.max_row_nnz <= 5) return f(I5(), Yes());
      return f(I8(), Yes());
    }
  }
  if (m.max_row_nnz <= 4) return f(I4(), No());
  if (m.max_row_nnz <= 5) return f(I5(), No());
  return f(I8(), No());
}

template <typename T, bool PATTERN, int ZMODE, bool HAS_PREV, int MAXNZ, bool OFF32>
hipError_t launch_step_t(hipStream_t s, const CsrMat& m, const T* vk, T* vm, T ca, T cb,
                         ProbeSrc src, const CsrStepPlan& plan, double* part) {
  const dim3 grid(plan.ngroups), block(kThreads);
  const CsrStepPlan p = banded(m, plan);
  if constexpr (MAXNZ == 0)
    csr_step_long_kernel<T, PATTERN, ZMODE, HAS_PREV, OFF32><<<grid, block, 0, s>>>(
        m.rowptr, m.col, m.val, m.nrows, vk, vm, ca, cb, src, hub_rows(m), p, part);
  else if constexpr (ZMODE <= 1)
    csr_step_wide_kernel<T, PATTERN, ZMODE, HAS_PREV, MAXNZ, OFF32><<<grid, block, 0, s>>>(
        m.rowptr, m.col, m.val, m.nrows, m.nnz, vk, vm, ca, cb, src, p, part);
  else
    csr_step_kernel<T, PATTERN, ZMODE, HAS_PREV, MAXNZ, OFF32><<<grid, block, 0, s>>>(
        m.rowptr, m.col, m.val, m.nrows, m.nnz, vk, vm, ca, cb, src, p, part);
  return hipGetLastError();
}

template <typename T, bool PATTERN, int ZMODE>
hipError_t launch_step_nz(hipStream_t s, const CsrMat& m, const T* vk, T* vm, T ca, T cb,
                          bool has_prev, ProbeSrc src, const CsrStepPlan& plan, double* part) {
  return dispatch_shape<T>(m, m.ncols, [&](auto mz, auto off32) {
    constexpr int MZ = decltype(mz)::value;
    constexpr bool O = decltype(off32)::value;
    return has_prev
               ? launch_step_t<T, PATTERN, ZMODE, true, MZ, O>(s, m, vk, vm, ca, cb, src, plan, part)
               : launch_step_t<T, PATTERN, ZMODE, false, MZ, O>(s, m, vk, vm, ca, cb, src, plan,
                                                                part);
  });
}

template <typename T>
hipError_t launch_step_any(hipStream_t s, const CsrMat& m, const T* vk, T* vm, T ca, T cb,
                           bool has_prev, int zmode, ProbeSrc src, const CsrStepPlan& plan,
                           double* part) {
  const bool pat = m.val == nullptr;
  if (pat) {
    if (zmode == 0) return launch_step_nz<T, true, 0>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
    if (zmode == 1) return launch_step_nz<T, true, 1>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
    return launch_step_nz<T, true, 2>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
  }
  if (zmode == 0) return launch_step_nz<T, false, 0>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
  if (zmode == 1) return launch_step_nz<T, false, 1>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
  return launch_step_nz<T, false, 2>(s, m, vk, vm, ca, cb, has_prev, src, plan, part);
}

// The two products of a Gram step for one pattern/valued and z-mode choice.
template <typename T, bool PATTERN, int ZMODE>
hipError_t launch_gram_z(hipStream_t s, const CsrMat& X, const CsrMat& XT, const T* vk, T* vm,
                         T* W, T ca, T cb, bool has_prev, ProbeSrc src,
                         const CsrStepPlan& pr, const CsrStepPlan& pc, double* part) {
  auto pass1 = [&](auto off32) {
    gram_pass1_kernel<T, PATTERN, decltype(off32)::value><<<pr.ngroups, kThreads, 0, s>>>(
        X.rowptr, X.col, X.val, X.nrows, X.ncols, vk, W, hub_rows(X), banded(X, pr));
    return hipGetLastError();
  };
  const int rsh = XT.nnz > 0 && XT.max_row_nnz <= 5 ? 3 : 2;  // as the CSR step's groups
  auto pass2 = [&](auto prev, auto off32) {
    gram_pass2_kernel<T, PATTERN, ZMODE, decltype(prev)::value, decltype(off32)::value>
        <<<pc.ngroups, kThreads, 0, s>>>(XT.rowptr, XT.col, XT.val, XT.nrows, XT.ncols, W, vk, vm,
                                         ca, cb, src, hub_rows(XT), rsh, banded(XT, pc),
                                         part);
    return hipGetLastError();
  };
  using Yes = std::true_type;
  using No = std::false_type;
  const hipError_t e = block_off32<T>(X.ncols) ? pass1(Yes()) : pass1(No());
  if (e != hipSuccess) return e;
  if (block_off32<T>(XT.ncols)) return has_prev ? pass2(Yes(), Yes()) : pass2(No(), Yes());
  return has_prev ? pass2(Yes(), No()) : pass2(No(), No());
}

// ---- two recurrence steps per launch ------------------------------------------
// For operators whose rows have at most 5 entries and whose columns lie
// within a bandwidth of the row (every column of a row in tile j lies in
// tiles j - w .. j + w), one launch applies the recurrence (Section 2.2, eq.
// eqn:recurrence) twice:
//   sub-step 1 on tile j: V_{s+1} = ca1 A V_s + cb1 V_s (- V_{s-1}) over V_{s-1}
//   sub-step 2 on tile j: V_{s+2} = ca2 A V_{s+1} + cb2 V_{s+1} - V_s  over V_s
// each tile through csr_step_wg, the single-step kernel's body, so every
// vector entry is bitwise the single-step path's (only the association of
// the FP64 moment sums follows the tiles).
//
// Work order: the tiles are split into eight contiguous ranges, one per XCD
// (read from the hardware XCC_ID register), and the workgroups of an XCD
// take tickets from that XCD's counter: sub-step 1 of its first L tiles,
// then alternately one sub-step 2 and the sub-step 1 L tiles ahead; the
// sub-steps 2 run from the range's tile w upward and its first w tiles come
// last.  With L > 2 w every sub-step 2 of the range was issued after the
// sub-steps 1 it gathers from inside the range; the first w tiles, which
// also gather from the top of the range below, wait for it at the end.
// Sub-steps 1 never wait, so every wait ends whether or not all workgroups
// are resident; waits are bounded by the real-time clock and an abort flag
// besides.  The lag L (chosen > 2 w + 64) leaves a tile's neighbours time to
// finish before its sub-step 2 claims them; V_{s+1} and V_s are then still
// in the memory-side cache, so the block vectors cross HBM about four times
// per two steps instead of six.
//
// Coherence: within an XCD a writer's stores complete (to the XCD's L2)
// before its tile flag is set, and a waiter polls the flags past its L1 and
// invalidates its L1 before gathering.  Tiles read by another XCD (the
// first and last w of a range) are released and acquired at device scope.
struct Fused2Args {
  const int32_t* rowptr;
  const int32_t* col;
  const float* val;
  int64_t d, nnz;
  float* x;  // V_{s-1} in, V_{s+1} out
  float* y;  // V_s in, V_{s+2} out
  float ca1, cb1, ca2, cb2;
  ProbeSrc src;
  int rows_per_tile, ntiles, window, lag;
  int two;        // 1: both sub-steps; 0: sub-step 1 only
  double* part1;  // [2][ntiles][64] partials of sub-step 1
  double* part2;  // [2][ntiles][64] partials of sub-step 2
  int* tickets;   // [8] ticket counters, zero at launch
  int* done;      // [ntiles] sub-step 1 completion flags, zero at launch
  int* abort_flag;
  long long spin_ticks;
};

// Ticket k of an XCD's range of per tiles -> (sub-step, tile in the range).
__device__ __forceinline__ void fused_ticket(int k, int per, int lag, int w, int two, int& sub,
                                             int& t) {
  if (!two) {
    sub = 1;
    t = k;
    return;
  }
  const int L = min(lag, per);
  if (k < L) {
    sub = 1;
    t = k;
    return;
  }
  const int m = k - L;
  const int pairs = per - L;
  int j;
  if (m < 2 * pairs) {
    if (m & 1) {
      sub = 1;
      t = (m >> 1) + L;
      return;
    }
    j = m >> 1;
  } else {
    j = pairs + (m - 2 * pairs);
  }
  sub = 2;
  t = j + w < per ? j + w : j + w - per;
}

// Thread 0 waits for the flags of tiles t0 .. t1; far: some lie in another
// XCD's range (acquire at device scope), else the L1 is invalidated.
__device__ __forceinline__ bool fused_wait(const Fused2Args& a, int t0, int t1, bool far) {
  __shared__ int ok;
  if (threadIdx.x == 0) {
    ok = 1;
    const long long c0 = (long long)__builtin_amdgcn_s_memrealtime();
    for (int t = t0; t <= t1 && ok; ++t) {
      while (__hip_atomic_load(a.done + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
        if (__hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
            (long long)__builtin_amdgcn_s_memrealtime() - c0 > a.spin_ticks) {
          __hip_atomic_store(a.abort_flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    if (far)
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    else
      asm volatile("buffer_inv sc0" ::: "memory");
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(ok) != 0;
}

template <bool PATTERN, int Z1, int Z2, bool PREV1, int MAXNZ, bool OFF32>
__global__ __launch_bounds__(kThreads) void csr_fused2_kernel(Fused2Args a) {
  __shared__ int tk;
  const int xcd = xcc_of_wg();
  const int per = a.ntiles >> 3;
  const int base = xcd * per;
  const int total = a.two ? 2 * per : per;
  const int w = a.window;
  CsrStepPlan plan;
  plan.ngroups = a.ntiles;
  plan.rows_per_group = a.rows_per_tile;
  plan.band = nullptr;
  // Thread 0 sets the flag of the sub-step-1 tile just done and claims the
  // next ticket in one block at the loop head, and the ticket is made
  // wave-uniform: the loop's control flow is then uniform, so no lane of
  // wave 0 can be split off into a loop of its own (two adjacent thread-0
  // blocks let the compiler send the other lanes straight back to the
  // barrier, where they re-read the old ticket).
  int pending = -1;
  bool pending_far = false;
  while (true) {
    if (threadIdx.x == 0) {
      if (pending >= 0) {
        if (pending_far)
          __hip_atomic_store(a.done + pending, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        else
          __hip_atomic_store(a.done + pending, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      tk = atomicAdd(a.tickets + xcd, 1);
    }
    __syncthreads();
    const int k = __builtin_amdgcn_readfirstlane(tk);
    __syncthreads();  // tk is rewritten by the next claim
    if (k >= total) break;
    int sub, t;
    fused_ticket(k, per, a.lag, w, a.two, sub, t);
    const int bid = t * 8 + xcd;  // the workgroup index whose band is tile base + t
    if (sub == 1) {
      RecEpi<float, Z1, PREV1, true, 4> epi(a.ca1, a.cb1, a.x, a.src);
      csr_step_wg<float, PATTERN, MAXNZ, OFF32>(a.rowptr, a.col, a.val, a.d, a.nnz,
                                                RowReader<float, OFF32>(a.y, a.d, lane_id()), epi,
                                                plan, a.part1, bid);
      // every wave's stores complete (in L2) before the flag is set
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      pending = base + t;
      pending_far = t < w || t >= per - w;
    } else {
      pending = -1;
      const int tile = base + t;
      const int t0 = max(0, tile - w), t1 = min(a.ntiles - 1, tile + w);
      if (!fused_wait(a, t0, t1, t0 < base || t1 >= base + per)) break;
      RecEpi<float, Z2, true, false, 4> epi(a.ca2, a.cb2, a.y, a.src);
      csr_step_wg<float, PATTERN, MAXNZ, OFF32>(a.rowptr, a.col, a.val, a.d, a.nnz,
                                                RowReader<float, OFF32>(a.x, a.d, lane_id()), epi,
                                                plan, a.part2, bid);
    }
  }
}

}  // namespace

CsrStepPlan plan_csr(int64_t d, int max_groups) {
  // the cap is a multiple of 8 so that every XCD band gets whole workgroups
  const int64_t cap = max_groups > 0 ? std::max<int64_t>(8, max_groups / 8 * 8) : 2048;
  int64_t g = (d + 255) / 256;
  g = (g + 7) / 8 * 8;
  if (g > cap) g = cap;
  if (g < 8) g = 8;
  CsrStepPlan p;
  p.ngroups = (int)g;
  p.rows_per_group = (int)((d + g - 1) / g);
  return p;
}

template <typename T>
hipError_t launch_probe_init(hipStream_t s, T* v0, int64_t d, ProbeSrc src,
                             const CsrStepPlan& plan, double* part0) {
  probe_init_kernel<T><<<dim3(plan.ngroups), dim3(kThreads), 0, s>>>(
      v0, d, src, plan.rows_per_group, plan.ngroups, part0);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_csr_step(hipStream_t s, const CsrMat& m, const T* vk, T* vm, T ca, T cb,
                           bool has_prev, int zmode, ProbeSrc src, const CsrStepPlan& plan,
                           double* part) {
  return launch_step_any<T>(s, m, vk, vm, ca, cb, has_prev, zmode, src, plan, part);
}

template <typename T>
hipError_t launch_gram_csr_step(hipStream_t s, const CsrMat& X, const CsrMat& XT, const T* vk,
                                T* vm, T* W, T ca, T cb, bool has_prev, int zmode, ProbeSrc src,
                                const CsrStepPlan& plan_rows, const CsrStepPlan& plan_cols,
                                double* part) {
#define MLCT_GZ(P, Z)                                                                       \
  return launch_gram_z<T, P, Z>(s, X, XT, vk, vm, W, ca, cb, has_prev, src, plan_rows,      \
                                plan_cols, part)
  if (X.val == nullptr) {
    if (zmode == 0) MLCT_GZ(true, 0);
    if (zmode == 1) MLCT_GZ(true, 1);
    MLCT_GZ(true, 2);
  }
  if (zmode == 0) MLCT_GZ(false, 0);
  if (zmode == 1) MLCT_GZ(false, 1);
  MLCT_GZ(false, 2);
#undef MLCT_GZ
}

hipError_t launch_slq_spmm(hipStream_t s, const CsrMat& m, const double* w, double* u,
                           const double* sdev, const CsrStepPlan& plan, double* part) {
  return dispatch_shape<double>(m, m.ncols, [&](auto mz, auto off32) {
    constexpr int MZ = decltype(mz)::value;
    constexpr bool O = decltype(off32)::value;
    if (m.val == nullptr)
      slq_spmm_kernel<true, MZ, O><<<plan.ngroups, kThreads, 0, s>>>(
          m.rowptr, m.col, m.val, m.nrows, m.nnz, w, u, sdev, hub_rows(m), banded(m, plan), part);
    else
      slq_spmm_kernel<false, MZ, O><<<plan.ngroups, kThreads, 0, s>>>(
          m.rowptr, m.col, m.val, m.nrows, m.nnz, w, u, sdev, hub_rows(m), banded(m, plan), part);
    return hipGetLastError();
  });
}

hipError_t launch_csr_bands(hipStream_t s, const int32_t* rowptr, int64_t d, int ngroups,
                            int32_t* band) {
  csr_band_kernel<<<(ngroups + 1 + 255) / 256, 256, 0, s>>>(rowptr, d, ngroups, band);
  return hipGetLastError();
}

hipError_t launch_hub_find(hipStream_t s, const int32_t* rowptr, int64_t d, int32_t* out,
                           int32_t* count, int cap) {
  const int64_t blocks = std::min<int64_t>((d + 255) / 256, 4096);
  hub_find_kernel<<<(int)blocks, 256, 0, s>>>(rowptr, d, out, count, cap);
  return hipGetLastError();
}

hipError_t launch_probe_init_batched(hipStream_t s, const BatchBlock* tab, int nblocks,
                                     int64_t total_groups) {
  probe_init_batched_kernel<<<(unsigned)total_groups, kThreads, 0, s>>>(tab, nblocks);
  return hipGetLastError();
}

hipError_t launch_csr_step_batched(hipStream_t s, const BatchBlock* tab, const int32_t* xblk,
                                   const int32_t* xg0, const int64_t* xbase,
                                   const XcdLaunch& xl, int64_t groups, int step, bool pattern,
                                   int maxnz, int zmode) {
  const bool hp = step > 1;
  const unsigned grid = (unsigned)groups;
#define MLCT_BATCH(P, Z, H, M) \
  csr_step_batched_kernel<P, Z, H, M><<<grid, kThreads, 0, s>>>(tab, xblk, xg0, xbase, xl, step)
#define MLCT_BATCH_M(P, Z, H)                  \
  if (maxnz <= 4) MLCT_BATCH(P, Z, H, 4);      \
  else if (maxnz <= 5) MLCT_BATCH(P, Z, H, 5); \
  else if (maxnz <= 8) MLCT_BATCH(P, Z, H, 8); \
  else MLCT_BATCH(P, Z, H, 0)
#define MLCT_BATCH_H(P, Z) \
  if (hp) { MLCT_BATCH_M(P, Z, true); } else { MLCT_BATCH_M(P, Z, false); }
#define MLCT_BATCH_Z(P) \
  if (zmode == 0) { MLCT_BATCH_H(P, 0); } else { MLCT_BATCH_H(P, 1); }
  if (pattern) { MLCT_BATCH_Z(true); } else { MLCT_BATCH_Z(false); }
#undef MLCT_BATCH_Z
#undef MLCT_BATCH_H
#undef MLCT_BATCH_M
#undef MLCT_BATCH
  return hipGetLastError();
}

hipError_t launch_csr_batch_persistent(hipStream_t s, const BatchBlock* tab,
                                       const int32_t* xblk, const int32_t* xg0,
                                       const int64_t* xbase, const XcdLaunch& xl, int steps,
                                       const int64_t* slots_at, int* cnt, int nblocks,
                                       int* abort_flag, int per_xcd, bool pattern, int maxnz,
                                       int zmode, long long spin_ticks) {
  const int64_t nz = nblocks + 1;
  fill_zero_i32_kernel<<<(unsigned)((nz + 255) / 256), 256, 0, s>>>(cnt, nblocks);
  fill_zero_i32_kernel<<<1, 64, 0, s>>>(abort_flag, 1);
  PersistLaunch pl;
  for (int x = 0; x < 8; ++x) {
    pl.first[x] = xl.first[x];
    pl.count[x] = xl.count[x];
  }
  pl.per_xcd = per_xcd;
  pl.steps = steps;
  pl.slots_at = slots_at;
  pl.cnt = cnt;
  pl.abort_flag = abort_flag;
  pl.spin_ticks = spin_ticks;
  void* args[] = {(void*)&tab, (void*)&xblk, (void*)&xg0, (void*)&xbase, (void*)&pl};
  const dim3 grid((unsigned)(8 * per_xcd)), block(kThreads);
#define MLCT_PERSIST(P, Z, M)                                                          \
  return hipLaunchCooperativeKernel((const void*)csr_batch_persistent_kernel<P, Z, M>, \
                                    grid, block, args, 0, s)
#define MLCT_PERSIST_M(P, Z)                  \
  if (maxnz <= 4) MLCT_PERSIST(P, Z, 4);      \
  else if (maxnz <= 5) MLCT_PERSIST(P, Z, 5); \
  else if (maxnz <= 8) MLCT_PERSIST(P, Z, 8); \
  else MLCT_PERSIST(P, Z, 0)
#define MLCT_PERSIST_Z(P) \
  if (zmode == 0) { MLCT_PERSIST_M(P, 0); } else { MLCT_PERSIST_M(P, 1); }
  if (pattern) { MLCT_PERSIST_Z(true); } else { MLCT_PERSIST_Z(false); }
#undef MLCT_PERSIST_Z
#undef MLCT_PERSIST_M
#undef MLCT_PERSIST
}

int csr_batch_persistent_per_xcd(bool pattern, int maxnz, int zmode) {
  int per_cu = 0;
  hipError_t e = hipSuccess;
#define MLCT_OCC(P, Z, M)                           \
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor( \
      &per_cu, (const void*)csr_batch_persistent_kernel<P, Z, M>, kThreads, 0)
#define MLCT_OCC_M(P, Z)                  \
  if (maxnz <= 4) MLCT_OCC(P, Z, 4);      \
  else if (maxnz <= 5) MLCT_OCC(P, Z, 5); \
  else if (maxnz <= 8) MLCT_OCC(P, Z, 8); \
  else MLCT_OCC(P, Z, 0)
#define MLCT_OCC_Z(P) \
  if (zmode == 0) { MLCT_OCC_M(P, 0); } else { MLCT_OCC_M(P, 1); }
  if (pattern) { MLCT_OCC_Z(true); } else { MLCT_OCC_Z(false); }
#undef MLCT_OCC_Z
#undef MLCT_OCC_M
#undef MLCT_OCC
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return per_cu * cus / 8;
}


hipError_t launch_csr_fused2(hipStream_t s, const CsrMat& m, float* x, float* y, float ca1,
                             float cb1, bool prev1, float ca2, float cb2, bool two, int zm1,
                             int zm2, ProbeSrc src, int rows_per_tile, int ntiles, int window,
                             double* part1, double* part2, int* sync, int* abort_flag,
                             int grid, int lag, int prev_total, long long spin_ticks) {
  // sync: [8] tickets, [ntiles] flags, cleared for every launch (after the
  // previous launch's counters are checked)
  hipError_t e = launch_fused_sync(s, sync, 8 + (int64_t)ntiles, prev_total, abort_flag);
  if (e != hipSuccess) return e;
  Fused2Args a;
  a.rowptr = m.rowptr;
  a.col = m.col;
  a.val = m.val;
  a.d = m.nrows;
  a.nnz = m.nnz;
  a.x = x;
  a.y = y;
  a.ca1 = ca1;
  a.cb1 = cb1;
  a.ca2 = ca2;
  a.cb2 = cb2;
  a.src = src;
  a.rows_per_tile = rows_per_tile;
  a.ntiles = ntiles;
  a.window = window;
  a.lag = lag;
  a.two = two ? 1 : 0;
  a.part1 = part1;
  a.part2 = part2;
  a.tickets = sync;
  a.done = sync + 8;
  a.abort_flag = abort_flag;
  a.spin_ticks = spin_ticks;
  const bool pat = m.val == nullptr;
  const bool off32 = block_off32<float>(m.ncols);
  const int mz = m.max_row_nnz <= 4 ? 4 : 5;
  const dim3 g(grid), b(kThreads);
#define MLCT_F(P, Z1, Z2, PV, M, O) csr_fused2_kernel<P, Z1, Z2, PV, M, O><<<g, b, 0, s>>>(a)
#define MLCT_F_O(P, Z1, Z2, PV, M) \
  if (off32) { MLCT_F(P, Z1, Z2, PV, M, true); } else { MLCT_F(P, Z1, Z2, PV, M, false); }
#define MLCT_F_M(P, Z1, Z2, PV) \
  if (mz == 4) { MLCT_F_O(P, Z1, Z2, PV, 4) } else { MLCT_F_O(P, Z1, Z2, PV, 5) }
#define MLCT_F_PV(P, Z1, Z2) \
  if (prev1) { MLCT_F_M(P, Z1, Z2, true) } else { MLCT_F_M(P, Z1, Z2, false) }
#define MLCT_F_Z(P)                                            \
  if (zm1 == 0 && zm2 == 0) { MLCT_F_PV(P, 0, 0) }             \
  else if (zm1 == 0) { MLCT_F_PV(P, 0, 1) }                    \
  else { MLCT_F_PV(P, 1, 1) }
  if (pat) { MLCT_F_Z(true) } else { MLCT_F_Z(false) }
#undef MLCT_F_Z
#undef MLCT_F_PV
#undef MLCT_F_M
#undef MLCT_F_O
#undef MLCT_F
  return hipGetLastError();
}

template hipError_t launch_probe_init<float>(hipStream_t, float*, int64_t, ProbeSrc,
                                             const CsrStepPlan&, double*);
template hipError_t launch_probe_init<double>(hipStream_t, double*, int64_t, ProbeSrc,
                                              const CsrStepPlan&, double*);
template hipError_t launch_csr_step<float>(hipStream_t, const CsrMat&, const float*, float*,
                                           float, float, bool, int, ProbeSrc,
                                           const CsrStepPlan&, double*);
template hipError_t launch_csr_step<double>(hipStream_t, const CsrMat&, const double*,
                                            double*, double, double, bool, int, ProbeSrc,
                                            const CsrStepPlan&, double*);
template hipError_t launch_gram_csr_step<float>(hipStream_t, const CsrMat&, const CsrMat&,
                                                const float*, float*, float*, float, float, bool,
                                                int, ProbeSrc, const CsrStepPlan&,
                                                const CsrStepPlan&, double*);
template hipError_t launch_gram_csr_step<double>(hipStream_t, const CsrMat&, const CsrMat&,
                                                 const double*, double*, double*, double, double,
                                                 bool, int, ProbeSrc, const CsrStepPlan&,
                                                 const CsrStepPlan&, double*);

}  // namespace mlct
