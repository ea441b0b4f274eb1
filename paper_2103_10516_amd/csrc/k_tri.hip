// Exact triangle-count moments over a 0/1 pattern CSR (Section 2.1 example
// and footnote, Section 5.4).  Per probe z, two integer SpMMs:
//   pass 1: y = A z   (int16 rows with exact escapes, stored)
//   pass 2: w = A y   (int32, never stored), and in int64
//           w1 += z_i y_i, w2 += y_i^2, w3 += y_i w_i
//
// Layout: probes in groups of up to 512, 64 a panel.  z is one sign word of
// 64 bits per row and panel (bit p: probe p is -1), the panels of a row side
// by side; y is one array of d x 128 int16 per two panels (of d x 64 for a last
// odd one).  A wave works on four
// rows at a time, 16 lanes (a slot) each, as the recurrence on long rows does;
// the rows longer than kHubLen are cut into chunks that the slots of their
// band's workgroup share.  All sums are exact integers, so their order is
// free.
#include <algorithm>
#include <climits>

#include "device.hpp"

namespace mlct {

namespace {

constexpr int kWaves = 8;
constexpr int kThreads = kWaves * 64;
constexpr int kSlots = kWaves * 4;
// probes of a panel, panels of a group
constexpr int kPanel = 64;

// |y_i| is at most the row's length: values past +-32767 can only sit in rows
// that long, which are hub rows.  They are stored as this sentinel, the exact
// value in the hub's row of a side table.
constexpr int32_t kY16Sentinel = -32768;
struct HubSide {
  const int32_t* rows;  // sorted hub row ids
  int n;
  int32_t* side;        // [panel][n][64], in the order of y's rows
  __device__ __forceinline__ int slot(int64_t i) const {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (rows[mid] < i) lo = mid + 1; else hi = mid;
    }
    return lo;
  }
};

typedef short s2 __attribute__((ext_vector_type(2)));
typedef int i4 __attribute__((ext_vector_type(4)));

// y's unit u: panels 2u and 2u + 1 side by side in rows of 128, or a last odd
// panel in rows of 64.
__host__ __device__ inline int64_t unit_base(int64_t d, int u) { return (int64_t)u * 2 * d * kPanel; }

// y's rows hold a panel's probes as 32-bit pairs (p, p + 16) of each half
// panel, the form in which pass 1 takes them from its bit planes: the probe
// at position s of a row.
__host__ __device__ constexpr int probe_at(int s) {
  return (s & 32) + ((s & 31) >> 1) + 16 * (s & 1);
}

// z packed: a wave makes the words of 64 probes for 64 rows (lane p: probe
// p's signs of the 64 rows) and transposes the 64 x 64 bits, so that lane i
// holds row i's word (a ballot per row took 8 times the instructions: 36 ->
// 6 us for 64 probes of 10^6 rows).  Probes past src.active get +1, which
// only their own, discarded, sums see.
__global__ __launch_bounds__(256) void tri_init_kernel(uint64_t* __restrict__ zbits, int64_t d,
                                                       ProbeSrc src, int panels,
                                                       uint32_t* __restrict__ escapes) {
  const int lane = lane_id();
  if (blockIdx.x == 0 && threadIdx.x == 0) *escapes = 0;
  const int64_t nchunk = (d + 63) >> 6;
  const int64_t nw = (int64_t)gridDim.x * 4;
  for (int64_t u = (int64_t)blockIdx.x * 4 + wave_id(); u < nchunk * panels; u += nw) {
    const int panel = (int)(u % panels);
    const int64_t c = u / panels;
    const int p = panel * kPanel + lane;
    uint64_t x = 0;
    if (p < src.active)
      x = sm_output(sm_output(src.seed, (uint64_t)(src.first_id + p)), (uint64_t)c);
    uint64_t m = 0x00000000FFFFFFFFull;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
      const uint64_t o = __shfl_xor(x, s, 64);
      x = (lane & s) ? ((x & ~m) | ((o & ~m) >> s)) : ((x & m) | ((o & m) << s));
      m ^= m << (s >> 1);
    }
    const int64_t i = c * 64 + lane;
    if (i < d) zbits[i * panels + panel] = x;
  }
}

// Sum over the entries of mix(i, j) - mix(j, i) modulo 2^64, one partial per
// workgroup: 0 for a symmetric pattern (and with probability 2^-64 for
// another), which lets pass 2 take each edge once.
// A unit of work is a row, or a chunk of a row longer than kHubLen.
__global__ __launch_bounds__(256) void tri_sym_kernel(const int32_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ col, int64_t d,
                                                      HubRows hubs, int chunks,
                                                      uint64_t* __restrict__ part) {
  __shared__ uint64_t sh;
  if (threadIdx.x == 0) sh = 0;
  __syncthreads();
  uint64_t s = 0;
  const int64_t nslot = (int64_t)gridDim.x * 16;
  for (int64_t u = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); u < d + chunks; u += nslot) {
    const bool row = u < d;
    const uint64_t i = row ? (uint64_t)u : (uint64_t)hubs.cr[u - d];
    // (64-bit entries: the last row may end at INT32_MAX)
    const int64_t b = row ? rowptr[u] : hubs.cs[u - d];
    int n = (int)((row ? rowptr[u + 1] : hubs.ce[u - d]) - b);
    if (row && n > kHubLen) n = 0;
    for (int t = (int)(threadIdx.x & 15); t < n; t += 16) {
      const uint64_t j = (uint64_t)(uint32_t)col[b + t];
      s += sm_mix((i << 32 | j) + kGamma) - sm_mix((j << 32 | i) + kGamma);
    }
  }
  atomicAdd((unsigned long long*)&sh, (unsigned long long)s);
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = sh;
}

__global__ __launch_bounds__(256) void tri_sym_sum_kernel(const uint64_t* __restrict__ part, int n,
                                                          uint64_t* __restrict__ out) {
  __shared__ uint64_t sh;
  if (threadIdx.x == 0) sh = 0;
  __syncthreads();
  uint64_t s = 0;
  for (int b = threadIdx.x; b < n; b += 256) s += part[b];
  atomicAdd((unsigned long long*)&sh, (unsigned long long)s);
  __syncthreads();
  if (threadIdx.x == 0) *out = sh;
}

// (h, l) = a + b + c, bitwise
__device__ __forceinline__ void csa(uint32_t& h, uint32_t& l, uint32_t a, uint32_t b, uint32_t c) {
  const uint32_t u = a ^ b;
  h = (a & b) | (u & c);
  l = u ^ c;
}

// Vertical counters of 32 probes: bit b of plane k is bit k of probe b's
// count of set bits among the words added so far (at most 256).
struct Planes {
  uint32_t p[9] = {};
  __device__ __forceinline__ void add16(const uint32_t (&x)[16]) {
    uint32_t t[8], f[4], e[2], c;
#pragma unroll
    for (int i = 0; i < 8; ++i) csa(t[i], p[0], p[0], x[2 * i], x[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 4; ++i) csa(f[i], p[1], p[1], t[2 * i], t[2 * i + 1]);
#pragma unroll
    for (int i = 0; i < 2; ++i) csa(e[i], p[2], p[2], f[2 * i], f[2 * i + 1]);
    csa(c, p[3], p[3], e[0], e[1]);
#pragma unroll
    for (int k = 4; k < 9; ++k) {
      const uint32_t n = p[k] & c;
      p[k] ^= c;
      c = n;
    }
  }
  // the counts as 16-bit pairs (probe i, probe i + 16); nb: planes in use
  __device__ __forceinline__ void counts(int nb, uint32_t (&c)[16]) const {
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = 0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      if (k >= nb) break;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        c[i] |= (i >= k ? p[k] >> (i - k) : p[k] << (k - i)) & (0x00010001u << k);
    }
  }
};

__device__ __forceinline__ s2 as_s2(uint32_t v) { return __builtin_bit_cast(s2, v); }
__device__ __forceinline__ uint32_t as_u32(s2 v) { return __builtin_bit_cast(uint32_t, v); }
// c + the low / high half of v
__device__ __forceinline__ int add_lo(s2 v, int c) {
  return __builtin_amdgcn_sdot2(v, s2{1, 0}, c, false);
}
__device__ __forceinline__ int add_hi(s2 v, int c) {
  return __builtin_amdgcn_sdot2(v, s2{0, 1}, c, false);
}

// Pass 1.  A lane holds 32 probes' signs of a gathered row in one word and
// counts the set bits of a row's entries in vertical counters (carry-save
// adders: about 2.5 logic operations per word), so y = length - 2 count for
// 512 probes costs about 2 instructions per entry, where summing +-1 with
// lane = probe took 18 for 64; the passes were bound by issuing those.
// Measured (Chung-Lu d = 10^6, 16M entries, us for 512 probes, with the launch
// for the long rows' chunks before): 4,490 -> 739, of which y's store 365.
__global__ __launch_bounds__(kThreads, 4) void tri_pass1_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t d,
    const uint32_t* __restrict__ zbits, int panels, int16_t* __restrict__ y, HubSide hs,
    HubRows hubs, CsrStepPlan plan, uint32_t* __restrict__ escapes) {
  const int lane = lane_id(), wave = wave_id();
  const int q = lane >> 4, l16 = lane & 15;
  const int words = 2 * panels;  // of 32 probes, per row
  const bool act = l16 < words;
  const int g = xcd_band(blockIdx.x, plan.ngroups);
  const int64_t r0 = plan.band ? (int64_t)plan.band[g] : (int64_t)g * plan.rows_per_group;
  const int64_t r1 = plan.band ? (int64_t)plan.band[g + 1]
                               : min<int64_t>(r0 + plan.rows_per_group, d);
  __shared__ union {
    uint32_t sc[kSlots][16][17];
    i4 out[kWaves][64][5];  // the lanes' 64 bytes of y (padded)
  } sh;
  const uint32_t row_bytes = (uint32_t)words * 4;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(zbits), (short)0,
                                                      (int)((uint32_t)d * row_bytes), 0x00020000);
  // lanes past the group's words repeat lane 0's (and are not used)
  const uint32_t lane_off = act ? (uint32_t)l16 * 4 : 0;
  // past the array, whatever the lane adds
  const uint32_t out = 0u - row_bytes;
  const int pairs = panels >> 1;

  // offsets of the slot's next 16 entries (past its end: out of range, reads 0)
  auto load16 = [&](int s, int n, int base) -> int {
    const bool in = base + l16 < n;
    return in ? (int)((uint32_t)col[(int64_t)s + base + l16] * row_bytes) : (int)out;
  };
  auto gather = [&](auto nc, Planes& pl, int o, auto&& after) {
    constexpr int N = decltype(nc)::value;
    uint32_t x[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) x[t] = 0;
    static_for<N>([&](auto t) {
      constexpr int I = decltype(t)::value;
      x[I] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (uint32_t)bcast16<I>(o) + lane_off, 0, 0);
    });
    after();
    __builtin_amdgcn_sched_barrier(0);
    pl.add16(x);
  };
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  using I16 = std::integral_constant<int, 16>;
  // counts of the slots' entries (n <= kHubChunk); returns the wave's largest n
  auto count_row = [&](Planes& pl, int s, int n, int o, auto&& last) {
    int mx = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mx = max(mx, read_lane(n, k * 16));
    int base = 0;
    while (mx - base > 16) {
      int on = 0;
      gather(I16(), pl, o, [&] { on = load16(s, n, base + 16); });
      o = on;
      base += 16;
    }
    if (mx - base > 8) gather(I16(), pl, o, last);
    else if (mx - base > 4) gather(I8(), pl, o, last);
    else gather(I4(), pl, o, last);
    return mx;
  };

  if (hubs.n > 0 && r1 > r0) {
    // hub rows: one chunk per slot and round, then one row per slot
    uint32_t(&sc)[kSlots][16][17] = sh.sc;  // counts of a chunk (padded)
    __shared__ int carry[16][33];
    const int slot = wave * 4 + q;
    int hr = hub_lower(hubs, r0);
    const int h1 = hub_lower(hubs, r1);
    if (h1 > hr) {
      const int ce = hubs.c0[h1];
      for (int c0 = hubs.c0[hr]; c0 < ce; c0 += kSlots) {
        const int c = c0 + slot;
        const int cs = c < ce ? hubs.cs[c] : 0;
        const int n = c < ce ? hubs.ce[c] - cs : 0;
        Planes pl;
        count_row(pl, cs, n, load16(cs, n, 0), [] {});
        uint32_t cnt[16];
        pl.counts(9, cnt);
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[slot][l16][i] = cnt[i];
        __syncthreads();
        const int h = hr + slot;
        const int b = h < h1 ? hubs.c0[h] : INT_MAX;
        bool ended = false;
        const bool mine = b < c0 + kSlots;
        int tot[32];
        if (mine) {
          const int e = hubs.c0[h + 1];
          ended = e <= c0 + kSlots;
#pragma unroll
          for (int i = 0; i < 32; ++i) tot[i] = b < c0 ? carry[l16][i] : 0;
          const int j1 = min(e, c0 + kSlots) - c0;
          for (int j = max(b - c0, 0); j < j1; ++j) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const uint32_t v = sc[j][l16][i];
              tot[2 * i] += (int)(v & 0xFFFFu);
              tot[2 * i + 1] += (int)(v >> 16);
            }
          }
          if (ended && act) {
            const int64_t row = hubs.rows[h];
            const int len = rowptr[row + 1] - rowptr[row];
            const int u = l16 >> 2;
            int16_t* yr = y + unit_base(d, u) + (l16 & 1) * 32 +
                          (u < pairs ? row * 2 * kPanel + ((l16 >> 1) & 1) * kPanel : row * kPanel);
            int32_t* sd = hs.side + ((int64_t)(l16 >> 1) * hs.n + h) * kPanel + (l16 & 1) * 32;
#pragma unroll
            for (int i = 0; i < 32; ++i) {
              const int v = len - 2 * tot[i];
              int st = v;
              if (v < -32767 || v > 32767) {
                st = kY16Sentinel;
                sd[i] = v;
                atomicOr(escapes, 1u << (l16 >> 1));
              }
              yr[i] = (int16_t)st;
            }
          }
        }
        const int done = __syncthreads_count(ended && l16 == 0);
        if (mine && !ended) {
#pragma unroll
          for (int i = 0; i < 32; ++i) carry[l16][i] = tot[i];
        }
        hr += done;
      }
    }
  }

  __syncthreads();  // the hub rows' counts are done with
  const int64_t ngrp = r1 > r0 ? (r1 - r0 + 3) / 4 : 0;
  const int64_t nk = ngrp > wave ? (ngrp - wave + kWaves - 1) / kWaves : 0;
  if (nk > 0) {
    auto extent = [&](int64_t k, int64_t& row, bool& live, int& s, int& n) {
      row = r0 + (k * kWaves + wave) * 4 + q;
      live = row < r1;
      row = live ? row : r1 - 1;
      s = rowptr[row];
      n = live ? rowptr[row + 1] - s : 0;
      if (n > kHubLen) {
        live = false;
        n = 0;
      }
    };
    int64_t row, row_n = 0;
    bool live, live_n = false;
    int s, n, s_n = 0, n_n = 0;
    extent(0, row, live, s, n);
    if (nk > 1) extent(1, row_n, live_n, s_n, n_n);
    int o = load16(s, n, 0), o_n = 0;
    for (int64_t k = 0; k < nk; ++k) {
      Planes pl;
      int64_t row_f = row;
      bool live_f = false;
      int s_f = 0, n_f = 0;
      const int mx = count_row(pl, s, n, o, [&] {
        o_n = load16(s_n, n_n, 0);
        if (k + 2 < nk) extent(k + 2, row_f, live_f, s_f, n_f);
      });
      uint32_t c[16];
      pl.counts(32 - __builtin_clz(mx | 1), c);
      // Four rows of a unit are consecutive in memory: the lanes exchange their
      // 64-byte pieces through LDS so that a store covers 1 KB in a piece (16
      // bytes a lane at 64-byte steps left y's 1 GB at 1.9 TB/s).
      const s2 nn = {(short)n, (short)n};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        i4 v;  // |y| <= n <= 256
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (int)as_u32(nn - as_s2(c[4 * i + e] << 1));
        sh.out[wave][lane][i] = v;
      }
      const uint64_t rows = __ballot(live);
      const int64_t row0 = r0 + (k * kWaves + wave) * 4;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (u < pairs) {
          const i4 v = sh.out[wave][q * 16 + u * 4 + (l16 >> 2)][l16 & 3];
          if (live) reinterpret_cast<i4*>(y + unit_base(d, u) + row0 * 2 * kPanel)[lane] = v;
        } else if (u == pairs && (panels & 1)) {
          const int r = (lane >> 3) & 3, c8 = lane & 7;
          const i4 v = sh.out[wave][r * 16 + u * 4 + (c8 >> 2)][c8 & 3];
          if (lane < 32 && ((rows >> (16 * r)) & 1))
            reinterpret_cast<i4*>(y + unit_base(d, u) + row0 * kPanel)[lane] = v;
        }
      }
      __builtin_amdgcn_wave_barrier();
      row = row_n;
      live = live_n;
      s = s_n;
      n = n_n;
      o = o_n;
      row_n = row_f;
      live_n = live_f;
      s_n = s_f;
      n_n = n_f;
    }
  }
}

// Pass 2, unit u0 + blockIdx.y of PW panels: w3 = sum_i y_i sum_j y_j over the entries (i, j).
// Bound by the gathers of y's rows and by the latency of walking the pattern,
// which two panels at a time share.  A symmetric pattern takes each
// edge once, from the row with the larger index (w3 = 2 sum_{j < i} y_i y_j +
// the diagonal): half the gathers, and where rows come in order of falling
// degree, the half that falls on the cached rows of the hubs.  A part of a row
// without such entries costs its column load alone.  CHECK: some row is longer
// than 32,767, and gathered values are tested for sentinels in the panels for
// which pass 1 set its bit of escapes.
// Measured (as above): 3,930 -> 1,897; without the halving about 3,300, with
// one panel at a time 2,850, without any gather 1,720 at one panel.  Fetching
// columns and own rows further ahead made no difference.
// (four waves: two panels take 160 registers, three waves per SIMD)
constexpr int kWaves2 = 4;
constexpr int kThreads2 = kWaves2 * 64;
constexpr int kSlots2 = kWaves2 * 4;
template <int PW, bool CHECK, bool OFF32>
__global__ __launch_bounds__(kThreads2) void tri_pass2_kernel(
    const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t d,
    const uint64_t* __restrict__ zbits, const int16_t* __restrict__ y, HubSide hs, HubRows hubs,
    CsrStepPlan plan, const uint64_t* __restrict__ asym, const uint32_t* __restrict__ escapes,
    int panels, int u0, int64_t active, unsigned long long* __restrict__ w) {
  constexpr int kVals = 4 * PW, kProbes = PW * kPanel;  // values per lane, per row
  using X = typename std::conditional<PW == 2, uint4, uint2>::type;
  __shared__ unsigned long long sw[3][kProbes];
  const int lane = lane_id(), wave = wave_id();
  const int q = lane >> 4, l16 = lane & 15;
  const int g = xcd_band(blockIdx.x, plan.ngroups);
  const int64_t r0 = plan.band ? (int64_t)plan.band[g] : (int64_t)g * plan.rows_per_group;
  const int64_t r1 = plan.band ? (int64_t)plan.band[g + 1]
                               : min<int64_t>(r0 + plan.rows_per_group, d);
  const bool sym = *asym == 0;
  const int p0 = 2 * (u0 + (int)blockIdx.y);  // the unit's first panel
  const int pl = PW == 2 ? l16 >> 3 : 0;       // the lane's panel in it
  const bool escaped = CHECK && ((*escapes >> p0) & (PW == 2 ? 3u : 1u));
  y += unit_base(d, u0 + (int)blockIdx.y);
  hs.side += (int64_t)(p0 + pl) * hs.n * kPanel;
  const int pos = (kVals * l16) & (kPanel - 1);  // its first position in the panel
  for (int e = threadIdx.x; e < 3 * kProbes; e += kThreads2) (&sw[0][0])[e] = 0;
  __syncthreads();
  constexpr uint32_t kRowBytes = kProbes * sizeof(int16_t);
  constexpr int kOut = OFF32 ? (int)(0u - kRowBytes) : -1;  // an entry not summed
  __amdgpu_buffer_rsrc_t rsrc;
  if constexpr (OFF32)
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<int16_t*>(y), (short)0,
                                             (int)((uint32_t)d * kRowBytes), 0x00020000);
  auto row_of = [&](int o) { return OFF32 ? (int)((uint32_t)o / kRowBytes) : o; };
  auto exact = [&](int64_t row, int e) { return hs.side[(int64_t)hs.slot(row) * kPanel + pos + e]; };

  // the slot's next 16 entries of row i from `base` on; dg: its lane's entry
  // is the diagonal (symmetric form)
  auto load16 = [&](int64_t i, int s, int n, int base, int& dg) -> int {
    int o = kOut;
    if (base + l16 < n) {
      const int j = col[(int64_t)s + base + l16];
      if (!sym || j < i) o = OFF32 ? (int)((uint32_t)j * kRowBytes) : j;
      if (sym && j == i) dg += 1;
    }
    return o;
  };
  typedef int Sum __attribute__((ext_vector_type(kVals)));
  auto gather = [&](auto nc, Sum& acc, int o, auto&& after) {
    constexpr int N = decltype(nc)::value;
    // none of the part's entries counts: nothing to gather
    if (__ballot(o != kOut) == 0) {
      after();
      return;
    }
    // at most 8 KB of gathers in flight a wave (registers)
    constexpr int B = N * PW > 16 ? 16 / PW : N;
    static_for<N / B>([&](auto h) {
      constexpr int H = decltype(h)::value * B;
      X x[B];
      static_for<B>([&](auto t) {
        constexpr int I = decltype(t)::value;
        const int ot = bcast16<H + I>(o);
        if constexpr (OFF32 && PW == 2) {
          x[I] = __builtin_bit_cast(X, __builtin_amdgcn_raw_buffer_load_b128(
                                           rsrc, (uint32_t)ot + (uint32_t)l16 * 16, 0, 0));
        } else if constexpr (OFF32) {
          x[I] = __builtin_bit_cast(X, __builtin_amdgcn_raw_buffer_load_b64(
                                           rsrc, (uint32_t)ot + (uint32_t)l16 * 8, 0, 0));
        } else {
          x[I] = X{};
          if (ot >= 0) x[I] = *reinterpret_cast<const X*>(y + (int64_t)ot * kProbes + l16 * kVals);
        }
      });
      if constexpr (H + B == N) after();
      __builtin_amdgcn_sched_barrier(0);
      static_for<B>([&](auto t) {
        constexpr int I = decltype(t)::value;
#pragma unroll
        for (int e = 0; e < kVals / 2; ++e) {
          const s2 v = as_s2(reinterpret_cast<const uint32_t*>(&x[I])[e]);
          acc[2 * e] = add_lo(v, acc[2 * e]);
          acc[2 * e + 1] = add_hi(v, acc[2 * e + 1]);
        }
      });
    });
    if (CHECK && escaped) {
      // add what the exact values have past the sentinels just summed
#pragma nounroll
      for (int t = 0; t < N; ++t) {
        const int ot = __builtin_amdgcn_ds_bpermute(((lane & 48) + t) << 2, o);
        if (ot == kOut) continue;
        const int j = row_of(ot);
#pragma unroll
        for (int e = 0; e < kVals; ++e)
          if (y[(int64_t)j * kProbes + l16 * kVals + e] == kY16Sentinel)
            acc[e] += exact(j, e) - kY16Sentinel;
      }
    }
  };
  using I4 = std::integral_constant<int, 4>;
  using I8 = std::integral_constant<int, 8>;
  using I16 = std::integral_constant<int, 16>;
  auto sum_row = [&](Sum& acc, int64_t i, int s, int n, int o, int& dg, auto&& last) {
    int mx = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mx = max(mx, read_lane(n, k * 16));
    int base = 0;
    while (mx - base > 16) {
      int on = 0;
      gather(I16(), acc, o, [&] { on = load16(i, s, n, base + 16, dg); });
      o = on;
      base += 16;
    }
    if (mx - base > 8) gather(I16(), acc, o, last);
    else if (mx - base > 4) gather(I8(), acc, o, last);
    else gather(I4(), acc, o, last);
  };
  // a slot's diagonal entries from its lanes' counts
  auto diag_of = [&](int dg) {
    if (__ballot(dg != 0) == 0) return 0;
    for (int s = 8; s >= 1; s >>= 1) dg += __shfl_xor(dg, s, 64);
    return dg;
  };
  // the lane's probes: pairs (p, p + 16) from p = probe_at(pos) on
  const int zsh = probe_at(pos);
  int m1[kVals] = {};  // |sum z_i y_i| <= the number of entries
  int m2[kVals] = {};  // below 2^31 between flushes
  long long m3[kVals] = {};
  struct Own {
    X y;
    uint64_t z;
  };
  auto own_row = [&](int64_t row) {
    return Own{*reinterpret_cast<const X*>(y + row * kProbes + l16 * kVals),
               zbits[row * panels + p0 + pl]};
  };
  // sw's index of the lane's e-th value
  auto probe_of = [&](int e) { return pl * kPanel + zsh + probe_at(e); };
  // z_i y_i, y_i^2 and y_i times row i's sum; BIG: a hub row
  auto add_row = [&](auto big, int64_t row, const Own& own, const Sum& sum, int diag) {
    const uint32_t zb = (uint32_t)(own.z >> zsh);
#pragma unroll
    for (int e = 0; e < kVals; ++e) {
      int v = as_s2(reinterpret_cast<const uint32_t*>(&own.y)[e / 2])[e & 1];
      if (decltype(big)::value && CHECK && escaped && v == kY16Sentinel) v = exact(row, e);
      const int neg = -(int)((zb >> probe_at(e)) & 1u);  // -1 where z = -1
      m1[e] += (v ^ neg) - neg;
      if constexpr (decltype(big)::value)
        atomicAdd(&sw[1][probe_of(e)], (unsigned long long)((long long)v * v));
      else
        m2[e] += v * v;
      m3[e] += (long long)v * sum[e];
      if (diag) atomicAdd(&sw[2][probe_of(e)], (unsigned long long)((long long)diag * v * v));
    }
  };
  auto flush = [&] {
#pragma unroll
    for (int e = 0; e < kVals; ++e) {
      atomicAdd(&sw[1][probe_of(e)], (unsigned long long)(long long)m2[e]);
      m2[e] = 0;
    }
  };

  if (hubs.n > 0 && r1 > r0) {
    __shared__ Sum ss[kSlots2][16], carry[16];
    __shared__ int sd[kSlots2], cdiag;
    const int slot = wave * 4 + q;
    int hr = hub_lower(hubs, r0);
    const int h1 = hub_lower(hubs, r1);
    if (h1 > hr) {
      const int ce = hubs.c0[h1];
      for (int c0 = hubs.c0[hr]; c0 < ce; c0 += kSlots2) {
        const int c = c0 + slot;
        const int cs = c < ce ? hubs.cs[c] : 0;
        const int n = c < ce ? hubs.ce[c] - cs : 0;
        const int64_t ci = c < ce ? hubs.cr[c] : 0;
        Sum acc = Sum(0);
        int dg = 0;
        const int o = load16(ci, cs, n, 0, dg);
        sum_row(acc, ci, cs, n, o, dg, [] {});
        ss[slot][l16] = acc;
        const int dsum = diag_of(dg);
        if (l16 == 0) sd[slot] = dsum;
        __syncthreads();
        const int h = hr + slot;
        const int b = h < h1 ? hubs.c0[h] : INT_MAX;
        const bool mine = b < c0 + kSlots2;
        bool ended = false;
        Sum tot = Sum(0);
        int td = 0;
        if (mine) {
          const int e = hubs.c0[h + 1];
          ended = e <= c0 + kSlots2;
          if (b < c0) {
            tot = carry[l16];
            td = cdiag;
          }
          const int j1 = min(e, c0 + kSlots2) - c0;
          for (int j = max(b - c0, 0); j < j1; ++j) {
            tot += ss[j][l16];
            td += sd[j];
          }
          if (ended) {
            const int64_t row = hubs.rows[h];
            add_row(std::true_type(), row, own_row(row), tot, td);
          }
        }
        const int done = __syncthreads_count(ended && l16 == 0);
        if (mine && !ended) {
          carry[l16] = tot;
          if (l16 == 0) cdiag = td;
        }
        hr += done;
      }
    }
  }

  const int64_t ngrp = r1 > r0 ? (r1 - r0 + 3) / 4 : 0;
  const int64_t nk = ngrp > wave ? (ngrp - wave + kWaves2 - 1) / kWaves2 : 0;
  if (nk > 0) {
    auto extent = [&](int64_t k, int64_t& row, bool& live, int& s, int& n) {
      row = r0 + (k * kWaves2 + wave) * 4 + q;
      live = row < r1;
      row = live ? row : r1 - 1;
      s = rowptr[row];
      n = live ? rowptr[row + 1] - s : 0;
      if (n > kHubLen) {
        live = false;
        n = 0;
      }
    };
    int64_t row, row_n = 0;
    bool live, live_n = false;
    int s, n, s_n = 0, n_n = 0, dg = 0, dg_n = 0;
    extent(0, row, live, s, n);
    if (nk > 1) extent(1, row_n, live_n, s_n, n_n);
    int o = load16(row, s, n, 0, dg), o_n = kOut;
    for (int64_t k = 0; k < nk; ++k) {
      Sum acc = Sum(0);
      Own own = {};
      int64_t row_f = row;
      bool live_f = false;
      int s_f = 0, n_f = 0;
      dg_n = 0;
      sum_row(acc, row, s, n, o, dg, [&] {
        own = own_row(row);
        o_n = load16(row_n, s_n, n_n, 0, dg_n);
        if (k + 2 < nk) extent(k + 2, row_f, live_f, s_f, n_f);
      });
      const int diag = diag_of(dg);
      if (live) add_row(std::false_type(), row, own, acc, diag);
      // a row that is no hub adds at most 2^16 to m2
      if ((k & 16383) == 16383) flush();
      row = row_n;
      live = live_n;
      s = s_n;
      n = n_n;
      o = o_n;
      dg = dg_n;
      row_n = row_f;
      live_n = live_f;
      s_n = s_f;
      n_n = n_f;
    }
  }
  flush();
#pragma unroll
  for (int e = 0; e < kVals; ++e) {
    atomicAdd(&sw[0][probe_of(e)], (unsigned long long)(long long)m1[e]);
    // in the symmetric form each edge counts from both ends
    atomicAdd(&sw[2][probe_of(e)], (unsigned long long)(m3[e] * (sym ? 2 : 1)));
  }
  __syncthreads();
  // exact in any order, so the workgroups add to the result as they end
  for (int e = threadIdx.x; e < 3 * kProbes; e += kThreads2) {
    const int64_t p = (int64_t)p0 * kPanel + e / 3;
    if (p < active) atomicAdd(w + p * 3 + e % 3, sw[e % 3][e / 3]);
  }
}

// Control variates of Section 5.4: ordinary least squares of w3 on
// [1, w1, w2] (centred normal equations), then
// T_cv = (mean(w3 - a1 w1 - a2 w2) + a1 tr(A) + a2 nnz) / 6 with tr(A) = 0.
// If the centred 2x2 system is singular no control variate is used.
// One workgroup, fixed-order sums.
constexpr int kCvThreads = 256;

__device__ double cv_block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int st = kCvThreads / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  const double r = sh[0];
  __syncthreads();
  return r;
}

__device__ long long cv_block_sum_i(long long v, long long* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int st = kCvThreads / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st) sh[threadIdx.x] += sh[threadIdx.x + st];
    __syncthreads();
  }
  const long long r = sh[0];
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(kCvThreads) void tri_cv_kernel(const long long* __restrict__ w,
                                                            int64_t m, int64_t nnz,
                                                            mlct_tri_result* __restrict__ out) {
  __shared__ double sh[kCvThreads];
  __shared__ long long shi[kCvThreads];
  long long t1 = 0, t2 = 0, t3 = 0;
  for (int64_t p = threadIdx.x; p < m; p += kCvThreads) {
    t1 += w[p * 3];
    t2 += w[p * 3 + 1];
    t3 += w[p * 3 + 2];
  }
  const long long s1 = cv_block_sum_i(t1, shi), s2 = cv_block_sum_i(t2, shi);
  const long long s3 = cv_block_sum_i(t3, shi);
  const double m1 = (double)s1 / m, m2 = (double)s2 / m, m3 = (double)s3 / m;
  double c11 = 0, c12 = 0, c22 = 0, c13 = 0, c23 = 0;
  for (int64_t p = threadIdx.x; p < m; p += kCvThreads) {
    const double x1 = (double)w[p * 3] - m1, x2 = (double)w[p * 3 + 1] - m2;
    const double x3 = (double)w[p * 3 + 2] - m3;
    c11 += x1 * x1;
    c12 += x1 * x2;
    c22 += x2 * x2;
    c13 += x1 * x3;
    c23 += x2 * x3;
  }
  c11 = cv_block_sum(c11, sh);
  c12 = cv_block_sum(c12, sh);
  c22 = cv_block_sum(c22, sh);
  c13 = cv_block_sum(c13, sh);
  c23 = cv_block_sum(c23, sh);
  if (threadIdx.x == 0) {
    double a1 = 0.0, a2 = 0.0;
    const double det = c11 * c22 - c12 * c12;
    if (m >= 3 && det > 1e-12 * c11 * c22 && c11 > 0 && c22 > 0) {
      a1 = (c22 * c13 - c12 * c23) / det;
      a2 = (c11 * c23 - c12 * c13) / det;
    }
    out->sum_w3 = s3;
    out->estimate = (double)s3 / (6.0 * (double)m);
    out->estimate_cv = (m3 - a1 * m1 - a2 * m2 + a2 * (double)nnz) / 6.0;
    out->a1 = a1;
    out->a2 = a2;
  }
}

}  // namespace

hipError_t launch_tri_init(hipStream_t s, int64_t d, ProbeSrc src, int panels, uint64_t* zbits,
                           uint32_t* escapes) {
  const int64_t units = ((d + 63) / 64) * panels;
  const int grid = (int)std::min<int64_t>((units + 3) / 4, 4096);
  tri_init_kernel<<<grid, 256, 0, s>>>(zbits, d, src, panels, escapes);
  return hipGetLastError();
}

hipError_t launch_tri_sym(hipStream_t s, const CsrMat& m, int ngroups, void* part, uint64_t* asym) {
  uint64_t* p = static_cast<uint64_t*>(part);
  tri_sym_kernel<<<ngroups, 256, 0, s>>>(m.rowptr, m.col, m.nrows, hub_rows(m), m.hub_chunks, p);
  tri_sym_sum_kernel<<<1, 256, 0, s>>>(p, ngroups, asym);
  return hipGetLastError();
}

hipError_t launch_tri_pass1(hipStream_t s, const CsrMat& m, const CsrStepPlan& plan,
                            const uint64_t* zbits, int panels, int16_t* y, int32_t* side,
                            uint32_t* escapes) {
  tri_pass1_kernel<<<plan.ngroups, kThreads, 0, s>>>(
      m.rowptr, m.col, m.nrows, reinterpret_cast<const uint32_t*>(zbits), panels, y,
      HubSide{m.hub_rows, m.hub_n, side}, hub_rows(m), banded(m, plan), escapes);
  return hipGetLastError();
}

hipError_t launch_tri_pass2(hipStream_t s, const CsrMat& m, const CsrStepPlan& plan, int panels,
                            const uint64_t* zbits, const int16_t* y, int32_t* side,
                            const uint64_t* asym, const uint32_t* escapes, int64_t active,
                            long long* w) {
  const HubSide hs{m.hub_rows, m.hub_n, side};
  auto go = [&](auto pw, int u0, int units) {
    constexpr int PW = decltype(pw)::value;
    const dim3 grid(plan.ngroups, units);
#define MLCT_TRI2(C, O)                                                                  \
  tri_pass2_kernel<PW, C, O><<<grid, kThreads2, 0, s>>>(                                 \
      m.rowptr, m.col, m.nrows, zbits, y, hs, hub_rows(m), banded(m, plan), asym, escapes, \
      panels, u0, active, reinterpret_cast<unsigned long long*>(w))
    // (further panels are taken only while all of y stays within 1 GiB, so that
    // two of them always have 32-bit offsets)
    if constexpr (PW == 1) {
      if ((uint64_t)m.ncols * kPanel * sizeof(int16_t) > 0xFFFFFFFFull) {
        if (m.max_row_nnz > 32767) MLCT_TRI2(true, false);
        else MLCT_TRI2(false, false);
        return;
      }
    }
    if (m.max_row_nnz > 32767) MLCT_TRI2(true, true);
    else MLCT_TRI2(false, true);
#undef MLCT_TRI2
  };
  if (panels >= 2) go(std::integral_constant<int, 2>(), 0, panels / 2);
  if (panels & 1) go(std::integral_constant<int, 1>(), panels / 2, 1);
  return hipGetLastError();
}

hipError_t launch_tri_cv(hipStream_t s, const long long* w, int64_t m, int64_t nnz,
                         mlct_tri_result* out) {
  tri_cv_kernel<<<1, kCvThreads, 0, s>>>(w, m, nnz, out);
  return hipGetLastError();
}

}  // namespace mlct
