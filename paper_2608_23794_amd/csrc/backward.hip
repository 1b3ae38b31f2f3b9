// Gradients of the static layer (Secs. 3.2-3.4) and of the coverage loss
// (Sec. 3.4 Eq. 7).
//
// With dy the gradient of the loss with respect to y, the layer's backward is
//   dalpha[b][e][i] = sum_p dy[b][e][p] x[b][s_ei][p]                (Eq. 5)
//   dz_i  = alpha_i (dalpha_i - sum_j alpha_j dalpha_j)               (Eq. 4)
//   dw[e][i]  = sum_b dz_bei / tau_be
//   dtau_be   = -sum_i dz_bei w_ei / tau_be^2
//   the gate's parameters from dtau; its inputs z_i = d[b][s_ei] from dtau
//   dx[b][c][p] = sum_{(e,i): s_ei = c} alpha_bei dy[b][e][p]
//               + [c uncovered] dy[b][E-1][p] / |U|                    (Eq. 6)
//               + dd[b][c] / HW                                        (GAP)
// where dd[b][c] sums the gate-input gradients of every support entry on c.
//
// Launches:
//  - pooling and the forward's gate (pool.hip, gate.hip): d, the softmax
//    statistics and the coefficients;
//  - the support entries in buckets of (64 channels, 64 experts), with the
//    uncovered channels as bitmaps, rebuilt per call from the prepared rows (the
//    buckets in a fixed order, a bucket's entries in any: what reads them gives each
//    a place of its own or sorts them); for the MLP gate and the generic dx also every
//    channel's list;
//  - dalpha (the sampled product of dy and x; the matrix-core kernel of
//    bwdmfma.hip for bfloat16, but for its limits, a wave per (image, expert) elsewhere);
//  - 16 lanes per (expert, group of images) for the row sums, dtau, the
//    softplus-linear gate's dg and the group's share of dw and the gate's slopes,
//    then the sums over the groups; the MLP gate's rows in blocks (below);
//  - dd (a float32 product of dg and the slopes, or from the channel lists a thread
//    per (image, channel)) and dx (the matrix-core kernel of bwdmfma.hip for bfloat16,
//    but for its limits, a thread per element elsewhere).
#include <algorithm>
#include <climits>
#include <type_traits>

#include "moce_internal.h"

namespace moce {
namespace {

constexpr int kBwThreads = 256;
constexpr int kBwWaves = kBwThreads / kWave;
constexpr int kBwMaxK = 1024;     // a support row in registers, 16 entries per lane
constexpr int kCovMaxC = 32768;   // a logit row's support positions in LDS

template <typename T> __device__ __forceinline__ float ld(const T* p, int64_t i);
template <> __device__ __forceinline__ float ld<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float ld<uint16_t>(const uint16_t* p, int64_t i) { return bf16_to_f32(p[i]); }
template <typename T> __device__ __forceinline__ void st_elem(T* p, int64_t i, float v);
template <> __device__ __forceinline__ void st_elem<float>(float* p, int64_t i, float v) { p[i] = v; }
template <> __device__ __forceinline__ void st_elem<uint16_t>(uint16_t* p, int64_t i, float v) { p[i] = f32_to_bf16(v); }

// element (b, channel c of nc, position p) of an NCHW or channels-last tensor
template <bool NHWC>
__device__ __forceinline__ int64_t at(int64_t b, int64_t c, int64_t p, int64_t nc, int64_t HW) {
  return NHWC ? (b * HW + p) * nc + c : (b * nc + c) * HW + p;
}

__device__ __forceinline__ float alpha_of(float w, float rt, float m, float rzs) {
  return coef_alpha(coef_e(coef_z(w, rt), m), rzs);
}

// ---------------------------------------------------------------- support entries by channel
// k_bw_part: the support entries of each chunk of 64 experts (a contiguous range
// of the rows) sorted into buckets by 64 channels, in the chunk's own range of
// the entry arrays, so that no workgroup waits for another's counts; bbeg[chunk]
// [block] is where a bucket starts, and the next bucket's start ends it.  The
// matrix-core dx walks these buckets.
// k_bw_lists: from the buckets, each channel's entries (the inverse support map)
// ascending by expert, as a row holds a channel once, and the channels with
// none.  A workgroup per 64 channels; its lists start after every entry on a
// lower channel, whose number its buckets' starts add up to.
// Two launches (11 us at stage 4, 5 at stage 1; the lists, which few callers need,
// 8 us at stage 3) in the place of nine of 4 to 11 us; with one
// workgroup per 64 channels reading every entry it was one of 55 us at stage 4.
constexpr int kPrepThreads = 1024;
constexpr int kPrepWindow = 8192;        // bucket counters in LDS at a time (32 KB)
constexpr int kPrepHold = 8;             // entries a thread reads ahead
constexpr int kListChunks = kWave;       // chunks whose experts k_bw_lists marks at a time, a lane each

__global__ void __launch_bounds__(kPrepThreads)
k_bw_part(const int32_t* __restrict__ s, const float* __restrict__ w, const float* __restrict__ a,
          int32_t* __restrict__ bbeg, uint2* __restrict__ bw, uint2* __restrict__ ba, int R, int k, int nblk) {
  extern __shared__ int32_t cnt[];       // [min(nblk, kPrepWindow)]
  __shared__ int32_t wsum[kPrepThreads / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int e0 = blockIdx.x * kBwBucketEx;
  const int n = min(kBwBucketEx, R - e0) * k;
  const int64_t base = (int64_t)e0 * k;
  int32_t* beg = bbeg + (int64_t)blockIdx.x * (nblk + 1);
  int run = (int)base;
  for (int win = 0; win < nblk; win += kPrepWindow) {
    const int nw = min(kPrepWindow, nblk - win);
    __syncthreads();
    for (int i = tid; i < nw; i += kPrepThreads) cnt[i] = 0;
    __syncthreads();
    // the chunk's entries kPrepHold a thread at a time, every read in flight
    // before any is used (reads past the end repeat the last entry)
    for (int t0 = tid; t0 < n; t0 += kPrepHold * kPrepThreads) {
      int c[kPrepHold];
#pragma unroll
      for (int u = 0; u < kPrepHold; ++u) c[u] = s[base + min(t0 + u * kPrepThreads, n - 1)];
#pragma unroll
      for (int u = 0; u < kPrepHold; ++u) {
        const int blk = c[u] / kBwBucketCh - win;
        if (t0 + u * kPrepThreads < n && blk >= 0 && blk < nw) atomicAdd(&cnt[blk], 1);
      }
    }
    __syncthreads();
    // exclusive scan of the window's counts, kPrepThreads at a time
    for (int i0 = 0; i0 < nw; i0 += kPrepThreads) {
      const int v = i0 + tid < nw ? cnt[i0 + tid] : 0;
      int incl = v;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += t;
      }
      if (lane == kWave - 1) wsum[wv] = incl;
      __syncthreads();
      int before = run, tot = 0;
      for (int j = 0; j < kPrepThreads / kWave; ++j) {
        before += j < wv ? wsum[j] : 0;
        tot += wsum[j];
      }
      if (i0 + tid < nw) {
        beg[win + i0 + tid] = before + incl - v;
        cnt[i0 + tid] = before + incl - v;
      }
      run += tot;
      __syncthreads();
    }
    for (int t0 = tid; t0 < n; t0 += kPrepHold * kPrepThreads) {
      int c[kPrepHold], q[kPrepHold];
      uint32_t wv0[kPrepHold], av[kPrepHold];
#pragma unroll
      for (int u = 0; u < kPrepHold; ++u) {
        const int64_t i = base + min(t0 + u * kPrepThreads, n - 1);
        c[u] = s[i];
        wv0[u] = __float_as_uint(w[i]);
        av[u] = __float_as_uint(a[i]);
      }
#pragma unroll
      for (int u = 0; u < kPrepHold; ++u) {
        const int blk = c[u] / kBwBucketCh - win;
        q[u] = t0 + u * kPrepThreads < n && blk >= 0 && blk < nw ? atomicAdd(&cnt[blk], 1) : -1;
      }
#pragma unroll
      for (int u = 0; u < kPrepHold; ++u)
        if (q[u] >= 0) {
          const int t = t0 + u * kPrepThreads;
          bw[q[u]] = make_uint2((uint32_t)(c[u] & 255) | ((uint32_t)(t / k) << 8), wv0[u]);
          ba[q[u]] = make_uint2(av[u], (uint32_t)(base + t));
        }
    }
  }
  if (tid == 0) beg[nblk] = run;
}

// unc[block]: a bit per channel of the block with no entry.  An entry's place in its
// channel's list is the number of the channel's experts below its own: per chunk a
// bit for each expert, the chunks' counts summed over a wave's lanes, kListChunks
// chunks at a time.  (Sorting each list, by rank in registers up to 256 entries and by
// insertion in one lane above, took 8393 us at C 2689, E 2689, k 336 and 47 at C 218,
// E 54, k 218; now 37 and 11.)
__global__ void __launch_bounds__(kPrepThreads)
k_bw_lists(const int32_t* __restrict__ bbeg, const uint2* __restrict__ bw, const uint2* __restrict__ ba,
           int32_t* __restrict__ off, int32_t* __restrict__ inv, uint64_t* __restrict__ unc, int R, int k, int C,
           int nblk) {
  // [chunk][channel]: which of the chunk's experts hold the channel; where their entries go
  __shared__ unsigned long long mask[kListChunks][kBwBucketCh + 1];
  __shared__ int32_t place[kListChunks][kBwBucketCh + 1];
  __shared__ int32_t cur[kBwBucketCh];   // a channel's entries, then where its next ones go
  __shared__ int32_t red[kPrepThreads / kWave];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int blk = blockIdx.x, c0 = blk * kBwBucketCh, nc = min(kBwBucketCh, C - c0);
  const int nch = (R + kBwBucketEx - 1) / kBwBucketEx;
  if (tid < kBwBucketCh) cur[tid] = 0;
  // entries on lower channels
  int below = 0;
  for (int ch = tid; ch < nch; ch += kPrepThreads)
    below += bbeg[(int64_t)ch * (nblk + 1) + blk] - ch * kBwBucketEx * k;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o, kWave);
  if (lane == 0) red[wv] = below;
  __syncthreads();
  below = 0;
  for (int j = 0; j < kPrepThreads / kWave; ++j) below += red[j];
  // f(entry, chunk of the group) over the buckets of a group of chunks, a wave per
  // bucket or, of few, several
  constexpr int waves = kPrepThreads / kWave;
  const int per = max(1, waves / max(1, nch));
  auto each = [&](int g0, auto&& f) __attribute__((always_inline)) {
    for (int j = wv / per; j < min(kListChunks, nch - g0); j += waves / per) {
      const int32_t* bg = bbeg + (int64_t)(g0 + j) * (nblk + 1) + blk;
      const int b0 = bg[0], b1 = bg[1];
#pragma unroll 4
      for (int q = b0 + wv % per * kWave + lane; q < b1; q += per * kWave) f(q, j);
    }
  };
  auto masks = [&](int g0) __attribute__((always_inline)) {
    for (int i = tid; i < min(kListChunks, nch - g0) * (kBwBucketCh + 1); i += kPrepThreads) mask[0][i] = 0;
    __syncthreads();
    each(g0, [&](int q, int j) __attribute__((always_inline)) {
      const uint32_t v = bw[q].x;
      atomicOr(&mask[j][v & (kBwBucketCh - 1)], 1ull << (v >> 8));
    });
    __syncthreads();
  };
  // the lane's chunk's entries on channel ci
  auto count = [&](int g0, int ci) __attribute__((always_inline)) {
    return g0 + lane < nch ? __popcll(mask[lane][ci]) : 0;
  };
  for (int g0 = 0; g0 < nch; g0 += kListChunks) {
    masks(g0);
    for (int ci = wv; ci < nc; ci += kPrepThreads / kWave) {
      int v = count(g0, ci);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
      if (lane == 0) cur[ci] += v;
    }
    __syncthreads();
  }
  if (wv == 0) {
    const int v = lane < nc ? cur[lane] : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int t = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += t;
    }
    cur[lane] = below + incl - v;
    if (lane < nc) off[c0 + lane] = below + incl - v;
    if (lane == kWave - 1 && c0 + nc == C) off[C] = below + incl;
    const uint64_t none = __ballot(lane < nc && v == 0);
    if (lane == 0) unc[blk] = none;
  }
  __syncthreads();
  for (int g0 = 0; g0 < nch; g0 += kListChunks) {
    if (nch > kListChunks) masks(g0);
    for (int ci = wv; ci < nc; ci += kPrepThreads / kWave) {
      const int v = count(g0, ci), at = cur[ci];
      int incl = v;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int t = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += t;
      }
      place[lane][ci] = at + incl - v;
      if (lane == kWave - 1) cur[ci] = at + incl;
    }
    __syncthreads();
    each(g0, [&](int q, int j) __attribute__((always_inline)) {
      const uint32_t v = bw[q].x;
      const int c = (int)(v & (kBwBucketCh - 1));
      inv[place[j][c] + __popcll(mask[j][c] & ((1ull << (v >> 8)) - 1ull))] = (int32_t)ba[q].y;
    });
    __syncthreads();
  }
}

// ---------------------------------------------------------------- dalpha, generic
// A wave per (image, routed expert); lanes over support positions.  Bound by the lines
// that the lanes' planes are: 823 us channels-first and 241 channels-last for 32 float32
// images of C 512, E 128, k 64, 28 x 28, whose x and dy are 64 MB.
template <typename T, bool NHWC>
__global__ void __launch_bounds__(kBwThreads)
k_bw_dalpha(const T* __restrict__ x, const T* __restrict__ dy, const int32_t* __restrict__ s,
            float* __restrict__ dal, int64_t B, int C, int E, int R, int k, int HW) {
  const int64_t row = (int64_t)blockIdx.x * kBwWaves + (threadIdx.x >> 6);
  if (row >= B * R) return;
  const int lane = threadIdx.x & 63;
  const int64_t b = row / R;
  const int e = (int)(row - b * R);
  for (int i0 = 0; i0 < k; i0 += kWave) {
    const int i = i0 + lane;
    const int c = i < k ? s[(int64_t)e * k + i] : 0;
    float acc = 0.f;
    for (int p = 0; p < HW; ++p) {
      const float g = ld<T>(dy, at<NHWC>(b, e, p, E, HW));
      acc += g * ld<T>(x, at<NHWC>(b, c, p, C, HW));
    }
    if (i < k) dal[row * k + i] = acc;
  }
}

// ---------------------------------------------------------------- rows and their sums
// sum over the wave: DPP moves within rows of 16 lanes, then the four rows
__device__ __forceinline__ float row16_sum(float v) {
  auto mov = [](float u, auto ctrl) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(u), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += mov(v, std::integral_constant<int, 0xb1>{});    // quad_perm [1, 0, 3, 2]
  v += mov(v, std::integral_constant<int, 0x4e>{});    // quad_perm [2, 3, 0, 1]
  v += mov(v, std::integral_constant<int, 0x141>{});   // row_half_mirror
  v += mov(v, std::integral_constant<int, 0x140>{});   // row_mirror
  return v;
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  v = row16_sum(v);
  auto row = [&](int l) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
  };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// LPR = 16 lanes (64 for k > 256) per (routed expert, group of gs images), so
// that a reduction serves four experts: the lanes keep the expert's row (logits,
// channels, slopes) in registers and walk the images, the next one's reads in
// flight.  Per image dalpha arrives as nsplit partial sums;
// S1 = sum_i alpha_i dalpha_i; with Aw = sum_i alpha_i w_i,
// sum_i dz_i w_i = sum_i alpha_i (dalpha_i - S1) (w_i - Aw), centred twice so that
// nothing cancels; dtau = -that / tau^2 (rt = 1/tau).  Softplus-linear gate:
// g = c_e + sum_i a_ei z_i, dg = dtau sigmoid(g).  Over the group's images the lanes
// sum dw[e][i] += alpha_bei (dalpha_bei - S1_be) rt_be, da[e][i] += dg_be d[b][s_ei] and
// dc[e] += dg_be: dalpha is read once, where a kernel for the rows and one for the
// sums read it twice (59 us of the stage-4 backward, 24 us with a wave a row; now 18).
// psum[group]: [R k] dw, then for the linear gate [R k] da, [R] dc.
template <int LPR, int PER>
__global__ void __launch_bounds__(kBwThreads)
k_bw_rows(const float* __restrict__ dal, const float* __restrict__ w, const float* __restrict__ stats,
          const float* __restrict__ d, const int32_t* __restrict__ s, const float* __restrict__ a,
          const float* __restrict__ cc, float* __restrict__ dtau_o, float* __restrict__ dg_o,
          float* __restrict__ psum, int64_t B, int C, int R, int k, int nsplit, int gs) {
  auto row_sum = [](float v) __attribute__((always_inline)) {
    if constexpr (LPR == 16)
      return row16_sum(v);
    else
      return wave_sum_dpp(v);
  };
  const int er = blockIdx.x * (kBwThreads / LPR) + threadIdx.x / LPR;
  const bool live = er < R;
  const int e = min(er, R - 1);
  const int lane = threadIdx.x % LPR;
  const int64_t n = B * R, rk = (int64_t)R * k;
  const int64_t b0 = (int64_t)blockIdx.y * gs, b1 = min<int64_t>(B, b0 + gs);
  float wv[PER], av[PER], sw[PER], sa[PER];
  int ch[PER], ix[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    ix[j] = min(lane + j * LPR, k - 1);
    wv[j] = w[(int64_t)e * k + ix[j]];
    ch[j] = s[(int64_t)e * k + ix[j]];
    av[j] = a ? a[(int64_t)e * k + ix[j]] : 0.f;
    sw[j] = sa[j] = 0.f;
  }
  const float ce = a ? cc[e] : 0.f;
  float sc = 0.f;
  struct In {
    float rt, m, rzs, da[PER], dv[PER];
  };
  auto load = [&](int64_t b, In& x) __attribute__((always_inline)) {
    const int64_t row = b * R + e;
    x.rt = stats[row];
    x.m = stats[n + row];
    x.rzs = stats[2 * n + row];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      x.da[j] = dal[row * k + ix[j]];
      x.dv[j] = a ? d[b * C + ch[j]] : 0.f;
    }
  };
  In x, xn;
  load(b0, x);
  for (int64_t b = b0; b < b1; ++b) {
    const int64_t row = b * R + e;
    load(min(b + 1, b1 - 1), xn);
    for (int sp = 1; sp < nsplit; ++sp)   // partial sums along the positions
#pragma unroll
      for (int j = 0; j < PER; ++j) x.da[j] += dal[(sp * n + row) * k + ix[j]];
    float al[PER], s1 = 0.f, aw = 0.f, g = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = lane + j * LPR < k;
      al[j] = in ? alpha_of(wv[j], x.rt, x.m, x.rzs) : 0.f;
      s1 += in ? al[j] * x.da[j] : 0.f;
      aw += in ? al[j] * wv[j] : 0.f;
      g += in ? av[j] * x.dv[j] : 0.f;
    }
    s1 = row_sum(s1);
    aw = row_sum(aw);
    float t = 0.f;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const bool in = lane + j * LPR < k;
      const float v = al[j] * (x.da[j] - s1);
      t += in ? v * (wv[j] - aw) : 0.f;
      sw[j] += v * x.rt;
    }
    const float dtau = -row_sum(t) * x.rt * x.rt;
    if (a) {
      const float dg = dtau / (1.f + expf(-(row_sum(g) + ce)));
#pragma unroll
      for (int j = 0; j < PER; ++j) sa[j] += dg * x.dv[j];
      sc += dg;
      if (lane == 0 && live) dg_o[row] = dg;
    } else if (lane == 0 && live) {
      dtau_o[row] = dtau;
    }
    x = xn;
  }
  if (!live) return;
  float* out = psum + blockIdx.y * (a ? 2 * rk + R : rk);
#pragma unroll
  for (int j = 0; j < PER; ++j)
    if (lane + j * LPR < k) {
      out[(int64_t)e * k + lane + j * LPR] = sw[j];
      if (a) out[rk + (int64_t)e * k + lane + j * LPR] = sa[j];
    }
  if (a && lane == 0) out[2 * rk + e] = sc;
}

// the groups' sums added in order: 32 entries a workgroup, eight threads each
// over every eighth group.  The first wave also counts U for the vector dx (unc: null
// where that does not run).
__global__ void __launch_bounds__(256)
k_bw_sums_reduce(const float* __restrict__ psum, int ng, int64_t rk, int64_t n, float* __restrict__ dw,
                 float* __restrict__ da, float* __restrict__ dc, const uint64_t* __restrict__ unc, int C,
                 int32_t* __restrict__ nU) {
  __shared__ float sums[8][32];
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  if (unc && blockIdx.x == 0 && threadIdx.x < kWave) {
    const int all = bwd_count_uncovered(unc, C);
    if (threadIdx.x == 0) *nU = all;
  }
  const int64_t q = (int64_t)blockIdx.x * 32 + x;
  float acc = 0.f;
#pragma unroll 8
  for (int g = y; g < ng; g += 8) acc += psum[g * n + min(q, n - 1)];
  sums[y][x] = acc;
  __syncthreads();
  if (y != 0 || q >= n) return;
  for (int j = 1; j < min(8, ng); ++j) acc += sums[j][x];
  if (q < rk)
    dw[q] = acc;
  else if (q < 2 * rk)
    da[q - rk] = acc;
  else
    dc[q - 2 * rk] = acc;
}

// ---------------------------------------------------------------- dd
// dd[b][c] = sum over the entries (e, i) on channel c of the gate-input gradient.
//
// Softplus-linear gate: dg_be a_ei, a product of dg [B][R] with the slopes as a
// matrix [R][C], on the matrix cores in float32: per chunk of 64 experts the
// bucket's slopes are scattered into a zeroed tile (each has a place of its own,
// so the result does not depend on the entries' order) and multiplied with the
// chunk's dg.  A workgroup per (64 channels, 32 images).  (A thread per (image,
// channel) over the channel's entries, three dependent reads each, took 49 us
// at stage 4.)  A dg that is not finite would reach every channel through the
// tile's zeros, so a workgroup that meets one sums over the entries alone.  The
// workgroups of the first images also write the uncovered channels' bitmaps (again,
// where the lists are built).
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
constexpr int kDdImages = 32;
constexpr int64_t kDdSliceThreads = 2049;   // for image_slices: at most 65535 groups of 32 images a launch
constexpr int kDdPitch = kBwBucketEx + 4;
constexpr int kDdHold = 4;
constexpr int kDdChunks = 64;
constexpr uint32_t kDdNone = 0xffffdeadu;   // no entry at this place of the tile

__global__ void __launch_bounds__(kBwThreads)
k_bw_dd_linear(const int32_t* __restrict__ bbeg, const uint2* __restrict__ bw, const uint2* __restrict__ ba,
               const float* __restrict__ dg, float* __restrict__ dd, uint64_t* __restrict__ unc, int64_t B, int C,
               int R, int nblk) {
  __shared__ __align__(16) float at[kBwBucketCh * kDdPitch];    // [channel][expert]
  __shared__ __align__(16) float gt[kDdImages * kDdPitch];      // [image][expert]
  __shared__ uint64_t orw[kBwWaves];
  __shared__ int2 rng[kDdChunks];                               // the first chunks' buckets
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int blk = blockIdx.x, c0 = blk * kBwBucketCh, nc = min(kBwBucketCh, C - c0);
  const int64_t b0 = (int64_t)blockIdx.y * kDdImages;
  const int im = wv & 1, cm = wv >> 1;   // this wave's 16 images and 32 channels
  const int nch = (R + kBwBucketEx - 1) / kBwBucketEx;
  f32x4 acc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  uint64_t seen = 0;
  int bad = 0;
  for (int ch = tid; ch < min(nch, kDdChunks); ch += kBwThreads) {
    const int32_t* bg = bbeg + (int64_t)ch * (nblk + 1) + blk;
    rng[ch] = make_int2(bg[0], bg[1]);
  }
  // the entries and dg of two chunks ahead in registers
  constexpr int GP = kDdImages * kBwBucketEx / kBwThreads;
  struct In {
    uint32_t ew[kDdHold], ea[kDdHold];
    float gr[GP];
    int eb, en;
  };
  auto load = [&](int chunk, In& x) __attribute__((always_inline)) {
    const int ch = min(chunk, nch - 1);
    const int32_t* bg = bbeg + (int64_t)ch * (nblk + 1) + blk;
    const int2 r = ch < kDdChunks ? rng[ch] : make_int2(bg[0], bg[1]);
    x.eb = r.x;
    x.en = r.y - r.x;
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int q = tid + u * kBwThreads, e = ch * kBwBucketEx + q % kBwBucketEx;
      const int64_t b = b0 + q / kBwBucketEx;
      x.gr[u] = dg[min(b, B - 1) * R + min(e, R - 1)];
    }
#pragma unroll
    for (int u = 0; u < kDdHold; ++u) {
      const int q = x.eb + min(tid + u * kBwThreads, max(x.en - 1, 0));
      x.ew[u] = bw[q].x;
      x.ea[u] = ba[q].x;
    }
  };
  In x0, x1;
  __syncthreads();
  load(0, x0);
  load(1, x1);
  auto chunk = [&](int ch, In& x) __attribute__((always_inline)) {
    for (int i = tid; i < kBwBucketCh * kDdPitch / 4; i += kBwThreads)
      reinterpret_cast<float4*>(at)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < GP; ++u) {
      const int q = tid + u * kBwThreads, e = q % kBwBucketEx, i = q / kBwBucketEx;
      bad |= (__float_as_uint(x.gr[u]) & 0x7f800000u) == 0x7f800000u;
      gt[i * kDdPitch + e] = b0 + i < B && ch * kBwBucketEx + e < R ? x.gr[u] : 0.f;
    }
    __syncthreads();
    auto put = [&](uint32_t v0, uint32_t v1) __attribute__((always_inline)) {
      const int c = v0 & (kBwBucketCh - 1);
      at[c * kDdPitch + (v0 >> 8)] = __uint_as_float(v1);
      seen |= 1ull << c;
    };
#pragma unroll
    for (int u = 0; u < kDdHold; ++u)
      if (tid + u * kBwThreads < x.en) put(x.ew[u], x.ea[u]);
    for (int q = tid + kDdHold * kBwThreads; q < x.en; q += kBwThreads) put(bw[x.eb + q].x, ba[x.eb + q].x);
    load(ch + 2, x);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kBwBucketEx / 16; ++c) {
      const float4 xg = *reinterpret_cast<const float4*>(gt + (16 * im + n) * kDdPitch + 16 * c + 4 * g);
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float4 y = *reinterpret_cast<const float4*>(at + (32 * cm + 16 * t + n) * kDdPitch + 16 * c + 4 * g);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xg.x, y.x, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xg.y, y.y, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xg.z, y.z, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xg.w, y.w, acc[t], 0, 0, 0);
      }
    }
    __syncthreads();
  };
  for (int ch = 0; ch < nch; ch += 2) {
    chunk(ch, x0);
    if (ch + 1 < nch) chunk(ch + 1, x1);
  }
  if (__syncthreads_or(bad)) {
    constexpr int N = kDdImages * kBwBucketCh / kBwThreads;   // images per thread
    float sum[N] = {};
    const int c = tid % kBwBucketCh, i0 = tid / kBwBucketCh;
#pragma unroll 1
    for (int ch = 0; ch < nch; ++ch) {
      for (int i = tid; i < kBwBucketCh * kDdPitch; i += kBwThreads) reinterpret_cast<uint32_t*>(at)[i] = kDdNone;
      __syncthreads();
      const int32_t* bg = bbeg + (int64_t)ch * (nblk + 1) + blk;
      for (int q = bg[0] + tid; q < bg[1]; q += kBwThreads) {
        const uint32_t v = bw[q].x;
        at[(v & (kBwBucketCh - 1)) * kDdPitch + (v >> 8)] = __uint_as_float(ba[q].x);
      }
      __syncthreads();
#pragma unroll 1
      for (int e = 0; e < kBwBucketEx; ++e) {
        const float a = at[c * kDdPitch + e];
        if (__float_as_uint(a) == kDdNone) continue;
#pragma unroll
        for (int u = 0; u < N; ++u)
          sum[u] += dg[min(b0 + i0 + u * (kDdImages / N), B - 1) * R + ch * kBwBucketEx + e] * a;
      }
      __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int64_t b = b0 + i0 + u * (kDdImages / N);
      if (b < B && c < nc) dd[b * C + c0 + c] = sum[u];
    }
  } else {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int c = 32 * cm + 16 * t + n;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t b = b0 + 16 * im + 4 * g + r;
        if (b < B && c < nc) dd[b * C + c0 + c] = acc[t][r];
      }
    }
  }
  if (blockIdx.y != 0) return;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) seen |= __shfl_xor((unsigned long long)seen, o, kWave);
  if (lane == 0) orw[wv] = seen;
  __syncthreads();
  if (tid == 0) {
    const uint64_t all = nc == 64 ? ~0ull : (1ull << nc) - 1ull;
    unc[blk] = ~(orw[0] | orw[1] | orw[2] | orw[3]) & all;
  }
}

// A thread per (image, channel) over the channel's list: dzg[b][e][i] of the MLP gate,
// or, where the lists are there for the vector dx, dg_be a_ei (dd_by_lists).
template <bool MLP>
__global__ void __launch_bounds__(kBwThreads)
k_bw_dd_lists(const int32_t* __restrict__ off, const int32_t* __restrict__ inv, const float* __restrict__ dzg,
              const float* __restrict__ dg, const float* __restrict__ a, float* __restrict__ dd, int64_t B, int C, int R,
              int k) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= B * C) return;
  const int64_t b = t / C, rk = (int64_t)R * k;
  const int c = (int)(t - b * C);
  float acc = 0.f;
#pragma unroll 8
  for (int j = off[c]; j < off[c + 1]; ++j) {
    const int ent = inv[j];
    acc += MLP ? dzg[b * rk + ent] : dg[b * R + ent / k] * a[ent];
  }
  dd[t] = acc;
}

// Whether the linear gate's dd comes from the channel lists (where they are built) or
// from the product, by what both take in ns: the lists 0.006 an entry and image with
// the device full, or 4000 and 600 for each of a channel's entries, one after another;
// the product 1 for a workgroup and chunk, or 2000 and 1500 a chunk, three barriers.
// At 10 images, C 1614, E 1614, k 21 the lists take 16 us and the product 38; at 128,
// C 2048, E 512, k 128 49 and 14.
bool dd_by_lists(const Shape& sh) {
  const double entries = (double)sh.R * sh.k, chunks = (sh.R + kBwBucketEx - 1) / kBwBucketEx;
  const double groups = (double)((sh.C + kBwBucketCh - 1) / kBwBucketCh) * (double)((sh.B + kDdImages - 1) / kDdImages);
  const double lists = std::max(0.006 * sh.B * entries, 4000. + 600. * entries / sh.C);
  return lists < std::max(groups * chunks, 2000. + 1500. * chunks);
}

// ---------------------------------------------------------------- dx, generic
// A thread per element of dx: the channel's entries in inverse-map order,
// then the residual share and the descriptor term: every entry's dy passes through the
// vector L1, 230 us channels-first and 593 channels-last at the float32 shape of
// k_bw_dalpha.  |U| is read where a lane needs it (nU, without routed experts C): counted
// from the bitmaps by every wave it took the kernel from 136 us to 181 at 24 float32
// images, C 2576, E 322, k 1, 785 positions channels-first.
template <typename T, bool NHWC>
__global__ void __launch_bounds__(kBwThreads)
k_bw_dx(const T* __restrict__ dy, const float* __restrict__ alpha, const int32_t* __restrict__ off,
        const int32_t* __restrict__ inv, const int32_t* __restrict__ nU, const float* __restrict__ dd,
        T* __restrict__ dx, int64_t B, int C, int E, int R, int k, int HW) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = B * C * (int64_t)HW;
  if (t >= total) return;
  int64_t b, c, p;
  if (NHWC) {
    c = t % C;
    const int64_t r = t / C;
    p = r % HW;
    b = r / HW;
  } else {
    p = t % HW;
    const int64_t r = t / HW;
    c = r % C;
    b = r / C;
  }
  const int64_t rk = (int64_t)R * k;
  float acc = 0.f;
  const int j0 = off[c], j1 = off[c + 1];
  for (int j = j0; j < j1; ++j) {
    const int ent = inv[j];
    const int e = ent / k;
    acc += alpha[b * rk + ent] * ld<T>(dy, at<NHWC>(b, e, p, E, HW));
  }
  if (j0 == j1) acc += ld<T>(dy, at<NHWC>(b, R, p, E, HW)) / (float)(R > 0 ? *nU : C);
  if (R > 0) acc += dd[b * C + c] / (float)HW;
  st_elem<T>(dx, t, acc);
}

// ---------------------------------------------------------------- the MLP gate
// Rows r = (b, e) in blocks of kMlpBwRows per workgroup.  Per row:
// z_i = d[b][s_ei], hpre = W1 z + b1, h = ReLU(hpre), g = w2 . h + b2,
// sigma = sigmoid(g), dg = dtau (tmax - tmin) sigma (1 - sigma),
// dh_j = dg w2_j [hpre_j > 0], dzg_i = sum_j W1[j][i] dh_j (written per row);
// the workgroup accumulates dW1 += dh z^T, db1 += dh, dw2 += dg h, db2 += dg
// and writes them as one partial per workgroup.
//
// The three products (Z W1^T, dh W1 and dh^T Z) run on the matrix cores in
// float32 (16x16x4), k padded to KP with zeros.  The four lane groups of an
// operand take a product's inner index four consecutive values each, so that the
// operands along a row are 16-byte LDS reads; rows of KP + 4 floats spread both
// these and the reads down a column over the banks.  Wave w owns rows 16 w ..
// 16 w + 15 of the block in the first two products and rows j = 16 (w + 4 t) of
// dW1, held in registers across blocks.  With the rows in vector FMAs over LDS
// this was 423 us for 64 x 255 rows at k = 64; now bound by the start (W1, the
// gathers of z) of one block a workgroup.
constexpr int kMlpBwRows = 64;
constexpr int kMlpBwMaxK = 128;
constexpr int kMlpBwMaxParts = 256;

__host__ __device__ constexpr int mlp_bw_kp(int k) { return k <= 32 ? 32 : k <= 64 ? 64 : 128; }
__host__ __device__ constexpr int mlp_bw_lds_floats(int KP) { return (KP + 2 * kMlpBwRows) * (KP + 4) + 2 * KP + 12 * KP; }

template <int KP>
__global__ void __launch_bounds__(kBwThreads)
k_bw_mlp(const float* __restrict__ d, const int32_t* __restrict__ s, const float* __restrict__ dtau,
         const float* __restrict__ W1, const float* __restrict__ b1, const float* __restrict__ w2, float b2,
         float tmin, float tmax, float* __restrict__ dzg, float* __restrict__ part, int64_t B, int C, int R, int k) {
  constexpr int P = KP + 4;          // row pitch
  constexpr int NB = KP / 16;        // 16-wide blocks of k
  constexpr int JT = (NB + 3) / 4;   // row blocks of dW1 per wave
  extern __shared__ __align__(16) float lds[];
  float* w1s = lds;                  // [KP][P]
  float* zs = w1s + KP * P;          // [rows][P]
  float* hs = zs + kMlpBwRows * P;   // [rows][P]: dh
  float* bs = hs + kMlpBwRows * P;   // b1, w2
  float* red = bs + 2 * KP;          // the waves' sums at the end
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  // (reads clamped, then masked, so that they are all in flight together)
#pragma unroll 8
  for (int q = tid; q < KP * KP; q += kBwThreads) {
    const int j = q / KP, i = q % KP;
    const float v = W1[min(j, k - 1) * k + min(i, k - 1)];
    w1s[j * P + i] = j < k && i < k ? v : 0.f;
  }
  for (int q = tid; q < KP; q += kBwThreads) {
    bs[q] = q < k ? b1[q] : 0.f;
    bs[KP + q] = q < k ? w2[q] : 0.f;
  }
  f32x4 aw[JT][NB];                  // dW1 rows 16 (wv + 4 t) + 4 g + r, column 16 nb + n
  float pb1[NB], pw2[NB];            // unit 16 nb + n, over the rows this lane sees
  double pb2 = 0.;                   // one sum over every row, of either sign: float64, as in the reduction
#pragma unroll
  for (int t = 0; t < JT; ++t)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) aw[t][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) pb1[nb] = pw2[nb] = 0.f;
  const int64_t nrows = B * R;
  const int64_t nblk = (nrows + kMlpBwRows - 1) / kMlpBwRows;
  const float span = tmax - tmin;
  for (int64_t blk = blockIdx.x; blk < nblk; blk += gridDim.x) {
    const int64_t r0 = blk * kMlpBwRows;
    __syncthreads();   // the previous block's rows are consumed
    // z: channels first, then the descriptors, each all in flight
    constexpr int ZP = kMlpBwRows * KP / kBwThreads;
    constexpr int ZC = ZP < 16 ? ZP : 16;
#pragma unroll
    for (int u0 = 0; u0 < ZP; u0 += ZC) {
      int ch[ZC];
      int64_t rb[ZC];
#pragma unroll
      for (int u = 0; u < ZC; ++u) {
        const int q = tid + (u0 + u) * kBwThreads, i = q % KP;
        const int64_t row = min(r0 + q / KP, nrows - 1);
        rb[u] = row / R;
        ch[u] = s[(row - rb[u] * R) * k + min(i, k - 1)];
      }
      float zv[ZC];
#pragma unroll
      for (int u = 0; u < ZC; ++u) zv[u] = d[rb[u] * C + ch[u]];
#pragma unroll
      for (int u = 0; u < ZC; ++u) {
        const int q = tid + (u0 + u) * kBwThreads, rr = q / KP, i = q % KP;
        zs[rr * P + i] = r0 + rr < nrows && i < k ? zv[u] : 0.f;
      }
    }
    float dt[4];   // dtau of the wave's rows 4 g + r
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = r0 + 16 * wv + 4 * g + r;
      const float v = dtau[min(row, nrows - 1)];
      dt[r] = row < nrows ? v : 0.f;
    }
    __syncthreads();
    // hpre of the wave's 16 rows
    f32x4 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const float4 a = *reinterpret_cast<const float4*>(zs + (16 * wv + n) * P + 16 * c + 4 * g);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float4 w = *reinterpret_cast<const float4*>(w1s + (16 * nb + n) * P + 16 * c + 4 * g);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, w.x, acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, w.y, acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, w.z, acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, w.w, acc[nb], 0, 0, 0);
      }
    }
    // g, dg, dh: this lane holds rows 4 g + r, units 16 nb + n
    float gp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float bj = bs[16 * nb + n], wj = bs[KP + 16 * nb + n];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[nb][r] += bj;
        gp[r] += wj * fmaxf(acc[nb][r], 0.f);
      }
    }
    float dg[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float sg = 1.f / (1.f + expf(-(row16_sum(gp[r]) + b2)));
      dg[r] = dt[r] * span * sg * (1.f - sg);
      pb2 += n == 0 ? dg[r] : 0.f;
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float wj = bs[KP + 16 * nb + n];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float hp = acc[nb][r];
        pw2[nb] += dg[r] * fmaxf(hp, 0.f);
        const float dh = hp > 0.f ? dg[r] * wj : 0.f;
        pb1[nb] += dh;
        hs[(16 * wv + 4 * g + r) * P + 16 * nb + n] = dh;
      }
    }
    __syncthreads();
    // dzg = dh W1 of the wave's rows
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const float4 a = *reinterpret_cast<const float4*>(hs + (16 * wv + n) * P + 16 * c + 4 * g);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const float* w = w1s + (16 * c + 4 * g) * P + 16 * nb + n;
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, w[0], acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, w[P], acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, w[2 * P], acc[nb], 0, 0, 0);
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, w[3 * P], acc[nb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t row = r0 + 16 * wv + 4 * g + r;
      if (row < nrows)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          if (16 * nb + n < k) dzg[row * k + 16 * nb + n] = acc[nb][r];
    }
    // dW1 += dh^T z over the block's rows
#pragma unroll
    for (int c = 0; c < kMlpBwRows / 16; ++c) {
      const float* hr = hs + (16 * c + 4 * g) * P + n;
      const float* zr = zs + (16 * c + 4 * g) * P + n;
      float hv[JT][4];
#pragma unroll
      for (int t = 0; t < JT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) hv[t][r] = 16 * (wv + 4 * t) < KP ? hr[r * P + 16 * (wv + 4 * t)] : 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float zv = zr[r * P + 16 * nb];
#pragma unroll
          for (int t = 0; t < JT; ++t) aw[t][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(hv[t][r], zv, aw[t][nb], 0, 0, 0);
        }
    }
  }
  // partial layout per workgroup: [k*k dW1][k db1][k dw2][1 db2]
  const int kk = k * k;
  float* out = part + (int64_t)blockIdx.x * (kk + 2 * k + 1);
#pragma unroll
  for (int t = 0; t < JT; ++t)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = 16 * (wv + 4 * t) + 4 * g + r, i = 16 * nb + n;
        if (j < k && i < k) out[j * k + i] = aw[t][nb][r];
      }
  // db1, dw2, db2: over the four lane groups, then the four waves
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    pb1[nb] += __shfl_xor(pb1[nb], 16, kWave);
    pb1[nb] += __shfl_xor(pb1[nb], 32, kWave);
    pw2[nb] += __shfl_xor(pw2[nb], 16, kWave);
    pw2[nb] += __shfl_xor(pw2[nb], 32, kWave);
    if (g == 0) {
      red[wv * KP + 16 * nb + n] = pb1[nb];
      red[(4 + wv) * KP + 16 * nb + n] = pw2[nb];
    }
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) pb2 += __shfl_xor(pb2, off, kWave);
  double* redd = reinterpret_cast<double*>(red + 8 * KP);
  if (lane == 0) redd[wv] = pb2;
  __syncthreads();
  if (tid < k) {
    out[kk + tid] = (red[tid] + red[KP + tid]) + (red[2 * KP + tid] + red[3 * KP + tid]);
    out[kk + k + tid] = (red[4 * KP + tid] + red[5 * KP + tid]) + (red[6 * KP + tid] + red[7 * KP + tid]);
  }
  if (tid == 0) out[kk + 2 * k] = (float)((redd[0] + redd[1]) + (redd[2] + redd[3]));
}

// sums the per-workgroup partials into dW1, db1, dw2, db2: 32 entries a
// workgroup, eight threads each over every eighth partial (one thread over all
// of 512 took 161 us)
__global__ void __launch_bounds__(256)
k_bw_mlp_reduce(const float* __restrict__ part, int nparts, int k, float* __restrict__ dW1, float* __restrict__ db1,
                float* __restrict__ dw2, float* __restrict__ db2) {
  __shared__ double sums[8][32];
  const int n = k * k + 2 * k + 1;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const int q = blockIdx.x * 32 + x;
  double acc = 0.;
#pragma unroll 8
  for (int j = y; j < nparts; j += 8) acc += (double)part[(int64_t)j * n + min(q, n - 1)];
  sums[y][x] = acc;
  __syncthreads();
  if (y != 0 || q >= n) return;
  for (int j = 1; j < 8; ++j) acc += sums[j][x];
  const float v = (float)acc;
  if (q < k * k)
    dW1[q] = v;
  else if (q < k * k + k)
    db1[q - k * k] = v;
  else if (q < k * k + 2 * k)
    dw2[q - k * k - k] = v;
  else
    *db2 = v;
}

// ---------------------------------------------------------------- coverage loss
// Row statistics of the full logits: m_e = max_c L[e][c], Z_e = sum_c exp(L - m_e).
__global__ void __launch_bounds__(kBwThreads)
k_cov_rows(const float* __restrict__ L, float* __restrict__ mz, int C) {
  __shared__ float red[kBwWaves];
  const int e = blockIdx.x;
  const float* row = L + (int64_t)e * C;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  float m = -INFINITY;
  for (int c = tid; c < C; c += kBwThreads) m = fmaxf(m, row[c]);
  m = wave_max(m);
  if (lane == 0) red[wv] = m;
  __syncthreads();
  m = red[0];
  for (int j = 1; j < kBwWaves; ++j) m = fmaxf(m, red[j]);
  __syncthreads();
  float z = 0.f;
  for (int c = tid; c < C; c += kBwThreads) z += expf(row[c] - m);
  z = wave_sum(z);
  if (lane == 0) red[wv] = z;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
    for (int j = 0; j < kBwWaves; ++j) t += red[j];
    mz[2 * e] = m;
    mz[2 * e + 1] = t;
  }
}

// u[c] = (1/R) sum_e exp(L[e][c] - m_e) / Z_e: 32 channels a workgroup, 32
// threads each over every 32nd row, added in a fixed order (a thread over all
// rows took 80 us for 255 rows of 1024)
__global__ void __launch_bounds__(1024)
k_cov_cols(const float* __restrict__ L, const float* __restrict__ mz, float* __restrict__ u, int R, int C) {
  __shared__ float sums[32][33];
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const int c = blockIdx.x * 32 + x;
  float acc = 0.f;
#pragma unroll 8
  for (int e = y; e < R; e += 32) acc += expf(L[(int64_t)e * C + min(c, C - 1)] - mz[2 * e]) / mz[2 * e + 1];
  sums[y][x] = acc;
  __syncthreads();
  if (y != 0 || c >= C) return;
  for (int j = 1; j < 32; ++j) acc += sums[j][x];
  u[c] = acc / (float)R;
}

// the sum of every thread's v over the workgroup (red: kBwWaves floats; in a
// fixed order, so every workgroup forms the same bits)
__device__ __forceinline__ float block_sum(float v, float* red) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  v = wave_sum(v);
  __syncthreads();
  if (lane == 0) red[wv] = v;
  __syncthreads();
  float t = 0.f;
  for (int j = 0; j < kBwWaves; ++j) t += red[j];
  return t;
}

// A workgroup per row e.  Each forms the column statistics ub = mean u,
// num = sum (u - ub)^2, den = ub^2 + eps for itself (a launch for one workgroup
// of them cost more than reading u again); loss = num / den, and
//   du_c = 2 (u_c - ub) / den - num 2 ub / (C den^2),
//   dL[e][c] = lambda / R p_ec (du_c - sum_c' p_ec' du_c') + dw[e][i] where c = s_ei.
__global__ void __launch_bounds__(kBwThreads)
k_cov_grad(const float* __restrict__ L, const float* __restrict__ mz, const float* __restrict__ u, float eps,
           float* __restrict__ loss, const int32_t* __restrict__ s, const float* __restrict__ dw,
           float* __restrict__ dL, int R, int C, int k, float lambda) {
  extern __shared__ int32_t pos[];  // [C]: support position of channel c in this row, or -1
  __shared__ float red[kBwWaves];
  const int e = blockIdx.x;
  const int tid = threadIdx.x;
  const float* row = L + (int64_t)e * C;
  const float m = mz[2 * e], rz = 1.f / mz[2 * e + 1];
  if (dw) {
    for (int c = tid; c < C; c += kBwThreads) pos[c] = -1;
    __syncthreads();
    for (int i = tid; i < k; i += kBwThreads) pos[s[(int64_t)e * k + i]] = i;
  }
  float su = 0.f;
#pragma unroll 8
  for (int c = tid; c < C; c += kBwThreads) su += u[c];
  const float ub = block_sum(su, red) / (float)C;
  float sq = 0.f;
#pragma unroll 8
  for (int c = tid; c < C; c += kBwThreads) {
    const float dv = u[c] - ub;
    sq += dv * dv;
  }
  const float num = block_sum(sq, red), den = ub * ub + eps;
  if (loss && e == 0 && tid == 0) *loss = num / den;
  const float c1 = 2.f / den, c0 = num * 2.f * ub / ((float)C * den * den);
  float t = 0.f;
#pragma unroll 4
  for (int c = tid; c < C; c += kBwThreads) {
    const float p = expf(row[c] - m) * rz;
    t += p * (c1 * (u[c] - ub) - c0);
  }
  const float tt = block_sum(t, red);
  const float scale = lambda / (float)R;
  for (int c = tid; c < C; c += kBwThreads) {
    const float p = expf(row[c] - m) * rz;
    float g = scale * p * ((c1 * (u[c] - ub) - c0) - tt);
    if (dw) {
      const int i = pos[c];
      if (i >= 0) g += dw[(int64_t)e * k + i];
    }
    dL[(int64_t)e * C + c] = g;
  }
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

// lanes per row of the rows' kernel, and its image groups: about 2048 waves (8 a
// CU), at most 1024 groups.  (A group's images are a serial chain: with at most 64
// groups the backward of 58145 images, C 23, E 2, k 1, one position took 560 us, with
// 256 199, with 1024 127; of 8775, C 10, E 3, k 1 106, 55 and 47.)
int rows_lanes(int k) { return k <= 256 ? 16 : kWave; }
void backward_sum_groups(const Shape& sh, int* ng, int* gs) {
  const int64_t waves = std::max<int64_t>(1, ((int64_t)sh.R * rows_lanes(sh.k) + kWave - 1) / kWave);
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>({sh.B, (int64_t)1024, (2048 + waves - 1) / waves}));
  *gs = (int)((sh.B + want - 1) / want);
  *ng = (int)((sh.B + *gs - 1) / *gs);
}

bool backward_supported(const Shape& sh, int gate_kind) {
  return sh.k <= kBwMaxK && (gate_kind != MOCE_GATE_MLP_SIGMOID || sh.k <= kMlpBwMaxK);
}

size_t backward_mlp_parts(const Shape& sh) {
  const int64_t nblk = (sh.B * sh.R + kMlpBwRows - 1) / kMlpBwRows;
  return (size_t)std::max<int64_t>(1, std::min<int64_t>(nblk, kMlpBwMaxParts));
}

size_t backward_mlp_part_floats(const Shape& sh) { return (size_t)sh.k * sh.k + 2 * (size_t)sh.k + 1; }

hipError_t launch_backward(const Shape& sh, const void* x, const void* dy, const int32_t* s, const float* w,
                           const moce_gate_params& g, void* dx, float* dw, const moce_gate_grads& gg,
                           const BwdWs& ws, hipStream_t st) {
  const int64_t B = sh.B, HW = sh.HW;
  const int C = (int)sh.C, E = sh.E, R = sh.R, k = sh.k;
  const bool bf = sh.elem == MOCE_BF16, nhwc = sh.layout == MOCE_NHWC;
  const bool mlp = g.kind == MOCE_GATE_MLP_SIGMOID;
  hipError_t err;
  // the support entries by channel
  const int nblk = (C + kBwBucketCh - 1) / kBwBucketCh;
  if (R > 0) {
    const size_t lds = (size_t)std::min(nblk, kPrepWindow) * sizeof(int32_t);
    k_bw_part<<<blocks_for(R, kBwBucketEx), kPrepThreads, lds, st>>>(s, w, mlp ? w : g.a, ws.bbeg, ws.bw, ws.ba,
                                                                     R, k, nblk);
  }
  // channel lists: for the MLP gate's dd and the generic dx
  const bool lists = R == 0 || mlp || !bwd_dx_on_mfma(sh);
  if (lists)
    k_bw_lists<<<nblk, kPrepThreads, 0, st>>>(ws.bbeg, ws.bw, ws.ba, ws.off, ws.inv, ws.unc, R, k, C, nblk);
  if ((err = hipGetLastError()) != hipSuccess) return err;
  // |U| for the vector dx, in the place of the temperatures, which nothing here reads
  int32_t* nU = reinterpret_cast<int32_t*>(ws.tau);
  if (R > 0) {
    // forward quantities: d, the softmax statistics and the coefficients
    if ((err = launch_pool(sh, x, ws.d, st)) != hipSuccess) return err;
    // the coefficients themselves only for the generic dx (the matrix-core dx
    // rebuilds them from the statistics)
    float* alpha_out = bwd_dx_on_mfma(sh) ? nullptr : ws.alpha;
    if ((err = launch_gate(sh, ws.d, s, w, g, ws.tau, alpha_out, ws.stats, st)) != hipSuccess) return err;
    // dalpha
    if (!bwd_mfma_dalpha(sh, x, dy, ws, st, &err)) {
      auto launch = [&](auto* xx) {
        using T = std::remove_const_t<std::remove_pointer_t<decltype(xx)>>;
        const auto gy = static_cast<const T*>(dy);
        const auto kern = nhwc ? k_bw_dalpha<T, true> : k_bw_dalpha<T, false>;
        return image_slices(B, (int64_t)R * kWave, 1, [&](int64_t b0, int64_t n) {
          kern<<<blocks_for(n * R, kBwWaves), kBwThreads, 0, st>>>(xx + b0 * C * HW, gy + b0 * E * HW, s,
                                                                  ws.dal + b0 * R * k, n, C, E, R, k, (int)HW);
          return hipGetLastError();
        });
      };
      err = bf ? launch(static_cast<const uint16_t*>(x)) : launch(static_cast<const float*>(x));
    }
    if (err != hipSuccess) return err;
    // rows and their sums over groups of images
    int ng, gs;
    backward_sum_groups(sh, &ng, &gs);
    {
      int nsplit = 1, split_len = 0;
      bwd_dalpha_splits(sh, &nsplit, &split_len);
      const dim3 grid(blocks_for(R, kBwThreads / rows_lanes(k)), ng);
      const float* a = mlp ? nullptr : g.a;
      const float* cc = mlp ? nullptr : g.c;
      const auto kern = k <= 32    ? k_bw_rows<16, 2>
                        : k <= 64  ? k_bw_rows<16, 4>
                        : k <= 128 ? k_bw_rows<16, 8>
                        : k <= 256 ? k_bw_rows<16, 16>
                        : k <= 512 ? k_bw_rows<64, 8>
                                   : k_bw_rows<64, 16>;
      kern<<<grid, kBwThreads, 0, st>>>(ws.dal, w, ws.stats, ws.d, s, a, cc, ws.dtau, ws.dg, ws.psum, B, C, R, k, nsplit,
                                        gs);
      const int64_t rk = (int64_t)R * k, n = mlp ? rk : 2 * rk + R;
      k_bw_sums_reduce<<<blocks_for(n, 32), 256, 0, st>>>(ws.psum, ng, rk, n, dw, mlp ? nullptr : gg.da,
                                                          mlp ? nullptr : gg.dc, lists ? ws.unc : nullptr, C, nU);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    if (mlp) {
      const int nparts = (int)backward_mlp_parts(sh);
      const int KP = mlp_bw_kp(k);
      const size_t lds = (size_t)mlp_bw_lds_floats(KP) * sizeof(float);
      const auto kern = KP == 32 ? k_bw_mlp<32> : KP == 64 ? k_bw_mlp<64> : k_bw_mlp<128>;
      if ((err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)) !=
          hipSuccess)
        return err;
      kern<<<nparts, kBwThreads, lds, st>>>(ws.d, s, ws.dtau, g.W1, g.b1, g.w2, g.b2, g.tau_min, g.tau_max, ws.dzg,
                                            ws.part, B, C, R, k);
      const int nq = (int)backward_mlp_part_floats(sh);
      k_bw_mlp_reduce<<<blocks_for(nq, 32), 256, 0, st>>>(ws.part, nparts, k, gg.dW1, gg.db1, gg.dw2, gg.db2);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    const bool dd_lists = mlp || (lists && dd_by_lists(sh));
    if (dd_lists)
      err = image_slices(B, C, 1, [&](int64_t b0, int64_t n) {
        const auto kern = mlp ? k_bw_dd_lists<true> : k_bw_dd_lists<false>;
        kern<<<blocks_for(n * C, kBwThreads), kBwThreads, 0, st>>>(ws.off, ws.inv, ws.dzg + b0 * R * k, ws.dg + b0 * R,
                                                                  g.a, ws.dd + b0 * C, n, C, R, k);
        return hipGetLastError();
      });
    else
      err = image_slices(B, kDdSliceThreads, 1, [&](int64_t b0, int64_t n) {
        k_bw_dd_linear<<<dim3(nblk, blocks_for(n, kDdImages)), kBwThreads, 0, st>>>(
            ws.bbeg, ws.bw, ws.ba, ws.dg + b0 * R, ws.dd + b0 * C, ws.unc, n, C, R, nblk);
        return hipGetLastError();
      });
    if (err != hipSuccess) return err;
  }
  // dx
  if (bwd_mfma_dx(sh, dy, ws, dx, st, &err)) return err;
  auto launch = [&](auto* o) {
    using T = std::remove_pointer_t<decltype(o)>;
    const auto gy = static_cast<const T*>(dy);
    const auto kern = nhwc ? k_bw_dx<T, true> : k_bw_dx<T, false>;
    return image_slices(B, C * HW, 1, [&](int64_t b0, int64_t n) {
      kern<<<blocks_for(n * C * HW, kBwThreads), kBwThreads, 0, st>>>(gy + b0 * E * HW, ws.alpha + b0 * R * k, ws.off,
                                                                     ws.inv, nU, ws.dd + b0 * C, o + b0 * C * HW,
                                                                     n, C, E, R, k, (int)HW);
      return hipGetLastError();
    });
  };
  return bf ? launch(static_cast<uint16_t*>(dx)) : launch(static_cast<float*>(dx));
}

bool logit_backward_supported(int64_t C) { return C >= 1 && C <= kCovMaxC; }

hipError_t launch_logit_backward(int R, int C, int k, const float* L, const int32_t* s, const float* dw, float eps,
                                 float lambda, float* loss, float* dL, float* ws, hipStream_t st) {
  float* mz = ws;                 // [2 R]
  float* u = mz + 2 * (size_t)R;  // [C]
  const size_t lds = dw ? (size_t)C * sizeof(int32_t) : 0;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_cov_grad, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  k_cov_rows<<<R, kBwThreads, 0, st>>>(L, mz, C);
  k_cov_cols<<<blocks_for(C, 32), 1024, 0, st>>>(L, mz, u, R, C);
  k_cov_grad<<<R, kBwThreads, lds, st>>>(L, mz, u, eps, loss, s, dw, dL, R, C, k, lambda);
  return hipGetLastError();
}

}  // namespace moce
