// Input-conditioned supports (Sec. 4.5, Eq. 11), the inference path.
//
// The variant keeps the temperature gate and the residual, and replaces the
// static supports by per-example ones: a router reads the whole pooled
// descriptor z, h = ReLU(Wh z + bh) (d outputs), and adds a rank-d offset to
// the routing logits, L(X)[e][c] = L[e][c] + <q_e * h, v_c>.  Each example then
// takes its own top-k channels per routed expert, the gate reads z at that
// support, the coefficients are the softmax of L(X) at the support over the
// temperature, and the residual averages the channels in no support of that
// example.
//
// Launches: pooling (pool.hip), the router (a wave per (image, bottleneck
// unit)), then for C <= 2048, k <= 160 and d <= 32 logits, selection, gate and
// U(X) by dyntop.hip, elsewhere selection (a workgroup per (image, block of EB
// experts): the block's logit rows are formed in LDS and each wave takes a row's
// top k by a radix select over order-preserving 32-bit keys, then sorts the k by
// (logit descending, channel ascending)), the per-example uncovered set (a
// workgroup per image) and the gate and coefficients (a wave per (image,
// expert)); and the mix (a workgroup per (image, tile of positions) with the tile
// of every channel in LDS).
#include <algorithm>
#include <climits>
#include <initializer_list>
#include <type_traits>

#include "dyn_keys.h"
#include "moce_internal.h"

namespace moce {
namespace {

constexpr int kDynThreads = 256;
constexpr int kDynWaves = kDynThreads / kWave;
constexpr size_t kDynLds = 160 * 1024;
constexpr int kDynMaxD = 64;     // bottleneck width
constexpr int kDynMaxC = 4096;   // the gather stages C rows of 16 bytes a unit, the selection rows of C logits

// ---------------------------------------------------------------- router
__global__ void __launch_bounds__(kDynThreads)
k_dyn_router(const float* __restrict__ d, const float* __restrict__ Wh, const float* __restrict__ bh,
             float* __restrict__ h, int64_t B, int C, int dd) {
  const int64_t wave = (int64_t)blockIdx.x * kDynWaves + (threadIdx.x >> 6);
  if (wave >= B * dd) return;  // whole waves
  const int lane = threadIdx.x & 63;
  const int64_t b = wave / dd;
  const int t = (int)(wave - b * dd);
  float acc = 0.f;
#pragma unroll 8
  for (int c = lane; c < C; c += kWave) acc += Wh[(int64_t)t * C + c] * d[b * C + c];
  acc = wave_sum(acc);
  if (lane == 0) h[wave] = fmaxf(acc + bh[t], 0.f);
}

// vT[t][c] = v[c][t]: the channel embeddings transposed, 32 x 32 tiles
// through LDS
__global__ void __launch_bounds__(1024)
k_dyn_transpose(const float* __restrict__ v, float* __restrict__ vT, int C, int dd) {
  __shared__ float tile[32][33];
  const int c0 = blockIdx.x * 32, t0 = blockIdx.y * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  if (c0 + ty < C && t0 + tx < dd) tile[ty][tx] = v[(int64_t)(c0 + ty) * dd + t0 + tx];
  __syncthreads();
  if (t0 + ty < dd && c0 + tx < C) vT[(int64_t)(t0 + ty) * C + c0 + tx] = tile[tx][ty];
}

// ---------------------------------------------------------------- selection
// (key a, channel a) comes before (key b, channel b): larger logit first,
// then the lower channel
__device__ __forceinline__ bool before(uint32_t ka, int ca, uint32_t kb, int cb) {
  return ka > kb || (ka == kb && ca < cb);
}
__device__ __forceinline__ void lds_wait() { __builtin_amdgcn_s_waitcnt(0xc07f); }  // lgkmcnt(0)

// LDS per wave for one row's selection: the radix histogram and the list of
// the selected (key, channel) pairs, kl = the power of two >= k entries
constexpr int kDynMaxK = 512;
__host__ __device__ inline int list_len(int k) {
  int P = 1;
  while (P < k) P <<= 1;
  return P;
}
__host__ __device__ inline int wave_words(int k) { return 256 + 2 * list_len(k); }

// The top k of one logit row by one wave: the k-th largest key by a radix
// select, most significant byte first, then the keys above it and the
// lowest-channel ones equal to it, sorted into the canonical order (logit
// descending, channel ascending).  hist: 256 words of LDS; lkey, lch: P
// entries each (P = list_len(k)), which may overlap hist.
__device__ __forceinline__ void select_row(const float* row, uint32_t* hist, uint32_t* lkey, int32_t* lch, int C,
                                           int k, int P, int lane, int32_t* __restrict__ Sout,
                                           float* __restrict__ Wout) {
    // the k-th largest key, most significant byte first: after each round,
  // `prefix` holds the known high bytes and kk the rank still to find
  // among the keys with that prefix
  uint32_t prefix = 0, mask = 0;
  int kk = k;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int i = lane; i < 256; i += kWave) hist[i] = 0;
    lds_wait();
    for (int c = lane; c < C; c += kWave) {
      const uint32_t key = fkey(row[c]);
      if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    lds_wait();
    // lane l holds bins 4 l .. 4 l + 3; counts above a lane's bins by a
    // suffix sum over the lanes
    uint32_t cnt[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) cnt[j] = hist[4 * lane + j];
    const uint32_t mine = cnt[0] + cnt[1] + cnt[2] + cnt[3];
    uint32_t incl = mine;  // sum over lanes >= this one
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t o = __shfl_down(incl, off, kWave);
      if (lane + off < kWave) incl += o;
    }
    uint32_t above = incl - mine;
    int digit = -1;
    uint32_t before_digit = 0;
    if (above < (uint32_t)kk && (uint32_t)kk <= incl) {
#pragma unroll
      for (int j = 3; j >= 0; --j) {
        if (digit < 0 && above + cnt[j] >= (uint32_t)kk) {
          digit = 4 * lane + j;
          before_digit = above;
        }
        above += cnt[j];
      }
    }
    const uint64_t found = __ballot(digit >= 0);
    const int src = __builtin_ctzll(found);
    digit = __shfl(digit, src, kWave);
    before_digit = __shfl(before_digit, src, kWave);
    kk -= (int)before_digit;
    prefix |= (uint32_t)digit << shift;
    mask |= 255u << shift;
    lds_wait();
  }
  // every key above the k-th is taken, and the lowest-channel kk of those
  // equal to it; gathered in channel order
  const uint32_t kstar = prefix;
  const uint64_t below = (1ull << lane) - 1ull;
  int taken = 0, eq_seen = 0;
  for (int c0 = 0; c0 < C; c0 += kWave) {
    const int c = c0 + lane;
    const uint32_t key = c < C ? fkey(row[c]) : 0u;
    const bool eq = c < C && key == kstar;
    const uint64_t beq = __ballot(eq);
    const bool sel = (c < C && key > kstar) || (eq && eq_seen + __popcll(beq & below) < kk);
    const uint64_t bsel = __ballot(sel);
    if (sel && taken + __popcll(bsel & below) < P) {
      const int pos = taken + __popcll(bsel & below);
      lkey[pos] = key;
      lch[pos] = c;
    }
    taken += __popcll(bsel);
    eq_seen += __popcll(beq);
  }
  // bitonic sort of the k (padded to a power of two with entries that sort
  // last) into the canonical order
  for (int i = k + lane; i < P; i += kWave) {
    lkey[i] = 0u;
    lch[i] = INT_MAX;
  }
  lds_wait();
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = lane; i < P / 2; i += kWave) {
        const int lo = 2 * stride * (i / stride) + (i % stride), hi = lo + stride;
        const uint32_t ka = lkey[lo], kb = lkey[hi];
        const int ca = lch[lo], cb = lch[hi];
        // runs of `size` alternate between the canonical order and its reverse
        const bool forward = (lo & size) == 0;
        if (forward ? before(kb, cb, ka, ca) : before(ka, ca, kb, cb)) {
          lkey[lo] = kb;
          lch[lo] = cb;
          lkey[hi] = ka;
          lch[hi] = ca;
        }
      }
      lds_wait();
    }
  }
  for (int i = lane; i < k; i += kWave) {
    Sout[i] = lch[i];
    Wout[i] = fkey_value(lkey[i]);
  }
  lds_wait();
}

// EB experts of one image per workgroup of EB waves (a row each); DD >= the
// bottleneck width
template <int EB, int DD>
__global__ void __launch_bounds__(EB * kWave)
k_dyn_select(const float* __restrict__ h, const float* __restrict__ L, const float* __restrict__ q,
             const float* __restrict__ vT, int32_t* __restrict__ S, float* __restrict__ W, int C, int R, int k,
             int dd, int nblk) {
  extern __shared__ float sm[];
  float* rows = sm;              // [EB][C] the block's logit rows of this image
  float* qh = rows + EB * C;     // [EB][DD] q_e * h, zero past dd
  const int P = list_len(k);
  uint32_t* wsm = reinterpret_cast<uint32_t*>(qh + EB * DD) + (threadIdx.x >> 6) * (256 + 2 * P);
  uint32_t* hist = wsm;
  uint32_t* lkey = hist + 256;
  int32_t* lch = reinterpret_cast<int32_t*>(lkey + P);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t b = blockIdx.x / nblk;
  const int e0 = (int)(blockIdx.x % nblk) * EB;
  const int ne = min(EB, R - e0);
  for (int i = threadIdx.x; i < EB * DD; i += blockDim.x) {
    const int e = i / DD, t = i - e * DD;
    const float qv = q[(int64_t)min(e0 + e, R - 1) * dd + min(t, dd - 1)];
    const float hv = h[b * dd + min(t, dd - 1)];
    qh[i] = t < dd ? qv * hv : 0.f;
  }
  __syncthreads();
  // logits: a thread per channel, v_c in registers (from the transposed
  // embeddings vT[d][C], so a wave's reads of one t are consecutive), every
  // expert of the block
  for (int c = threadIdx.x; c < C; c += blockDim.x) {
    float vr[DD];
#pragma unroll
    for (int t = 0; t < DD; ++t) {
      const float x = vT[(int64_t)min(t, dd - 1) * C + c];
      vr[t] = t < dd ? x : 0.f;
    }
#pragma unroll 4
    for (int e = 0; e < EB; ++e) {
      float off = 0.f;
#pragma unroll
      for (int t = 0; t < DD; ++t) off += qh[e * DD + t] * vr[t];
      rows[e * C + c] = L[(int64_t)min(e0 + e, R - 1) * C + c] + off;
    }
  }
  __syncthreads();
  // each wave: one row
  for (int e = wv; e < ne; e += EB) {
    const int64_t item = b * R + e0 + e;
    select_row(rows + e * C, hist, lkey, lch, C, k, P, lane, S + item * k, W + item * k);
  }
}

// ---------------------------------------------------------------- U(X)
// A workgroup per image: the channels in none of the image's supports, in
// ascending order, by a block-wide compaction.
__global__ void __launch_bounds__(1024)
k_dyn_uncovered(const int32_t* __restrict__ S, int32_t* __restrict__ U, int32_t* __restrict__ nU, int C, int R,
                int k) {
  extern __shared__ unsigned char cov[];  // [C] flags, then 16 wave counts
  int32_t* wcnt = reinterpret_cast<int32_t*>(cov + ((C + 15) & ~15));
  const int64_t b = blockIdx.x;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int c = threadIdx.x; c < C; c += blockDim.x) cov[c] = 0;
  __syncthreads();
  const int64_t n = (int64_t)R * k;
#pragma unroll 8
  for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
    const int32_t c = S[b * n + j];
    if ((uint32_t)c < (uint32_t)C) cov[c] = 1;
  }
  __syncthreads();
  const uint64_t below = (1ull << lane) - 1ull;
  int base = 0;
  for (int c0 = 0; c0 < C; c0 += blockDim.x) {
    const int c = c0 + threadIdx.x;
    const bool f = c < C && !cov[c];
    const uint64_t bf = __ballot(f);
    if (lane == 0) wcnt[wv] = __popcll(bf);
    __syncthreads();
    int off = base;
    for (int w = 0; w < wv; ++w) off += wcnt[w];
    if (f) U[b * C + off + __popcll(bf & below)] = c;
    int tot = 0;
    for (int w = 0; w < nw; ++w) tot += wcnt[w];
    base += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) nU[b] = base;
}

// ---------------------------------------------------------------- gate
// A wave per (image, routed expert): z at the example's support, the gate's
// temperature, and the coefficients from the example's logits there (the
// library's coefficient operations; the largest scaled logit from the
// largest logit, as 1/tau > 0).
__global__ void __launch_bounds__(kDynThreads)
k_dyn_gate(const float* __restrict__ d, const int32_t* __restrict__ S, const float* __restrict__ W,
           moce_gate_params g, float* __restrict__ tau, float* __restrict__ alpha, int64_t B, int C, int R, int k) {
  __shared__ float zsm[kDynWaves][kDynMaxK];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t item = (int64_t)blockIdx.x * kDynWaves + wv;
  if (item >= B * R) return;  // whole waves; no block barrier below
  const int64_t b = item / R;
  const int e = (int)(item - b * R);
  const int32_t* s = S + item * k;
  const float* w = W + item * k;
  float* z = zsm[wv];
  for (int i = lane; i < k; i += kWave) z[i] = d[b * C + min(max(s[i], 0), C - 1)];
  lds_wait();
  float t;
  if (g.kind == MOCE_GATE_SOFTPLUS_LINEAR) {
    float acc = 0.f;
    for (int i = lane; i < k; i += kWave) acc += g.a[(int64_t)e * k + i] * z[i];
    t = softplusf(wave_sum(acc) + g.c[e]) + 1e-3f;
  } else {
    float acc = 0.f;
    for (int j = lane; j < k; j += kWave) {
      float hj = g.b1[j];
      for (int i = 0; i < k; ++i) hj += g.W1[(int64_t)j * k + i] * z[i];
      acc += g.w2[j] * fmaxf(hj, 0.f);
    }
    const float gg = wave_sum(acc) + g.b2;
    t = g.tau_min + (g.tau_max - g.tau_min) / (1.f + expf(-gg));
  }
  const float rt = 1.f / t;
  float wm = -INFINITY;
  for (int i = lane; i < k; i += kWave) wm = fmaxf(wm, w[i]);
  const float m = coef_z(wave_max(wm), rt);
  float zs = 0.f;
  for (int i = lane; i < k; i += kWave) zs += coef_e(coef_z(w[i], rt), m);
  const float rzs = 1.f / wave_sum(zs);
  for (int i = lane; i < k; i += kWave) alpha[item * k + i] = coef_alpha(coef_e(coef_z(w[i], rt), m), rzs);
  if (lane == 0) tau[item] = t;
}

// ---------------------------------------------------------------- mix
template <typename T> __device__ __forceinline__ void st(T* p, float v);
template <> __device__ __forceinline__ void st<float>(float* p, float v) { *p = v; }
template <> __device__ __forceinline__ void st<uint16_t>(uint16_t* p, float v) { *p = f32_to_bf16(v); }

// The gather over per-example supports.  A workgroup takes NU units of 16 bytes
// of positions (PU = 8 bfloat16 or 4 float32 each) of one image and stages them
// for every channel in LDS, unit by unit ([NU][C] rows of 16 bytes, so that
// random channels spread over the bank groups); one 16-byte read then serves a
// support entry at PU positions, and an entry read from memory serves all PU NU.
// LPE = 4 lanes share an expert where k is large: they read 64 consecutive bytes
// of its support and coefficient rows a round, and their partial sums meet in a
// reduce-scatter that leaves each lane a quarter of the positions.  The
// residual (the mean over U(X)) is summed by one wave, lanes splitting U.  Bound
// by the bank conflicts of the random 16-byte reads and by the unpacking.
constexpr int kMixThreads = 1024;     // at most
constexpr int kMixSplitK = 32;        // entries from which four lanes share an expert
constexpr int kMixMinThreads = 128;   // two waves: the last one also sums the residual
constexpr int kMixTarget = 512;       // workgroups that a few tiles are shared out to

template <typename T> struct Unit;
template <> struct Unit<uint16_t> {
  static constexpr int PU = 8;
  __device__ static void fma(float* acc, const uint4& v, float a) {
    acc[0] += a * bf16_lo(v.x);
    acc[1] += a * bf16_hi(v.x);
    acc[2] += a * bf16_lo(v.y);
    acc[3] += a * bf16_hi(v.y);
    acc[4] += a * bf16_lo(v.z);
    acc[5] += a * bf16_hi(v.z);
    acc[6] += a * bf16_lo(v.w);
    acc[7] += a * bf16_hi(v.w);
  }
};
template <> struct Unit<float> {
  static constexpr int PU = 4;
  __device__ static void fma(float* acc, const uint4& v, float a) {
    acc[0] += a * __uint_as_float(v.x);
    acc[1] += a * __uint_as_float(v.y);
    acc[2] += a * __uint_as_float(v.z);
    acc[3] += a * __uint_as_float(v.w);
  }
};

// the value of lane l ^ M (M = 1, 2) within a quad
template <int M>
__device__ __forceinline__ float quad_xor(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), M == 1 ? 0xb1 : 0x4e, 0xf, 0xf, true));
}

struct DynMixArgs {
  const void* x;
  const int32_t* S;
  const float* alpha;
  const int32_t *U, *nU;
  void* y;
  int C, HW, E, k, ntiles;
  int nes, eper;   // workgroups that share a tile's experts, and their share
  int vec;   // rows of S and alpha can be read in 16-byte pieces
};

template <typename T, bool NHWC, int NU, int LPE>
__global__ void __launch_bounds__(kMixThreads)
k_dyn_gather(DynMixArgs p) {
  constexpr int PU = Unit<T>::PU, NP = PU * NU;
  extern __shared__ __align__(16) unsigned char xl[];   // [NU][C] rows of 16 bytes
  const int C = p.C, HW = p.HW, E = p.E, R = E - 1, k = p.k;
  const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;
  // (only with one unit a workgroup: the range of experts cost the others 8 us of 53 at
  // 128 images, C 2048, E 512, k 128, 7 x 7)
  constexpr bool SHARED = NU == 1;
  const unsigned tile = SHARED ? blockIdx.x / p.nes : blockIdx.x;
  const int es = SHARED ? (int)(blockIdx.x % p.nes) : 0;
  const int64_t b = tile / p.ntiles;
  const int p0 = (int)(tile % p.ntiles) * NP;
  const T* xb = static_cast<const T*>(p.x) + b * (int64_t)C * HW;
  uint4* rows = reinterpret_cast<uint4*>(xl);
  // ---- x; positions past the image repeat its last one
  if (NHWC && (sizeof(T) == 4 || C % 2 == 0)) {
    // two (float32: one) consecutive channels at the PU positions of a unit
    constexpr int CP = 4 / (int)sizeof(T);
    const int nc = C / CP;
    for (int i = tid; i < NU * nc; i += nt) {
      const int u = i / nc, c = (i - u * nc) * CP;
      uint32_t w[PU];
#pragma unroll
      for (int j = 0; j < PU; ++j)
        w[j] = *reinterpret_cast<const uint32_t*>(xb + (int64_t)min(p0 + u * PU + j, HW - 1) * C + c);
      if constexpr (sizeof(T) == 4) {
        rows[u * C + c] = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
        constexpr uint32_t kLo = 0x05040100u, kHi = 0x07060302u;   // low, high halves of (src1, src0)
        rows[u * C + c] = make_uint4(__builtin_amdgcn_perm(w[1], w[0], kLo), __builtin_amdgcn_perm(w[3], w[2], kLo),
                                     __builtin_amdgcn_perm(w[5], w[4], kLo), __builtin_amdgcn_perm(w[7], w[6], kLo));
        rows[u * C + c + 1] = make_uint4(__builtin_amdgcn_perm(w[1], w[0], kHi), __builtin_amdgcn_perm(w[3], w[2], kHi),
                                         __builtin_amdgcn_perm(w[5], w[4], kHi), __builtin_amdgcn_perm(w[7], w[6], kHi));
      }
    }
  } else if (!NHWC && HW % PU == 0) {
    for (int i = tid; i < NU * C; i += nt) {
      const int c = i / NU, u = i - c * NU;
      rows[u * C + c] = *reinterpret_cast<const uint4*>(xb + (int64_t)c * HW + min(p0 + u * PU, HW - PU));
    }
  } else {
    T* el = reinterpret_cast<T*>(xl);
    for (int i = tid; i < NP * C; i += nt) {
      const int c = NHWC ? i % C : i / NP, j = NHWC ? i / C : i % NP;
      const int q = min(p0 + j, HW - 1);
      el[((j / PU) * C + c) * PU + j % PU] = xb[NHWC ? (int64_t)q * C + c : (int64_t)c * HW + q];
    }
  }
  __syncthreads();

  T* yb = static_cast<T*>(p.y) + b * (int64_t)E * HW;
  // n results of output o at positions p0 + q0 ..; of whole planes in pieces of up to 16
  // bytes (one image of C 1408, E 1408, k 6, 56 x 56 in bfloat16: 27 us, by elements 52)
  auto store = [&](int o, int q0, const float* v, auto count) __attribute__((always_inline)) {
    constexpr int n = decltype(count)::value;
    if constexpr (!NHWC && n > 1 && (LPE == 1 || NU == 1)) {   // (four lanes an expert and more units: no register left)
      if (HW % PU == 0) {
        constexpr int PC = n < PU ? n : PU;   // positions a piece
        T* yo = yb + (int64_t)o * HW + p0 + q0;
#pragma unroll
        for (int j = 0; j < n; j += PC) {
          if (p0 + q0 + j >= HW) break;
          struct alignas(PC * sizeof(T)) { T e[PC]; } w;
#pragma unroll
          for (int i = 0; i < PC; ++i) st<T>(&w.e[i], v[j + i]);
          *reinterpret_cast<decltype(w)*>(yo + j) = w;
        }
        return;
      }
    }
#pragma unroll
    for (int j = 0; j < n; ++j) {
      const int q = p0 + q0 + j;
      if (q < HW) st<T>(NHWC ? yb + (int64_t)q * E + o : yb + (int64_t)o * HW + q, v[j]);
    }
  };
  // ---- the routed outputs
  const int PER = nt / LPE;   // experts a pass
  const int sub = tid % LPE;
  const int nch = (k + 4 * LPE - 1) / (4 * LPE);
  const int e0 = SHARED ? es * p.eper : 0, e1 = SHARED ? min(R, e0 + p.eper) : R;
  for (int o = e0 + tid / LPE; o < e1; o += PER) {
    const int32_t* Sr = p.S + (b * R + o) * k;
    const float* ar = p.alpha + (b * R + o) * k;
    // entries i0 .. i0 + 3 of a round; past the row: channel 0 with coefficient 0
    auto fetch = [&](int j, int (&c)[4], float (&a)[4]) __attribute__((always_inline)) {
      const int i0 = (min(j, nch - 1) * LPE + sub) * 4;
      if (p.vec) {
        const int ic = min(i0, k - 4);
        const int4 c4 = *reinterpret_cast<const int4*>(Sr + ic);
        const float4 a4 = *reinterpret_cast<const float4*>(ar + ic);
        const bool in = i0 < k;
        c[0] = c4.x; c[1] = c4.y; c[2] = c4.z; c[3] = c4.w;
        a[0] = in ? a4.x : 0.f; a[1] = in ? a4.y : 0.f; a[2] = in ? a4.z : 0.f; a[3] = in ? a4.w : 0.f;
      } else {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const int ic = min(i0 + t, k - 1);
          c[t] = Sr[ic];
          const float av = ar[ic];
          a[t] = i0 + t < k ? av : 0.f;
        }
      }
    };
    float acc[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) acc[q] = 0.f;
    int c[4], cn[4];
    float a[4], an[4];
    fetch(0, c, a);
    for (int j = 0; j < nch; ++j) {
      fetch(j + 1, cn, an);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const uint4* r = rows + min(max(c[t], 0), C - 1);
        if ((j * LPE + sub) * 4 + t < k) {   // a zero coefficient past the row must not meet an infinity
#pragma unroll
          for (int u = 0; u < NU; ++u) Unit<T>::fma(acc + u * PU, r[u * C], a[t]);
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        c[t] = cn[t];
        a[t] = an[t];
      }
    }
    if constexpr (LPE == 4) {
      float h[NP / 2], r[NP / 4];
      const bool s2 = sub & 2, s1 = sub & 1;
#pragma unroll
      for (int q = 0; q < NP / 2; ++q)
        h[q] = (s2 ? acc[q + NP / 2] : acc[q]) + quad_xor<2>(s2 ? acc[q] : acc[q + NP / 2]);
#pragma unroll
      for (int q = 0; q < NP / 4; ++q)
        r[q] = (s1 ? h[q + NP / 4] : h[q]) + quad_xor<1>(s1 ? h[q] : h[q + NP / 4]);
      store(o, sub * (NP / 4), r, std::integral_constant<int, NP / 4>{});
    } else {
      store(o, 0, acc, std::integral_constant<int, NP>{});
    }
  }
  // ---- the residual, by the wave with the fewest experts
  if ((SHARED && es != p.nes - 1) || tid < nt - kWave) return;
  float acc[NP];
#pragma unroll
  for (int q = 0; q < NP; ++q) acc[q] = 0.f;
  const int n = p.nU[b];
  for (int u = lane; u < n; u += kWave) {
    const uint4* r = rows + min(max(p.U[b * C + u], 0), C - 1);
#pragma unroll
    for (int t = 0; t < NU; ++t) Unit<T>::fma(acc + t * PU, r[t * C], 1.f);
  }
  const float inv = n > 0 ? 1.f / (float)n : 0.f;
  float mine = 0.f;
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const float v = wave_sum(acc[q]);
    mine = lane == q ? v : mine;
  }
  mine *= inv;
  if (lane < NP) store(R, lane, &mine, std::integral_constant<int, 1>{});
}

// experts (and waves) per selection workgroup: as many of 8, 4 and 2 as let two
// workgroups share a CU's LDS, else as one fits (2 holds the largest C and k)
size_t select_lds(const Shape& sh, int eb, int DD) {
  return ((size_t)eb * sh.C + (size_t)eb * DD) * 4 + (size_t)eb * wave_words(sh.k) * 4;
}
int select_eb(const Shape& sh, int DD) {
  for (int eb : {8, 4, 2})
    if (2 * select_lds(sh, eb, DD) <= kDynLds) return eb;
  for (int eb : {8, 4, 2})
    if (select_lds(sh, eb, DD) <= kDynLds) return eb;
  return 0;
}

template <int DD>
hipError_t launch_select_dd(const Shape& sh, const float* h, const float* L, const float* q, const float* vT,
                            int32_t* S, float* W, int dd, hipStream_t st) {
  using K = void (*)(const float*, const float*, const float*, const float*, int32_t*, float*, int, int, int, int,
                     int);
  const int eb = select_eb(sh, DD);
  if (eb == 0) return hipErrorInvalidValue;
  const int nblk = (sh.R + eb - 1) / eb;
  const size_t lds = select_lds(sh, eb, DD);
  const K kern = eb == 8 ? k_dyn_select<8, DD> : eb == 4 ? k_dyn_select<4, DD> : k_dyn_select<2, DD>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(sh.B * nblk)), dim3(eb * kWave), lds, st, h, L, q, vT, S, W, (int)sh.C,
                     sh.R, sh.k, dd, nblk);
  return hipGetLastError();
}

template <typename T, bool NHWC, int NU>
hipError_t launch_gather_nu(const Shape& sh, DynMixArgs p, hipStream_t st) {
  constexpr int NP = Unit<T>::PU * NU;
  p.ntiles = (int)((sh.HW + NP - 1) / NP);
  const size_t lds = (size_t)NU * sh.C * 16;
  // four lanes an expert where they have whole rounds of 16 entries to share
  auto kern = sh.k >= kMixSplitK ? k_dyn_gather<T, NHWC, NU, 4> : k_dyn_gather<T, NHWC, NU, 1>;
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  // Threads for the experts' lanes and the residual's wave, and, so that the loads of x
  // of few workgroups still fill a CU, 2048 over the workgroups that share one by LDS
  // and by their number.  Always 1024 left most waves of few experts without work: 1424
  // bfloat16 images of C 15, E 7, k 8, 785 positions channels-first 371 us (135 with 128
  // threads); with 256 for all, 17 of C 1204, E 602, k 38, 7 x 7 98 (85 with 1024).
  //
  // Few tiles leave most CUs idle: their experts are shared out, two waves' worth or more
  // a workgroup (23 images, C 853, E 853, k 426, one position: 730 us for the whole forward
  // with a workgroup a tile, 568 with the tiles shared out to 512, 590 to 1024).
  const int lpe = sh.k >= kMixSplitK ? 4 : 1;
  const int64_t all = sh.B * p.ntiles;
  p.nes = 1;
  if (NU == 1) p.nes = (int)std::max<int64_t>(1, std::min<int64_t>(kMixTarget / all, (int64_t)sh.R * lpe / kMixMinThreads));
  p.eper = std::max(1, (sh.R + p.nes - 1) / p.nes);
  p.nes = std::max(1, (sh.R + p.eper - 1) / p.eper);
  const int64_t tiles = all * p.nes, lanes = (int64_t)p.eper * lpe + kWave;
  const int64_t share = std::max<int64_t>(1, std::min<int64_t>(kDynLds / lds, (tiles + 255) / 256));
  int threads = kMixMinThreads;
  while (threads < kMixThreads && threads < std::max(lanes, 2048 / share)) threads *= 2;
  // a launch holds fewer than 2^32 threads (the excess would be dropped without an
  // error): smaller workgroups where there are that many tiles
  while (threads > kMixMinThreads && tiles * threads >= (int64_t)1 << 32) threads /= 2;
  hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(threads), lds, st, p);
  return hipGetLastError();
}

template <typename T, bool NHWC>
hipError_t launch_gather_t(const Shape& sh, const DynMixArgs& p, hipStream_t st) {
  // as many units a workgroup as the LDS holds, each entry then serving more
  // positions, while every CU still has a workgroup and the image more than half of
  // one's units (20000 float32 images of C 36, E 9, k 24, one position: 418 us with four
  // units, 403 with one)
  const int64_t units = (sh.HW + Unit<T>::PU - 1) / Unit<T>::PU;
  auto fits = [&](int nu) {
    return (size_t)nu * sh.C * 16 <= 128 * 1024 && sh.B * ((units + nu - 1) / nu) >= 256 && units > nu / 2;
  };
  return fits(4) ? launch_gather_nu<T, NHWC, 4>(sh, p, st) : fits(2) ? launch_gather_nu<T, NHWC, 2>(sh, p, st)
                                                               : launch_gather_nu<T, NHWC, 1>(sh, p, st);
}

hipError_t launch_dyn_gather(const Shape& sh, const void* x, const int32_t* S, const float* alpha, const int32_t* U,
                             const int32_t* nU, void* y, hipStream_t st) {
  DynMixArgs p{};
  p.x = x;
  p.S = S;
  p.alpha = alpha;
  p.U = U;
  p.nU = nU;
  p.y = y;
  p.C = (int)sh.C;
  p.HW = (int)sh.HW;
  p.E = sh.E;
  p.k = sh.k;
  p.vec = sh.k % 4 == 0 && ((reinterpret_cast<uintptr_t>(S) | reinterpret_cast<uintptr_t>(alpha)) & 15) == 0;
  const bool nhwc = sh.layout == MOCE_NHWC;
  if (sh.elem == MOCE_BF16)
    return nhwc ? launch_gather_t<uint16_t, true>(sh, p, st) : launch_gather_t<uint16_t, false>(sh, p, st);
  return nhwc ? launch_gather_t<float, true>(sh, p, st) : launch_gather_t<float, false>(sh, p, st);
}

}  // namespace

bool dynamic_supported(const Shape& sh, int dd) {
  if (dd < 1 || dd > kDynMaxD || sh.k > kDynMaxK) return false;
  if (sh.C > kDynMaxC) return false;
  return select_eb(sh, dd <= 32 ? 32 : 64) > 0;
}

hipError_t launch_dynamic(const Shape& sh, const void* x, const float* L, const moce_router& r,
                          const moce_gate_params& g, void* y, float* d, float* h, float* vT, int32_t* S, float* W,
                          int32_t* U, int32_t* nU, float* tau, float* alpha, hipStream_t st) {
  hipError_t e = launch_pool(sh, x, d, st);
  if (e != hipSuccess) return e;
  if (sh.R > 0) {
    const int64_t waves = sh.B * r.d;
    hipLaunchKernelGGL(k_dyn_router, dim3((unsigned)((waves + kDynWaves - 1) / kDynWaves)), dim3(kDynThreads), 0,
                       st, d, r.Wh, r.bh, h, sh.B, (int)sh.C, r.d);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const bool top = dyn_top_eligible(sh, r.d);
  if (top) {
    // logits, selection, U(X) and the softplus-linear gate
    e = launch_dyn_top(sh, h, L, r, g, d, S, W, tau, alpha, U, nU, st);
    if (e != hipSuccess) return e;
  } else {
    if (sh.R > 0) {
      hipLaunchKernelGGL(k_dyn_transpose, dim3((unsigned)((sh.C + 31) / 32), (unsigned)((r.d + 31) / 32)),
                         dim3(1024), 0, st, r.v, vT, (int)sh.C, r.d);
      e = hipGetLastError();
      if (e != hipSuccess) return e;
      e = r.d <= 32 ? launch_select_dd<32>(sh, h, L, r.q, vT, S, W, r.d, st)
                    : launch_select_dd<64>(sh, h, L, r.q, vT, S, W, r.d, st);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_dyn_uncovered, dim3((unsigned)sh.B), dim3(1024), ((sh.C + 15) & ~15) + 16 * 4, st, S, U, nU,
                       (int)sh.C, sh.R, sh.k);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (sh.R > 0 && !(top && g.kind == MOCE_GATE_SOFTPLUS_LINEAR)) {
    const int64_t items = sh.B * sh.R;
    hipLaunchKernelGGL(k_dyn_gate, dim3((unsigned)((items + kDynWaves - 1) / kDynWaves)), dim3(kDynThreads), 0, st, d,
                       S, W, g, tau, alpha, sh.B, (int)sh.C, sh.R, sh.k);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (tilemix_dynamic_eligible(sh)) return launch_tilemix_dynamic(sh, x, S, alpha, U, nU, y, st);
  return launch_dyn_gather(sh, x, S, alpha, U, nU, y, st);
}

}  // namespace moce
