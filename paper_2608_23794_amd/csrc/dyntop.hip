// Input-conditioned supports (Sec. 4.5, Eq. 11): logits, per-example top k and
// the gate in one kernel, for C <= 2048, k <= 160 and a router of at most 32
// units.
//
// A workgroup of 16 waves owns a run of 16-expert blocks of one image.
//  - Logits.  L(X)[e][c] - L[e][c] = <q_e * h, v_c> is a product over the router's
//    units: each wave holds v of its share of the channels as float32 MFMA operands
//    for the whole run and forms the block's [channels][16 experts] tile with
//    16x16x4 float32 products (the same arithmetic precision as a vector FMA
//    chain), adds L and writes the order-preserving keys to the block's LDS
//    rows.
//  - Selection.  Each wave takes a row into registers (C / 64 keys a lane).
//    64 of its keys, sorted across the lanes, are the candidate thresholds: a
//    threshold that at least k and at most CAP keys reach is found by counting
//    (one or two counts for logits of any smooth distribution; bisection over the
//    key range otherwise, and over the channels among keys equal to the
//    threshold), the keys that reach it are compacted into LDS, and a bitonic
//    sort of 64 NE (key, channel) pairs puts them in the canonical order (logit
//    descending, channel ascending).  A pair travels as one float64 whose bits
//    order like the pair, so a compare-exchange is one v_max_f64.
//  - Gate.  The sorted pairs sit in the lanes: the softplus-linear temperature
//    and the coefficients are formed there (the MLP gate has a kernel of its
//    own).
//  - Coverage.  The selected channels are marked in a bitmap of the workgroup,
//    one per (image, run), which k_dyn_uncovered_bits turns into U(X).
//
// A wave that has taken its row into registers leaves the LDS rows free, so it
// goes on to form its share of the next block's rows as soon as it is done,
// beside the waves that still select; a schedule in which even and odd waves run
// the two halves in opposite order was 3% slower (the row then stays in
// registers through the products).  Bound by the selection's vector
// instructions (about 1300 a row of 2048 keys and k = 128) and the barriers: 255
// to 280 us for 128 images x 511 experts at those sizes, k = 128, against 1115 us for
// the separate kernels (logits on the vector ALUs, a radix select with LDS
// atomics, an LDS bitonic sort, the gate and U(X) in launches of their own).
#include <algorithm>
#include <type_traits>

#include "dyn_keys.h"
#include "moce_internal.h"

namespace moce {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTopEB = 16;           // experts per block: the MFMA's N
constexpr int kTopThreads = kTopEB * kWave;   // a wave per row of a block
constexpr int kTopD = 32;            // router units, zero-padded
constexpr int kTopMaxC = 2048;
constexpr int kTopMaxK = 160;
constexpr size_t kTopLds = 160 * 1024;

// list entries per wave: 64 NE, but 240 where 256 and the rows of 2048 channels
// would pass the LDS
constexpr int list_cap(int NE) { return NE == 4 ? 240 : 64 * NE; }

// the value of lane l ^ M
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane) {
  if constexpr (M == 1) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);   // quad_perm [1, 0, 3, 2]
  } else if constexpr (M == 2) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);   // quad_perm [2, 3, 0, 1]
  } else if constexpr (M == 4) {
    const int m = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true);         // row_half_mirror: l ^ 7
    return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1b, 0xf, 0xf, true);            // quad_perm [3, 2, 1, 0]: l ^ 3
  } else if constexpr (M == 8) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);  // row_ror 8
  } else if constexpr (M == 16) {
    return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401f);
  } else {
    return (uint32_t)__shfl_xor((int)v, 32, kWave);
  }
}

// sum over the wave: DPP moves within rows of 16 lanes, then the four rows
__device__ __forceinline__ float wave_sum_dpp(float v) {
  auto mov = [](float u, auto ctrl) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(u), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += mov(v, std::integral_constant<int, 0xb1>{});    // l ^ 1
  v += mov(v, std::integral_constant<int, 0x4e>{});    // l ^ 2
  v += mov(v, std::integral_constant<int, 0x141>{});   // the other quad of 8 lanes
  v += mov(v, std::integral_constant<int, 0x140>{});   // the other half of the row
  auto row = [&](int l) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
  };
  return (row(0) + row(16)) + (row(32) + row(48));
}

// max(a, -b), max(a, b) and min(a, b) of float64 values that are never NaN
// (the library's fmax would canonicalize both operands first).  The wait
// states cover a cross-lane read of the result by the next instruction.
__device__ __forceinline__ double max_neg(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, -%2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double max64(double a, double b) {
  double r;
  asm("v_max_f64 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double min64(double a, double b) {
  double r;
  asm("v_min_f64 %0, %1, %2\n\ts_nop 1" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ double flip(double v, uint32_t sign) {
  const uint64_t u = __double_as_longlong(v);
  return __longlong_as_double(((uint64_t)((uint32_t)(u >> 32) ^ sign) << 32) | (uint32_t)u);
}
template <int M>
__device__ __forceinline__ double lane_xor64(double v, int lane) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t lo = lane_xor<M>((uint32_t)u, lane), hi = lane_xor<M>((uint32_t)(u >> 32), lane);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
// sign bit in the lanes whose bit LS is set
template <int LS>
__device__ __forceinline__ uint32_t lane_sign(int lane) {
  if constexpr (LS == 0 || LS >= kWave)
    return 0u;
  else
    return ((uint32_t)lane << (31 - __builtin_ctz(LS))) & 0x80000000u;
}

// Bitonic sort, descending, of 64 NE values, element lane NE + j in v[j].
// Signs take the place of directions.  In the merge of runs of SIZE every
// second run is sorted the other way round, by holding it negated; in a step
// between lanes l and l ^ LS the lower lane keeps the larger value, so the
// upper lanes hold theirs negated and both keep the maximum of their own and
// the other's negated one.  Between steps the sign bits change by one XOR.
// A sign pattern is a set of lane bits, whose parity is the sign, and an
// element bit.
template <int LANES>
__device__ __forceinline__ uint32_t sign_of(int lane) {   // parity of the lane's bits LANES, as a sign bit
  uint32_t s = 0u;
  if constexpr (LANES & 1) s ^= lane_sign<1>(lane);
  if constexpr (LANES & 2) s ^= lane_sign<2>(lane);
  if constexpr (LANES & 4) s ^= lane_sign<4>(lane);
  if constexpr (LANES & 8) s ^= lane_sign<8>(lane);
  if constexpr (LANES & 16) s ^= lane_sign<16>(lane);
  if constexpr (LANES & 32) s ^= lane_sign<32>(lane);
  return s;
}
// from sign pattern (FL lanes, FJ element bit) to (TL, TJ)
template <int FL, int FJ, int TL, int TJ, int NE>
__device__ __forceinline__ void resign(double (&v)[NE], int lane) {
  if constexpr (FL == TL && FJ == TJ) return;
  const uint32_t s = sign_of<FL ^ TL>(lane);
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const bool f = ((j & FJ) != 0) != ((j & TJ) != 0);
    if (FL != TL || f) v[j] = flip(v[j], f ? s ^ 0x80000000u : s);
  }
}
template <int SIZE, int STRIDE, int FL, int FJ, int NE>
__device__ __forceinline__ void sort_step(double (&v)[NE], int lane) {
  constexpr int DL = SIZE >= NE && SIZE < kWave * NE ? SIZE / NE : 0;   // direction of the runs
  constexpr int DJ = SIZE < NE ? SIZE : 0;
  constexpr int TL = STRIDE >= NE ? DL ^ (STRIDE / NE) : DL;
  resign<FL, FJ, TL, DJ, NE>(v, lane);
  if constexpr (STRIDE >= NE) {
#pragma unroll
    for (int j = 0; j < NE; ++j) v[j] = max_neg(v[j], lane_xor64<STRIDE / NE>(v[j], lane));
  } else {
#pragma unroll
    for (int j = 0; j < NE; ++j)
      if ((j & STRIDE) == 0) {
        const double a = v[j], b = v[j | STRIDE];
        v[j] = max64(a, b);
        v[j | STRIDE] = min64(a, b);
      }
  }
  if constexpr (STRIDE > 1)
    sort_step<SIZE, STRIDE / 2, TL, DJ, NE>(v, lane);
  else if constexpr (SIZE < kWave * NE)
    sort_step<SIZE * 2, SIZE, TL, DJ, NE>(v, lane);
  else
    resign<TL, DJ, 0, 0, NE>(v, lane);
}
template <int NE>
__device__ __forceinline__ void sort_pairs(double (&v)[NE], int lane) {
  sort_step<2, 1, 0, 0, NE>(v, lane);
}

// the same over the lanes for one 32-bit key each, complement in the place of
// negation
template <int LANES>
__device__ __forceinline__ uint32_t fill_of(int lane) {
  return (uint32_t)((int32_t)sign_of<LANES>(lane) >> 31);
}
template <int SIZE, int LS, int FL>
__device__ __forceinline__ void key_step(uint32_t& v, int lane) {
  constexpr int TL = (SIZE < kWave ? SIZE : 0) ^ LS;
  v ^= fill_of<FL ^ TL>(lane);
  v = max(v, ~lane_xor<LS>(v, lane));
  if constexpr (LS > 1)
    key_step<SIZE, LS / 2, TL>(v, lane);
  else if constexpr (SIZE < kWave)
    key_step<SIZE * 2, SIZE, TL>(v, lane);
  else
    v ^= fill_of<TL>(lane);
}

// (key, channel) as the bits of a positive normal float64: larger key first,
// then the lower channel (channel < 4096)
__device__ __forceinline__ double pack_pair(uint32_t key, uint32_t ch) {
  const uint32_t hi = 0x3ff00000u | (key >> 12), lo = (key << 20) | ((4095u - ch) << 8);
  return __longlong_as_double(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void unpack_pair(double v, uint32_t& key, int& ch) {
  const uint64_t u = __double_as_longlong(v);
  const uint32_t hi = (uint32_t)(u >> 32), lo = (uint32_t)u;
  key = (hi << 12) | (lo >> 20);
  ch = 4095 - (int)((lo >> 8) & 0xfffu);
}

// element i of a, by a 32-bit byte offset (the arrays here hold at most 2^24
// elements)
__device__ __forceinline__ const float& at(const float* a, int i) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a) + (uint32_t)(4 * i));
}

struct TopArgs {
  const float *h, *L, *q, *v, *d;
  const float *a, *c;        // softplus-linear gate, or null: W is written instead of tau and alpha
  int32_t* S;
  float *W, *tau, *alpha;
  int32_t* cov;              // the images' bitmaps, nsplit of nwords words, every covs words
  int C, R, k, dd, nblk, nbp, nsplit, nwords;
  int rank0;                 // first threshold: this rank of the 64 sampled keys
  int target;                // keys a threshold should let through
  int covs;
};

// The keys of one row that a wave holds, NK a lane: key 4 j + q of a lane is
// channel 256 j + chl + q.
template <int NK, int NE>
__device__ __forceinline__ void select_row(uint32_t (&r)[NK], uint32_t* list, const TopArgs& p, int64_t item,
                                           int e, const float* db, uint32_t* covl, int chl, int lane) {
  constexpr int CAP = list_cap(NE);
  constexpr int CN = NK * kWave;
  const int k = p.k;
  asm volatile("" : "+v"(chl), "+v"(lane));   // opaque: nothing derived from them is held outside this row
  auto chan = [&](int i) __attribute__((always_inline)) { return 256 * (i >> 2) + chl + (i & 3); };
  auto count = [&](uint32_t t) __attribute__((always_inline)) {
    int n = 0;
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      n += __popcll(__ballot(r[i] >= t));
      if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // few masks at a time in scalar registers
    }
    return n;
  };
  // 64 keys from four parts of the row, sorted, largest first
  uint32_t smp = r[0];
  smp = lane >= 16 ? r[NK / 4] : smp;
  smp = lane >= 32 ? r[NK / 2] : smp;
  smp = lane >= 48 ? r[3 * NK / 4] : smp;
  key_step<2, 1, 0>(smp, lane);
  // a threshold reached by k .. CAP keys, between lo (reached by more) and hi
  // (by fewer than k); every round narrows (lo, hi)
  uint64_t lo = 0, hi = 1ull << 32;
  int rank = p.rank0;
  uint64_t t = (uint32_t)__builtin_amdgcn_readlane((int)smp, rank);
  bool ties = false;
  for (;;) {
    if (t <= lo || t >= hi) {
      if (hi == 1ull << 32) {   // no key above the row's largest
        uint32_t m = 0u;
        asm volatile("" : "+v"(m));   // formed here, not ahead of the loop
#pragma unroll
        for (int i = 0; i < NK; ++i) m = max(m, r[i]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off, kWave));
        hi = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)m) + 1;
      }
      t = lo + (hi - lo) / 2;
    }
    if (hi - lo <= 1) {
      ties = true;
      break;
    }
    const int n = count((uint32_t)t);
    if (n > CAP)
      lo = t;
    else if (n < k)
      hi = t;
    else
      break;
    const int step = max(1, abs(n - p.target) * kWave / CN);
    rank += n > CAP ? -step : step;
    t = rank >= 0 && rank < kWave ? (uint32_t)__builtin_amdgcn_readlane((int)smp, rank) : 0u;
  }
  // among more than CAP keys equal to lo, with fewer than k above it, the
  // lowest channels: cb such that the keys above lo and those equal to it on
  // channels below cb are exactly k
  int cb = 0;
  uint32_t lo32 = (uint32_t)lo;
  if (ties) {
    if (lo32 == ~0u) {   // NaN bits: leave room for a bound above the key
#pragma unroll
      for (int i = 0; i < NK; ++i) r[i] = min(r[i], ~1u);
      lo32 = ~1u;
    }
    int c0 = 0, c1 = CN;   // fewer than k below c0, at least k below c1
    while (c1 - c0 > 1) {
      const int cm = (c0 + c1) / 2;
      int n = 0;
      // key > lo, or key = lo on a channel below cm, as one comparison with a
      // per-key bound (opaque, so that no comparison is held across rounds)
      int left = cm - chl;
      uint32_t l2 = lo32;
      asm volatile("" : "+v"(left), "+v"(l2));
#pragma unroll
      for (int i = 0; i < NK; ++i) {
        n += __popcll(__ballot(r[i] >= l2 + (256 * (i >> 2) + (i & 3) < left ? 0u : 1u)));
        if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
      }
      if (n >= k)
        c1 = cm;
      else
        c0 = cm;
    }
    cb = c1;
  }
  // compaction
  int base = 0;
  auto put = [&](int i, bool in) __attribute__((always_inline)) {
    const uint64_t m = __ballot(in);
    const int pos = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
    if (in) {
      list[2 * pos] = r[i];
      list[2 * pos + 1] = (uint32_t)chan(i);
    }
    base += __popcll(m);
    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);
  };
  if (!ties) {
    const uint32_t t32 = (uint32_t)t;
#pragma unroll
    for (int i = 0; i < NK; ++i) put(i, r[i] >= t32);
  } else {
#pragma unroll
    for (int i = 0; i < NK; ++i) put(i, r[i] >= lo32 + (chan(i) < cb ? 0u : 1u));
  }
  // the gate's row, in flight beside the sort
  const int i0 = lane * NE;
  float av[NE], cv = 0.f;
  if (p.a) {
#pragma unroll
    for (int j = 0; j < NE; ++j) av[j] = at(p.a, e * k + min(i0 + j, k - 1));
    cv = p.c[e];
  }
  // the canonical order
  double v[NE];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    const int idx = lane * NE + j;
    const uint2 en = *reinterpret_cast<const uint2*>(list + 2 * min(idx, CAP - 1));
    v[j] = idx < base ? pack_pair(en.x, en.y) : pack_pair(0u, 4095u);
  }
  sort_pairs<NE>(v, lane);
  float w[NE];
  int ch[NE];
#pragma unroll
  for (int j = 0; j < NE; ++j) {
    uint32_t key;
    unpack_pair(v[j], key, ch[j]);
    ch[j] = min(ch[j], p.C - 1);
    w[j] = fkey_value(key);
  }
#pragma unroll
  for (int j = 0; j < NE; ++j)
    if (i0 + j < k) atomicOr(&covl[ch[j] >> 5], 1u << (ch[j] & 31));
  if (p.a) {
    float dv[NE], g = 0.f;
#pragma unroll
    for (int j = 0; j < NE; ++j) dv[j] = at(db, ch[j]);
#pragma unroll
    for (int j = 0; j < NE; ++j)
      if (i0 + j < k) g += av[j] * dv[j];
    const float tv = softplusf(wave_sum_dpp(g) + cv) + 1e-3f;
    const float rt = 1.f / tv;
    // the first logit is the largest, and 1/tau > 0
    const float m = coef_z(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(w[0]))), rt);
    float zs = 0.f;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
      w[j] = i0 + j < k ? coef_e(coef_z(w[j], rt), m) : 0.f;
      zs += w[j];
    }
    const float rzs = 1.f / wave_sum_dpp(zs);
#pragma unroll
    for (int j = 0; j < NE; ++j) w[j] = coef_alpha(w[j], rzs);
    if (lane == 0) p.tau[item] = tv;
  }
  // stores last: a later load would wait for them
  float* out = p.a ? p.alpha : p.W;
#pragma unroll
  for (int j = 0; j < NE; ++j)
    if (i0 + j < k) {
      p.S[item * k + i0 + j] = ch[j];
      out[item * k + i0 + j] = w[j];
    }
}

// CB: the rows hold 256 CB channels (C padded); NE: sorted entries per lane; LM:
// 2 where C fills the rows, the router has kTopD units and L and q can be read in
// 16-byte pieces, 1 where all but the first, 0 elsewhere.
// LDS: 16 rows of 256 CB keys in 16-byte chunks, chunk x of row n at
// x ^ (n & 7) so that eight consecutive lanes of a tile's store (one row each)
// fall on distinct bank groups; the lists; the coverage bitmap.
template <int CB, int NE, int LM>
__global__ void __launch_bounds__(kTopThreads)
k_dyn_topk(TopArgs p) {
  constexpr int CN = 256 * CB;
  constexpr int NK = 4 * CB;
  constexpr int TPW = CB;               // 16-channel tiles per wave
  constexpr int NPRE = TPW < 2 ? TPW : 2;   // tiles whose L is read ahead
  constexpr int CAP = list_cap(NE);
  extern __shared__ __align__(16) uint32_t sm[];
  uint32_t* rows = sm;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t* list = rows + kTopEB * CN + wv * 2 * CAP;
  uint32_t* covl = rows + kTopEB * CN + 2 * kTopEB * CAP;
  const int64_t b = blockIdx.x / p.nsplit;
  const int blk0 = (int)(blockIdx.x % p.nsplit) * p.nbp;
  const int blk1 = min(blk0 + p.nbp, p.nblk);
  const int n = lane & 15, g = lane >> 4;
  const int C = p.C, dd = p.dd;
  for (int i = threadIdx.x; i < p.nwords; i += kTopThreads) covl[i] = 0u;
  // operands held for the whole run: v of channel 16 tile + n, units 8 g .. 8 g + 7
  // (the same permutation of the units on both sides)
  float va[TPW][8];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int c = (wv * TPW + t) * 16 + n;
#pragma unroll
    for (int j = 0; j < 8; ++j) va[t][j] = at(p.v, min(c, C - 1) * dd + min(8 * g + j, dd - 1));
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int c = (wv * TPW + t) * 16 + n;
    // read unconditionally (clamped into v), then masked: a select of the load
    // would become a branch around it
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      uint32_t m = -(uint32_t)((c < C) & (8 * g + j < dd));
      asm volatile("" : "+v"(m));
      va[t][j] = __uint_as_float(__float_as_uint(va[t][j]) & m);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  const float* hb = p.h + b * dd;
  auto logits = [&](int blk) __attribute__((always_inline)) {
    // opaque per block: the tiles' addresses and bounds are recomputed instead
    // of being held in registers across the run
    int gq = g, ws = wv;
    asm volatile("" : "+v"(gq), "+s"(ws));
    const int e = min(blk * kTopEB + n, p.R - 1);
    float qh[8];
    [[maybe_unused]] const int lim = dd - 8 * gq;
    if constexpr (LM > 0) {   // all kTopD units, in 16-byte pieces
#pragma unroll
      for (int j = 0; j < 8; j += 4) {
        const float4 q4 = *reinterpret_cast<const float4*>(&at(p.q, e * kTopD + 8 * gq + j));
        const float4 h4 = *reinterpret_cast<const float4*>(&at(hb, 8 * gq + j));
        qh[j] = q4.x * h4.x;
        qh[j + 1] = q4.y * h4.y;
        qh[j + 2] = q4.z * h4.z;
        qh[j + 3] = q4.w * h4.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int u = min(8 * gq + j, dd - 1);
        const float x = at(p.q, e * dd + u) * at(hb, u);
        qh[j] = __uint_as_float(__float_as_uint(x) & (uint32_t)((j - lim) >> 31));   // 0 past dd
      }
    }
    auto load_l = [&](int t, float (&lv)[4]) __attribute__((always_inline)) {
      const int c = (ws * TPW + t) * 16 + 4 * gq;  // this lane's four channels of expert n
      if constexpr (LM > 0) {
        const float4 l4 = *reinterpret_cast<const float4*>(&at(p.L, e * C + (LM == 2 ? c : min(c, C - 4))));
        lv[0] = l4.x;
        lv[1] = l4.y;
        lv[2] = l4.z;
        lv[3] = l4.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) lv[i] = at(p.L, e * C + min(c + i, C - 1));
      }
    };
    float lb[NPRE][4];
#pragma unroll
    for (int t = 0; t < NPRE; ++t) load_l(t, lb[t]);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int tile = ws * TPW + t;
      [[maybe_unused]] const int c = tile * 16 + 4 * gq;
      float (&lv)[4] = lb[t % NPRE];
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(va[t][j], qh[j], acc, 0, 0, 0);
      u32x4 key;   // 0 past C, below every real key
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        key[i] = fkey(lv[i] + acc[i]);
        if constexpr (LM < 2) key[i] &= (uint32_t)((LM == 1 ? c - C : c + i - C) >> 31);
      }
      *reinterpret_cast<u32x4*>(rows + n * CN + (((tile * 4 + gq) ^ (n & 7)) << 2)) = key;
      if (t + NPRE < TPW) load_l(t + NPRE, lb[t % NPRE]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  logits(blk0);
  __syncthreads();
  for (int blk = blk0; blk < blk1; ++blk) {
    uint32_t r[NK];
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      const u32x4 x = *reinterpret_cast<const u32x4*>(rows + wv * CN + 256 * j + 4 * lane);
#pragma unroll
      for (int i = 0; i < 4; ++i) r[4 * j + i] = x[i];
    }
    __syncthreads();  // every row is in registers: the next block's may be written
    const int e = blk * kTopEB + wv;
    if (e < p.R)
      select_row<NK, NE>(r, list, p, b * p.R + e, e, p.d + b * C, covl, 4 * (lane ^ (wv & 7)), lane);
    if (blk + 1 < blk1) logits(blk + 1);
    __syncthreads();
  }
  uint32_t* cov = reinterpret_cast<uint32_t*>(p.cov + b * p.covs) + (blockIdx.x % p.nsplit) * p.nwords;
  for (int i = threadIdx.x; i < p.nwords; i += kTopThreads) cov[i] = covl[i];
}

// U(X) of an image from its runs' bitmaps: a wave per image, a word of 32
// channels a lane (C <= 2048), channels in ascending order.  The bitmaps may lie in
// the image's row of U, which the wave overwrites once it has read them all.
__global__ void __launch_bounds__(256)
k_dyn_uncovered_bits(const int32_t* cov, int covs, int32_t* U, int32_t* __restrict__ nU, int64_t B, int C,
                     int nsplit, int nwords) {
  const int64_t b = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= B) return;
  const int lane = threadIdx.x & 63;
  uint32_t w = 0u;
#pragma unroll 4
  for (int s = 0; s < nsplit; ++s) w |= (uint32_t)cov[b * covs + s * nwords + min(lane, nwords - 1)];
  const int left = C - 32 * lane;   // channels of this word
  w = left <= 0 ? 0u : ~w & (left >= 32 ? ~0u : (1u << left) - 1u);
  const int n = __popc(w);
  int incl = n;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int o = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += o;
  }
  int32_t* out = U + b * C + (incl - n);
  for (int i = 0; w; ++i) {
    const int bit = __ffs(w) - 1;
    out[i] = 32 * lane + bit;
    w &= w - 1;
  }
  if (lane == 63) nU[b] = incl;
}

int row_blocks(int64_t C) { return C <= 256 ? 1 : C <= 512 ? 2 : C <= 1024 ? 4 : 8; }
int entries_per_lane(int k) { return k <= 32 ? 1 : k <= 64 ? 2 : 4; }

template <int CB, int NE>
hipError_t launch_top(const TopArgs& p, int64_t B, bool lv, hipStream_t st) {
  constexpr size_t fixed = ((size_t)kTopEB * 256 * CB + (size_t)2 * kTopEB * list_cap(NE)) * 4;
  static_assert(fixed + kTopMaxC / 8 <= kTopLds, "rows, lists and bitmap fit a CU's LDS");
  const size_t lds = fixed + (size_t)p.nwords * 4;
  auto kern = lv ? (p.C == 256 * CB ? k_dyn_topk<CB, NE, 2> : k_dyn_topk<CB, NE, 1>) : k_dyn_topk<CB, NE, 0>;
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(B * p.nsplit)), dim3(kTopThreads), lds, st, p);
  return hipGetLastError();
}

}  // namespace

bool dyn_top_eligible(const Shape& sh, int dd) {
  return sh.R > 0 && dd <= kTopD && sh.C >= 4 && sh.C <= kTopMaxC && sh.k <= kTopMaxK;
}

hipError_t launch_dyn_top(const Shape& sh, const float* h, const float* L, const moce_router& r,
                          const moce_gate_params& g, const float* d, int32_t* S, float* W, float* tau, float* alpha,
                          int32_t* U, int32_t* nU, hipStream_t st) {
  int cus = 256, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  const int rb = row_blocks(sh.C), ne = entries_per_lane(sh.k);
  TopArgs p{};
  p.h = h;
  p.L = L;
  p.q = r.q;
  p.v = r.v;
  p.d = d;
  const bool lin = g.kind == MOCE_GATE_SOFTPLUS_LINEAR;
  p.a = lin ? g.a : nullptr;
  p.c = g.c;
  p.S = S;
  p.W = W;
  p.tau = tau;
  p.alpha = alpha;
  // the bitmaps in the longer of the image's row of U and of the logits' or coefficients'
  // array that nothing holds yet
  const int64_t rk = (int64_t)sh.R * sh.k;
  p.cov = rk > sh.C ? reinterpret_cast<int32_t*>(lin ? W : alpha) : U;
  p.covs = (int)std::max(rk, sh.C);
  p.C = (int)sh.C;
  p.R = sh.R;
  p.k = sh.k;
  p.dd = r.d;
  p.nblk = (sh.R + kTopEB - 1) / kTopEB;
  p.nwords = (int)((sh.C + 31) / 32);
  // blocks per workgroup: the fewest block times of all rounds of workgroups
  // over the CUs (one workgroup each), a workgroup's start costing about one;
  // no more runs than there is room for bitmaps (with that of U alone, 32, one image
  // of C 2048, R 2047, k 8 took 71 us, runs of four blocks on 32 CUs; now 45)
  int64_t best = 0;
  for (int nbp = 1; nbp <= p.nblk; ++nbp) {
    const int64_t ns = (p.nblk + nbp - 1) / nbp;
    if (ns * p.nwords > p.covs) continue;
    const int64_t cost = ((sh.B * ns + cus - 1) / cus) * (nbp + 1);
    if (best == 0 || cost < best) {
      best = cost;
      p.nbp = nbp;
      p.nsplit = (int)ns;
    }
  }
  // the first threshold: the sampled key whose expected count lies between k and the list's length
  const int cn = 256 * rb, cap = list_cap(ne);
  p.target = (sh.k + cap) / 2;
  p.rank0 = std::min(kWave - 1, std::max(0, (p.target * (kWave + 1) + cn / 2) / cn - 1));
  const bool lv = sh.C % 4 == 0 && r.d == kTopD &&
                  ((reinterpret_cast<uintptr_t>(L) | reinterpret_cast<uintptr_t>(r.q) | reinterpret_cast<uintptr_t>(h)) & 15) == 0;
  hipError_t e;
#define MOCE_TOP(T) (ne == 1 ? launch_top<T, 1>(p, sh.B, lv, st) : ne == 2 ? launch_top<T, 2>(p, sh.B, lv, st) : launch_top<T, 4>(p, sh.B, lv, st))
  e = rb == 1 ? MOCE_TOP(1) : rb == 2 ? MOCE_TOP(2) : rb == 4 ? MOCE_TOP(4) : MOCE_TOP(8);
#undef MOCE_TOP
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dyn_uncovered_bits, dim3((unsigned)((sh.B + 3) / 4)), dim3(256), 0, st, p.cov, p.covs, U, nU, sh.B, p.C,
                     p.nsplit, p.nwords);
  return hipGetLastError();
}

}  // namespace moce
