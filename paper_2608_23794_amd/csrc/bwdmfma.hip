// Matrix-core kernels of the backward.
//
// dalpha[b][e][i] = sum_p dy[b][e][p] x[b][s_ei][p] is a sampled product: for
// a block of Et experts and 256 channels it is the dense block
// G[e][c] = sum_p dy[b][e][p] x[b][c][p], of which only the support entries
// are kept.  With k/C small the dense block wastes most of its products, but
// the matrix cores run them at many times the rate of a gather through LDS
// (one LDS read per product), so the dense block is the faster way to the
// sparse result; both operands are the bfloat16 inputs themselves, exact in
// the products, accumulated in float32.
//
// A workgroup owns (expert block, channel block) and walks a set of units
// (image, range of positions).  Per unit, 32-position steps of both operands
// are staged in LDS (double-buffered, one barrier per step) and each of the
// 4 WE waves (WE = 1 or 2: at most two waves a SIMD, for the registers of
// the accumulators, operands and the loads in flight) accumulates a 64 x 64
// block as 4 x 4 MFMA 16x16x32 tiles.  A
// byte table [channel][expert] of support positions (0xff: not an entry),
// built once per workgroup from the prepared rows, picks the entries out of
// the accumulators at the end of a unit.
//
// Layouts in LDS:
//  - NCHW (positions contiguous): a row of 32 positions per feature (64
//    bytes), its four 16-byte chunks XOR-swizzled by (row >> 2) & 3, read as
//    one 16-byte operand per lane;
//  - channels-last: the 32 positions as rows of features (512 bytes for the
//    256 channels, at least 256 for the experts), 32-byte blocks
//    XOR-swizzled by the position, read as operands with the transposing LDS
//    load (two 8-byte loads per operand).
// Both swizzles make the operand reads and the staging writes free of bank
// conflicts.
#include <algorithm>
#include <climits>

#include "moce_internal.h"

namespace moce {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kDaWC = 4;       // channel waves: 4 x 64 = 256 channels per workgroup
constexpr int kDaCt = 64 * kDaWC;
constexpr int kDaKs = 32;      // positions per step
constexpr int kDaMaxK = 255;   // support positions fit a byte, 0xff marks "no entry"
constexpr int kDaTargetBlocks = 512;

// 32-byte block swizzle of the channels-last staging rows (16 blocks a row)
__device__ __forceinline__ int rowswz(int p) { return (p & 3) | ((p >> 1) & 4); }

template <int WE, bool NHWC, int VEC>
struct DaCfg {
  static constexpr int Et = 64 * WE;
  static constexpr int T = 64 * WE * kDaWC;
  // staging bytes of one step: A (experts) then B (channels)
  // channels-last rows: at least 256 bytes, so that the 8 values of the
  // block swizzle stay within the row
  static constexpr int APitch = NHWC ? (Et > 128 ? Et : 128) * 2 : 64;
  static constexpr int ABytes = NHWC ? kDaKs * APitch : Et * kDaKs * 2;
  static constexpr int BBytes = NHWC ? kDaKs * 256 * 2 : kDaCt * kDaKs * 2;
  static constexpr int Stage = ABytes + BBytes;
  static constexpr int TableBytes = kDaCt * Et;
  static constexpr int Lds = TableBytes + 2 * Stage;
  // 16-byte (NHWC) or VEC-position (NCHW) loads per step
  static constexpr int NA = NHWC ? kDaKs * Et / 8 : Et * (kDaKs / VEC);
  static constexpr int NB = NHWC ? kDaKs * kDaCt / 8 : kDaCt * (kDaKs / VEC);
  static constexpr int LPT = (NA + NB + T - 1) / T;
  static constexpr int WORDS = NHWC ? 4 : VEC / 2;  // 32-bit words per load
};

template <int WE, bool NHWC, int VEC>
__global__ void __launch_bounds__(64 * WE * kDaWC)
k_bwd_dalpha_mfma(const uint16_t* __restrict__ x, const uint16_t* __restrict__ dy, const int32_t* __restrict__ s,
                  float* __restrict__ dal, int B, int C, int E, int R, int k, int HW, int nsplit, int split_len,
                  int nCB, int G) {
  using Cf = DaCfg<WE, NHWC, VEC>;
  constexpr int Et = Cf::Et, T = Cf::T;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  unsigned char* table = lds;
  unsigned char* stage0 = lds + Cf::TableBytes;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int we = wave / kDaWC, wc = wave % kDaWC;
  const int g = blockIdx.x % G;
  const int rest = blockIdx.x / G;
  const int cb = rest % nCB, eb = rest / nCB;
  const int e0 = eb * Et, c0 = cb * kDaCt;

  // ---- the support-position table of this block: each wave takes 16 rows,
  // lanes along the row, all 16 loads of a chunk issued before any is used
  for (int q = tid; q < Cf::TableBytes / 16; q += T)
    reinterpret_cast<u32x4*>(table)[q] = u32x4{~0u, ~0u, ~0u, ~0u};
  __syncthreads();
  for (int i0 = 0; i0 < k; i0 += 64) {
    const int i = i0 + lane;
    int cv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int e = e0 + wave * 16 + r;
      cv[r] = s[(int64_t)min(e, R - 1) * k + min(i, k - 1)];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int el = wave * 16 + r;
      const int cl = cv[r] - c0;
      if (e0 + el < R && i < k && cl >= 0 && cl < kDaCt)
        table[cl * Et + ((((el >> 2) ^ (cl & 15))) << 2) + (el & 3)] = (unsigned char)i;
    }
  }

  // ---- the units (image, position range) of this workgroup as one stream of
  // 32-position steps: the next step's loads are in flight while the current
  // one is multiplied, across unit boundaries too
  const int nunits = B * nsplit;
  auto unit_steps = [&](int u) {
    const int sp = u % nsplit;
    const int pb = sp * split_len, pe = min(HW, pb + split_len);
    return (pe - pb + kDaKs - 1) / kDaKs;
  };
  typedef uint32_t Regs[Cf::LPT][Cf::WORDS];
  // global -> registers for step ks of unit u (zeros outside the positions, experts and channels)
  auto load = [&](int u, int ks, Regs& reg) {
    const int b = u / nsplit, sp = u - b * nsplit;
    const int pb = sp * split_len, pe = min(HW, pb + split_len);
    const int p0 = pb + ks * kDaKs;
    const uint16_t* xb = x + (int64_t)b * C * HW;
    const uint16_t* yb = dy + (int64_t)b * E * HW;
#pragma unroll
    for (int j = 0; j < Cf::LPT; ++j) {
      const int q = tid + j * T;
#pragma unroll
      for (int w = 0; w < Cf::WORDS; ++w) reg[j][w] = 0;
      if (q < Cf::NA + Cf::NB) {
        const bool isA = q < Cf::NA;
        const int qq = isA ? q : q - Cf::NA;
        if (NHWC) {
          const int F = isA ? Et : kDaCt;
          const int p = qq / (F / 8), f8 = qq - p * (F / 8);
          const int f = (isA ? e0 : c0) + f8 * 8;
          const int nf = isA ? E : C;
          const int pp = p0 + p;
          if (pp < pe && f < nf) {
            const uint16_t* src = (isA ? yb : xb) + (int64_t)pp * nf + f;
            const u32x4 v = *reinterpret_cast<const u32x4*>(src);
            reg[j][0] = v.x;
            reg[j][1] = v.y;
            reg[j][2] = v.z;
            reg[j][3] = v.w;
          }
        } else {
          constexpr int CH = kDaKs / VEC;
          const int row = qq / CH, ch = qq - row * CH;
          const int f = (isA ? e0 : c0) + row;
          const int nf = isA ? E : C;
          const int pp = p0 + ch * VEC;
          if (pp < pe && f < nf) {
            const uint16_t* src = (isA ? yb : xb) + (int64_t)f * HW + pp;
            if (VEC == 8) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(src);
              reg[j][0] = v.x;
              reg[j][1] = v.y;
              reg[j][2] = v.z;
              reg[j][3] = v.w;
            } else {
              const u32x2 v = *reinterpret_cast<const u32x2*>(src);
              reg[j][0] = v.x;
              reg[j][1] = v.y;
            }
          }
        }
      }
    }
  };
  // registers -> LDS stage buffer
  auto store = [&](unsigned char* stg, const Regs& reg) {
#pragma unroll
    for (int j = 0; j < Cf::LPT; ++j) {
      const int q = tid + j * T;
      if (q >= Cf::NA + Cf::NB) continue;
      const bool isA = q < Cf::NA;
      const int qq = isA ? q : q - Cf::NA;
      unsigned char* base = stg + (isA ? 0 : Cf::ABytes);
      if (NHWC) {
        const int F = isA ? Et : kDaCt;
        const int p = qq / (F / 8), f8 = qq - p * (F / 8);
        const int blk = (f8 >> 1) ^ rowswz(p);
        *reinterpret_cast<u32x4*>(base + p * (isA ? Cf::APitch : 512) + (blk << 5) + ((f8 & 1) << 4)) =
            u32x4{reg[j][0], reg[j][1], reg[j][2], reg[j][3]};
      } else {
        constexpr int CH = kDaKs / VEC;
        const int row = qq / CH, ch = qq - row * CH;
        // byte offset of positions ch*VEC.. within the row's 64 bytes
        const int off = ch * VEC * 2;
        const int chunk = (off >> 4) ^ ((row >> 2) & 3);
        unsigned char* dst = base + row * 64 + (chunk << 4) + (off & 15);
        if (VEC == 8)
          *reinterpret_cast<u32x4*>(dst) = u32x4{reg[j][0], reg[j][1], reg[j][2], reg[j][3]};
        else
          *reinterpret_cast<u32x2*>(dst) = u32x2{reg[j][0], reg[j][1]};
      }
    }
  };
  // operand of the 16-feature tile starting at feature fl of region `base`
  auto operand = [&](const unsigned char* base, int pitch, int fl) -> bf16x8 {
    if (NHWC) {
      const int G4 = lane >> 4, t = (lane >> 2) & 3, q = lane & 3;
      const int nb = fl >> 4;
      const int p1 = 8 * G4 + t, p2 = p1 + 4;
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4*)(base + p1 * pitch + ((nb ^ rowswz(p1)) << 5) + (q << 3)));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_s16x4*)(base + p2 * pitch + ((nb ^ rowswz(p2)) << 5) + (q << 3)));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const s16x8 v = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      return __builtin_bit_cast(bf16x8, v);
    } else {
      const int row = fl + (lane & 15);
      const int chunk = (lane >> 4) ^ ((row >> 2) & 3);
      return *reinterpret_cast<const bf16x8*>(base + row * 64 + (chunk << 4));
    }
  };

  f32x4 acc[4][4];
#pragma unroll
  for (int me = 0; me < 4; ++me)
#pragma unroll
    for (int nc = 0; nc < 4; ++nc) acc[me][nc] = f32x4{0.f, 0.f, 0.f, 0.f};

  // steps as (unit, step within the unit); u >= nunits: past the end
  auto advance = [&](int& su, int& sk) {
    if (su >= nunits) return;
    if (++sk >= unit_steps(su)) {
      su += G;
      sk = 0;
    }
  };
  // step i is multiplied from LDS buffer i & 1 while step i + 1 waits in
  // registers (loaded an iteration earlier) and step i + 2 is being loaded
  Regs r0, r1;
  int u = g, ks = 0;             // step i
  int u1 = u, k1 = ks;           // step i + 1
  advance(u1, k1);
  int u2 = u1, k2 = k1;          // step i + 2
  advance(u2, k2);
  load(u, ks, r0);
  store(stage0, r0);
  if (u1 < nunits) load(u1, k1, r1);
  __syncthreads();  // the table and the first step
  int cur = 0;
  auto body = [&](Regs& rfree, Regs& rnext) {
    if (u2 < nunits) load(u2, k2, rfree);
    const unsigned char* stg = stage0 + cur * Cf::Stage;
    bf16x8 a[4], bb[4];
#pragma unroll
    for (int me = 0; me < 4; ++me) a[me] = operand(stg, Cf::APitch, 64 * we + 16 * me);
#pragma unroll
    for (int nc = 0; nc < 4; ++nc) bb[nc] = operand(stg + Cf::ABytes, 512, 64 * wc + 16 * nc);
#pragma unroll
    for (int me = 0; me < 4; ++me)
#pragma unroll
      for (int nc = 0; nc < 4; ++nc)
        acc[me][nc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[me], bb[nc], acc[me][nc], 0, 0, 0);
    if (ks + 1 == unit_steps(u)) {
      // ---- the support entries of unit u out of the accumulators
      const int b = u / nsplit, sp = u - b * nsplit;
      float* out = dal + (((int64_t)sp * B + b) * R) * k;
#pragma unroll
      for (int me = 0; me < 4; ++me)
#pragma unroll
        for (int nc = 0; nc < 4; ++nc) {
          const int cl = 64 * wc + 16 * nc + (lane & 15);
          const int el = 64 * we + 16 * me + 4 * (lane >> 4);
          const uint32_t word =
              *reinterpret_cast<const uint32_t*>(table + cl * Et + ((((el >> 2) ^ (cl & 15))) << 2));
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t pos = (word >> (8 * r)) & 0xffu;
            if (pos != 0xffu) out[(int64_t)(e0 + el + r) * k + pos] = acc[me][nc][r];
          }
          acc[me][nc] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (u1 < nunits) store(stage0 + (cur ^ 1) * Cf::Stage, rnext);
    __syncthreads();
    cur ^= 1;
    u = u1;
    ks = k1;
    u1 = u2;
    k1 = k2;
    advance(u2, k2);
  };
  while (u < nunits) {
    body(r0, r1);   // r0 held step i (already in LDS); step i + 1 sits in r1
    if (u >= nunits) break;
    body(r1, r0);
  }
}

template <int WE, bool NHWC, int VEC>
hipError_t launch_da(const Shape& sh, const uint16_t* x, const uint16_t* dy, const int32_t* s, float* dal,
                     int nsplit, int split_len, hipStream_t st) {
  using Cf = DaCfg<WE, NHWC, VEC>;
  const int nEB = (sh.R + Cf::Et - 1) / Cf::Et;
  const int nCB = (int)((sh.C + kDaCt - 1) / kDaCt);
  const int units = (int)sh.B * nsplit;
  int G = std::max(1, kDaTargetBlocks / (nEB * nCB));
  G = std::min(units, (G + 7) / 8 * 8);
  auto kern = k_bwd_dalpha_mfma<WE, NHWC, VEC>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, Cf::Lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(nEB * nCB * G), dim3(Cf::T), Cf::Lds, st, x, dy, s, dal, (int)sh.B, (int)sh.C,
                     sh.E, sh.R, sh.k, (int)sh.HW, nsplit, split_len, nCB, G);
  return hipGetLastError();
}

bool dalpha_mfma_eligible(const Shape& sh) {
  if (sh.elem != MOCE_BF16 || sh.R < 1 || sh.k > kDaMaxK) return false;
  if (sh.layout == MOCE_NHWC) return sh.C % 8 == 0 && sh.E % 8 == 0;
  return sh.HW % 4 == 0;
}

// Position splits of the product (units of work along the positions when
// the images alone give too few workgroups); dal then holds one partial sum
// per split.  1 wherever the matrix-core kernel does not apply.
void bwd_dalpha_split(const Shape& sh, int* nsplit, int* split_len) {
  *nsplit = 1;
  *split_len = (int)std::min<int64_t>(sh.HW, INT32_MAX / 2);
  if (!dalpha_mfma_eligible(sh)) return;
  const int WE = std::min(2, (sh.R + 63) / 64);
  const int64_t blocks = sh.B * ((sh.R + 64 * WE - 1) / (64 * WE)) * ((sh.C + kDaCt - 1) / kDaCt);
  const int64_t steps = (sh.HW + kDaKs - 1) / kDaKs;
  const int64_t want = std::min<int64_t>(steps, std::max<int64_t>(1, kDaTargetBlocks / std::max<int64_t>(1, blocks)));
  const int64_t len = (steps + want - 1) / want * kDaKs;
  *split_len = (int)len;
  *nsplit = (int)((sh.HW + len - 1) / len);
}

}  // namespace

void bwd_dalpha_splits(const Shape& sh, int* nsplit, int* split_len) { bwd_dalpha_split(sh, nsplit, split_len); }

bool bwd_mfma_dalpha(const Shape& sh, const void* x, const void* dy, const int32_t* s, const BwdWs& ws,
                     hipStream_t st, hipError_t* err) {
  if (!dalpha_mfma_eligible(sh)) return false;
  int nsplit, split_len;
  bwd_dalpha_split(sh, &nsplit, &split_len);
  const int WE = std::min(2, (sh.R + 63) / 64);
  auto xx = static_cast<const uint16_t*>(x);
  auto yy = static_cast<const uint16_t*>(dy);
#define MOCE_DA(W, N, V) launch_da<W, N, V>(sh, xx, yy, s, ws.dal, nsplit, split_len, st)
  if (sh.layout == MOCE_NHWC)
    *err = WE == 1 ? MOCE_DA(1, true, 8) : MOCE_DA(2, true, 8);
  else if (sh.HW % 8 == 0)
    *err = WE == 1 ? MOCE_DA(1, false, 8) : MOCE_DA(2, false, 8);
  else
    *err = WE == 1 ? MOCE_DA(1, false, 4) : MOCE_DA(2, false, 4);
#undef MOCE_DA
  return true;
}

// ---- dx on the matrix cores -------------------------------------------------
//
// dx[b][c][p] = sum_e coef_b[c][e] dy[b][e][p] + dd[b][c] / HW, where
// coef_b[c][e] is alpha_b[e][i] for the support entry (e, i) on channel c,
// 1/|U| for e = E-1 (the residual) when c is uncovered, and 0 elsewhere.
// The coefficients enter the product as two bf16 parts (hi = bf16(alpha),
// lo = bf16(alpha - hi): 16 significant bits), dy as it is.
//
// The entries come in buckets by (64 channels, 64 experts) with their logits
// (k_bw_part), the residual expert's channels as a bitmap; the coefficients are
// rebuilt here from the logits and the image's softmax statistics.  A workgroup
// of four waves owns (image, 64 positions, 128 channels) and walks the expert
// chunks: the chunk's dy tile (64 x 64) and its coefficient tile (128 x 64, two
// parts) sit in LDS; the coefficient tile starts zero, receives its buckets'
// entries by scatter and is cleared entry by entry once multiplied, so a chunk
// costs LDS writes in proportion to its entries, not to its area.  The next
// chunk's reads are in flight beside the products.  A step is a chain of
// barriers (scatter, multiply, clear), so the tile is kept small enough for
// three workgroups a CU to fill each other's gaps: one of 256 channels with
// double-buffered tiles, alone on its CU, took 74 us at stage 4 (40k cycles a
// workgroup, a third of them vector and a fifth matrix instructions).  The
// results leave through LDS as whole rows.
namespace {

constexpr int kDxCt = 128;   // channels per workgroup
constexpr int kDxEk = 64;    // experts per chunk
constexpr int kDxP = 64;     // positions per workgroup
constexpr int kDxThreads = 256;
constexpr int kDxEPT = 4;    // bucket entries a thread holds for the next scatter
constexpr int kDxCoefPart = kDxCt * kDxEk * 2;   // bytes of one part of the coefficient tile
constexpr int kDxDyBuf = kDxP * kDxEk * 2;
constexpr int kDxStats = kDxEk * 16;             // the softmax statistics of a chunk's experts
constexpr int kDxRanges = 32;                    // chunks whose buckets' ranges sit in LDS
constexpr int kDxLds = 2 * kDxCoefPart + 2 * kDxDyBuf + 2 * kDxStats + kDxRanges * 2 * 8;
constexpr int kDxSub = kDxCt / kBwBucketCh;      // bucket rows per workgroup
constexpr int kDxSubThreads = kDxThreads / kDxSub;
constexpr int kDxMaxBuckets = 4096;
static_assert(kDxEk == kBwBucketEx, "a chunk is a bucket column");

__device__ __forceinline__ int dyswz(int r) { return ((r >> 1) & 1) | ((r >> 2) & 2); }

// byte offset of (channel cl, expert el) in one coefficient part: rows of 64
// experts (128 bytes), 16-byte chunks XOR-swizzled by the channel
__device__ __forceinline__ int coef_off(int cl, int el) {
  return cl * 128 + ((((el >> 3) ^ (cl & 7))) << 4) + ((el & 7) << 1);
}

template <bool NHWC, int VEC>
__global__ void __launch_bounds__(kDxThreads, 3)
k_bwd_dx_mfma(const uint16_t* __restrict__ dy, uint16_t* __restrict__ dx, const float* __restrict__ dd,
              const int32_t* __restrict__ bbeg, const uint2* __restrict__ bw, const float* __restrict__ stats,
              const uint64_t* __restrict__ unc, int B, int C, int E, int HW, int nEC,
              int nPC) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  unsigned char* hiP = lds;                           // [2 part][128][64] bf16
  unsigned char* loP = hiP + kDxCoefPart;
  unsigned char* dyL = lds + 2 * kDxCoefPart;         // [2 buf][64][64] bf16
  float4* stL = reinterpret_cast<float4*>(dyL + 2 * kDxDyBuf);   // [2 buf][64] (rt, m, rzs, -)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t units = (int64_t)B * nPC;
  const int cb = (int)(blockIdx.x / units);
  const int64_t bp = blockIdx.x - (int64_t)cb * units;
  const int b = (int)(bp / nPC), pc = (int)(bp - (int64_t)b * nPC);
  const int c0 = cb * kDxCt, p0 = pc * kDxP;
  const uint16_t* yb = dy + (int64_t)b * E * HW;
  const int R = E - 1;
  const int nch = (R + kDxEk - 1) / kDxEk;            // chunks with routed experts: nEC or nEC - 1
  const float inv_nU = 1.f / (float)bwd_count_uncovered(unc, C);

  // zero the coefficient tile once; every scatter is undone after use
  for (int q = tid; q < 2 * kDxCoefPart / 16; q += kDxThreads)
    reinterpret_cast<u32x4*>(hiP)[q] = u32x4{0u, 0u, 0u, 0u};

  // the softmax statistics of chunk ec's experts, an expert a thread, in
  // registers until the chunk's turn
  float4 sreg = make_float4(0.f, 0.f, 0.f, 0.f);
  auto load_stats = [&](int ec) {
    if (tid < kDxEk) {
      const int64_t n = (int64_t)B * R, i = (int64_t)b * R + min(ec * kDxEk + tid, R - 1);
      sreg = make_float4(stats[i], stats[n + i], stats[2 * n + i], 0.f);
    }
  };
  auto store_stats = [&](int buf) {
    if (tid < kDxEk) stL[buf * kDxEk + tid] = sreg;
  };
  // the entries of the two buckets of a chunk, kDxSubThreads threads each: the
  // first kDxEPT a thread in registers, the rest read again where they are used
  const int sub = tid / kDxSubThreads, st0 = tid % kDxSubThreads;
  const int nblk = (C + kBwBucketCh - 1) / kBwBucketCh;
  const int blk = cb * kDxSub + sub;
  // (first entry, number) of a chunk's bucket, the first chunks' from LDS so
  // that the entries are one round trip away
  int2* rngL = reinterpret_cast<int2*>(stL + 2 * kDxEk);   // [chunk][kDxSub]
  auto bucket = [&](int ec, int bk) {
    if (ec >= nch || bk >= nblk) return make_int2(0, 0);
    const int32_t* bg = bbeg + (int64_t)ec * (nblk + 1) + bk;
    return make_int2(bg[0], bg[1] - bg[0]);
  };
  for (int q = tid; q < min(nEC, kDxRanges) * kDxSub; q += kDxThreads)
    rngL[q] = bucket(q / kDxSub, cb * kDxSub + q % kDxSub);
  struct Ents {
    uint2 w[kDxEPT];   // (channel, expert), logit
    int n, base;
  };
  auto load_entries = [&](int ec, Ents& E) {
    const int2 r = ec < kDxRanges ? rngL[ec * kDxSub + sub] : bucket(ec, blk);
    E.base = r.x;
    E.n = r.y;
#pragma unroll
    for (int r = 0; r < kDxEPT; ++r) {
      const int j = E.base + min(st0 + r * kDxSubThreads, max(E.n - 1, 0));
      E.w[r] = bw[j];
    }
  };
  // a coefficient's two bf16 parts into its place
  auto put2 = [&](int o, float a) {
    const uint16_t hi = f32_to_bf16(a);
    *reinterpret_cast<uint16_t*>(hiP + o) = hi;
    *reinterpret_cast<uint16_t*>(loP + o) = f32_to_bf16(a - bf16_to_f32(hi));
  };
  // scatter (or, with clear, zero) the entries of chunk ec
  auto scatter = [&](int ec, const Ents& E, bool clear) __attribute__((always_inline)) {
    const float4* sb = stL + (ec & 1) * kDxEk;
    auto put = [&](uint2 v) __attribute__((always_inline)) {
      const int el = (int)(v.x >> 8), o = coef_off(v.x & (kDxCt - 1), el);
      if (clear) {
        *reinterpret_cast<uint16_t*>(hiP + o) = 0;
        *reinterpret_cast<uint16_t*>(loP + o) = 0;
      } else {
        const float4 q = sb[el];
        put2(o, coef_alpha(coef_e(coef_z(__uint_as_float(v.y), q.x), q.y), q.z));
      }
    };
#pragma unroll
    for (int r = 0; r < kDxEPT; ++r)
      if (st0 + r * kDxSubThreads < E.n) put(E.w[r]);
    for (int q = st0 + kDxEPT * kDxSubThreads; q < E.n; q += kDxSubThreads) put(bw[E.base + q]);
    // the residual's channels (the last chunk's: never cleared for a later one)
    if (!clear && ec == R / kDxEk && st0 < kBwBucketCh && blk < nblk && ((unc[blk] >> st0) & 1))
      put2(coef_off(sub * kBwBucketCh + st0, R % kDxEk), inv_nU);
  };
  // dy tile of expert chunk ec: NHWC rows of positions (64 experts each, 16-byte
  // chunks swizzled by the row), NCHW rows of experts (64 positions each,
  // 32-byte blocks swizzled for the transposing read)
  constexpr int DYL = kDxP * kDxEk / (NHWC ? 8 : VEC) / kDxThreads;   // loads per thread
  constexpr int DYW = NHWC ? 4 : VEC / 2;   // words per load
  uint32_t dyr[DYL][DYW];
  auto load_dy = [&](int ec) {
    const int e0 = ec * kDxEk;
#pragma unroll
    for (int j = 0; j < DYL; ++j) {
#pragma unroll
      for (int w = 0; w < DYW; ++w) dyr[j][w] = 0;
      if (NHWC) {
        const int q = tid + j * kDxThreads, row = q >> 3, oct = q & 7;
        const int p = p0 + row, e = e0 + oct * 8;
        if (p < HW && e < E) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(yb + (int64_t)p * E + e);
          dyr[j][0] = v.x;
          dyr[j][1] = v.y;
          dyr[j][2] = v.z;
          dyr[j][3] = v.w;
        }
      } else {
        const int q = tid + j * kDxThreads;
        constexpr int PER = kDxP / VEC;     // loads per expert row
        const int row = q / PER, piece = q - row * PER;
        const int e = e0 + row, p = p0 + piece * VEC;
        if (e < E && p < HW) {
          const uint16_t* src = yb + (int64_t)e * HW + p;
          if (VEC == 8) {
            const u32x4 v = *reinterpret_cast<const u32x4*>(src);
            dyr[j][0] = v.x;
            dyr[j][1] = v.y;
            dyr[j][2] = v.z;
            dyr[j][3] = v.w;
          } else {
            const u32x2 v = *reinterpret_cast<const u32x2*>(src);
            dyr[j][0] = v.x;
            dyr[j][1] = v.y;
          }
        }
      }
    }
  };
  auto store_dy = [&](int buf) {
    unsigned char* base = dyL + buf * kDxDyBuf;
#pragma unroll
    for (int j = 0; j < DYL; ++j) {
      if (NHWC) {
        const int q = tid + j * kDxThreads, row = q >> 3, oct = q & 7;
        *reinterpret_cast<u32x4*>(base + row * 128 + ((oct ^ (row & 7)) << 4)) =
            u32x4{dyr[j][0], dyr[j][1], dyr[j][2], dyr[j][3]};
      } else {
        const int q = tid + j * kDxThreads;
        constexpr int PER = kDxP / VEC;
        const int row = q / PER, piece = q - row * PER;
        const int byte = piece * VEC * 2;               // within the 128-byte row
        const int blk = (byte >> 5) ^ dyswz(row);
        unsigned char* dst = base + row * 128 + (blk << 5) + (byte & 31);
        if (VEC == 8)
          *reinterpret_cast<u32x4*>(dst) = u32x4{dyr[j][0], dyr[j][1], dyr[j][2], dyr[j][3]};
        else
          *reinterpret_cast<u32x2*>(dst) = u32x2{dyr[j][0], dyr[j][1]};
      }
    }
  };

  f32x4 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // the entries of the chunk multiplied (to be cleared) and of the next; the
  // sets change roles by the unrolled steps, not by copies, which would wait for
  // the loads
  Ents E0, E1;
  load_dy(0);
  load_stats(0);
  store_stats(0);
  __syncthreads();  // the zeroed tile, chunk 0's statistics, the buckets' ranges
  load_entries(0, E0);
  store_dy(0);
  auto step = [&](int ec, const Ents& E0, Ents& E1) __attribute__((always_inline)) {
    const int cur = ec & 1;
    scatter(ec, E0, false);
    if (ec + 1 < nEC) {
      load_entries(ec + 1, E1);
      load_dy(ec + 1);
      load_stats(ec + 1);
    }
    __syncthreads();  // chunk ec's coefficients and dy are in place
    const unsigned char* dyP = dyL + cur * kDxDyBuf;
#pragma unroll
    for (int ks = 0; ks < kDxEk / 32; ++ks) {
      const int oct = ks * 4 + (lane >> 4);
      if (NHWC) {
        // D[p][c]: A = dy rows (positions), B = coefficient rows (channels)
        bf16x8 a[4], bh[2], bl[2];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const int row = mt * 16 + (lane & 15);
          a[mt] = *reinterpret_cast<const bf16x8*>(dyP + row * 128 + ((oct ^ (row & 7)) << 4));
        }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int cl = (wave * 2 + nt) * 16 + (lane & 15);
          const int o = cl * 128 + ((oct ^ (cl & 7)) << 4);
          bh[nt] = *reinterpret_cast<const bf16x8*>(hiP + o);
          bl[nt] = *reinterpret_cast<const bf16x8*>(loP + o);
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt) {
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bh[nt], acc[mt][nt], 0, 0, 0);
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bl[nt], acc[mt][nt], 0, 0, 0);
          }
      } else {
        // D[c][p]: A = coefficient rows (channels), B = dy rows (experts) read transposed
        bf16x8 ah[2], al[2], bb[4];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const int cl = (wave * 2 + mt) * 16 + (lane & 15);
          const int o = cl * 128 + ((oct ^ (cl & 7)) << 4);
          ah[mt] = *reinterpret_cast<const bf16x8*>(hiP + o);
          al[mt] = *reinterpret_cast<const bf16x8*>(loP + o);
        }
        const int G4 = lane >> 4, t = (lane >> 2) & 3, q = lane & 3;
        const int r1 = ks * 32 + 8 * G4 + t, r2 = r1 + 4;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4*)(dyP + r1 * 128 + ((nt ^ dyswz(r1)) << 5) + (q << 3)));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4*)(dyP + r2 * 128 + ((nt ^ dyswz(r2)) << 5) + (q << 3)));
          typedef short s16x8 __attribute__((ext_vector_type(8)));
          const s16x8 v = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          bb[nt] = __builtin_bit_cast(bf16x8, v);
        }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
          for (int nt = 0; nt < 4; ++nt) {
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah[mt], bb[nt], acc[nt][mt], 0, 0, 0);
            acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al[mt], bb[nt], acc[nt][mt], 0, 0, 0);
          }
      }
    }
    if (ec + 1 < nEC) {   // into the buffers chunk ec - 1 used
      store_dy(cur ^ 1);
      store_stats(cur ^ 1);
    }
    __syncthreads();  // every wave is done with the tile
    if (ec + 1 < nEC) {
      scatter(ec, E0, true);
      __syncthreads();  // the tile is zero again
    }
  };
  for (int ec = 0; ec < nEC; ec += 2) {
    step(ec, E0, E1);
    if (ec + 1 < nEC) step(ec + 1, E1, E0);
  }

  // ---- epilogue: + dd / HW, rounded to bf16, staged as rows (of channels for
  // each position, or of positions for each channel) and written 16 or 8 bytes a
  // thread; channels-last rows that are not a multiple of 16 bytes go out singly
  const float rhw = 1.f / (float)HW;
  unsigned char* stg = lds;
  constexpr int PITCH = (NHWC ? kDxCt : kDxP) * 2 + 16;
  static_assert((NHWC ? kDxP : kDxCt) * PITCH <= 2 * kDxCoefPart + 2 * kDxDyBuf, "the staged results fit");
  if (NHWC) {
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int cl = (wave * 2 + nt) * 16 + (lane & 15), c = c0 + cl;
      const float add = dd[(int64_t)b * C + min(c, C - 1)] * rhw;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<uint16_t*>(stg + (mt * 16 + 4 * (lane >> 4) + r) * PITCH + cl * 2) =
              f32_to_bf16(acc[mt][nt][r] + add);
    }
    __syncthreads();
    if (C % 8 == 0) {
      for (int q = tid; q < kDxP * (kDxCt / 8); q += kDxThreads) {
        const int row = q / (kDxCt / 8), c8 = q % (kDxCt / 8), p = p0 + row, c = c0 + c8 * 8;
        if (p < HW && c < C)
          *reinterpret_cast<u32x4*>(dx + ((int64_t)b * HW + p) * C + c) =
              *reinterpret_cast<const u32x4*>(stg + row * PITCH + c8 * 16);
      }
    } else {
      for (int q = tid; q < kDxP * kDxCt; q += kDxThreads) {
        const int row = q / kDxCt, cl = q % kDxCt, p = p0 + row, c = c0 + cl;
        if (p < HW && c < C) dx[((int64_t)b * HW + p) * C + c] = *reinterpret_cast<const uint16_t*>(stg + row * PITCH + cl * 2);
      }
    }
  } else {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int cl = (wave * 2 + mt) * 16 + 4 * (lane >> 4) + r;
        const float add = dd[(int64_t)b * C + min(c0 + cl, C - 1)] * rhw;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
          *reinterpret_cast<uint16_t*>(stg + cl * PITCH + (nt * 16 + (lane & 15)) * 2) = f32_to_bf16(acc[nt][mt][r] + add);
      }
    __syncthreads();
    constexpr int PR = kDxP / VEC;   // pieces of VEC positions per row
    for (int q = tid; q < kDxCt * PR; q += kDxThreads) {
      const int cl = q / PR, pc8 = q % PR, p = p0 + pc8 * VEC, c = c0 + cl;
      if (c >= C || p >= HW) continue;
      uint16_t* dst = dx + ((int64_t)b * C + c) * HW + p;
      const unsigned char* src = stg + cl * PITCH + pc8 * VEC * 2;
      if (VEC == 8)
        *reinterpret_cast<u32x4*>(dst) = *reinterpret_cast<const u32x4*>(src);
      else
        *reinterpret_cast<u32x2*>(dst) = *reinterpret_cast<const u32x2*>(src);
    }
  }
}

bool dx_mfma_eligible(const Shape& sh) {
  if (sh.elem != MOCE_BF16 || sh.R < 1) return false;
  if ((sh.C + 255) / 256 * ((sh.E + kDxEk - 1) / kDxEk) > kDxMaxBuckets) return false;
  if (sh.layout == MOCE_NHWC) return sh.E % 8 == 0;
  return sh.HW % 4 == 0;
}

}  // namespace

bool bwd_dx_on_mfma(const Shape& sh) { return dx_mfma_eligible(sh); }

bool bwd_mfma_dx(const Shape& sh, const void* dy, const BwdWs& ws, void* dx, hipStream_t st, hipError_t* err) {
  if (!dx_mfma_eligible(sh)) return false;
  const int nEC = (sh.E + kDxEk - 1) / kDxEk;
  const int nCB = (int)((sh.C + kDxCt - 1) / kDxCt);
  const int nPC = (int)((sh.HW + kDxP - 1) / kDxP);
  const unsigned grid = (unsigned)(nCB * sh.B * nPC);
  auto y = static_cast<const uint16_t*>(dy);
  auto o = static_cast<uint16_t*>(dx);
  using K = void (*)(const uint16_t*, uint16_t*, const float*, const int32_t*, const uint2*, const float*,
                     const uint64_t*, int, int, int, int, int, int);
  const K kern = sh.layout == MOCE_NHWC ? k_bwd_dx_mfma<true, 8>
                 : sh.HW % 8 == 0      ? k_bwd_dx_mfma<false, 8>
                                       : k_bwd_dx_mfma<false, 4>;
  if ((*err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kDxLds)) !=
      hipSuccess)
    return true;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kDxThreads), kDxLds, st, y, o, ws.dd, ws.bbeg, ws.bw, ws.stats,
                     ws.unc, (int)sh.B, (int)sh.C, sh.E, (int)sh.HW, nEC, nPC);
  *err = hipGetLastError();
  return true;
}

}  // namespace moce
