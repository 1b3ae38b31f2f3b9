// Matrix-core kernels of the backward.
//
// dalpha[b][e][i] = sum_p dy[b][e][p] x[b][s_ei][p] is a sampled product: for
// 64 experts and 128 channels it is the dense block
// G[e][c] = sum_p dy[b][e][p] x[b][c][p], of which only the support entries
// are kept.  With k/C small the dense block wastes most of its products, but
// the matrix cores run them at many times the rate of a gather through LDS
// (one LDS read per product), so the dense block is the faster way to the
// sparse result; both operands are the bfloat16 inputs themselves, exact in
// the products, accumulated in float32.
//
// A workgroup of four waves owns (image, 64 experts, a run of 128-channel
// blocks, a range of positions); a wave takes 32 channels of each block by all
// 64 experts, so x passes through LDS of its own, for the layout only, and the
// waves need no barriers where dy stays: in registers where one 64-position
// stage holds all positions, in LDS up to four stages; else dy is staged with
// two barriers a stage.  The block is then written to the wave's LDS and the
// entries of its buckets (k_bw_part) are picked out of it, a lane each, into the
// rows of dalpha.  Picking them out of the accumulators by a byte table took 64
// conditional stores a lane and unit, and the loads of the next unit, which share
// the in-order counter, waited for them: 87 us at stage 4; with 32 x 64 tiles
// sharing x between waves, 67 us, bound by the LDS reads of both operands.
//
// Layouts in LDS, 64 positions a stage:
//  - NCHW (positions contiguous): a row of 64 positions per feature (128
//    bytes), its 16-byte chunks XOR-swizzled by the row, read as one 16-byte
//    operand per lane;
//  - channels-last: the 64 positions as rows of the features (128 bytes of dy,
//    32-byte blocks XOR-swizzled by the position; 64 of x, 80 apart), read as
//    operands with the transposing LDS load (two 8-byte loads per operand).
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

constexpr int kDaEt = kBwBucketEx;      // experts per workgroup: a bucket column
constexpr int kDaCt = 2 * kBwBucketCh;  // channels per block: two bucket rows
constexpr int kDaCw = 32;               // channels per wave
constexpr int kDaP = 64;                // positions per stage
constexpr int kDaThreads = 256;
constexpr int kDaTargetBlocks = 1024;   // workgroups wanted, about two rounds of two a CU
constexpr int kDaPitchG = kDaEt + 4;    // floats of a channel's row of the block
constexpr int kDaRanges = 127;          // buckets whose entries' ranges sit in LDS
constexpr int kDaStages = 4;            // stages of dy held in LDS
constexpr int kDaABytes = kDaEt * kDaP * 2;                  // a stage of dy
constexpr int kDaWBytes = kDaCw * kDaPitchG * 4;             // a wave's block, over its x stage
constexpr int kDaRBytes = (kDaRanges + 1) * 4;
static_assert(kDaP * 80 <= kDaWBytes && kDaCw * 128 <= kDaWBytes, "the block lies over the wave's x stage");

// block swizzle of dy's channels-last rows (4 blocks of 32 bytes)
__device__ __forceinline__ int dyswz(int r) { return ((r >> 1) & 1) | ((r >> 2) & 2); }

// The unit of a workgroup of n units, `per` an image, in a grid of xcd_grid(n, per):
// workgroup u runs on XCD u mod 8 and takes the (u / 8)-th of that XCD's run of the units,
// an eighth of them or, where the batch has no more than one image a run, an image of up
// to 32, a round on the XCD's CUs: the units of one image, which are consecutive, share an
// L2, at any number of images.
// (With whole images dealt to the XCDs in turn, one image ran on one of them: the
// backward took 504 us in the place of 406 at 5 images of C 4088, E 4088, k 7, 360
// positions channels-first, 267 in the place of 103 at one of C 2504, E 1248, k 12,
// 785 positions channels-last.  With eighths of one image's 13 and 26 units dalpha took 34
// us in the place of 21 and dx 15 in the place of 10, C 136, E 64, k 136, 785 positions.)
__device__ __forceinline__ int xcd_unit() { return (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3); }
int64_t xcd_grid(int64_t units, int64_t per) {
  return 8 * std::max<int64_t>((units + 7) / 8, std::min<int64_t>(per, 32));
}

struct DaArgs {
  const uint16_t *x, *dy;
  const int32_t* bbeg;
  const uint2 *bw, *ba;
  float* dal;
  int B, C, E, R, k, HW, nsplit, split_len, nblk, nCB, nEB, csplit, cper, per;
  int nres;     // stages of dy in LDS
  int staged;   // the workgroup holds whole rows of dalpha in LDS and writes them at the end
};

// VEC: elements a global load holds (8 or 4 where rows are aligned to 16 or 8
// bytes, else 1).  MODE: 0: one stage, dy in registers; 1: dy's stages in LDS;
// 2: dy staged.
template <bool NHWC, int VEC, int MODE>
__global__ void __launch_bounds__(kDaThreads, 2)
k_bwd_dalpha_mfma(DaArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  unsigned char* aL = lds;                                          // [nres] stages of dy
  unsigned char* wL = lds + a.nres * kDaABytes + wave * kDaWBytes;  // this wave's x stage, then its block
  float* gL = reinterpret_cast<float*>(wL);
  int32_t* rngL = reinterpret_cast<int32_t*>(lds + a.nres * kDaABytes + 4 * kDaWBytes);
  float* rowL = reinterpret_cast<float*>(rngL) + kDaRBytes / 4;
  const int u = xcd_unit(), b = u / a.per;
  if (b >= a.B) return;
  int r = u % a.per;
  const int sp = r % a.nsplit;
  r /= a.nsplit;
  const int cs = r % a.csplit, eb = r / a.csplit;
  const int e0 = eb * kDaEt;
  const int cb0 = cs * a.cper, cb1 = min(a.nCB, cb0 + a.cper);
  const int pb = sp * a.split_len, pe = min(a.HW, pb + a.split_len);
  const int nst = MODE == 0 ? 1 : (pe - pb + kDaP - 1) / kDaP;
  const int C = a.C, E = a.E, HW = a.HW;
  const uint16_t* xb = a.x + (int64_t)b * C * HW;
  const uint16_t* yb = a.dy + (int64_t)b * E * HW;

  // Loads are clamped into the tensor and what lies outside the stage is zeroed
  // when it goes to LDS: a load under a lane condition is waited for in its own
  // branch, one round trip each.
  //
  // 8 consecutive elements from src[i], of which those from lim on are not used
  auto load8 = [](const uint16_t* src, int i, int lim) __attribute__((always_inline)) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if constexpr (VEC == 8) {
      v = *reinterpret_cast<const u32x4*>(src + min(i, lim - 8));
    } else if constexpr (VEC == 4) {
      const u32x2 lo = *reinterpret_cast<const u32x2*>(src + min(i, lim - 4));
      const u32x2 hi = *reinterpret_cast<const u32x2*>(src + min(i + 4, lim - 4));
      v = u32x4{lo.x, lo.y, hi.x, hi.y};
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j / 2] |= (uint32_t)src[min(i + j, lim - 1)] << (16 * (j & 1));
    }
    return v;
  };
  // piece q of a stage: channels-last the 8 features f of position p, else the 8
  // positions p of feature f; F features a stage
  auto where = [&](int f0, int p0, int q, int F, int& f, int& p) __attribute__((always_inline)) {
    f = f0 + (NHWC ? q % (F / 8) * 8 : q / (kDaP / 8));
    p = p0 + (NHWC ? q / (F / 8) : q % (kDaP / 8) * 8);
  };
  auto piece = [&](const uint16_t* src, int f0, int nt, int p0, int q, int F) __attribute__((always_inline)) {
    int f, p;
    where(f0, p0, q, F, f, p);
    if constexpr (NHWC)
      return load8(src + (int64_t)min(p, HW - 1) * nt, f, nt);
    else
      return load8(src + (int64_t)min(f, nt - 1) * HW, p, HW);
  };
  auto put = [&](unsigned char* base, int f0, int nt, int p0, int q, int F, u32x4 v) __attribute__((always_inline)) {
    int f, p;
    where(f0, p0, q, F, f, p);
    // elements in use: all 8 or none where the limits are multiples of 8
    const int left = NHWC ? (p < pe ? nt - f : 0) : (f < nt ? pe - p : 0);
    if constexpr (VEC == 8) {
      const uint32_t m = left > 0 ? ~0u : 0u;
      v = u32x4{v.x & m, v.y & m, v.z & m, v.w & m};
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[j] &= left > 2 * j + 1 ? ~0u : left == 2 * j + 1 ? 0xffffu : 0u;
    }
    if constexpr (NHWC) {
      const int pp = q / (F / 8), f8 = q % (F / 8);
      const int off = F == kDaEt ? pp * 128 + (((f8 >> 1) ^ dyswz(pp)) << 5) + ((f8 & 1) << 4) : pp * 80 + f8 * 16;
      *reinterpret_cast<u32x4*>(base + off) = v;
    } else {
      const int row = q / (kDaP / 8), ch = q % (kDaP / 8);
      *reinterpret_cast<u32x4*>(base + row * 128 + ((ch ^ (row & 7)) << 4)) = v;
    }
  };
  // operand of 16 features from fl of a stage's 32-position slice ks
  auto operand = [&](const unsigned char* base, bool isA, int fl, int ks) __attribute__((always_inline)) -> bf16x8 {
    if constexpr (NHWC) {
      const int G4 = lane >> 4, t = (lane >> 2) & 3, q = lane & 3;
      const int nb = fl >> 4;
      const int p1 = 32 * ks + 8 * G4 + t, p2 = p1 + 4;
      auto at = [&](int p) {
        return base + (isA ? p * 128 + ((nb ^ dyswz(p)) << 5) : p * 80 + (nb << 5)) + (q << 3);
      };
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at(p1));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at(p2));
      typedef short s16x8 __attribute__((ext_vector_type(8)));
      const s16x8 v = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
      return __builtin_bit_cast(bf16x8, v);
    } else {
      const int row = fl + (lane & 15);
      return *reinterpret_cast<const bf16x8*>(base + row * 128 + (((4 * ks + (lane >> 4)) ^ (row & 7)) << 4));
    }
  };

  const int32_t* bg = a.bbeg + (int64_t)eb * (a.nblk + 1);
  const int nbk = min(2 * cb1, a.nblk) - 2 * cb0;   // buckets
  for (int i = tid; i <= min(nbk, kDaRanges); i += kDaThreads) rngL[i] = bg[2 * cb0 + i];
  // where bucket i's entries start
  auto start = [&](int i) { return i <= kDaRanges ? rngL[min(i, nbk)] : bg[2 * cb0 + min(i, nbk)]; };
  constexpr int NA = kDaEt * kDaP / 8 / kDaThreads;
  u32x4 ra[NA];
  auto load_a = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NA; ++j) ra[j] = piece(yb, e0, E, pb + st * kDaP, tid + j * kDaThreads, kDaEt);
  };
  auto put_a = [&](int st, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
      put(aL + slot * kDaABytes, e0, E, pb + st * kDaP, tid + j * kDaThreads, kDaEt, ra[j]);
  };
  // a stage's loads of x, and with a block's first stage the entries of the
  // wave's bucket (which it shares with its neighbour)
  constexpr int NB = kDaCw * kDaP / 8 / kWave;
  constexpr int H = 4;
  struct Stage {
    u32x4 b[NB];
    uint2 ew[H], ea[H];
  };
  auto load = [&](int cb, int st, Stage& s) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
      s.b[j] = piece(xb, cb * kDaCt + wave * kDaCw, C, pb + st * kDaP, lane + j * kWave, kDaCw);
    if (st == 0) {
      const int bk = 2 * (cb - cb0) + (wave >> 1);
      const int q0 = start(bk), q1 = start(bk + 1);
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int q = min(q0 + lane + h * kWave, max(q1 - 1, 0));
        s.ew[h] = a.bw[q];
        s.ea[h] = a.ba[q];
      }
    }
  };
  float* out = a.dal + ((int64_t)sp * a.B + b) * a.R * a.k;
  // the stages of all blocks as one stream: stage i goes to LDS while stages
  // i + 1 and i + 2 are in registers or on their way (two sets, by the unrolled
  // steps)
  const int nb = cb1 - cb0, n = nb * nst;
  Stage s0, s1;
  int cl = cb0, sl = 0;     // the next stage to load
  auto next_load = [&](Stage& s) __attribute__((always_inline)) {
    if (cl >= cb1) return;
    load(cl, sl, s);
    if (++sl == nst) {
      sl = 0;
      ++cl;
    }
  };
  load_a(0);
  __syncthreads();   // the ranges
  next_load(s0);
  next_load(s1);
  bf16x8 av[2][4];
  if constexpr (MODE != 2) {
    put_a(0, 0);
    for (int st = 1; st < nst; ++st) {
      load_a(st);
      put_a(st, st);
    }
    __syncthreads();
  }
  auto read_a = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int me = 0; me < 4; ++me) av[ks][me] = operand(aL + slot * kDaABytes, true, 16 * me, ks);
  };
  if constexpr (MODE == 0) read_a(0);
  f32x4 acc[4][2];
  uint2 ew[H], ea[H];
  int cb = cb0, st = 0;
  auto step = [&](int i, Stage& s) __attribute__((always_inline)) {
    if (st == 0) {
#pragma unroll
      for (int me = 0; me < 4; ++me)
#pragma unroll
        for (int nc = 0; nc < 2; ++nc) acc[me][nc] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int h = 0; h < H; ++h) {
        ew[h] = s.ew[h];
        ea[h] = s.ea[h];
      }
    }
    if constexpr (MODE == 2) {
      __syncthreads();   // the previous stage of dy is consumed
      put_a(st, 0);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
      put(wL, cb * kDaCt + wave * kDaCw, C, pb + st * kDaP, lane + j * kWave, kDaCw, s.b[j]);
    if constexpr (MODE == 2) {
      __syncthreads();
      load_a(st + 1 < nst ? st + 1 : 0);
    }
    __builtin_amdgcn_wave_barrier();   // (no instruction: the wave's own LDS steps stay in this order)
    next_load(s);
    if constexpr (MODE != 0) read_a(MODE == 1 ? st : 0);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 bv[2];
#pragma unroll
      for (int nc = 0; nc < 2; ++nc) bv[nc] = operand(wL, false, 16 * nc, ks);
#pragma unroll
      for (int me = 0; me < 4; ++me)
#pragma unroll
        for (int nc = 0; nc < 2; ++nc)
          acc[me][nc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[ks][me], bv[nc], acc[me][nc], 0, 0, 0);
    }
    if (++st < nst) return;
    // the block, a row of experts per channel, over the x stage (a wave's LDS
    // operations run in order), then its entries
    const int bk = 2 * (cb - cb0) + (wave >> 1);
    const int q0 = start(bk), q1 = start(bk + 1);
    st = 0;
    ++cb;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int me = 0; me < 4; ++me)
#pragma unroll
      for (int nc = 0; nc < 2; ++nc)
        *reinterpret_cast<f32x4*>(gL + (16 * nc + (lane & 15)) * kDaPitchG + 16 * me + 4 * (lane >> 4)) = acc[me][nc];
    __builtin_amdgcn_wave_barrier();
    auto take = [&](uint2 w, uint2 v, bool in) __attribute__((always_inline)) {
      if (!in || ((w.x >> 5) & 1) != (uint32_t)(wave & 1)) return;
      const float g = gL[(w.x & (kDaCw - 1)) * kDaPitchG + (w.x >> 8)];
      if (a.staged)
        rowL[v.y - (uint32_t)(e0 * a.k)] = g;
      else
        out[v.y] = g;
    };
#pragma unroll
    for (int h = 0; h < H; ++h) take(ew[h], ea[h], q0 + lane + h * kWave < q1);
    for (int q = q0 + lane + H * kWave; q < q1; q += kWave) take(a.bw[q], a.ba[q], true);
    __builtin_amdgcn_wave_barrier();
  };
  for (int i = 0; i < n; i += 2) {
    step(i, s0);
    if (i + 1 < n) step(i + 1, s1);
  }
  if (a.staged) {
    __syncthreads();
    const int m = min(kDaEt, a.R - e0) * a.k;
    for (int i = tid; i < m; i += kDaThreads) out[(int64_t)e0 * a.k + i] = rowL[i];
  }
}

// a launch holds fewer than 2^32 threads; the excess would be dropped without an
// error
bool launch_holds(int64_t workgroups, int threads) { return workgroups < ((int64_t)1 << 32) / threads; }

// Position splits of the product (units of work along the positions when
// images, expert blocks and channel blocks give too few workgroups).
void da_split(const Shape& sh, int* nsplit, int* split_len) {
  const int64_t blocks = sh.B * ((sh.R + kDaEt - 1) / kDaEt) * ((sh.C + kDaCt - 1) / kDaCt);
  const int64_t stages = (sh.HW + kDaP - 1) / kDaP;
  const int64_t want = std::min<int64_t>(stages, std::max<int64_t>(1, kDaTargetBlocks / std::max<int64_t>(1, blocks)));
  const int64_t len = (stages + want - 1) / want * kDaP;
  *split_len = (int)len;
  *nsplit = (int)((sh.HW + len - 1) / len);
}

// Runs of channel blocks (cper blocks each): long ones keep dy, but enough workgroups first.
void da_runs(const Shape& sh, int nsplit, int* csplit, int* cper) {
  const int64_t base = sh.B * ((sh.R + kDaEt - 1) / kDaEt) * nsplit;
  const int nCB = (int)((sh.C + kDaCt - 1) / kDaCt);
  const int want = (int)std::min<int64_t>(nCB, std::max<int64_t>(1, (kDaTargetBlocks + base - 1) / base));
  *cper = (nCB + want - 1) / want;
  *csplit = (nCB + *cper - 1) / *cper;
}

// bfloat16 layers with routed experts, up to what one launch holds (2^24 images of a
// block each, far past what needs channel runs or position splits).  Where rows
// allow wide loads (16 bytes channels-last, 8 channels-first) always; elsewhere by
// what both kernels take in ns, fitted to their times over 700 ragged shapes.  The
// vector kernel: 0.028 (channels-last 0.038) for a row, position and 64 entries and for
// each entry, a line of its own, 0.001 (0.0002), or 0.0024 (0.0007) where an image is more
// than the L1 and its lines in flight hold (64 and 200 KB; 27 images of C 2328, E 144, k
// 32, 785 positions channels-first: the whole backward 648 us with it and 490 with the
// product); or, with few rows, the latency of a position, 100, and 270 channels-last where x is larger than an L2 (364 images of C 176,
// E 3, k 22, 785 positions: the whole backward 353 us with it and 233 with the product).
// The product: 3.5 (8-byte loads) to 13 (single elements, dy
// staged again for every block) for a dense unit of 64 experts by 128 channels by 64
// positions, however few of the entries it holds, 3 for an image's 64 experts, 0.007 for
// an entry; or, with few workgroups, the chain of one: its stages and the rounds of 64
// bucket entries past those it holds.  Where the two meet: 18 images of C 3416, E 854, k
// 8, 784 positions channels-last 481 us with the vector kernel and 1311 with this one;
// 409 of C 2560, E 640, k 32, 21 positions channels-first 682 and 462; 32 of C 105, E 52,
// k 105, 25 positions 8 and 31.
bool dalpha_mfma_eligible(const Shape& sh) {
  const int64_t nEB = (sh.R + kDaEt - 1) / kDaEt;
  if (sh.elem != MOCE_BF16 || sh.R < 1 || !launch_holds(xcd_grid(sh.B * nEB, nEB), kDaThreads)) return false;
  const bool nhwc = sh.layout == MOCE_NHWC;
  if (nhwc ? sh.C % 8 == 0 && sh.E % 8 == 0 : sh.HW % 4 == 0) return true;
  int nsplit, len, csplit, cper;
  da_split(sh, &nsplit, &len);
  da_runs(sh, nsplit, &csplit, &cper);
  const int64_t stages = (std::min<int64_t>(sh.HW, len) + kDaP - 1) / kDaP;
  const double units = (double)nEB * ((sh.C + kDaCt - 1) / kDaCt) * ((sh.HW + kDaP - 1) / kDaP);
  const double unit = nhwc && sh.C % 4 == 0 && sh.E % 4 == 0 ? 3.5
                      : stages == 1                          ? (nhwc ? 6.5 : 4.)
                      : stages <= kDaStages                  ? 7.
                                                             : (nhwc ? 13. : 10.);
  const double k64 = (sh.k + kWave - 1) / kWave;
  const int64_t image = sh.C * sh.HW * 2;
  const double entry = nhwc ? (image > 200'000 ? 0.0007 : 0.0002) : image > 65'536 ? 0.0024 : 0.001;
  const double row = sh.B * (double)sh.R * ((nhwc ? 0.038 : 0.028) * k64 + entry * sh.k);
  const double latency = nhwc && sh.B * image > 6'000'000 ? 270. : 100.;
  const double vec = std::max(4000., sh.HW * std::max(row, k64 * latency));
  const double bucket = (double)std::min(sh.R, kDaEt) * sh.k * kBwBucketCh / std::max<int64_t>(sh.C, kBwBucketCh);
  const double chain = 4000. + cper * (400. * stages + 500. * std::max(0., bucket / kWave - 4.));
  return std::max(sh.B * (units * unit + 3. * nEB + 0.0068 * sh.R * sh.k), chain) <= vec;
}

// dal holds one partial sum per split; 1 wherever the matrix-core kernel does not
// apply.
void bwd_dalpha_split(const Shape& sh, int* nsplit, int* split_len) {
  *nsplit = 1;
  *split_len = (int)std::min<int64_t>(sh.HW, INT32_MAX / 2);
  if (dalpha_mfma_eligible(sh)) da_split(sh, nsplit, split_len);
}

template <bool NHWC, int VEC>
hipError_t launch_da(const DaArgs& a, hipStream_t st) {
  const int stages = (std::min(a.HW, a.split_len) + kDaP - 1) / kDaP;
  auto kern = stages == 1            ? k_bwd_dalpha_mfma<NHWC, VEC, 0>
              : stages <= kDaStages ? k_bwd_dalpha_mfma<NHWC, VEC, 1>
                                    : k_bwd_dalpha_mfma<NHWC, VEC, 2>;
  const int lds = a.nres * kDaABytes + 4 * kDaWBytes + kDaRBytes + (a.staged ? kDaEt * a.k * 4 : 0);
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)xcd_grid((int64_t)a.B * a.per, a.per)), dim3(kDaThreads), lds, st, a);
  return hipGetLastError();
}

}  // namespace

void bwd_dalpha_splits(const Shape& sh, int* nsplit, int* split_len) { bwd_dalpha_split(sh, nsplit, split_len); }

bool bwd_mfma_dalpha(const Shape& sh, const void* x, const void* dy, const BwdWs& ws, hipStream_t st, hipError_t* err) {
  if (!dalpha_mfma_eligible(sh)) return false;
  DaArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.dy = static_cast<const uint16_t*>(dy);
  a.bbeg = ws.bbeg;
  a.bw = ws.bw;
  a.ba = ws.ba;
  a.dal = ws.dal;
  a.B = (int)sh.B;
  a.C = (int)sh.C;
  a.E = sh.E;
  a.R = sh.R;
  a.k = sh.k;
  a.HW = (int)sh.HW;
  bwd_dalpha_split(sh, &a.nsplit, &a.split_len);
  a.nblk = (int)((sh.C + kBwBucketCh - 1) / kBwBucketCh);
  a.nCB = (int)((sh.C + kDaCt - 1) / kDaCt);
  a.nEB = (sh.R + kDaEt - 1) / kDaEt;
  da_runs(sh, a.nsplit, &a.csplit, &a.cper);
  a.per = a.nEB * a.csplit * a.nsplit;
  // whole rows gathered in LDS where the workgroup sees every channel and two
  // still share a CU: single entries, written as their channel blocks
  // come, left the L2 as 206 MB of partial lines for 33 MB of dalpha at stage 4
  const int stages = (std::min(a.HW, a.split_len) + kDaP - 1) / kDaP;
  a.nres = stages <= kDaStages ? stages : 1;
  a.staged = a.csplit == 1 && a.nres * kDaABytes + 4 * kDaWBytes + kDaRBytes + kDaEt * sh.k * 4 <= 80 * 1024;
  if (sh.layout == MOCE_NHWC)
    *err = sh.C % 8 == 0 && sh.E % 8 == 0   ? launch_da<true, 8>(a, st)
           : sh.C % 4 == 0 && sh.E % 4 == 0 ? launch_da<true, 4>(a, st)
                                            : launch_da<true, 1>(a, st);
  else
    *err = sh.HW % 8 == 0 ? launch_da<false, 8>(a, st) : sh.HW % 4 == 0 ? launch_da<false, 4>(a, st) : launch_da<false, 1>(a, st);
  return true;
}

// ---- dx on the matrix cores -------------------------------------------------
//
// dx[b][c][p] = sum_e coef_b[c][e] dy[b][e][p] + dd[b][c] / HW, where
// coef_b[c][e] is alpha_b[e][i] for the support entry (e, i) on channel c,
// 1/|U| for e = E-1 (the residual) when c is uncovered, and 0 elsewhere.
// The coefficients enter the product as two bf16 parts (hi = bf16(alpha),
// lo = bf16(alpha - hi): 16 significant bits) or, for rows that only the generic
// kernel with its float32 coefficients would take otherwise, as three that sum to
// them exactly; dy as it is.
//
// The entries come in buckets by (64 channels, 64 experts) with their logits
// (k_bw_part), the residual expert's channels as a bitmap; the coefficients are
// rebuilt here from the logits and the image's softmax statistics.  A workgroup
// of four waves owns (image, 64 positions, 128 channels) and walks the expert
// chunks: the chunk's dy tile (64 x 64) and its coefficient tile (128 x 64, its
// parts) sit in LDS; the coefficient tile starts zero, receives its buckets'
// entries by scatter and is cleared entry by entry once multiplied, so a chunk
// costs LDS writes in proportion to its entries, not to its area.  The next
// chunk's reads are in flight beside the products.  A step is a chain of
// barriers (scatter, multiply, clear), so the tile is kept small enough for
// three workgroups a CU to fill each other's gaps: 54 us at stage 4 and 49 at
// stage 1, where one of 256 channels with double-buffered tiles, alone on its CU,
// took 74 at stage 4 (40k cycles a workgroup, a third of them vector and a fifth
// matrix instructions).  The results leave through LDS as whole rows.  dy's rows
// are read 16 or 8 bytes a load where E (channels-last) or H W allow, by single
// elements elsewhere, where the whole backward takes 157 us in the place of 267
// with the vector dx (219 images, C 1024, E 256, k 32, 7 x 7 channels-first); where
// a chunk holds too few entries for that, dx_mfma_eligible leaves the call to it.
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
constexpr int dx_lds(int parts) { return parts * kDxCoefPart + 2 * kDxDyBuf + 2 * kDxStats + kDxRanges * 2 * 8; }
// parts of a coefficient: two where rows allow 16-byte (channels-last) or 8-byte
// loads; three, whose sum is the float32 coefficient itself, elsewhere
constexpr int dx_parts(bool nhwc, int vec) { return vec == 8 || (!nhwc && vec == 4) ? 2 : 3; }
constexpr int kDxSub = kDxCt / kBwBucketCh;      // bucket rows per workgroup
constexpr int kDxSubThreads = kDxThreads / kDxSub;
constexpr uint32_t kDxNone = 0xffffdeadu;        // no entry at this place of a float32 tile
constexpr int64_t kDxMaxTiles = 4096;            // of 256 channels by 64 experts
static_assert(kDxEk == kBwBucketEx, "a chunk is a bucket column");

// byte offset of (channel cl, expert el) in one coefficient part: rows of 64
// experts (128 bytes), 16-byte chunks XOR-swizzled by the channel
__device__ __forceinline__ int coef_off(int cl, int el) {
  return cl * 128 + ((((el >> 3) ^ (cl & 7))) << 4) + ((el & 7) << 1);
}

template <bool NHWC, int VEC>
__global__ void __launch_bounds__(kDxThreads, dx_parts(NHWC, VEC) == 2 ? 3 : 2)
k_bwd_dx_mfma(const uint16_t* __restrict__ dy, uint16_t* __restrict__ dx, const float* __restrict__ dd,
              const int32_t* __restrict__ bbeg, const uint2* __restrict__ bw, const float* __restrict__ stats,
              const uint64_t* __restrict__ unc, int B, int C, int E, int HW, int nEC,
              int nPC) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int NP = dx_parts(NHWC, VEC);
  unsigned char* coP = lds;                           // [NP][128][64] bf16
  unsigned char* dyL = lds + NP * kDxCoefPart;        // [2 buf][64][64] bf16
  float4* stL = reinterpret_cast<float4*>(dyL + 2 * kDxDyBuf);   // [2 buf][64] (rt, m, rzs, -)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // the channel blocks of one position block run together, so that dy's tile is
  // read from the XCD's L2
  const int nCB = (C + kDxCt - 1) / kDxCt;
  const int u = xcd_unit(), b = u / (nCB * nPC);
  if (b >= B) return;
  const int cb = u % (nCB * nPC) % nCB, pc = u % (nCB * nPC) / nCB;
  const int c0 = cb * kDxCt, p0 = pc * kDxP;
  const uint16_t* yb = dy + (int64_t)b * E * HW;
  const int R = E - 1;
  const int nch = (R + kDxEk - 1) / kDxEk;            // chunks with routed experts: nEC or nEC - 1
  const float inv_nU = 1.f / (float)bwd_count_uncovered(unc, C);

  // zero the coefficient tile once; every scatter is undone after use
  for (int q = tid; q < NP * kDxCoefPart / 16; q += kDxThreads)
    reinterpret_cast<u32x4*>(coP)[q] = u32x4{0u, 0u, 0u, 0u};

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
  // a coefficient's bf16 parts into its place
  auto put_parts = [&](int o, float a) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const uint16_t v = f32_to_bf16(a);
      *reinterpret_cast<uint16_t*>(coP + i * kDxCoefPart + o) = v;
      a -= bf16_to_f32(v);
    }
  };
  // scatter (or, with clear, zero) the entries of chunk ec
  auto scatter = [&](int ec, const Ents& E, bool clear) __attribute__((always_inline)) {
    const float4* sb = stL + (ec & 1) * kDxEk;
    auto put = [&](uint2 v) __attribute__((always_inline)) {
      const int el = (int)(v.x >> 8), o = coef_off(v.x & (kDxCt - 1), el);
      if (clear) {
#pragma unroll
        for (int i = 0; i < NP; ++i) *reinterpret_cast<uint16_t*>(coP + i * kDxCoefPart + o) = 0;
      } else {
        const float4 q = sb[el];
        put_parts(o, coef_alpha(coef_e(coef_z(__uint_as_float(v.y), q.x), q.y), q.z));
      }
    };
#pragma unroll
    for (int r = 0; r < kDxEPT; ++r)
      if (st0 + r * kDxSubThreads < E.n) put(E.w[r]);
    for (int q = st0 + kDxEPT * kDxSubThreads; q < E.n; q += kDxSubThreads) put(bw[E.base + q]);
    // the residual's channels (the last chunk's: never cleared for a later one)
    if (!clear && ec == R / kDxEk && st0 < kBwBucketCh && blk < nblk && ((unc[blk] >> st0) & 1))
      put_parts(coef_off(sub * kBwBucketCh + st0, R % kDxEk), inv_nU);
  };
  // dy tile of expert chunk ec: NHWC rows of positions (64 experts each, 16-byte
  // chunks swizzled by the row), NCHW rows of experts (64 positions each,
  // 32-byte blocks swizzled for the transposing read)
  constexpr int PW = VEC == 1 ? 8 : VEC;    // elements of a thread's piece, one load or (VEC = 1) one each
  constexpr int DYL = kDxP * kDxEk / PW / kDxThreads;   // pieces per thread
  constexpr int DYW = PW / 2;               // words per piece
  uint32_t dyr[DYL][DYW];
  // (clamped reads; experts and positions outside the tensor meet zero
  // coefficients or are not written, but must not bring a NaN: store_dy zeroes
  // the experts)
  auto load_dy = [&](int ec) {
    const int e0 = ec * kDxEk;
#pragma unroll
    for (int j = 0; j < DYL; ++j) {
      const int q = tid + j * kDxThreads;
      const int row = q / (64 / PW), o = q % (64 / PW) * PW;   // (position, experts) or (expert, positions)
      if (VEC == 1) {
        // rows of any alignment: single elements
        const uint16_t* src = yb + (NHWC ? (int64_t)min(p0 + row, HW - 1) * E : (int64_t)min(e0 + row, E - 1) * HW);
        const int first = (NHWC ? e0 : p0) + o, last = (NHWC ? E : HW) - 1;
#pragma unroll
        for (int i = 0; i < DYW; ++i)
          dyr[j][i] = src[min(first + 2 * i, last)] | (uint32_t)src[min(first + 2 * i + 1, last)] << 16;
        continue;
      }
      const uint16_t* src = NHWC ? yb + (int64_t)min(p0 + row, HW - 1) * E + min(e0 + o, E - VEC)
                                 : yb + (int64_t)min(e0 + row, E - 1) * HW + min(p0 + o, HW - VEC);
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
  };
  int bad = 0;   // (three parts) an element that is not finite among those met
  auto store_dy = [&](int ec) {
    unsigned char* base = dyL + (ec & 1) * kDxDyBuf;
    const int e0 = ec * kDxEk;
#pragma unroll
    for (int j = 0; j < DYL; ++j) {
      const int q = tid + j * kDxThreads, row = q / (64 / PW), o = q % (64 / PW) * PW;
      if (NHWC && VEC != 8) {
        // E is no multiple of 8: some of the piece's experts may lie past the last
#pragma unroll
        for (int w = 0; w < DYW; ++w) {
          const int left = E - (e0 + o + 2 * w);
          dyr[j][w] &= left >= 2 ? ~0u : left == 1 ? 0xffffu : 0u;
        }
      } else {
        const uint32_t m = e0 + (NHWC ? o : row) < E ? ~0u : 0u;
#pragma unroll
        for (int w = 0; w < DYW; ++w) dyr[j][w] &= m;
      }
      if (NP == 3) {
#pragma unroll
        for (int w = 0; w < DYW; ++w)
          bad |= ((dyr[j][w] & 0x7f80u) == 0x7f80u) | ((dyr[j][w] & 0x7f800000u) == 0x7f800000u);
      }
      unsigned char* dst = NHWC ? base + row * 128 + (((o >> 3) ^ (row & 7)) << 4) + (o & 7) * 2
                                : base + row * 128 + (((o >> 4) ^ dyswz(row)) << 5) + (o & 15) * 2;
      if (PW == 8)
        *reinterpret_cast<u32x4*>(dst) = u32x4{dyr[j][0], dyr[j][1], dyr[j][2], dyr[j][3]};
      else
        *reinterpret_cast<u32x2*>(dst) = u32x2{dyr[j][0], dyr[j][1]};
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
        bf16x8 a[4], bc[NP][2];
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const int row = mt * 16 + (lane & 15);
          a[mt] = *reinterpret_cast<const bf16x8*>(dyP + row * 128 + ((oct ^ (row & 7)) << 4));
        }
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const int cl = (wave * 2 + nt) * 16 + (lane & 15);
          const int o = cl * 128 + ((oct ^ (cl & 7)) << 4);
#pragma unroll
          for (int i = 0; i < NP; ++i) bc[i][nt] = *reinterpret_cast<const bf16x8*>(coP + i * kDxCoefPart + o);
        }
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int i = 0; i < NP; ++i)
              acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], bc[i][nt], acc[mt][nt], 0, 0, 0);
      } else {
        // D[c][p]: A = coefficient rows (channels), B = dy rows (experts) read transposed
        bf16x8 ac[NP][2], bb[4];
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) {
          const int cl = (wave * 2 + mt) * 16 + (lane & 15);
          const int o = cl * 128 + ((oct ^ (cl & 7)) << 4);
#pragma unroll
          for (int i = 0; i < NP; ++i) ac[i][mt] = *reinterpret_cast<const bf16x8*>(coP + i * kDxCoefPart + o);
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
          for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int i = 0; i < NP; ++i)
              acc[nt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ac[i][mt], bb[nt], acc[nt][mt], 0, 0, 0);
      }
    }
    if (ec + 1 < nEC) {   // into the buffers chunk ec - 1 used
      store_dy(ec + 1);
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
  // An element of dy that is not finite would reach every channel through the
  // tile's zeros, where a sum over the channel's entries gives it to those alone:
  // a workgroup that meets one sums so (a tile of float32 coefficients by chunk, 8
  // outputs a thread at a time).
  if (NP == 3 && __syncthreads_or(bad)) {
    float* ct = reinterpret_cast<float*>(lds);
    constexpr int OUT = 8, PC = kDxEk + 1;   // outputs of a thread, pitch of the tile
    static_assert(kDxCt * PC * 4 <= 3 * kDxCoefPart, "the float32 tile fits");
    const int64_t n = (int64_t)B * R;
    const int cl = tid % kDxCt, c = c0 + cl, ib = cl / kBwBucketCh;
#pragma unroll 1
    for (int pp = tid / kDxCt; pp < kDxP; pp += OUT * (kDxThreads / kDxCt)) {
      float sum[OUT] = {};
      auto at_dy = [&](int e, int u) {
        const int p = min(p0 + pp + u * (kDxThreads / kDxCt), HW - 1);
        return bf16_to_f32(NHWC ? yb[(int64_t)p * E + e] : yb[(int64_t)e * HW + p]);
      };
#pragma unroll 1
      for (int ec = 0; ec < nch; ++ec) {
        for (int q = tid; q < kDxCt * PC; q += kDxThreads) reinterpret_cast<uint32_t*>(ct)[q] = kDxNone;
        __syncthreads();
        const int2 r = bucket(ec, blk);
        for (int q = r.x + st0; q < r.x + r.y; q += kDxSubThreads) {
          const uint2 v = bw[q];
          const int el = (int)(v.x >> 8);
          const int64_t i = (int64_t)b * R + ec * kDxEk + el;
          ct[(v.x & (kDxCt - 1)) * PC + el] =
              coef_alpha(coef_e(coef_z(__uint_as_float(v.y), stats[i]), stats[n + i]), stats[2 * n + i]);
        }
        __syncthreads();
#pragma unroll 1
        for (int el = 0; el < kDxEk; ++el) {
          const float a = ct[cl * PC + el];
          if (__float_as_uint(a) == kDxNone) continue;
#pragma unroll
          for (int u = 0; u < OUT; ++u) sum[u] += a * at_dy(ec * kDxEk + el, u);
        }
        __syncthreads();
      }
      const int cblk = cb * kDxSub + ib;
      if (c < C) {
        const bool none = (unc[cblk] >> (cl % kBwBucketCh)) & 1;
        const float add = dd[(int64_t)b * C + c] * rhw;
#pragma unroll
        for (int u = 0; u < OUT; ++u) {
          const int p = p0 + pp + u * (kDxThreads / kDxCt);
          const float v = (none ? sum[u] + at_dy(R, u) * inv_nU : sum[u]) + add;
          if (p < HW) dx[NHWC ? ((int64_t)b * HW + p) * C + c : ((int64_t)b * C + c) * HW + p] = f32_to_bf16(v);
        }
      }
    }
    return;
  }
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
      else if (VEC == 4)
        *reinterpret_cast<u32x2*>(dst) = *reinterpret_cast<const u32x2*>(src);
      else
        *dst = *reinterpret_cast<const uint16_t*>(src);
    }
  }
}

// bfloat16 layers with routed experts (without any, dx spreads the residual plane over
// the channels) but the largest numbers of chunks (more than kDxMaxTiles tiles of 256
// channels by 64 experts) and more workgroups than a launch holds.  Where rows allow
// wide loads always; elsewhere, where the tiles have three parts, by what both kernels
// take in ns, fitted to their times over 700 ragged shapes.  The vector kernel: 0.0036 for
// an element of dx, 0.00115 for an entry at a position channels-first, where its dy is
// read in order, 0.0021 channels-last, 400 for each of a channel's entries, one after
// another, and 10500 for itself and the channels' lists.  This one: 7.5 for a workgroup
// and 3.7 for each of its chunks, three barriers however few entries it holds (5.8 and
// 3.1 with 8-byte rows), 0.003 for an entry at 64 positions, 1500 a chunk for the chain of
// one workgroup and 5500.  Where the two meet: 7 images of C 2903, E 720, k 1, 785
// positions channels-first 54 us with the vector dx and 151 with this one; 192 of C 1328,
// E 328, k 8, 197 positions 280 and 323; 49152 of C 16, E 4, k 16, 64 positions
// channels-last 303 and 460.
bool dx_mfma_eligible(const Shape& sh) {
  const int64_t nCB = (sh.C + kDxCt - 1) / kDxCt, nEC = (sh.E + kDxEk - 1) / kDxEk, nPC = (sh.HW + kDxP - 1) / kDxP;
  if (sh.elem != MOCE_BF16 || sh.R < 1 || !launch_holds(xcd_grid(sh.B * nCB * nPC, nCB * nPC), kDxThreads)) return false;
  if ((nCB + 1) / 2 * nEC > kDxMaxTiles) return false;
  const bool nhwc = sh.layout == MOCE_NHWC;
  if (nhwc ? sh.E % 8 == 0 : sh.HW % 4 == 0) return true;
  const double entries = (double)sh.R * sh.k, chunks = (double)nEC;
  const double vec = 10500. + sh.B * (0.0036 * sh.C + (nhwc ? 0.0021 : 0.00115) * entries) * sh.HW + 400. * entries / sh.C;
  const bool four = nhwc && sh.E % 4 == 0;
  const double group = four ? 5.8 + 3.1 * chunks : 7.5 + 3.7 * chunks;
  const double mfma = 5500. + 1500. * chunks + sh.B * nPC * (nCB * group + 0.003 * entries);
  return vec >= mfma;
}

}  // namespace

bool bwd_dx_on_mfma(const Shape& sh) { return dx_mfma_eligible(sh); }

bool bwd_mfma_dx(const Shape& sh, const void* dy, const BwdWs& ws, void* dx, hipStream_t st, hipError_t* err) {
  if (!dx_mfma_eligible(sh)) return false;
  const int nEC = (sh.E + kDxEk - 1) / kDxEk;
  const int nCB = (int)((sh.C + kDxCt - 1) / kDxCt);
  const int nPC = (int)((sh.HW + kDxP - 1) / kDxP);
  const unsigned grid = (unsigned)xcd_grid(sh.B * nCB * nPC, (int64_t)nCB * nPC);
  auto y = static_cast<const uint16_t*>(dy);
  auto o = static_cast<uint16_t*>(dx);
  using K = void (*)(const uint16_t*, uint16_t*, const float*, const int32_t*, const uint2*, const float*,
                     const uint64_t*, int, int, int, int, int, int);
  // the widest piece that rows of E (channels-last) or H W elements allow
  const int64_t row = sh.layout == MOCE_NHWC ? sh.E : sh.HW;
  const bool nhwc = sh.layout == MOCE_NHWC;
  const int vec = row % 8 == 0 ? 8 : row % 4 == 0 ? 4 : 1, bytes = dx_lds(dx_parts(nhwc, vec));
  const K kern = nhwc ? (vec == 8 ? k_bwd_dx_mfma<true, 8> : vec == 4 ? k_bwd_dx_mfma<true, 4> : k_bwd_dx_mfma<true, 1>)
                      : (vec == 8   ? k_bwd_dx_mfma<false, 8>
                         : vec == 4 ? k_bwd_dx_mfma<false, 4>
                                    : k_bwd_dx_mfma<false, 1>);
  if ((*err = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes)) != hipSuccess)
    return true;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kDxThreads), bytes, st, y, o, ws.dd, ws.bbeg, ws.bw, ws.stats,
                     ws.unc, (int)sh.B, (int)sh.C, sh.E, (int)sh.HW, nEC, nPC);
  *err = hipGetLastError();
  return true;
}

}  // namespace moce
