// W4A4 GEMM with Runtime Smooth for many tokens on the 6-bit matrix rate: the
// same product as the main kernel (Section 3.2, Eq. 3, Fig. 4 step (3)),
//   Y[i, n] = fp16( alpha_i * beta_n / K * sum_b s_b * P_b[i, n] ),
// and, with one team of waves, the same bits: the partials P_b are exact here too,
// and each is added with one FMA by s_b in the same order. Two teams (split_teams)
// sum the two halves of K apart and add the two sums last.
//
// What bounds the int8 kernel is issue: per 32 x 32 x 64 of work two MFMAs (64
// clocks) and 20.5 vector instructions (82 clocks), of which 16 rescale (an
// exact subtraction that turns the seeded integer into a float, and the FMA).
// v_mfma_f32_32x32x64_f8f6f4 on E2M3 operands does that work in one MFMA and
// leaves the partial as a float, so the rescale is the FMA alone, and the codes
// are spread to six bits instead of eight (rrs_gemm_fp6.h). Per 32 x 32 x 64: one
// MFMA and a quarter of another (the start values), 10.4 vector instructions.
//
// Tokens are spread once, by a launch of their own (expand_tokens_kernel, into
// scratch memory of the caller), in MFMA operand order: in a 2048 x 12288 layer
// every token row would otherwise be spread for each of 96 column tiles. Weights
// are spread while they are staged; doing them beforehand would cost more (38 MB
// written and read at 4096 x 12288) than it saves below some 4000 tokens.
//
// A workgroup computes 64 WMC x 128: 2 WMC waves of 64 x 64, 2 x 2 blocks of
// 32 x 32. K advances in tiles of 128. Per tile and wave, the token rows of the
// upper block come from LDS, those of the lower block straight from global
// memory a tile ahead (LDS and L1 then carry about the same: LDS alone would be
// busy four clocks in five), the weights from LDS. LDS is double-buffered, with one
// barrier per tile in its middle: by then every fragment of the tile is in
// registers and the next tile is staged. While a block's MFMAs run, the vector
// unit rescales the block before.
//
// Measured, GEMM calls in graph replays, weights cold, row-major, int8 kernel -> this one
// with the token pass: 2048 x 4096 x 12288, g = 128 115 -> 94 us; 4096 x 4096 x 22016 402 ->
// 334; 8192 x 8192 x 28672, g = 64 2510 -> 1880; 512 x 8192 x 8192 69 -> 41 (two teams).
// Spreading 2048 x 4096 tokens takes 4.7 us. Counters at 2048 x 4096 x 12288, of the busy
// cycles: the MFMA unit 35 %, vector instructions 49 %; of a wave's time a quarter issues
// vector instructions, 7 % LDS, 28 % waits for data or the barrier, 31 % for its turn to
// issue.
// Tried and slower: one wave per SIMD with 128 x 96 (158 us: nothing covers its
// stalls), four waves per SIMD with 64 x 32 (104: 1.5 times the LDS reads), two
// register sets for the loads (no gain), fragment pairs as three 128-bit reads
// (the compiler moves the halves apart again).
#include <type_traits>

#include "rrs_gemm_fp6.h"

namespace rrs {
namespace {
using namespace fp6;

typedef const __attribute__((address_space(1))) uint8_t* gbytes;
typedef const __attribute__((address_space(1))) v4u* gv4u;
typedef const __attribute__((address_space(1))) v2u* gv2u;
typedef const __attribute__((address_space(1))) uint32_t* gu32;

constexpr int kGroupM = 4;  // row tiles per column strip

// LDS layout of one 32-row weight block of a 128-channel tile, in MFMA operand
// order: four sections of 32 rows x 16 bytes (dwords 0-3 of the six; section q
// holds channels [32 q, 32 q + 32)), then four of 32 rows x 8 bytes (dwords 4-5).
// Sections are padded by 32 bytes so that the four lanes that stage one row's
// four pieces write to different banks.
constexpr int kSec16 = 512 + 32;
constexpr int kSec8 = 256 + 32;
constexpr int kBlk8 = 4 * kSec16;
constexpr int kBlk = 4 * (kSec16 + kSec8);  // 3328

struct TileMap {
  int m0, n0;
  bool valid;
};

// XCD-aware tile order: workgroup ids are dealt round-robin to the 8 XCDs, so
// each XCD gets a contiguous run of tiles, in column strips of 4 row tiles.
// Workgroup w, of index `local` on its XCD.
template <int BM, int BN>
__device__ __forceinline__ TileMap map_tile(int M, int N, int w, int local) {
  const int tm = (M + BM - 1) / BM;
  const int tn = (N + BN - 1) / BN;
  const int T = tm * tn;
  const int per = (T + 7) >> 3;
  const int lin = (w & 7) * per + local;
  TileMap r;
  r.valid = local < per && lin < T;
  const int strip = kGroupM * tn;
  const int first_m = (lin / strip) * kGroupM;
  const int gm = min(tm - first_m, kGroupM);
  const int rem = lin % strip;
  r.m0 = (first_m + rem % gm) * BM;
  r.n0 = (rem / gm) * BN;
  return r;
}

// Tokens: packed codes -> MFMA operand order (rrs_gemm_fp6.h). One thread per
// 16-byte piece (32 codes); rows past M are written as zeros.
__global__ __launch_bounds__(256) void expand_tokens_kernel(const uint8_t* __restrict__ Xq, int M,
                                                            int K, uint8_t* __restrict__ out) {
  const int ntiles = K / 128;
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int q = t & 3, row32 = (t >> 2) & 31;
  const int kt = (t >> 7) % ntiles, mb = (t >> 7) / ntiles;
  const int nb = (int)token_blocks(M);
  if (mb >= nb) return;
  const int row = mb * 32 + row32;
  v4u x = {0, 0, 0, 0};
  if (row < M) x = *reinterpret_cast<const v4u*>(Xq + (size_t)row * (K / 2) + kt * 64 + q * 16);
  const Flip none{0, 0, 0};
  uint32_t d[6], g[6];
  v4u y, sg;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t neg = (x[i] >> 3) & 0x11111111u;
    y[i] = (x[i] ^ ((neg << 4) - neg)) + neg;  // |q|, up to 8: no carry
    sg[i] = neg;
  }
  spread16(y[0], y[1], none, d[0], d[1], d[2]);
  spread16(y[2], y[3], none, d[3], d[4], d[5]);
  spread16(sg[0], sg[1], none, g[0], g[1], g[2]);
  spread16(sg[2], sg[3], none, g[3], g[4], g[5]);
#pragma unroll
  for (int i = 0; i < 6; i += 3) {  // the sign bit sits five above the magnitude's lowest
    d[i] |= g[i] << 5;
    d[i + 1] |= __builtin_amdgcn_alignbit(g[i + 1], g[i], 27);
    d[i + 2] |= __builtin_amdgcn_alignbit(g[i + 2], g[i + 1], 27);
  }
  int sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_sdot8((int)x[i], 0x11111111, sum, false);
  uint8_t* o = out + ((size_t)mb * ntiles + kt) * kTokTile;
  *reinterpret_cast<v4u*>(o + q * 512 + row32 * 16) = v4u{d[0], d[1], d[2], d[3]};
  *reinterpret_cast<v2u*>(o + 2048 + q * 256 + row32 * 8) = v2u{d[4], d[5]};
  sum += __shfl_xor(sum, 1);                       // a 64-channel step
  const uint32_t hs = __builtin_bit_cast(uint16_t, (_Float16)(-0.125f * (float)sum));
  const uint32_t other = (uint32_t)__shfl_xor((int)hs, 2);
  if (q == 0)
    *reinterpret_cast<uint32_t*>(out + (size_t)nb * ntiles * kTokTile +
                                 ((size_t)mb * ntiles + kt) * kTokSum + row32 * 4) =
        hs | (other << 16);
}

constexpr int NB = 2;  // 32-column blocks per wave

template <int WMC>
struct Shape {
  static constexpr int kThreads = 128 * WMC;
  static constexpr int kRowsPer = kThreads / 4;  // weight rows staged at once
  static constexpr int BM = 64 * WMC;
  static constexpr int BN = 128;
  static constexpr int A_BYTES = WMC * kTokTile;  // the waves' upper blocks
  static constexpr int PA = (A_BYTES / 16 + kThreads - 1) / kThreads;
  static constexpr int PB = BN / kRowsPer;
  static constexpr bool kHalfA = A_BYTES / 16 % kThreads != 0;
  static constexpr int SA = A_BYTES;  // code sums, one word a row
  static constexpr int B0 = SA + BM * 4;
  static constexpr int STAGE = B0 + BN / 32 * kBlk;
  static_assert(BN % kRowsPer == 0 && BM <= kThreads, "staging");
  static_assert(!kHalfA || A_BYTES / 16 % kThreads == kThreads / 2, "half of the waves");
};

// GS = g / 32. kPerChannel: one sum over all of K and no rescale (Section 2.1).
// kGather (runtime channel reorder): position block p of the tokens pairs with
// block border[p] of every Wq row. KS = 2: two teams of 2 WMC waves on one tile,
// each over half of K.
template <int GS, int WMC, int KS, bool kPerChannel, bool kGather, bool kTiled>
__device__ __forceinline__ void gemm_fp6_tile(
    const TileMap tile, uint8_t* const lds_all, float* const scale_tab, int* const btab,
    const uint8_t* __restrict__ Xe, const float* __restrict__ a_scale,
    const float* __restrict__ s_group, const uint8_t* __restrict__ Wq,
    const float* __restrict__ w_scale, int M, int N, int K, uint16_t* __restrict__ Y,
    float out_scale, const int32_t* __restrict__ border) {
  using S = Shape<WMC>;
  constexpr int kThreads = S::kThreads;
  constexpr WqLayout lay{kTiled};
  constexpr int BM = S::BM, BN = S::BN;
  constexpr bool kKeep = kPerChannel || GS > 4;  // a sum spans several K tiles
  constexpr int GPT = GS >= 4 ? 1 : 4 / GS;      // groups per K tile
  constexpr int TPG = GS >= 4 ? GS / 4 : 1;      // K tiles per group
  const int m0 = tile.m0, n0 = tile.n0;
  // The team's share: its threads, its LDS and its K tiles, [k0, k0 + nt).
  const int team = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);
  const int t = threadIdx.x & (kThreads - 1);
  const int ntiles = K / 128;
  const int nt = ntiles / KS;
  const int k0 = team * nt;
  uint8_t* const lds = lds_all + team * 2 * S::STAGE;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave % WMC;
  const int wn = wave / WMC;
  const Flip flip = make_flip();

  // Staging slots. Tokens: 16-byte chunk t + kThreads i of the tile's upper
  // blocks. Weights: thread t handles piece q (32 channels) of rows t / 4 +
  // kRowsPer i. Rows past M or N take the last valid block or row instead: their
  // results are never stored.
  const int nblk = (int)token_blocks(M);
  const int q = t & 3;
  const int row0 = t >> 2;
  constexpr uint32_t wts = (uint32_t)lay.tile();
  constexpr uint32_t wqs = (uint32_t)lay.quarter();
  const uint32_t bstep = (uint32_t)ntiles * kTokTile;  // bytes of one 32-row block
  const uint8_t* abase = Xe + (size_t)(m0 >> 5) * bstep + (size_t)k0 * kTokTile;
  const uint8_t* sbase =
      Xe + (size_t)nblk * bstep + ((size_t)(m0 >> 5) * ntiles + k0) * kTokSum;
  const uint8_t* bbase = Wq + lay.row(n0, K) + (kGather ? 0 : (size_t)k0 * wts);
  const int lastb = nblk - 1 - (m0 >> 5);
  uint32_t aoff[S::PA], boff_[S::PB];
#pragma unroll
  for (int i = 0; i < S::PA; ++i) {
    const int c = t + kThreads * i;
    aoff[i] = (uint32_t)min(c / 192 * 2, lastb) * bstep + (uint32_t)(c % 192) * 16;
  }
  uint32_t soff = (uint32_t)min((t & (BM - 1)) >> 5, lastb) * (uint32_t)(ntiles * kTokSum) +
                  (uint32_t)(t & 31) * 4;
#pragma unroll
  for (int i = 0; i < S::PB; ++i)
    boff_[i] = (uint32_t)(lay.row(min(n0 + row0 + S::kRowsPer * i, N - 1), K) - lay.row(n0, K)) +
               (kGather ? 0u : q * wqs);
  const int st16 = S::B0 + (row0 >> 5) * kBlk + q * kSec16 + (row0 & 31) * 16;
  const int st8 = S::B0 + (row0 >> 5) * kBlk + kBlk8 + q * kSec8 + (row0 & 31) * 8;

  // Fragment reads: lane (l & 31) is the row, l >> 5 the half of a 64-channel step.
  const int half = lane >> 5, lr = lane & 31;
  const int a16 = wm * kTokTile + lane * 16;
  const int a8 = wm * kTokTile + 2048 + lane * 8;
  const int b16 = S::B0 + wn * NB * kBlk + half * kSec16 + lr * 16;
  const int b8 = S::B0 + wn * NB * kBlk + kBlk8 + half * kSec8 + lr * 8;
  // Opaque, so that the 8-byte reads of two steps are not merged into one
  // 16-byte read whose halves then have to be moved apart.
  int a8b = a8 + 512, b8b = b8 + 2 * kSec8;
  asm volatile("" : "+v"(a8b), "+v"(b8b));
  const int sa_rd = S::SA + (wm * 64 + lane) * 4;
  const uint8_t* dbase = Xe + (size_t)min((m0 >> 5) + wm * 2 + 1, nblk - 1) * bstep +
                         (size_t)k0 * kTokTile;
  uint32_t d16 = lane * 16, d8 = lane * 8;

  // A uniform pointer, opaque so that the loads keep it in scalar registers, and
  // an offset, opaque so that its widened copy is not hoisted.
  auto uni = [](const uint8_t* p) {
    gbytes g = (gbytes)(uintptr_t)p;
    asm volatile("" : "+s"(g));
    return g;
  };
  auto off = [](uint32_t& o) {
    asm volatile("" : "+v"(o));
    return o;
  };
  v4u ra[S::PA], rb[S::PB];
  uint32_t rs;
  auto boff = [&](int kt) -> uint32_t {
    if constexpr (kGather) {
      const uint32_t p = (uint32_t)btab[(k0 + kt) * 4 + q];
      return (p >> 2) * wts + (p & 3u) * wqs;
    } else {
      return (uint32_t)kt * wts;
    }
  };
  auto load_a = [&](int kt) {
    const gbytes pa = uni(abase + (size_t)kt * kTokTile);
    const gbytes ps = uni(sbase + (size_t)kt * kTokSum);
#pragma unroll
    for (int i = 0; i < S::PA; ++i) ra[i] = *(gv4u)(pa + off(aoff[i]));
    rs = *(gu32)(ps + off(soff));
  };
  auto load_b = [&](uint32_t bo) {
    const gbytes pb = uni(kGather ? bbase : bbase + bo);
#pragma unroll
    for (int i = 0; i < S::PB; ++i)
      rb[i] = *(gv4u)(pb + (kGather ? boff_[i] + bo : off(boff_[i])));
  };
  // Staging: the token chunks are copied; a weight piece is spread in two
  // halves, the second of which stores it.
  uint32_t wd[3];
  auto stage_a = [&](int stage) {
    uint8_t* s = lds + stage * S::STAGE;
#pragma unroll
    for (int k = 0; k < S::PA; ++k)
      if (!(S::kHalfA && k == S::PA - 1) || wave < WMC)
        *reinterpret_cast<v4u*>(s + t * 16 + k * kThreads * 16) = ra[k];
    *reinterpret_cast<uint32_t*>(s + S::SA + (t & (BM - 1)) * 4) = rs;
  };
  auto stage_b = [&](int stage, int i) {
    uint8_t* s = lds + stage * S::STAGE + (i >> 1) * (S::kRowsPer / 32) * kBlk;
    const v4u x = rb[i >> 1];
    if ((i & 1) == 0) {
      spread16(x[0], x[1], flip, wd[0], wd[1], wd[2]);
    } else {
      uint32_t e0, e1, e2;
      spread16(x[2], x[3], flip, e0, e1, e2);
      *reinterpret_cast<v4u*>(s + st16) = v4u{wd[0], wd[1], wd[2], e0};
      *reinterpret_cast<v2u*>(s + st8) = v2u{e1, e2};
    }
  };
  auto six = [](v4u lo, v2u hi) {
    return v6i{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1]};
  };
  // Fragments by step: fa the upper row block, fd the lower (two tiles), fb the
  // column blocks; ca: lane l's row sums (row l of the wave's 64).
  v6i fa[2], fd[2][2], fb[NB][2];
  v2u ca = {0u, 0u};
  auto read_a = [&](int stage) {
    const uint8_t* s = lds + stage * S::STAGE;
    fa[0] = six(*reinterpret_cast<const v4u*>(s + a16), *reinterpret_cast<const v2u*>(s + a8));
    fa[1] = six(*reinterpret_cast<const v4u*>(s + a16 + 1024),
                *reinterpret_cast<const v2u*>(s + a8b));
  };
  auto read_b = [&](int stage, int j) {
    const uint8_t* s = lds + stage * S::STAGE + j * kBlk;
    fb[j][0] = six(*reinterpret_cast<const v4u*>(s + b16), *reinterpret_cast<const v2u*>(s + b8));
    fb[j][1] = six(*reinterpret_cast<const v4u*>(s + b16 + 2 * kSec16),
                   *reinterpret_cast<const v2u*>(s + b8b));
  };
  auto read_s = [&](int stage) {
    ca[0] = *reinterpret_cast<const uint32_t*>(lds + stage * S::STAGE + sa_rd);
  };
  auto read_d = [&](int set, int kt) {
    const gbytes pd = uni(dbase + (size_t)kt * kTokTile);
    off(d16);
    off(d8);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const v4u lo = *(gv4u)(pd + d16 + ks * 1024);
      const v2u hi = *(gv2u)(pd + d8 + 2048 + ks * 512);
      fd[set][ks] = six(lo, hi);
    }
  };

  // The start values: D = sums x selection, a depth-8 product in which lanes 0-31
  // (the upper rows' sums) are depth 0-3 and lanes 32-63 (the lower rows') depth
  // 4-7, so the selection's ones choose the row half, and for g = 64 the step.
  auto sel = [&](int h, int step) {
    const uint32_t w = GS >= 4 ? 0x3C003C00u : step ? 0x3C000000u : 0x3C00u;
    return __builtin_bit_cast(v4h, v2u{half == h ? w : 0u, 0u});
  };
  const v4h selh[2][2] = {{sel(0, 0), sel(0, 1)}, {sel(1, 0), sel(1, 1)}};
  auto start = [&](int h, int step, const v16f& acc) {
    return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, ca), selh[h][step], acc, 0,
                                                0, 0);
  };

  const v16f zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  float f[2][NB][16];
  v16f pk[2][NB];  // kKeep: the sums carried over K tiles
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      pk[h][j] = zero;
#pragma unroll
      for (int r = 0; r < 16; ++r) f[h][j][r] = 0.0f;
    }
  auto rescale = [&](const v16f& p, int b, int r0, int r1, float s) {
#pragma unroll
    for (int r = r0; r < r1; ++r) {
      float& x = f[b / NB][b % NB][r];
      x = __builtin_fmaf(s, p[r], x);
      // Pin the update here: the compiler would sink a tile's rescales to its end.
      asm volatile("" : "+v"(x));
    }
  };
  auto row_of = [&](int h, int r) { return wm * 64 + h * 32 + 8 * (r >> 2) + 4 * half + (r & 3); };
  auto col_of = [&](int j) { return (wn * NB + j) * 32 + lr; };

  // Prologue: the output scales in LDS, tile 0 staged, tile 1 in flight.
  for (int i = threadIdx.x; i < BM + BN; i += KS * kThreads)
    scale_tab[i] = i < BM ? a_scale[min(m0 + i, M - 1)] : w_scale[min(n0 + i - BM, N - 1)];
  if constexpr (kGather) {
    // Entries are masked into range, so any table keeps every load in bounds.
    for (int i = threadIdx.x; i < K / kReorderBlock; i += KS * kThreads)
      btab[i] = border[i] & (K / kReorderBlock - 1);
    __syncthreads();
  }
  load_a(0);
  load_b(boff(0));
  stage_a(0);
#pragma unroll
  for (int i = 0; i < 2 * S::PB; ++i) stage_b(0, i);
  load_a(1);
  load_b(boff(1));
  read_d(0, 0);
  __syncthreads();
  read_a(0);
  read_b(0, 0);
  read_s(0);
  v16f cs = start(0, 0, zero);  // start values of the next row of blocks (g = 128)

  v16f pp = zero;  // the block whose group has just closed, and its scale
  float sp = 0.0f;
  uint32_t bnext = 0;
  constexpr int NBLK = 2 * NB;             // blocks 0, 1: upper rows; 2, 3: lower
  constexpr int kBar = NB;                 // the barrier stands before this block
  constexpr int kChunk = 64 * TPG / GPT;   // K tiles whose scales one register holds

  const int ngrp = nt * 128 / (GS * 32);
  for (int kc = 0; kc < nt; kc += kChunk) {
    float sv = 0.0f;
    if constexpr (!kPerChannel)
      sv = s_group[team * ngrp + min(kc / TPG * GPT + lane, ngrp - 1)];
    const int kend = min(kc + kChunk, nt);
    for (int kt0 = kc; kt0 < kend; kt0 += 2) {
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int kt = kt0 + p;
        const int grp = kt / TPG * GPT;
        float s0 = 0.0f, s1 = 0.0f;
        if constexpr (!kPerChannel) {
          const int svi = __builtin_bit_cast(int, sv);
          s0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(svi, grp & 63));
          if constexpr (GS < 4)
            s1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(svi, (grp + 1) & 63));
        }
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
          const int h = b / NB, j = b % NB;
          const int prev = (b + NBLK - 1) % NBLK;
          // Every fragment of this tile is in registers and the next tile is
          // staged in the other half of the LDS.
          if (b == kBar) __syncthreads();
          if (b == 0) {
            read_b(p, 1);
            read_d(p ^ 1, min(kt + 1, nt - 1));
          }
          if (b == kBar) {
            read_a(p ^ 1);
            if constexpr (GS == 4 && !kPerChannel) read_s(p ^ 1);
          }
          if (b == NBLK - 1) read_b(p ^ 1, 0);
          const v6i x0 = h ? fd[p][0] : fa[0], x1 = h ? fd[p][1] : fa[1];
          // The next tile is staged before the barrier, each part's registers
          // refilled at once.
          auto steps = [&](int part) {
            const int kn = min(kt + 2, nt - 1);
            if (b == 0 && part == 0) {
              if constexpr (kGather) bnext = boff(kn);
              stage_a(p ^ 1);
              load_a(kn);
            }
#pragma unroll
            for (int i = 0; i < 2 * S::PB; ++i)
              if (b < kBar && i * kBar / S::PB == 2 * b + part) stage_b(p ^ 1, i);
            if (b == kBar - 1 && part == 1) load_b(kGather ? bnext : boff(kn));
          };
          if constexpr (kKeep) {
            const bool gstart = !kPerChannel && kt % TPG == 0;
            const bool gend = !kPerChannel && (kt + 1) % TPG == 0;
            v16f c = pk[h][j];
            if (gstart) c = zero;
            c = start(h, 0, c);
            c = mfma64(x0, fb[j][0], c);
            steps(0);
            c = mfma64(x1, fb[j][1], c);
            steps(1);
            pk[h][j] = c;
            if (gend) rescale(c, b, 0, 16, s0);
            if (b == NBLK - 1) read_s(p ^ 1);
          } else if constexpr (GS == 4) {
            v16f c = mfma64(x0, fb[j][0], cs);
            if (j == NB - 1) cs = start(h ^ 1, 0, zero);
            rescale(pp, prev, 0, 8, sp);
            steps(0);
            __builtin_amdgcn_sched_barrier(0);
            c = mfma64(x1, fb[j][1], c);
            rescale(pp, prev, 8, 16, sp);
            steps(1);
            pp = c;
            sp = s0;
          } else {
            v16f c0 = start(h, 0, zero);
            rescale(pp, prev, 0, 8, sp);
            c0 = mfma64(x0, fb[j][0], c0);
            rescale(pp, prev, 8, 16, sp);
            steps(0);
            __builtin_amdgcn_sched_barrier(0);
            v16f c = start(h, 1, zero);
            rescale(c0, b, 0, 8, s0);
            c = mfma64(x1, fb[j][1], c);
            rescale(c0, b, 8, 16, s0);
            steps(1);
            pp = c;
            sp = s1;
            if (b == NBLK - 1) read_s(p ^ 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }
  if constexpr (!kKeep) rescale(pp, NBLK - 1, 0, 16, sp);
  if constexpr (kPerChannel) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) f[h][j][r] = pk[h][j][r];
  }

  // Two teams: each hands the half of the rows that it does not store (the upper
  // blocks, if it is the second) to the other through LDS, and adds what it gets.
  if constexpr (KS == 2) {
    __syncthreads();
    float4* const xch = reinterpret_cast<float4*>(lds_all);
    constexpr int kWave = NB * 4 * 64;  // float4s per wave
    static_assert(2 * 2 * WMC * kWave * 16 <= KS * 2 * S::STAGE, "the exchange fits");
    auto give = [&](const float (&x)[NB][16]) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; r += 4)
          xch[(team * 2 * WMC + wave) * kWave + (j * 4 + r / 4) * 64 + lane] =
              make_float4(x[j][r], x[j][r + 1], x[j][r + 2], x[j][r + 3]);
    };
    auto take = [&](float (&x)[NB][16]) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
          const float4 o =
              xch[((team ^ 1) * 2 * WMC + wave) * kWave + (j * 4 + r / 4) * 64 + lane];
          x[j][r] += o.x;
          x[j][r + 1] += o.y;
          x[j][r + 2] += o.z;
          x[j][r + 3] += o.w;
        }
    };
    if (team == 0) give(f[1]); else give(f[0]);
    __syncthreads();
    if (team == 0) take(f[0]); else take(f[1]);
  }

  // The products are in units of 1/64, and out_scale also undoes the 16 x 16 of
  // the int8 kernels' operands: 2^6 * 2^8, exact.
  const float inv = out_scale * 16384.0f;
  float4 ar4[2][4];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      ar4[h][k] = *reinterpret_cast<const float4*>(&scale_tab[row_of(h, 4 * k)]);
  auto store = [&](auto full) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int col = n0 + col_of(j);
      const float bc = scale_tab[BM + col_of(j)];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if (KS == 2 && h != team) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + row_of(h, r);
          const float4 a4 = ar4[h][r >> 2];
          const float ar = (r & 3) == 0 ? a4.x : (r & 3) == 1 ? a4.y : (r & 3) == 2 ? a4.z : a4.w;
          const uint16_t v =
              __builtin_bit_cast(uint16_t, (_Float16)((f[h][j][r] * (ar * inv)) * bc));
          if (decltype(full)::value || (row < M && col < N)) Y[(size_t)row * N + col] = v;
        }
      }
    }
  };
  if (m0 + BM <= M && n0 + BN <= N)
    store(std::true_type{});
  else
    store(std::false_type{});
}

// LDS of a tile: the stages, alpha of its rows then beta of its columns, the order.
template <int WMC, int KS, bool kGather>
struct Lds {
  __attribute__((aligned(16))) uint8_t stages[KS * 2 * Shape<WMC>::STAGE];
  __attribute__((aligned(16))) float scales[Shape<WMC>::BM + Shape<WMC>::BN];
  int order[kGather ? 16384 / kReorderBlock : 1];
};

template <int GS, int WMC, int KS, bool kPerChannel, bool kGather, bool kTiled>
__global__ __launch_bounds__(128 * WMC * KS, 2) void gemm_fp6_kernel(
    const uint8_t* __restrict__ Xe, const float* __restrict__ a_scale,
    const float* __restrict__ s_group, const uint8_t* __restrict__ Wq,
    const float* __restrict__ w_scale, int M, int N, int K, uint16_t* __restrict__ Y,
    float out_scale, const int32_t* __restrict__ border) {
  __shared__ Lds<WMC, KS, kGather> lds;
  const int w = blockIdx.x;
  const TileMap tile = map_tile<Shape<WMC>::BM, Shape<WMC>::BN>(M, N, w, w >> 3);
  if (!tile.valid) return;
  gemm_fp6_tile<GS, WMC, KS, kPerChannel, kGather, kTiled>(
      tile, lds.stages, lds.scales, lds.order, Xe, a_scale, s_group, Wq, w_scale, M, N, K, Y,
      out_scale, border);
}

// Tiles of 256 x 128 whose last round would leave half of the compute units or more
// idle: the tiles of the full rounds (workgroups below `full`) as above, each tile after
// them as two of 128 x 128 with two teams, which a compute unit finishes in about 0.7 of
// the time. Quantizer and GEMM, before -> now: 1500 x 4096 x 12288 (576 tiles) 96.3 -> 88.4
// us, per-channel 84.6 -> 78.5; 2500 x 8192 x 8192, g = 512 (640) 202 -> 190; 2560 x 4096 x
// 8192, g = 64 (640) 121.8 -> 111.5; 1024 x 4096 x 8704 / 10240 / 11264 (272 / 320 / 352)
// 65.4 / 64.0 / 62.9 -> 63.2 / 61.4 / 60.9.
template <int GS, bool kPerChannel, bool kGather, bool kTiled>
__global__ __launch_bounds__(512, 2) void gemm_fp6_tail_kernel(
    const uint8_t* __restrict__ Xe, const float* __restrict__ a_scale,
    const float* __restrict__ s_group, const uint8_t* __restrict__ Wq,
    const float* __restrict__ w_scale, int M, int N, int K, uint16_t* __restrict__ Y,
    float out_scale, const int32_t* __restrict__ border, int full) {
  __shared__ union {
    Lds<4, 1, kGather> whole;
    Lds<2, 2, kGather> half;
  } lds;
  const int w = blockIdx.x;
  if (w < full) {
    const TileMap tile = map_tile<256, 128>(M, N, w, w >> 3);
    if (!tile.valid) return;
    gemm_fp6_tile<GS, 4, 1, kPerChannel, kGather, kTiled>(
        tile, lds.whole.stages, lds.whole.scales, lds.whole.order, Xe, a_scale, s_group, Wq,
        w_scale, M, N, K, Y, out_scale, border);
  } else {
    const int u = (w - full) >> 3;
    TileMap tile = map_tile<256, 128>(M, N, w, (full >> 3) + (u >> 1));
    tile.m0 += (u & 1) * 128;
    if (!tile.valid || tile.m0 >= M) return;
    gemm_fp6_tile<GS, 2, 2, kPerChannel, kGather, kTiled>(
        tile, lds.half.stages, lds.half.scales, lds.half.order, Xe, a_scale, s_group, Wq,
        w_scale, M, N, K, Y, out_scale, border);
  }
}

// Tiles of 256 x 128 per XCD, and those of them after its full rounds of 32 where they
// are split in halves: at most 16, so that the halves take one round; K as split_teams.
struct TailSplit {
  int per, tail;
};
TailSplit tail_split(int M, int N, int K) {
  const long T = (long)((M + 255) / 256) * ((N + 127) / 128);
  const int per = (int)((T + 7) / 8);
  const int rest = per % 32;
  return {per, per > 32 && rest <= 16 && K >= 2048 ? rest : 0};
}

template <int WMC, int KS, bool kPerChannel, bool kGather, bool kTiled>
hipError_t launch_gemm(bool tail, const uint8_t* Xe, const float* a_scale, const float* s_group,
                       const uint8_t* Wq, const float* w_scale, int M, int N, int K, int g,
                       uint16_t* Y, float out_scale, hipStream_t stream, const int32_t* border) {
  using S = Shape<WMC>;
  const int T = ((M + S::BM - 1) / S::BM) * ((N + S::BN - 1) / S::BN);
  const int grid = 8 * ((T + 7) / 8);
  const TailSplit sp = tail ? tail_split(M, N, K) : TailSplit{0, 0};
  const int full = 8 * (sp.per - sp.tail);
  auto run = [&](auto gs) {
    constexpr int GS = decltype(gs)::value;
    if constexpr (WMC == 4)
      if (sp.tail) {
        gemm_fp6_tail_kernel<GS, kPerChannel, kGather, kTiled>
            <<<full + 16 * sp.tail, 512, 0, stream>>>(Xe, a_scale, s_group, Wq, w_scale, M, N, K, Y,
                                                      out_scale, border, full);
        return;
      }
    gemm_fp6_kernel<GS, WMC, KS, kPerChannel, kGather, kTiled>
        <<<grid, KS * S::kThreads, 0, stream>>>(Xe, a_scale, s_group, Wq, w_scale, M, N, K, Y,
                                                out_scale, border);
  };
  if constexpr (kPerChannel) {
    run(std::integral_constant<int, 4>{});
  } else {
    switch (g) {
      case 64: run(std::integral_constant<int, 2>{}); break;
      case 128: run(std::integral_constant<int, 4>{}); break;
      case 256: run(std::integral_constant<int, 8>{}); break;
      case 512: run(std::integral_constant<int, 16>{}); break;
      default: return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

// At most 256 tiles of 128 x 128: one per compute unit, whose two waves per SIMD
// then are two teams, each over half of K. A compute unit with one team per tile ran
// one wave per SIMD. GEMM with the token pass, one team / two: 512 x 8192 x 8192
// 47.5 -> 38.7 us; 777 x 16384 x 4096, g = 256 76 -> 63; 1000 x 4096 x 4096, g = 64
// 36 -> 28; 512 x 2048 x 8192 17.0 -> 15.5; at K = 1024 12.2 both. With more tiles
// the teams only share one barrier that two workgroups would not (2048 x 4096 x
// 12288 98 -> 108).
bool split_teams(int M, int N, int K) {
  return (long)((M + 127) / 128) * ((N + 127) / 128) <= 256 && K >= 2048;
}

// Otherwise 256 x 128 or 128 x 128 (also instead of a tail of halves), by the time of
// one K tile of 128 for the whole product, in ns: a round of 256 tiles of 256 x 128 takes
// 780, one of 512 tiles of 128 x 128 (two per compute unit) 890, a last round of up to
// 256 of those (one per unit) 620, a tail of halves 520 and 14 for each of an XCD's tiles
// (at 16, 1024 x 4096 x 12288, the 128 x 128 tiles stay: per-channel 54.4 us, with the
// tail 57). Measured: 2048 x K x 12288 (768 / 1536 tiles) 2.34 / 2.67 us per K tile,
// 512 x 8192 x 8192 (128 / 256 tiles, one team each) 51.7 / 45 us in all.
bool small_tiles(int M, int N, int K) {
  const long tn = (N + 127) / 128;
  const long t256 = (long)((M + 255) / 256) * tn, t128 = (long)((M + 127) / 128) * tn;
  const TailSplit sp = tail_split(M, N, K);
  const long large = sp.tail ? (sp.per - sp.tail) / 32 * 780 + 520 + 14 * sp.tail
                             : (t256 + 255) / 256 * 780;
  const long rest = t128 % 512;
  return t128 / 512 * 890 + (rest == 0 ? 0 : rest <= 256 ? 620 : 890) < large;
}

}  // namespace

// Where the main kernel would serve; with two teams also from 512 tiles of 64 x 64 of
// the mid-size kernel on (mid-size -> this one, weights in the caches, token pass
// included: 256 x 8192 x 8192, 512 tiles, 33 us both; 640 tiles: 320 x 4096 x 8192 26 ->
// 22, 128 x 4096 x 20480 27 -> 21; 768 tiles: 384 x 8192 x 8192 46 -> 34, 768 x 16384 x 4096 87 ->
// 60; below: 384 x 4096 x 4096, 384 tiles, 18.5 -> 20.7). The scratch stays below
// 1 GB.
size_t fp6_scratch_bytes(int M, int N, int K) {
  if (M <= 16) return 0;
  const long tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64);
  if (mid_kernel_fits(M, N) && !(split_teams(M, N, K) && tiles64 > 512)) return 0;
  const size_t n = expanded_bytes(M, K);
  return n <= ((size_t)1 << 30) ? n : 0;
}

GemmPath fp6_form(int M, int N, int K) {
  if (split_teams(M, N, K)) return GemmPath::kFp6Teams;
  if (small_tiles(M, N, K)) return GemmPath::kFp6Small;
  return tail_split(M, N, K).tail ? GemmPath::kFp6Tail : GemmPath::kFp6Large;
}

hipError_t launch_w4a4_gemm_fp6(GemmPath path, const uint8_t* Xq, const float* a_scale, const float* s_group,
                                const uint8_t* Wq, const float* w_scale, const int32_t* border,
                                int M, int N, int K, int g, uint16_t* Y, float out_scale,
                                void* scratch, hipStream_t stream, WqLayout lay) {
  uint8_t* Xe = static_cast<uint8_t*>(scratch);
  const unsigned groups = (unsigned)(token_blocks(M) * (size_t)(K / 128) / 2);  // K / 128 is even
  expand_tokens_kernel<<<groups, 256, 0, stream>>>(Xq, M, K, Xe);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const bool teams = path == GemmPath::kFp6Teams, small = path == GemmPath::kFp6Small;
  const bool tail = path == GemmPath::kFp6Tail;
#define RRS_ARGS \
  tail, Xe, a_scale, s_group, Wq, w_scale, M, N, K, g, Y, out_scale, stream, border
#define RRS_LAY(WMC_, KS_, PC_, GA_)                                       \
  (lay.tiled ? launch_gemm<WMC_, KS_, PC_, GA_, true>(RRS_ARGS)            \
             : launch_gemm<WMC_, KS_, PC_, GA_, false>(RRS_ARGS))
#define RRS_FORM(PC_, GA_)                                                 \
  return teams   ? RRS_LAY(2, 2, PC_, GA_)                                 \
         : small ? RRS_LAY(2, 1, PC_, GA_)                                 \
                 : RRS_LAY(4, 1, PC_, GA_)
  if (!s_group) RRS_FORM(true, false);
  if (border) RRS_FORM(false, true);
  RRS_FORM(false, false);
#undef RRS_FORM
#undef RRS_LAY
#undef RRS_ARGS
}

}  // namespace rrs
