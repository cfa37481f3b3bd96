// W4A4 GEMM with Runtime Smooth for 17 to a few hundred tokens, the same product
// as the main kernel (Section 3.2, Eq. 3, Fig. 4 step (3)):
//   Y[i, n] = fp16( alpha_i * beta_n / K * sum_b s_b * P_b[i, n] )
//   P_b[i, n] = sum_{j in group b} qx[i, j] * qw[j, n]   (exact int32)
//
// What bounds these calls: the main kernel's 256 x 128 tiles are too few to
// fill 256 compute units (173 tokens at N = 4096: 32 tiles), and each tile
// walks all of K behind a barrier per 128 channels, about 1 us each, however
// little it has to do. Here a tile is 16, 32 or 64 tokens x 64 columns and the
// four waves of a workgroup split K between them (wave w takes the tiles of
// 128 channels, or the groups where those are longer, w, w + 4, ...), so K
// is walked four times faster, nothing is staged in LDS and no barrier stands
// in the loop; the waves' fp32 sums are added at the end in a fixed order
// through LDS. Operands go from global memory (token codes: from L2) to registers
// two K tiles ahead: lane (r, q) takes 16 bytes of each row, quarter q of the
// tile's 64, so a load instruction reads 16 rows x 64 bytes (one contiguous
// 1 KB with the tiled Wq), and two v_mfma_i32_16x16x64_i8 use them. For g = 64
// the lane takes two pieces of 8 bytes, an eighth of each group's 32, so that
// every product stays inside one group.
//
// Measured in graph replays, cold weights, g = 128, row-major (tiled), the main kernel ->
// this one: 173 x 4096 x 4096 (M x K x N) 34.5 -> 10.9 us (34.4 -> 8.9); 300 x 8192 x 1024
// 62.3 -> 13.5 (62.3 -> 10.2); 128 x 8192 x 8192 63.8 -> 21.6 (63.7 -> 16.4); 100 x 4096 x
// 12288 35.9 -> 19.2 (35.4 -> 15.1); the few-token kernel -> this one: 64 x 4096 x 4096
// 12.0 -> 7.1 (10.9 -> 5.4); 49 x 4096 x 22016 24.3 -> 20.7 (21.3 -> 16.8); 64 x 8192 x
// 28672 48.4 -> 44.4 (38.8 -> 35.4); not at K = 8192 with 17 to 32 tokens, row-major (32 x
// 8192 x 28672 30.4 on the weight stream, 35.8 here: 64 bytes of each of 16 rows per load).
// At 173 x 4096 x 4096 a wave issues in half of its clocks; four waves beat eight on one
// tile (11.8 against 12.4 us: the sum of eight takes longer), loads four tiles ahead are
// slower even with registers for them (12.5 us at one workgroup per compute unit), and so
// are tiles of 32 columns (16.0: the tokens are read twice as often). The last trip's loads
// past the end cost 6 to 12 % and are left out.
//
// Codes are unpacked into the high nibble of each int8 lane (16 q), the 2^-8
// folded into the output scale, and a group's accumulators start from the bits
// of 1.5 * 2^23 (g <= 256), so that the int32 result read as a float is exactly
// 1.5 * 2^23 + 256 P and one subtraction recovers 256 P; for g = 512 they start
// from 0 and are converted. The per-channel scheme (Section 2.1) is the same
// loop with every group scale 1: the sums stay multiples of 256 below 2^32, so
// fp32 holds them exactly.
#include "rrs_stream.h"

namespace rrs {
namespace {

using stream::unpack_pair;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int NW = 4;          // waves per workgroup, each with its share of K
constexpr int DB = 2;          // K tiles in flight
constexpr int kCB = 4;         // blocks of 16 columns per tile
constexpr int BN = 16 * kCB;
constexpr int kRedStride = BN + 4;
constexpr int kMagic = 0x4B400000;  // bits of 1.5 * 2^23

// fp16(a0 b0) and fp16(a1 b1) in one register, with one rounding each, as every other kernel
// stores: the compiler folds their conversion into the product, but not where two halves are
// packed. (Packed by shifts and or: 173 x 4096 x 4096 10.85 us, so 10.72.)
__device__ __forceinline__ uint32_t halves_once(float a0, float b0, float a1, float b1) {
  uint32_t h;
  asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(h) : "v"(a0), "v"(b0));
  asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(h) : "v"(a1), "v"(b1));
  return h;
}

enum Mode { kSmooth, kPerChannel, kPartials };

// GS = g / 32; RB blocks of 16 tokens. kGather (runtime channel reorder):
// position block p of Xq pairs with block border[p] of every Wq row. kEighths: wave w
// takes the contiguous eighths 2 w and 2 w + 1 of K instead, and the eight sums are
// added in their order, which is the eight-wave weight stream's: the same bits.
template <int GS, int RB, Mode mode, bool kGather, bool kTiled, bool kEighths>
__global__ __launch_bounds__(64 * NW, 2) void gemm_mid_kernel(
    const uint8_t* __restrict__ Xq, const float* __restrict__ a_scale,
    const float* __restrict__ s_group, const uint8_t* __restrict__ Wq,
    const float* __restrict__ w_scale, int M, int N, int K, uint16_t* __restrict__ Y,
    int32_t* __restrict__ P, float out_scale, const int32_t* __restrict__ border) {
  constexpr WqLayout lay{kTiled};
  constexpr int BM = 16 * RB;
  constexpr int TPG = GS > 4 ? GS / 4 : 1;  // K tiles of 128 per group
  constexpr int kParts = kEighths ? 2 * NW : NW;
  __shared__ __attribute__((aligned(16))) float red[kParts * BM * kRedStride];
  __shared__ int btab[kGather ? 16384 / kReorderBlock : 1];

  const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
  const int T = tm * tn, per = (T + 7) >> 3;
  const int lin = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
  if (lin >= T) return;
  const int m0 = lin % tm * BM, n0 = lin / tm * BN;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 15, q = lane >> 4;
  const int ng = K / (128 * TPG);  // runs of whole groups, dealt to the waves in turn
  const int n = wave < ng ? TPG * ((ng - wave + NW - 1) / NW) : 0;
  auto tile_of = [&](int i) {
    i = min(i, max(n - 1, 0));
    if constexpr (kEighths) return wave * n + i;  // n = K / 512
    return min((wave + i / TPG * NW) * TPG + i % TPG, K / 128 - 1);
  };

  if constexpr (kGather) {
    for (int i = t; i < K / kReorderBlock; i += 64 * NW)
      btab[i] = border[i] & (K / kReorderBlock - 1);
    __syncthreads();
  }

  // Row offsets from the tile's first row; the bases stay in scalar registers.
  const uint8_t* abase = Xq + (size_t)m0 * (K / 2);
  const uint8_t* bbase = Wq + lay.row(n0, K);
  uint32_t pa[RB], pb[kCB];
#pragma unroll
  for (int i = 0; i < RB; ++i) pa[i] = (uint32_t)(min(16 * i + r, M - 1 - m0) * (K / 2));
#pragma unroll
  for (int j = 0; j < kCB; ++j)
    pb[j] = (uint32_t)(lay.row(min(n0 + 16 * j + r, N - 1), K) - lay.row(n0, K));
  typedef const __attribute__((address_space(1))) uint8_t* gbytes;

  // A lane holds 16 bytes of each row per K tile: for groups of 128 and more the
  // quarter q of the 64, for groups of 64 an eighth of each group's 32 bytes, so
  // that every product of depth 64 stays in one group.
  v4u ra[DB][RB], rb[DB][kCB];
  auto woff = [&](int p) -> uint32_t {  // byte offset of piece p in a weight row
    if constexpr (kGather) p = btab[p];
    return (uint32_t)((p >> 2) * lay.tile() + (p & 3) * lay.quarter());
  };
  auto ld16 = [](const uint8_t* base, uint32_t o) {
    gbytes g = (gbytes)(uintptr_t)base;
    asm volatile("" : "+s"(g), "+v"(o));
    const v4u v = *(const __attribute__((address_space(1))) v4u*)(g + o);
    return v;
  };
  auto ld8 = [](const uint8_t* base, uint32_t o) {
    gbytes g = (gbytes)(uintptr_t)base;
    asm volatile("" : "+s"(g), "+v"(o));
    const v2u v = *(const __attribute__((address_space(1))) v2u*)(g + o);
    return v;
  };
  auto load_a = [&](int set, int i) {
    const int kt = tile_of(i);
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      if constexpr (GS >= 4) {
        ra[set][k] = ld16(abase + kt * 64, pa[k] + q * 16);
      } else {
        const v2u x = ld8(abase + kt * 64, pa[k] + q * 8);
        const v2u y = ld8(abase + kt * 64 + 32, pa[k] + q * 8);
        ra[set][k] = v4u{x[0], x[1], y[0], y[1]};
      }
    }
  };
  auto load_b = [&](int set, int i) {
    const int kt = tile_of(i);
    const uint8_t* bk = kGather ? bbase : bbase + (size_t)kt * lay.tile();
    auto wo = [&](int p) { return kGather ? woff(kt * 4 + p) : (uint32_t)(p * lay.quarter()); };
    if constexpr (GS >= 4) {
      const uint32_t o = wo(q);
#pragma unroll
      for (int k = 0; k < kCB; ++k) rb[set][k] = ld16(bk, pb[k] + o);
    } else {
      const uint32_t o0 = wo(q >> 1) + (q & 1) * 8, o1 = wo(2 + (q >> 1)) + (q & 1) * 8;
#pragma unroll
      for (int k = 0; k < kCB; ++k) {
        const v2u x = ld8(bk, pb[k] + o0), y = ld8(bk, pb[k] + o1);
        rb[set][k] = v4u{x[0], x[1], y[0], y[1]};
      }
    }
  };

  v4f f[RB][kCB];
  constexpr bool kZeroSeed = GS > 8;
  constexpr int kSeed = kZeroSeed ? 0 : kMagic;
  const v4i seed = {kSeed, kSeed, kSeed, kSeed};
  v4i acc[RB][kCB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < kCB; ++j) {
      f[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
      acc[i][j] = seed;
    }

  auto rescale = [&](const v4i& c, int i, int j, float s, int grp, bool live) {
    if constexpr (mode == kPartials) {
      int32_t* Pg = P + (size_t)grp * (size_t)M * (size_t)N;
      const int col = n0 + 16 * j + r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = m0 + 16 * i + 4 * q + e;
        if (live && row < M && col < N) Pg[(size_t)row * N + col] = (c[e] - kSeed) >> 8;
      }
    } else {
      const v4f cf = __builtin_bit_cast(v4f, c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float pv = kZeroSeed ? (float)c[e] : cf[e] - 12582912.0f;
        f[i][j][e] = __builtin_fmaf(s, pv, f[i][j][e]);
      }
    }
  };
  // Step u of the unrolled trip: a trip starts with a group.
  auto compute = [&](int u, int i) {
    const int set = u % DB;
    const int kt = tile_of(i);
    const bool live = i < n;
    const int grp = GS >= 4 ? kt / TPG : kt * 2;
    float s0 = 0.0f, s1 = 0.0f;
    if constexpr (mode == kPerChannel) {
      s0 = s1 = live ? 1.0f : 0.0f;
    } else if constexpr (mode == kSmooth) {
      s0 = live ? s_group[grp] : 0.0f;
      if constexpr (GS < 4) s1 = live ? s_group[grp + 1] : 0.0f;
    }
    v4i a[RB][2];
#pragma unroll
    for (int k = 0; k < RB; ++k) {
      a[k][0] = unpack_pair(ra[set][k][0], ra[set][k][1]);
      a[k][1] = unpack_pair(ra[set][k][2], ra[set][k][3]);
    }
#pragma unroll
    for (int j = 0; j < kCB; ++j) {
      const v4i b0 = unpack_pair(rb[set][j][0], rb[set][j][1]);
      const v4i b1 = unpack_pair(rb[set][j][2], rb[set][j][3]);
      if constexpr (GS >= 4) {
        const bool first = u % TPG == 0, last = u % TPG == TPG - 1;
#pragma unroll
        for (int k = 0; k < RB; ++k)
          acc[k][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][0], b0, first ? seed : acc[k][j], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < RB; ++k)
          acc[k][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][1], b1, acc[k][j], 0, 0, 0);
        if (last) {
#pragma unroll
          for (int k = 0; k < RB; ++k) rescale(acc[k][j], k, j, s0, grp, live);
        }
      } else {
        v4i c[RB];
#pragma unroll
        for (int k = 0; k < RB; ++k)
          c[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][0], b0, seed, 0, 0, 0);
#pragma unroll
        for (int k = 0; k < RB; ++k) rescale(c[k], k, j, s0, grp, live);
#pragma unroll
        for (int k = 0; k < RB; ++k)
          c[k] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[k][1], b1, seed, 0, 0, 0);
#pragma unroll
        for (int k = 0; k < RB; ++k) rescale(c[k], k, j, s1, grp + 1, live);
      }
    }
  };

#pragma unroll
  for (int d = 0; d < DB; ++d) {
    load_b(d, d);
    load_a(d, d);
  }
  auto put = [&](int part) {  // a wave's sums to LDS
    float* mine = red + part * BM * kRedStride;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < kCB; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[(16 * i + 4 * q + e) * kRedStride + 16 * j + r] = f[i][j][e];
  };
  // Trips of U tiles; the last one requests nothing past itself. Tiles past a
  // wave's last repeat it and count with scale 0.
  constexpr int U = TPG > DB ? TPG : DB;
  int i0 = 0;
  for (; i0 + U < n; i0 += U) {
    if constexpr (kEighths) {
      if (i0 == n / 2) {  // a trip's start: n is a multiple of 2 U
        put(2 * wave);
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int j = 0; j < kCB; ++j) f[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      compute(u, i0 + u);
      load_b(u % DB, i0 + u + DB);
      load_a(u % DB, i0 + u + DB);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (n > 0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      compute(u, i0 + u);
      if (u + DB < U) {
        load_b(u % DB, i0 + u + DB);
        load_a(u % DB, i0 + u + DB);
      }
    }
  }
  if constexpr (mode == kPartials) return;

  // The waves' sums are added in a fixed order through LDS.
  put(kEighths ? 2 * wave + 1 : wave);
  __syncthreads();
  constexpr int kPieces = BM * BN / 4;
#pragma unroll
  for (int p = t; p < kPieces; p += 64 * NW) {
    const int row = p >> 4, c4 = (p & 15) * 4;
    v4f sum = *reinterpret_cast<const v4f*>(red + row * kRedStride + c4);
#pragma unroll
    for (int w = 1; w < kParts; ++w) sum += *reinterpret_cast<const v4f*>(red + (w * BM + row) * kRedStride + c4);
    const int gr = m0 + row, gc = n0 + c4;
    if (gr < M && gc < N) {
      const float sc = a_scale[gr] * out_scale;
      const v4f bc = *reinterpret_cast<const v4f*>(w_scale + gc);
      *reinterpret_cast<v2u*>(Y + (size_t)gr * N + gc) =
          v2u{halves_once(sum[0] * sc, bc[0], sum[1] * sc, bc[1]),
              halves_once(sum[2] * sc, bc[2], sum[3] * sc, bc[3])};
    }
  }
}

template <int GS, int RB, Mode mode, bool kGather, bool kTiled, bool kEighths = false>
hipError_t launch(const uint8_t* Xq, const float* a_scale, const float* s_group,
                  const uint8_t* Wq, const float* w_scale, int M, int N, int K, uint16_t* Y,
                  int32_t* P, float out_scale, hipStream_t stream, const int32_t* border) {
  const int T = ((M + 16 * RB - 1) / (16 * RB)) * ((N + BN - 1) / BN);
  gemm_mid_kernel<GS, RB, mode, kGather, kTiled, kEighths><<<8 * ((T + 7) / 8), 64 * NW, 0, stream>>>(
      Xq, a_scale, s_group, Wq, w_scale, M, N, K, Y, P, out_scale, border);
  return hipGetLastError();
}

}  // namespace

// Token blocks per tile: the smaller tile while its workgroups fit one to a compute
// unit (a second pass over the weights, out of L2, then costs less than idle units); past
// 256 it takes a second round, and the larger tile is ahead although half of the units
// idle. Measured, row-major, 16 / 32 / 64 tokens per tile (workgroups): 64 x 4096 x 4096
// 7.1 / 8.1 / 10.5 us (256 / 128 / 64); 32 x 16384 x 4096 20.8 / 24.2 (128 / 64); 300 x 8192
// x 1024 20.0 / 13.2 / 17.2 (304 / 160 / 80); 28 x 4096 x 9168, g = 256 13.4 / 10.0 (288 /
// 144); 22 x 16384 x 9440, g = 64 72.9 / 42.4 (296 / 148); 61 x 8192 x 4688, g = 256 22.8 /
// 15.9 / 20.7 (296 / 148 / 74); 49 x 8192 x 9104, g = 64 55.2 / 45.5 / 29.9 (572 / 286 /
// 143). Up to K = 1024 with the tiled layout there is too little work for that below 160
// large tiles (32 x 1024 x 8624 4.4 / 4.8; 58 x 1024 x 8944 with 32 or 64 tokens 4.8 / 5.2).
int mid_token_blocks(int M, int N, int K, bool tiled) {
  const long tn = (N + BN - 1) / BN;
  auto wgs = [&](int rb) { return (M + 16 * rb - 1) / (16 * rb) * tn; };
  for (int rb = 4; rb > 1; rb /= 2) {
    if (M <= 8 * rb) continue;  // half of the tile would be idle
    if (wgs(rb) >= 160 || (wgs(rb / 2) > 256 && !(tiled && K <= 1024))) return rb;
  }
  return 1;
}

namespace {

template <Mode mode, bool kGather, bool kTiled>
hipError_t launch_any(const uint8_t* Xq, const float* a_scale, const float* s_group,
                      const uint8_t* Wq, const float* w_scale, int M, int N, int K, int g,
                      uint16_t* Y, int32_t* P, float out_scale, hipStream_t stream,
                      const int32_t* border) {
  const int rb = mid_token_blocks(M, N, K, kTiled);
#define RRS_MID(GS_, RB_)                                                                       \
  launch<GS_, RB_, mode, kGather, kTiled>(Xq, a_scale, s_group, Wq, w_scale, M, N, K, Y, P, \
                                          out_scale, stream, border)
#define RRS_CASE(G_) \
  case G_:           \
    return rb == 4 ? RRS_MID(G_ / 32, 4) : rb == 2 ? RRS_MID(G_ / 32, 2) : RRS_MID(G_ / 32, 1)
  if constexpr (mode == kPerChannel) {
    return rb == 4 ? RRS_MID(4, 4) : rb == 2 ? RRS_MID(4, 2) : RRS_MID(4, 1);
  } else {
    switch (g) {
      RRS_CASE(64);
      RRS_CASE(128);
      RRS_CASE(256);
      RRS_CASE(512);
      default: return hipErrorInvalidValue;
    }
  }
#undef RRS_CASE
#undef RRS_MID
}

}  // namespace

// Against the main kernel's 256 x 128 tiles, one a compute unit: a tile of 64 x
// 64 costs about 1 us per 1000 K tiles of 128 over the whole chip, a round of
// 256 large ones 1 us per K tile. Measured, here / main: 512 x 8192 x 8192
// (1024 small tiles, one round) 63.1 / 64.4 us; 512 x 4096 x 12288 (1536, one
// round) 53.1 / 39.6; 256 x 4096 x 4096 (256, one round) 10.8 / 33.2.
bool mid_kernel_fits(int M, int N) {
  if (M <= 16) return false;
  const long small = (long)((M + 63) / 64) * ((N + 63) / 64);
  const long large = (long)((M + 255) / 256) * ((N + 127) / 128);
  return small <= 768 * ((large + 255) / 256);
}

hipError_t launch_w4a4_gemm_mid(const uint8_t* Xq, const float* a_scale, const float* s_group,
                                const uint8_t* Wq, const float* w_scale, const int32_t* border,
                                int M, int N, int K, int g, uint16_t* Y, float out_scale,
                                hipStream_t stream, WqLayout lay) {
  if (border)
    return lay.tiled ? launch_any<kSmooth, true, true>(Xq, a_scale, s_group, Wq, w_scale, M, N, K,
                                                       g, Y, nullptr, out_scale, stream, border)
                     : launch_any<kSmooth, true, false>(Xq, a_scale, s_group, Wq, w_scale, M, N, K,
                                                        g, Y, nullptr, out_scale, stream, border);
  return lay.tiled ? launch_any<kSmooth, false, true>(Xq, a_scale, s_group, Wq, w_scale, M, N, K, g,
                                                      Y, nullptr, out_scale, stream, nullptr)
                   : launch_any<kSmooth, false, false>(Xq, a_scale, s_group, Wq, w_scale, M, N, K,
                                                       g, Y, nullptr, out_scale, stream, nullptr);
}

hipError_t launch_w4a4_gemm_mid_eighths(const uint8_t* Xq, const float* a_scale,
                                        const float* s_group, const uint8_t* Wq,
                                        const float* w_scale, int M, int N, int K, int g,
                                        uint16_t* Y, float out_scale, hipStream_t stream) {
  if (K != 8192 || M > 32) return hipErrorInvalidValue;
  const int rb = mid_token_blocks(M, N, K, true);
#define RRS_MID(GS_, RB_)                                                                     \
  launch<GS_, RB_, kSmooth, false, true, true>(Xq, a_scale, s_group, Wq, w_scale, M, N, K, Y, \
                                               nullptr, out_scale, stream, nullptr)
  switch (g) {
    case 64: return rb == 2 ? RRS_MID(2, 2) : RRS_MID(2, 1);
    case 128: return rb == 2 ? RRS_MID(4, 2) : RRS_MID(4, 1);
    case 256: return rb == 2 ? RRS_MID(8, 2) : RRS_MID(8, 1);
    default: return hipErrorInvalidValue;
  }
#undef RRS_MID
}

hipError_t launch_w4a4_gemm_mid_per_channel(const uint8_t* Xq, const float* a_scale,
                                            const uint8_t* Wq, const float* w_scale, int M, int N,
                                            int K, uint16_t* Y, float out_scale,
                                            hipStream_t stream, WqLayout lay) {
  return lay.tiled ? launch_any<kPerChannel, false, true>(Xq, a_scale, nullptr, Wq, w_scale, M, N,
                                                          K, 128, Y, nullptr, out_scale, stream,
                                                          nullptr)
                   : launch_any<kPerChannel, false, false>(Xq, a_scale, nullptr, Wq, w_scale, M, N,
                                                           K, 128, Y, nullptr, out_scale, stream,
                                                           nullptr);
}

hipError_t launch_w4a4_gemm_mid_partials(const uint8_t* Xq, const uint8_t* Wq, int M, int N, int K,
                                         int g, int32_t* P, hipStream_t stream) {
  return launch_any<kPartials, false, false>(Xq, nullptr, nullptr, Wq, nullptr, M, N, K, g, nullptr,
                                             P, 0.0f, stream, nullptr);
}

}  // namespace rrs
