// INT4 codes as 6-bit floats for v_mfma_f32_32x32x64_f8f6f4 (E2M3 on both
// sides), which multiplies at twice the rate of the int8 instruction.
//
// E2M3 is linear up to 15 / 8: a field whose low four bits are the magnitude m and
// whose top bit is the sign holds +-m / 8. Tokens are stored that way
// (expand_tokens_kernel). Weights take the cheaper form, two's complement with
// the top bit flipped, that is u = q + 8 as the magnitude: four bits moved and
// one xor per code, for every q in [-8, 7]. The products then carry the offset:
//   sum q_x q_w = sum q_x u_w - 8 sum q_x
// (sums over the same channels); the last term, the same for all columns, is the
// accumulators' start value. Everything is exact: products are multiples of
// 1/64 and sums stay below 2^24 of these (per-channel: |sum| <= 64 * 16384, and
// a running sum exceeds it by at most one tile's offset).
#pragma once

#include "rrs_internal.h"

namespace rrs {
namespace fp6 {

typedef int v6i __attribute__((ext_vector_type(6)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// The flip of each field's top bit, per dword of a 96-bit run of 16 fields.
// Kept in registers (a VOP3 instruction reads at most one scalar register).
struct Flip {
  uint32_t k0, k1, k2;
};
__device__ __forceinline__ Flip make_flip() {
  Flip f{0x08208208u, 0x82082082u, 0x20820820u};
  asm volatile("" : "+v"(f.k0), "+v"(f.k1), "+v"(f.k2));
  return f;
}

// (a & b) ^ c and a ^ (b & c), one instruction each.
__device__ __forceinline__ uint32_t and_xor(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x6A);
}
__device__ __forceinline__ uint32_t xor_and(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x78);
}

// 16 codes (x0, x1) -> 96 bits of fields (d0, d1, d2): eight instructions.
// Nibbles 0, 3, 6 keep or shift by 2 into fields 12 bits apart, and so do
// 1, 4, 7 and 2, 5, so each output dword takes one unshifted and one shifted
// dword under a mask; the one field that straddles d0 and d1 is nibble 7 of x0,
// whose top half the funnel shift brings in. The order of the fields is the
// same for both operands, so every dot product is unchanged.
__device__ __forceinline__ void spread16(uint32_t x0, uint32_t x1, const Flip& f, uint32_t& d0,
                                         uint32_t& d1, uint32_t& d2) {
  const uint32_t a = x0 << 2;
  const uint32_t b = __builtin_amdgcn_alignbit(x1, x0, 30);  // x1 << 2 | x0 >> 30
  d0 = xor_and(and_xor(a, 0xC03C03C0u, f.k0), x0, 0x0F00F00Fu);
  d1 = xor_and(and_xor(b, 0x03C03C03u, f.k1), x1, 0xF00F00F0u);
  d2 = xor_and(and_xor(b, 0x3C03C03Cu, f.k2), x0, 0x00F00F00u);
}

// Token rows in MFMA operand order (expand_tokens_kernel writes it, the GEMM
// reads it): for each block of 32 rows and each tile of 128 channels 3072
// bytes, four sections of 32 rows x 16 bytes (dwords 0-3 of a row's six for
// channels [32 q, 32 q + 32)), then four of 32 rows x 8 bytes (dwords 4-5);
// after all tiles, for each block and tile 32 words of two f16, -1/8 of the
// row's code sums over the tile's two 64-channel steps.
constexpr int kTokTile = 3072;
constexpr int kTokSum = 128;
inline __host__ __device__ size_t token_blocks(int M) { return ((size_t)M + 31) / 32; }
inline __host__ __device__ size_t expanded_bytes(int M, int K) {
  return token_blocks(M) * (size_t)(K / 128) * (kTokTile + kTokSum);
}

// D = A B + C over 64 channels, both operands E2M3; the operands take six
// registers each (the builtin's last two elements are not read).
__device__ __forceinline__ v16f mfma64(const v6i& a, const v6i& b, const v16f& c) {
  const v8i a8 = __builtin_shufflevector(a, a, 0, 1, 2, 3, 4, 5, -1, -1);
  const v8i b8 = __builtin_shufflevector(b, b, 0, 1, 2, 3, 4, 5, -1, -1);
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 2, 2, 0, 0, 0, 0);
}

}  // namespace fp6
}  // namespace rrs
