// Which kernel a GEMM call takes: host code only, a function of the call's sizes,
// options and scratch, used by every entry point and by the query of the tests.
//
// Times below are the GEMM in graph replays, weights cold, in us.
#include "rrs_internal.h"

namespace rrs {
namespace {

// 17 to 32 tokens at K = 8192: the eight-wave weight stream reads whole rows of
// 512 bytes per wave, where the mid-size kernel's loads take 64 bytes of each of 16
// rows. Row-major it is ahead (stream / mid, 32 tokens, g = 128: N = 1024 8.1 / 11.6,
// 12288 16.5 / 18.4, 28672 29.9 / 36.0; the two tie at N = 16384). With the tiled layout both read
// contiguous tiles: it is ahead where there are few columns, g = 512 (the mid-size
// kernel then converts its sums) or the second block of tokens nearly empty.
bool stream_wide(const GemmCall& c) {
  if (c.M > 32 || c.K != 8192) return false;
  if (!c.tiled) return true;
  if (c.g == 512) return c.N <= 4096 || c.N >= 10240 || c.M <= 20;
  return c.N <= 4096 && (c.g == 128 || c.M <= 24);
}

// 17 to 64 tokens, long groups, from the width on where the mid-size kernel's tiles
// are 32 tokens and more (160 tiles of columns): a wave of the few-token kernel reads
// a group of a row at once, 128 or 256 bytes, and the mid-size kernel 64. Few-token /
// mid, row-major, g = 256, N = 12288: 32 x 4096 9.7 / 10.5, 32 x 16384 28.4 / 34.7, 64 x
// 16384 38.0 / 42.7; g = 512, tiled, 32 x 16384 x 20480 46.5 / 47.8. With two groups of
// 64 per wave (K = 512) the mid-size kernel's prologue and sum are all there is: 64 x
// 512 x 20480 9.1 / 11.4.
bool decode_wide(const GemmCall& c) {
  if (!decode_wide_fits(c.M, c.K, c.g, c.tiled) || c.N <= 64 * 159) return false;
  if (c.K == 512) return c.g == 64;
  if (c.K == 16384) return true;
  if (c.tiled || c.M > 32) return false;
  return c.K == 4096 || (c.K == 2048 && c.N > 64 * 191);
}

}  // namespace

GemmPath gemm_path(const GemmCall& c, bool scratch) {
  if (c.M <= 16) {
    // The per-channel scheme has no few-token kernel of its own, and the main
    // kernel's 256-row tiles took 35 us at K = N = 4096 whatever M is.
    if (c.per_channel) return GemmPath::kMid;
    if (c.reorder)
      return stream_gather_fits(c.M, c.K) ? GemmPath::kStreamGather : GemmPath::kDecodeGather;
    return stream_kernel_fits(c.M, c.K, c.g) ? GemmPath::kStream : GemmPath::kDecode;
  }
  if (!c.per_channel && !c.reorder) {
    if (stream_wide(c)) return GemmPath::kStream;
    if (decode_wide(c)) return GemmPath::kDecode;
  }
  const bool mid = mid_kernel_fits(c.M, c.N);
  // Without the rescale the mid-size kernel stays ahead where it fits (300 x 8192 x
  // 8192: 33 against 35.5 us).
  if (scratch && fp6_scratch_bytes(c.M, c.N, c.K) && !(c.per_channel && mid))
    return fp6_form(c.M, c.N, c.K);
  return mid ? GemmPath::kMid : GemmPath::kMain;
}

const char* gemm_path_name(GemmPath p) {
  switch (p) {
    case GemmPath::kStream: return "stream";
    case GemmPath::kStreamGather: return "stream_gather";
    case GemmPath::kDecode: return "decode";
    case GemmPath::kDecodeGather: return "decode_gather";
    case GemmPath::kMid: return "mid";
    case GemmPath::kMain: return "main";
    case GemmPath::kFp6Teams: return "fp6_teams";
    case GemmPath::kFp6Small: return "fp6_small";
    case GemmPath::kFp6Large: return "fp6_large";
    case GemmPath::kFp6Tail: return "fp6_tail";
  }
  return "";
}

}  // namespace rrs
