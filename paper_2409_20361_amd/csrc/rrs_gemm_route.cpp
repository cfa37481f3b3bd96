// Which kernel a GEMM call takes: host code only, a function of the call's sizes,
// options and scratch, used by every entry point and by the query of the tests.
//
// Times below are the GEMM in graph replays, weights cold, in us.
#include "rrs_internal.h"

namespace rrs {
namespace {

// Both layouts of the weights give the same bits, so a choice between kernels that add
// the groups' sums in different orders goes by sizes and options alone. (The main kernel
// and the 6-bit kernel's one-team forms add in the same order, and the per-channel scheme
// has no such sum.)

// 17 to 32 tokens at K = 8192: the eight-wave weight stream reads whole rows of
// 512 bytes per wave, where the mid-size kernel's row-major loads take 64 bytes of each of
// 16 rows. Stream / mid, 32 tokens, g = 128: N = 1024 8.1 / 11.6, 12288 16.5 / 18.4,
// 28672 29.9 / 36.0 (a tie at N = 16384). With the tiled layout both read contiguous tiles,
// and from some 6000 columns on the mid-size kernel is ahead (N = 28672 29.7 / 27.3; not
// with g = 512, whose sums it converts): its form by eighths of K, with the stream's bits.
bool stream_wide(const GemmCall& c) { return c.M <= 32 && c.K == 8192; }
bool mid_eighths(const GemmCall& c) { return c.tiled && c.N >= 6144 && c.g <= 256; }

// 17 to 64 tokens, long groups, from 160 tiles of columns on (129 at K = 512 and 16384, where
// the mid-size kernel's tiles grow; there not from 33 tokens on with g = 256, which the mid-size
// kernel multiplies faster with the tiled layout: 39 x 16384 x 9040 33.9 / 30.2): a wave of the
// few-token kernel reads a group of a row at once, 128 or 256 bytes, and the mid-size kernel
// 64. Few-token / mid, row-major, g = 256, N = 12288: 32 x 4096 9.7 / 10.5, 32 x 16384 28.4 /
// 34.7, 64 x 16384 38.0 / 42.7; g = 512, 29 x 16384 x 9040 27.3 / 31.1, 46 x 16384 x 9968 34.6
// / 37.4 (tiled between 5 % ahead and 13 % behind). With two groups of 64 per wave (K = 512)
// the mid-size kernel's prologue and sum are all there is: 64 x 512 x 20480 9.1 / 11.4, 49 x
// 512 x 9664 6.3 / 7.1. At K = 2048 the line is where the mean of both layouts turns.
bool decode_wide(const GemmCall& c) {
  const int columns = (c.N + 63) / 64;
  if (!decode_wide_fits(c.M, c.K, c.g)) return false;
  if (columns <= 128) return false;
  if (c.K == 512) return c.g == 64;
  if (c.K == 16384) return columns >= 160 || c.M <= 32 || c.g == 512;
  if (columns < 160) return false;
  if (c.M > 32) return false;
  return c.K == 4096 || (c.K == 2048 && columns >= (c.g == 512 ? 192 : 320));
}

// Time of a call in us (the launch that spreads the tokens included), to compare a
// path with the main kernel. A kernel works off its tiles in rounds over the compute
// units, `cap` tiles per XCD and round; a round takes a time per K tile of 128, by the
// group size (a column each for 64, 128, 256, 512 and per-channel), more with gathered
// row-major weights (pieces of 16 bytes) and, for the 6-bit paths, with the tiled layout
// (its 16-byte pieces are spread by other lanes). Output and token terms are per
// million elements. Fitted by least squares to 4000 calls with 65 to 8192 tokens, all of
// whose paths were measured: 4 to 8 % off (mid-size 13 %). With the comparison 76 of them
// are more than 2 % slower than the main kernel, without it 621, most of them with few
// columns or K up to 2048, where the token launch costs more than 6-bit operands
// save: 4096 x 2048 x 1120 (M x K x N) 21.3 us on the main kernel, 24.9 with two teams.
struct Fit {
  double tile[5], gather64, gather, tiled;  // per K tile of a round, and shares on top
  double fixed, out, tokens, round;
  double last, share, half;  // the last round: last + share x its filling (half: up to half)
};
constexpr Fit kMainFit = {{1.457, 1.083, 0.948, 0.873, 0.787}, 0.045, 0.092, 0, 3.45, 0.239, 0,
                          2.53, 0.801, 0.146, 0};
constexpr Fit kTeamsFit = {{0.559, 0.459, 0.451, 0.476, 0.436}, 0.34, 0.63, 0.055, 3.35, 0.671,
                           0.12, 4.46, 0.877, 0.141, 0};
constexpr Fit kSmallFit = {{1.03, 0.871, 0.819, 0.861, 0.784}, 0.359, 0.402, 0.12, 5.28, 0.288,
                           0.211, 1.70, 1.099, 0, 0.759};
constexpr Fit kLargeFit = {{1.026, 0.818, 0.806, 0.821, 0.735}, 0.191, 0.254, 0.011, 6.48, 0.249,
                           0.143, 2.03, 0.794, 0.184, 0};
constexpr Fit kTailFit = {{0.946, 0.768, 0.752, 0.767, 0.697}, 0.218, 0.334, 0.029, 8.41, 0.364,
                          0.185, 1.44, 0.479, 0.317, 0};

int ceil_div(int a, int b) { return (int)(((long)a + b - 1) / b); }

double fit_us(const Fit& f, const GemmCall& c, int bm, int cap) {
  const long tiles = (long)ceil_div(c.M, bm) * ceil_div(c.N, 128);
  const long per = (tiles + 7) / 8;
  const double full = (double)(per / cap), rest = (double)(per % cap) / cap;
  const double last = rest == 0 ? 0 : f.half > 0 && rest <= 0.5 ? f.half : f.last + f.share * rest;
  const int col = c.per_channel ? 4 : c.g == 64 ? 0 : c.g == 128 ? 1 : c.g == 256 ? 2 : 3;
  double tile = f.tile[col];
  if (c.reorder && !c.tiled) tile *= 1 + (c.g == 64 ? f.gather64 : f.gather);
  if (c.tiled) tile *= 1 + f.tiled;
  return f.fixed + 1e-6 * c.M * (f.out * c.N + f.tokens * c.K) + f.round * (full + (rest > 0)) +
         tile * (full + last) * (c.K / 128);
}

// The mid-size kernel: two tiles per compute unit. K tiles between the mean and the
// longest wave's (waves without any leave the others more), and 3.4 for the start and
// the sum; row-major weights cost more the fewer tokens share them, gathered ones once
// the caches no longer hold them.
double mid_us(const GemmCall& c) {
  const int rb = mid_token_blocks(c.M, c.N, c.K, c.tiled);
  const int i = rb == 4 ? 0 : rb == 2 ? 1 : 2;
  constexpr double kTile[3] = {0.313, 0.175, 0.145}, kRow[3] = {0.336, 0.564, 0.777};
  const long per = ((long)ceil_div(c.M, 16 * rb) * ceil_div(c.N, 64) + 7) / 8;
  const double full = (double)(per / 64), rest = (double)(per % 64) / 64;
  const int run = !c.per_channel && c.g > 128 ? c.g / 128 : 1;  // K tiles of a wave's turn
  const double kt = 0.545 * (c.K / 128) + 0.455 * 4 * run * ceil_div(c.K / 128 / run, 4) + 3.37;
  const double k = c.K < 4096 ? c.K / 4096.0 : 1.0;
  double tile = kTile[i];
  if (!c.per_channel && c.g == 64) tile *= 1.68;
  if (!c.tiled) tile *= 1 + kRow[i];
  if (c.reorder && !c.tiled) tile *= 1 + 0.413 * k * k;
  return 2.39 + 1.104e-6 * c.M * c.N +
         tile * kt * (full + (rest > 0 ? 0.326 + 0.773 * rest : 0));
}

double path_us(GemmPath p, const GemmCall& c) {
  switch (p) {
    case GemmPath::kMid: return mid_us(c);
    case GemmPath::kFp6Teams: return fit_us(kTeamsFit, c, 128, 32);
    case GemmPath::kFp6Small: return fit_us(kSmallFit, c, 128, 64);
    case GemmPath::kFp6Large: return fit_us(kLargeFit, c, 256, 32);
    case GemmPath::kFp6Tail: return fit_us(kTailFit, c, 256, 32);
    default: return fit_us(kMainFit, c, 256, 32);
  }
}

// The mean over both layouts, for a choice that must not depend on it.
double both_layouts_us(GemmPath p, GemmCall c) {
  c.tiled = !c.tiled;
  const double other = path_us(p, c);
  c.tiled = !c.tiled;
  return (path_us(p, c) + other) / 2;
}

// The share of the main kernel's fitted time that a path has to stay below, where the fits
// err to one side. Few columns and short K: the main kernel finds the tokens in the caches
// and is 5 to 8 % faster than fitted, the 6-bit kernels 4 to 13 % slower (7932 x 2048 x 400, g =
// 256, main 18.7, two teams 23.0 us; 7439 x 2048 x 992, g = 64, 28.0, 256 x 128 tiles 32.3).
// K = 512: with short groups or per-channel a second round of the mid-size kernel starts with
// a step that is not in the fit (g = 64, 4587 x 512 x 448, one round, main 11.0, mid-size
// 11.0; 771 x 512 x 2928, 1.2 rounds, 10.6 / 16.4); with groups of 512, one wave of four has
// them all, and the fit charges it too much (618 x 512 x 3072, tiled, 9.1 / 6.9). Of 1400 calls
// with at most 1280 columns or K = 512 95 were more than 4 % slower than on the main kernel,
// with the shares 16 of 1500.
double worth_it(GemmPath p, const GemmCall& c) {
  if (p == GemmPath::kMid) {
    if (c.K != 512) return 1.0;
    if (!c.per_channel && c.g >= 256) return c.g == 512 ? 1.04 : 1.0;
    const int bm = 16 * mid_token_blocks(c.M, c.N, c.K, c.tiled);
    return (long)ceil_div(c.M, bm) * ceil_div(c.N, 64) > 512 ? 0.8 : 1.0;
  }
  return c.N <= 1280 && c.K <= 4096 ? 0.9 : 1.0;
}

GemmPath unless_main_is_faster(GemmPath p, const GemmCall& c) {
  // Two workgroups of 128 x 128 per compute unit gather row-major weights for twice the
  // tiles, and from K = 4096 the caches no longer hold them: 547 x 8192 x 23696, g = 256,
  // 328 us, main 207; 548 x 4096 x 22016, g = 512, 142 / 104; 1020 x 4096 x 12288, g = 256,
  // 80 / 78. (g = 64, where the main kernel is slowest, stays: 1867 x 8192 x 8512 231 / 278.)
  // So does a single row of large tiles from K = 8192, each of which gathers weights of its
  // own: 134 x 8192 x 18400, g = 128, 82.4 / 78.0; 141 x 16384 x 17472 172 / 158 (187 x 4096
  // x 17040 41.3 / 42.7).
  const int gathered = p == GemmPath::kFp6Small                  ? 4096
                       : p == GemmPath::kFp6Large && c.M <= 256 ? 8192
                                                                : 0;
  if (gathered && c.K >= gathered && c.reorder && !c.tiled && c.g >= 128) return GemmPath::kMain;
  const bool same_order =
      c.per_channel || p == GemmPath::kFp6Small || p == GemmPath::kFp6Large;
  const double share = worth_it(p, c);
  const bool main = same_order
                        ? share * path_us(GemmPath::kMain, c) < path_us(p, c)
                        : share * both_layouts_us(GemmPath::kMain, c) < both_layouts_us(p, c);
  return main ? GemmPath::kMain : p;
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
    if (stream_wide(c)) return mid_eighths(c) ? GemmPath::kMidEighths : GemmPath::kStream;
    if (decode_wide(c)) return GemmPath::kDecode;
  }
  const bool mid = mid_kernel_fits(c.M, c.N);
  // Without the rescale the mid-size kernel stays ahead where it fits (300 x 8192 x
  // 8192: 33 against 35.5 us).
  if (scratch && fp6_scratch_bytes(c.M, c.N, c.K) && !(c.per_channel && mid))
    return unless_main_is_faster(fp6_form(c.M, c.N, c.K), c);
  return mid ? unless_main_is_faster(GemmPath::kMid, c) : GemmPath::kMain;
}

const char* gemm_path_name(GemmPath p) {
  switch (p) {
    case GemmPath::kStream: return "stream";
    case GemmPath::kStreamGather: return "stream_gather";
    case GemmPath::kDecode: return "decode";
    case GemmPath::kDecodeGather: return "decode_gather";
    case GemmPath::kMid: return "mid";
    case GemmPath::kMidEighths: return "mid_eighths";
    case GemmPath::kMain: return "main";
    case GemmPath::kFp6Teams: return "fp6_teams";
    case GemmPath::kFp6Small: return "fp6_small";
    case GemmPath::kFp6Large: return "fp6_large";
    case GemmPath::kFp6Tail: return "fp6_tail";
  }
  return "";
}

}  // namespace rrs
