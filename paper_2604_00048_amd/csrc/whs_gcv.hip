// GCV weight selection: launches of the grid-search kernel.
#include <hip/hip_runtime.h>

#include "whs_gcv.h"
#include "whs_kernels.h"

namespace whs {

constexpr int kGcvTile = 4;

// Grid values that a wavefront runs side by side where two share a SIMD: the
// most that fit in its registers.
constexpr int gcv_split(int D) { return D <= 3 ? 3 : 2; }
// Wavefronts of a block in the split form: 21 values of order 1 to 3 are seven
// groups, one pass of seven wavefronts (four in two passes: 5 % slower); the
// eleven groups of order 4 are three even passes of four.
constexpr int gcv_split_threads(int D) { return D <= 3 ? 512 : 256; }

// Rows per tile of a wavefront that is alone on its SIMD: at order 1 four rows of
// doubles are computed before the next four arrive (65,536 series of 1200 days, 21
// values: 1.56 ms, with eight 1.45; in float32 eight are level, and 131,072 series of
// 365 days take 0.29 ms for 0.27).
template <int D, typename TS>
constexpr int gcv_lone_tile() { return D == 1 && sizeof(TS) == 8 ? 8 : kGcvTile; }

// Wavefronts for one pass over the grid, spread evenly over as many passes as the
// block's limit of NT work-items asks for.
struct GcvBlock {
  int waves, passes;
};
template <int G, int SL, int NT>
static GcvBlock gcv_block(int n_grid) {
  const int per_wave = 64 >> SL;
  const int waves = ((n_grid + G - 1) / G + per_wave - 1) / per_wave;
  const int passes = (waves + NT / 64 - 1) / (NT / 64);
  return GcvBlock{(waves + passes - 1) / passes, passes};
}

// one: blocks of one wavefront, which takes all passes
template <int D, typename TS, int G, int SL, int NT, int W, int B = kGcvTile>
static hipError_t gcv_go(const GcvLaunch& L, hipStream_t stream, bool one = false) {
  GcvArgs a;
  a.P = L.P;
  a.T = L.T;
  a.S = L.S;
  a.nt = (L.T + B - 1) / B;
  a.n_grid = L.n_grid;
  a.w = L.w;
  a.x = L.x;
  a.grid = L.grid;
  a.lam_best = L.lam_best;
  a.scores = L.scores;
  a.info = L.info;
  int threads = 64 * (one ? 1 : gcv_block<G, SL, NT>(L.n_grid).waves);
  const int64_t blocks = (L.P + (1 << SL) - 1) >> SL;
  // a launch holds fewer than 2^32 work-items
  if (blocks * threads >= (int64_t)1 << 32) threads = 64;
  hipLaunchKernelGGL((k_gcv<D, B, TS, G, SL, NT, W>), dim3((unsigned)blocks), dim3(threads), 0, stream, a);
  return hipGetLastError();
}

// The form with the least time: eight series and their grid over the lanes of each
// wavefront while there are at most three such wavefronts per SIMD (8,192 series of
// 21 values); then blocks of 64 series, with the grid over their wavefronts or in one.
// Two wavefronts of the split form share a SIMD.  Its time, in turns of one of them,
// is the number of turns of the busiest SIMD: a CU takes eight blocks of one wavefront
// a round in two turns, four of two, two of three or four, and one of more in two
// turns.  A wavefront that is alone on its SIMD runs a pass of seven values (order 1
// and 2) in the time of 2.5 such turns, or one of three (order 3) or two values (order
// 4) in the time of 7/6.  Split and in one wavefront, us, float32, 365 days:
//   order 2,  7 values: 49,152 series 254 / 202, 81,920 409 / 405, 98,304 488 / 405
//   order 2, 14 values: 32,768 345 / 400, 49,152 515 / 400, 98,304 1030 / 808
//   order 2, 21 values: 49,152 521 / 610, 65,536 - / 616, 98,304 1039 / 1220
//   order 3,  7 values: 49,152 337 / 390, 65,536 442 / 392, 131,072 860 / 738
//   order 3, 14 values: 49,152 685 / 638, 65,536 912 / 654, 131,072 1819 / 1233
//   order 3, 21 values: 65,536 936 / 960, 131,072 1861 / 1930
template <int D, typename TS>
static hipError_t gcv_t(const GcvLaunch& L, hipStream_t stream) {
  constexpr int G = gcv_split(D), NT = gcv_split_threads(D);
  const int64_t lanes = ((L.P + 7) / 8) * ((L.n_grid + 7) / 8);
  if (lanes <= 3 * 1024) return gcv_go<D, TS, 1, 3, 512, 2>(L, stream);
  const int64_t nb = (L.P + 63) / 64;
  const int64_t cu = (nb + 255) / 256, rounds = (nb + 1023) / 1024;  // blocks of a CU; rounds of lone wavefronts
  const GcvBlock b = gcv_block<G, 6, NT>(L.n_grid);
  const int64_t turns = b.passes * (b.waves == 1   ? (cu + 3) / 4
                                    : b.waves == 2 ? cu / 4 * 2 + (cu % 4 < 2 ? cu % 4 : 2)
                                                   : cu * ((b.waves + 3) / 4));
  if constexpr (D <= 2) {
    if (5 * rounds * ((L.n_grid + 6) / 7) < 2 * turns)
      return gcv_go<D, TS, 7, 6, 64, 1, gcv_lone_tile<D, TS>()>(L, stream);
    return gcv_go<D, TS, G, 6, NT, 2>(L, stream);
  }
  return gcv_go<D, TS, G, 6, NT, 2>(L, stream, 7 * rounds * ((L.n_grid + G - 1) / G) < 6 * turns);
}

hipError_t launch_gcv(const GcvLaunch& L, hipStream_t stream) {
  switch (L.D) {
    case 1: return L.f64 ? gcv_t<1, double>(L, stream) : gcv_t<1, float>(L, stream);
    case 2: return L.f64 ? gcv_t<2, double>(L, stream) : gcv_t<2, float>(L, stream);
    case 3: return L.f64 ? gcv_t<3, double>(L, stream) : gcv_t<3, float>(L, stream);
    case 4: return L.f64 ? gcv_t<4, double>(L, stream) : gcv_t<4, float>(L, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace whs
