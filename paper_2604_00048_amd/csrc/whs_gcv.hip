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

template <int D, typename TS, int G, int SL, int NT, int W>
static hipError_t gcv_go(const GcvLaunch& L, hipStream_t stream) {
  GcvArgs a;
  a.P = L.P;
  a.T = L.T;
  a.S = L.S;
  a.nt = (L.T + kGcvTile - 1) / kGcvTile;
  a.n_grid = L.n_grid;
  a.w = L.w;
  a.x = L.x;
  a.grid = L.grid;
  a.lam_best = L.lam_best;
  a.scores = L.scores;
  a.info = L.info;
  // wavefronts for one pass over the grid, spread evenly over as many passes
  // as the block's limit asks for
  const int per_wave = 64 >> SL;
  const int waves = ((L.n_grid + G - 1) / G + per_wave - 1) / per_wave;
  const int passes = (waves + NT / 64 - 1) / (NT / 64);
  int threads = 64 * ((waves + passes - 1) / passes);
  const int64_t blocks = (L.P + (1 << SL) - 1) >> SL;
  // a launch holds fewer than 2^32 work-items: beyond, one wavefront takes all passes
  if (blocks * threads >= (int64_t)1 << 32) threads = 64;
  hipLaunchKernelGGL((k_gcv<D, kGcvTile, TS, G, SL, NT, W>), dim3((unsigned)blocks), dim3(threads), 0, stream, a);
  return hipGetLastError();
}

// The form with the least time by the figures beside the kernel: eight series
// and their grid over the lanes of each wavefront while there are at most three
// such wavefronts per SIMD (8,192 series of 21 values); then blocks of 64 series
// with the grid over their wavefronts.  Order 1 and 2 fit seven values in a
// wavefront that is alone on its SIMD, which is the better one where such
// wavefronts fill the chip: a round of 1,024 of them takes 60 parts of time to
// 17 of a round of 256 split blocks.  Orders 3 and 4 are faster split at every
// size (65,536 series of order 3: 8.6 against 9.6 ms, of order 4: 12.8 against
// 13.1 ms).
template <int D, typename TS>
static hipError_t gcv_t(const GcvLaunch& L, hipStream_t stream) {
  const int64_t lanes = ((L.P + 7) / 8) * ((L.n_grid + 7) / 8);
  if (lanes <= 3 * 1024) return gcv_go<D, TS, 1, 3, 512, 2>(L, stream);
  if constexpr (D <= 2) {
    const int64_t nb = (L.P + 63) / 64;
    if ((nb + 1023) / 1024 * 60 < (nb + 255) / 256 * 17) return gcv_go<D, TS, 7, 6, 64, 1>(L, stream);
  }
  return gcv_go<D, TS, gcv_split(D), 6, gcv_split_threads(D), 2>(L, stream);
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
