// Launch of the segmented solve and adjoint (whs_seg.h) and the rule that chooses them.
#include <hip/hip_runtime.h>

#include "whs_seg.h"
#include "whs_two_sweep.h"

namespace whs {

namespace {

constexpr int kCus = 256;  // MI355X

// Steps per tile.  One band: as the one-lane kernel's in FP32 storage; the
// adjoint of order 2 takes 22 (24 spilled 260 bytes per lane).  Several bands
// run in groups of 3 (solve) or 2 (adjoint) and one: the widest groups whose
// tiles stay deep enough for the checkpoints to cost less than the weights and
// the mask read again, and free of spills (3 bands of the adjoint at 12 steps
// spilled 232 bytes per lane).  The checkpoints (seg_fields per tile, none for a
// segment's first) stay below what checkpoint_bytes reports for the call: in
// doubles per step at order 2, 9 / 22 against 5 / 12 for one band, 11 / 13
// against 7 / 8 for two, 13 / 16 against 9 / 8 for three; at order 1, 3 / 24
// against 2 / 16, 4 / 13 against 3 / 8, 5 / 16 against 4 / 8.
template <int D, int C, bool BWD>
constexpr int seg_tile() { return C == 1 ? (D == 2 && BWD ? 22 : 24) : BWD ? 13 : 16; }

constexpr int seg_group(int bands, bool bwd) {
  const int widest = bwd ? 2 : 3;
  return bands >= widest ? widest : bands;
}

struct Shape {
  int sw_log2, nseg, tps, ne;
  int64_t groups;
};

// As many segments as leave every wavefront its own SIMD (1024 on the chip) and
// every segment a tile: 32 for up to 2048 series, then 16, 8, 4 and, up to
// 32,768 series, 2 (beyond, one lane per series fills the chip by itself).
template <int B>
bool shape(const LaunchDesc& L, Shape& s) {
  const int nt = (L.T + B - 1) / B;
  for (s.sw_log2 = 3, s.nseg = 32; s.nseg >= 2; s.nseg /= 2) {
    s.groups = (L.P + (1 << s.sw_log2) - 1) >> s.sw_log2;
    if ((s.groups << s.sw_log2) * s.nseg <= kCus * 4 * 64 && s.nseg <= nt) {
      s.tps = (nt + s.nseg - 1) / s.nseg;
      s.ne = (nt + s.tps - 1) / s.tps;
      return true;
    }
    if (s.sw_log2 < 6) ++s.sw_log2;
  }
  return false;
}

template <int D, int C, bool BWD, bool PERDIFF, bool WB, bool MB>
hipError_t launch(const LaunchDesc& L, int c0, hipStream_t stream) {
  constexpr int B = seg_tile<D, C, BWD>();
  // (tps - 1) nseg < T / B checkpoints of seg_fields, against the T / 12 (one
  // band, uneven dates) or T / 8 tiles of the same group that size the workspace
  static_assert(seg_fields<D, C>() * (C == 1 ? tile_depth<D, 1, true>() : tile_depth<D, C>()) <= ck_fields<D, C>() * B,
                "the checkpoints must fit the workspace of the call");
  Shape s;
  if (!shape<B>(L, s)) return hipErrorInvalidValue;
  SegArgs g;
  g.f.P = L.P;
  g.f.T = L.T;
  g.f.S = L.S;
  g.f.Ctot = L.C;
  g.f.c0 = c0;
  g.f.nt = (L.T + B - 1) / B;
  g.f.w = L.w;
  g.f.lam = L.lam;
  g.f.rhs = L.rhs;
  g.f.zin = L.zin;
  g.f.out = L.out;
  g.f.glam = L.glam;
  g.f.info = L.info;
  g.f.ck = L.ws;
  g.f.coef = nullptr;
  g.f.write_info = c0 == 0;  // later groups add their share of grad_lambda
  g.f.glam_accum = c0 > 0;
  g.sw_log2 = s.sw_log2;
  g.nseg = s.nseg;
  g.tps = s.tps;
  g.ne = s.ne;
  // two segments of 64 series make two wavefronts, every other shape four
  if (s.nseg == 2)
    hipLaunchKernelGGL((k_seg<D, C, B, float, BWD, PERDIFF, WB, 128, MB>), dim3((unsigned)s.groups), dim3(128), 0,
                       stream, g);
  else
    hipLaunchKernelGGL((k_seg<D, C, B, float, BWD, PERDIFF, WB, 256, MB>), dim3((unsigned)s.groups), dim3(256), 0,
                       stream, g);
  return hipGetLastError();
}

template <int D, bool BWD, bool PERDIFF>
hipError_t pick(const LaunchDesc& L, hipStream_t stream) {
  if (L.C == 1)
    return L.wbits ? launch<D, 1, BWD, PERDIFF, true, false>(L, 0, stream)
                   : launch<D, 1, BWD, PERDIFF, false, false>(L, 0, stream);
  for (int c0 = 0; c0 < L.C;) {
    const int n = seg_group(L.C - c0, BWD);
    hipError_t e;
    if constexpr (BWD) e = n == 2 ? launch<D, 2, BWD, PERDIFF, false, true>(L, c0, stream)
                                  : launch<D, 1, BWD, PERDIFF, false, true>(L, c0, stream);
    else e = n == 3   ? launch<D, 3, BWD, PERDIFF, false, true>(L, c0, stream)
             : n == 2 ? launch<D, 2, BWD, PERDIFF, false, true>(L, c0, stream)
                      : launch<D, 1, BWD, PERDIFF, false, true>(L, c0, stream);
    if (e != hipSuccess) return e;
    c0 += n;
  }
  return hipSuccess;
}

template <int D>
hipError_t pick_kind(const LaunchDesc& L, bool bwd, hipStream_t stream) {
  if (bwd) return L.perdiff ? pick<D, true, true>(L, stream) : pick<D, true, false>(L, stream);
  return L.perdiff ? pick<D, false, true>(L, stream) : pick<D, false, false>(L, stream);
}

}  // namespace

// Where it runs: daily grid, FP32 storage, order <= 2, blocks of 64 series, at
// least 512 steps, and a batch that one lane per series leaves waiting on its
// own recurrence.  3288 steps, order 2, a weight per difference
// row, solve / adjoint in us, one lane per series -> segments:
//      512 series   620 /  815 ->  48 /  69      16,384 series  681 / 869 -> 287 / 417
//    4,096 series   643 /  825 -> 103 / 153      32,768 series  722 / 914 -> 558 / 801
// (from 4096 series on the segments run at the memory's rate, about 28 and 40
// bytes per series-step at 5 TB/s, checkpoints included).  512 steps, 4,096
// series: 105 / 143 -> 22 / 29.  Ten bands, 16,384 series of 3288 steps: solve
// and adjoint 8.07 -> 4.11 ms.  At 65,536 series one lane per series already
// fills every SIMD and moves fewer checkpoint bytes.
// Not taken: FP64 storage, whose callers see the last digits, which another
// order of elimination changes on ill-conditioned series; fewer than 512
// steps, where a solve gives bit for bit what a plan's launch of one lane per
// series gives; order 3 and 4, whose state leaves no registers for the spike.
bool seg_path(const LaunchDesc& L) {
  if (L.fac || L.coef || L.f64 || L.D > 2 || L.S != 64 || L.T < 512) return false;
  if ((int64_t)L.T * L.C * 256 >= ((int64_t)1 << 30)) return false;  // 32-bit offsets, tiles past the end included
  Shape s;
  return shape<24>(L, s);
}

hipError_t launch_seg(const LaunchDesc& L, bool bwd, hipStream_t stream) {
  return L.D == 1 ? pick_kind<1>(L, bwd, stream) : pick_kind<2>(L, bwd, stream);
}

}  // namespace whs
