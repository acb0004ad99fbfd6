// Launch of the segmented solve and adjoint (whs_seg.h) and the rule that chooses them.
#include <hip/hip_runtime.h>

#include "whs_seg.h"

namespace whs {

namespace {

constexpr int kCus = 256;  // MI355X

// Steps per tile, as the one-lane kernel's in FP32 storage; the adjoint of
// order 2 takes 22 (24 spilled 260 bytes per lane).  The checkpoints
// (seg_fields per tile, none for a segment's first) stay below what
// checkpoint_bytes reports for one band: 9 / 22 doubles per step against its
// 5 / 12 at order 2, 3 / 24 against 2 / 16 at order 1.
template <int D, bool BWD>
constexpr int seg_tile() { return D == 2 && BWD ? 22 : 24; }

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

template <int D, bool BWD, bool PERDIFF, bool WB>
hipError_t launch(const LaunchDesc& L, hipStream_t stream) {
  constexpr int B = seg_tile<D, BWD>();
  Shape s;
  if (!shape<B>(L, s)) return hipErrorInvalidValue;
  SegArgs g;
  g.f.P = L.P;
  g.f.T = L.T;
  g.f.S = L.S;
  g.f.Ctot = L.C;
  g.f.c0 = 0;
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
  g.f.write_info = 1;
  g.f.glam_accum = 0;
  g.sw_log2 = s.sw_log2;
  g.nseg = s.nseg;
  g.tps = s.tps;
  g.ne = s.ne;
  // two segments of 64 series make two wavefronts, every other shape four
  if (s.nseg == 2)
    hipLaunchKernelGGL((k_seg<D, 1, B, float, BWD, PERDIFF, WB, 128>), dim3((unsigned)s.groups), dim3(128), 0, stream, g);
  else
    hipLaunchKernelGGL((k_seg<D, 1, B, float, BWD, PERDIFF, WB, 256>), dim3((unsigned)s.groups), dim3(256), 0, stream, g);
  return hipGetLastError();
}

template <int D, bool BWD>
hipError_t pick(const LaunchDesc& L, hipStream_t stream) {
  if (L.perdiff) return L.wbits ? launch<D, BWD, true, true>(L, stream) : launch<D, BWD, true, false>(L, stream);
  return L.wbits ? launch<D, BWD, false, true>(L, stream) : launch<D, BWD, false, false>(L, stream);
}

}  // namespace

// Where it runs: one band, daily grid, FP32 storage, order <= 2, blocks of 64
// series, at least 512 steps, and a batch that one lane per series leaves
// waiting on its own recurrence.  3288 steps, order 2, a weight per difference
// row, solve / adjoint in us, one lane per series -> segments:
//      512 series   620 /  815 ->  48 /  69      16,384 series  681 / 869 -> 287 / 417
//    4,096 series   643 /  825 -> 103 / 153      32,768 series  722 / 914 -> 558 / 801
// (from 4096 series on the segments run at the memory's rate, about 28 and 40
// bytes per series-step at 5 TB/s, checkpoints included).  512 steps, 4,096
// series: 105 / 143 -> 22 / 29.  At 65,536 series one lane per series already
// fills every SIMD and moves fewer checkpoint bytes.
// Not taken: FP64 storage, whose callers see the last digits, which another
// order of elimination changes on ill-conditioned series; fewer than 512
// steps, where a solve gives bit for bit what a plan's launch of one lane per
// series gives; order 3 and 4, whose state leaves no registers for the spike.
bool seg_path(const LaunchDesc& L) {
  if (L.fac || L.coef || L.f64 || L.C != 1 || L.D > 2 || L.S != 64 || L.T < 512) return false;
  if ((int64_t)L.T * L.S * 4 >= ((int64_t)1 << 30)) return false;
  Shape s;
  return shape<24>(L, s);
}

hipError_t launch_seg(const LaunchDesc& L, bool bwd, hipStream_t stream) {
  if (L.D == 1) return bwd ? pick<1, true>(L, stream) : pick<1, false>(L, stream);
  return bwd ? pick<2, true>(L, stream) : pick<2, false>(L, stream);
}

}  // namespace whs
