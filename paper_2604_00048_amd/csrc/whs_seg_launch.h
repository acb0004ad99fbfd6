// Host side of the segmented kernels: launch shapes, included by the files that
// instantiate them (one per order and mode, so that they compile side by side).
#pragma once

#include <hip/hip_runtime.h>

#include "whs_seg.h"
#include "whs_two_sweep.h"

namespace whs {

constexpr int kCus = 256;  // MI355X

// Steps per tile.  One band: as the one-lane kernel's in FP32 storage; the
// adjoint of order 2 takes 22 (24 spilled 260 bytes per lane).  Several bands
// (MB) run in groups of 3 (solve) or 2 (adjoint) and fewer: the widest groups whose
// tiles stay deep enough for the checkpoints to cost less than the weights and
// the mask read again, and free of spills (3 bands of the adjoint at 12 steps
// spilled 232 bytes per lane).  Every group of a call takes the same tile: its
// segments then end at the same rows, and every group factors a series alike and
// agrees on whether it is singular.  (That costs a last band alone some checkpoints,
// its tile would else be 24 and 22: ten bands of 16,384 series of 3288 days, solve
// and adjoint, 4.13 -> 4.16 ms.)
template <int D, int C, bool BWD, bool MB>
constexpr int seg_tile() { return !MB ? (D == 2 && BWD ? 22 : 24) : BWD ? 13 : 16; }

constexpr int seg_group(int bands, bool bwd) {
  const int widest = bwd ? 2 : 3;
  return bands >= widest ? widest : bands;
}

struct SegShape {
  int sw_log2, nseg, tps, ne;
  int64_t groups;
};

// As many segments as leave every wavefront its own SIMD (1024 on the chip) and
// every segment a tile: 32 for up to 2048 series, then 16, 8, 4 and, up to
// 32,768 series, 2.  Beyond, one lane per series fills the chip by itself.  Series-
// contiguous batches then take one segment, which saves them the copies and is the
// recurrence of one lane per series: the two layouts give the same results at every size.
template <int B>
inline bool seg_shape(const LaunchDesc& L, SegShape& s) {
  const int nt = (L.T + B - 1) / B;
  for (s.sw_log2 = 3, s.nseg = 32; s.nseg >= (L.S == 1 ? 1 : 2); s.nseg /= 2) {
    s.groups = (L.P + (1 << s.sw_log2) - 1) >> s.sw_log2;
    const bool room = (s.groups << s.sw_log2) * s.nseg <= kCus * 4 * 64 || s.nseg == 1;
    if (room && s.nseg <= nt) {
      s.tps = (nt + s.nseg - 1) / s.nseg;
      s.ne = (nt + s.tps - 1) / s.tps;
      return true;
    }
    if (s.sw_log2 < 6) ++s.sw_log2;
  }
  return false;
}

// workspace of one series-contiguous launch: the checkpoints, and one dword per
// tile with its weights as bits
template <int D, bool BWD>
inline size_t seg_contiguous_bytes(const LaunchDesc& L) {
  SegShape s;
  if (!seg_shape<seg_tile<D, 1, BWD, false>()>(L, s)) return ~(size_t)0;
  const size_t lanes = (size_t)s.groups * ((size_t)s.nseg << s.sw_log2);
  return lanes * ((size_t)(s.tps - 1) * seg_fields<D, 1>() * sizeof(double) + (size_t)s.tps * 4);
}

template <int D, int C, bool BWD, bool PERDIFF, bool WB, bool MB, bool CT = false>
hipError_t launch_seg_group(const LaunchDesc& L, int c0, hipStream_t stream) {
  constexpr int B = seg_tile<D, C, BWD, MB>();
  // The checkpoints fit the workspace of an interleaved call: (tps - 1) nseg < T / B
  // of seg_fields against the T / 12 (one band, uneven dates) or, as a call of several
  // bands always has a group of two, T / 8 tiles that size it.  In doubles per step
  // at order 2, 9 / 22 against 5 / 12 for one band; 13 / 16 (three), 11 / 13 (two)
  // and 9 / 13 (a last one) against 7 / 8; at order 1, 3 / 24 against 2 / 16, and
  // 5 / 16, 4 / 13 and 3 / 13 against 3 / 8.
  static_assert(MB ? seg_fields<D, C>() * tile_depth<D, 2>() <= ck_fields<D, 2>() * B
                   : seg_fields<D, C>() * tile_depth<D, 1, true>() <= ck_fields<D, 1>() * B,
                "the checkpoints must fit the workspace of an interleaved call");
  SegShape s;
  if (!seg_shape<B>(L, s)) return hipErrorInvalidValue;
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
  // one or two segments of 64 series make as many wavefronts, every other shape four
  if (CT && s.nseg == 1)
    hipLaunchKernelGGL((k_seg<D, C, B, float, BWD, PERDIFF, WB, CT ? 64 : 128, MB, CT>), dim3((unsigned)s.groups),
                       dim3(64), 0, stream, g);
  else if (s.nseg == 2)
    hipLaunchKernelGGL((k_seg<D, C, B, float, BWD, PERDIFF, WB, 128, MB, CT>), dim3((unsigned)s.groups), dim3(128), 0,
                       stream, g);
  else
    hipLaunchKernelGGL((k_seg<D, C, B, float, BWD, PERDIFF, WB, 256, MB, CT>), dim3((unsigned)s.groups), dim3(256), 0,
                       stream, g);
  return hipGetLastError();
}

template <int D, bool BWD, bool PERDIFF>
hipError_t run_seg(const LaunchDesc& L, hipStream_t stream) {
  if (L.S == 1) return launch_seg_group<D, 1, BWD, PERDIFF, false, false, true>(L, 0, stream);
  if (L.C == 1)
    return L.wbits ? launch_seg_group<D, 1, BWD, PERDIFF, true, false>(L, 0, stream)
                   : launch_seg_group<D, 1, BWD, PERDIFF, false, false>(L, 0, stream);
  for (int c0 = 0; c0 < L.C;) {
    const int n = seg_group(L.C - c0, BWD);
    hipError_t e;
    if constexpr (BWD) e = n == 2 ? launch_seg_group<D, 2, BWD, PERDIFF, false, true>(L, c0, stream)
                                  : launch_seg_group<D, 1, BWD, PERDIFF, false, true>(L, c0, stream);
    else e = n == 3   ? launch_seg_group<D, 3, BWD, PERDIFF, false, true>(L, c0, stream)
             : n == 2 ? launch_seg_group<D, 2, BWD, PERDIFF, false, true>(L, c0, stream)
                      : launch_seg_group<D, 1, BWD, PERDIFF, false, true>(L, c0, stream);
    if (e != hipSuccess) return e;
    c0 += n;
  }
  return hipSuccess;
}

}  // namespace whs
