// The rule that chooses the segmented solve and adjoint (whs_seg.h).
#include <hip/hip_runtime.h>

#include "whs_seg_launch.h"

namespace whs {

hipError_t run_seg_solve_d1(const LaunchDesc&, hipStream_t);
hipError_t run_seg_solve_d2(const LaunchDesc&, hipStream_t);
hipError_t run_seg_backward_d1(const LaunchDesc&, hipStream_t);
hipError_t run_seg_backward_d2(const LaunchDesc&, hipStream_t);

// Where it runs: daily grid, FP32 storage, order <= 2, blocks of 64 series, at
// least 96 steps (4 tiles), and a batch that one lane per series leaves waiting on its
// own recurrence.  3288 steps, order 2, a weight per difference row, solve /
// adjoint in us, one lane per series -> segments:
//      512 series   620 /  815 ->  48 /  69      16,384 series  681 / 869 -> 281 / 408
//    4,096 series   643 /  825 -> 103 / 147      32,768 series  722 / 914 -> 558 / 801
// (from 4096 series on the segments run at the memory's rate, about 28 and 40
// bytes per series-step at 5 TB/s, checkpoints included).  512 steps, 4,096
// series: 105 / 143 -> 22 / 29; 150 steps: 41 / 55 -> 17 / 22, 32,768 series 45 /
// 58 -> 35 / 47; at 64 steps, three tiles, 34 / 41 -> 27 / 30 on 4,096 series but
// level on 65,536 contiguous ones.  Ten bands, 16,384 series of 3288 steps: solve
// and adjoint 8.07 -> 4.16 ms.  At 65,536 series one lane per series already
// fills every SIMD and moves fewer checkpoint bytes.
// Series-contiguous arrays of one band take the same kernel, their row pieces
// turned through LDS, instead of three copies into the interleaved layout and
// back (or, where the call's workspace has no room for copies, the partition kernel):
//       64 series   611 /  812 ->  54 /  70      16,384 series   958 / 1315 ->  383 /  620
//    4,096 series   706 /  951 -> 120 / 213      65,536 series  2091 / 3093 -> 1532 / 2484
// (the last in one segment; slower than interleaved because a lane's pieces of 88
// to 96 bytes split lines of 128, and the lines that 65,536 lanes hold open in
// five arrays exceed the L2).
// Not taken: the one-band solve with a weight per series below 512 steps.  No
// crossover lies there: segments would be ahead from 96 steps on (4,096 series of 365
// steps 66 -> 16 us, of 511 89 -> 21; 32,768 of 511 92 -> 65).  It stays because a
// plan's launch of one lane per series gives its groups bit for bit what this call
// gives them, which is kept for groups of about a year, where it costs a call at most
// some 70 us; longer ones, where it would cost up to 0.6 ms, agree to rounding.
// Nor FP64 storage and orders 3 and 4, for which no segmented kernel has been built.
// Several bands: the segments take 3 (solve) or 2 (adjoint) to a launch, one lane
// per series 5 or 3 (solve) and 3, and every launch factors the series again.  With
// eight segments and more that never matters; with fewer the segments' time grows
// with the launches and the series while one lane per series waits the same time
// for any batch, so they are taken where their launches are few enough.  Times of
// one lane per series over those of the segments, lengths of 100 to 1000 steps:
//   two segments (20,000 and 32,768 series)
//     solve    a weight per series 1.08-1.43; per difference row, twice the launches
//              or more (4, 5, 10 bands) 0.83-1.23, fewer 1.01-1.55
//     adjoint  as many launches (2, 4 bands) 1.00-1.71; up to 1.33 times (7, 8, 10)
//              1.01-1.41, but 0.89-1.15 at order 1 with a weight per series; more (3,
//              5, 6, 9, 12) 0.61-1.24
//   four segments (16,384 series)
//     adjoint  three bands, a weight per difference row 0.90-1.14, others 1.16-2.58
static bool bands_pay(const LaunchDesc& L, bool bwd) {
  SegShape s;
  if (bwd ? !seg_shape<seg_tile<2, 2, true, true>()>(L, s) : !seg_shape<seg_tile<2, 2, false, true>()>(L, s))
    return false;
  if (s.nseg > 4) return true;
  const int widest = seg_group(L.C, bwd), one_lane = max_group(L.D, bwd, false, L.perdiff);
  const int n = (L.C + widest - 1) / widest, n1 = (L.C + one_lane - 1) / one_lane;
  if (!bwd) return s.nseg > 2 || n < 2 * n1;
  if (s.nseg > 2) return !L.perdiff || n < 2 * n1;
  return L.D == 1 && !L.perdiff ? n <= n1 : 2 * n < 3 * n1;
}

bool seg_path(const LaunchDesc& L, bool bwd) {
  if (L.fac || L.coef || L.f64 || L.D > 2 || L.T < 96 || L.P < 1 || L.P >= ((int64_t)1 << 31))
    return false;
  if (L.T < 512 && !bwd && !L.perdiff && L.C == 1) return false;
  if (L.S != 64 && !(L.S == 1 && L.C == 1)) return false;
  if ((int64_t)L.T * L.C * 256 >= ((int64_t)1 << 30)) return false;  // 32-bit offsets, tiles past the end included
  SegShape s;
  if (!seg_shape<24>(L, s)) return false;
  if (L.S == 64) return L.C == 1 || bands_pay(L, bwd);
  // up to 1024 series the partition kernel's 256 lanes per series are ahead (64
  // series 25 / 27 us against 54 / 70, 1024 series 70 / 80 against 62 / 100); a
  // call with the larger workspace keeps the interleaved call's results bit for bit,
  // which the partition kernel does not give
  if (L.in_place && L.P <= 1024 && chunk_path(L)) return false;
  // a series-contiguous call's workspace is sized without the padding to whole workgroups
  const size_t need = L.D == 1 ? (bwd ? seg_contiguous_bytes<1, true>(L) : seg_contiguous_bytes<1, false>(L))
                               : (bwd ? seg_contiguous_bytes<2, true>(L) : seg_contiguous_bytes<2, false>(L));
  return L.ws_bytes >= need;
}

hipError_t launch_seg(const LaunchDesc& L, bool bwd, hipStream_t stream) {
  if (bwd) return L.D == 1 ? run_seg_backward_d1(L, stream) : run_seg_backward_d2(L, stream);
  return L.D == 1 ? run_seg_solve_d1(L, stream) : run_seg_solve_d2(L, stream);
}

}  // namespace whs
