// Several segments per series: the fused solve and adjoint for batches too
// small to fill the chip with one lane per series.
//
// What bounds such a batch is the dependent chain of one series (2 T steps of
// the recurrence), not bytes or operations, so the rows of a series are cut
// into `nseg` consecutive segments, one lane each, all in one workgroup.  The
// last D rows of every segment but the last are separators.  Eliminating the
// interiors first and the separators last is Cholesky of a symmetric
// permutation of Omega (Sec. III-A), so it keeps the accuracy of the
// sequential sweep:
//
//   sweep 1     each lane factors its segment (interior, then its separator)
//               with the ordinary recurrence and carries, beside y = L^-1 b,
//               the D columns v = L^-1 E, E = Omega[segment, separator before].
//               The last D factor rows give Y = Omega_SS - E_R' A^-1 E_R, c and
//               the coupling F to the separator before; sums over the interior
//               give G = E' A^-1 E and h = E' A^-1 b.
//   interface   block-tridiagonal D x D system in the separators, solved by one
//               lane per series: diagonal Y_s - G_{s+1}, off-diagonal F_s,
//               right-hand side c_s - h_{s+1}.
//   sweep 2     each lane back-substitutes its segment from the two separators
//               it touches, tile by tile from checkpoints as the one-lane kernel
//               does, with y - v z_before in place of y.
//
// A workgroup holds SW series x nseg segments (lane = segment * SW + series):
// SW = 64 gives whole rows per wavefront, smaller SW more segments per series.
// NT = SW * nseg work-items, one wavefront per SIMD.  MB: a group of C bands of
// a call that has more.
#pragma once

#include <hip/hip_runtime.h>

#include "whs_fast.h"
#include "whs_step.h"

namespace whs {

struct SegArgs {
  FastArgs f;
  int sw_log2;  // series per workgroup: 1 << sw_log2
  int nseg;     // segments per series; (1 << sw_log2) * nseg work-items per workgroup
  int tps;      // tiles per segment
  int ne;       // segments that hold rows
};

// doubles of checkpoints per lane: every tile of a segment but its first
template <int D, int C>
constexpr int seg_fields() { return ck_fields<D, C>() + D * D; }

template <int D, int C, int B, typename TS, bool BWD, bool PERDIFF, bool WB, int NT, bool MB = false>
struct Seg {
  static constexpr int NF = seg_fields<D, C>();
  static constexpr int NY = D * (D + 1) / 2;
  // LDS fields of one lane: Y, c, F, G, h
  static constexpr int fY = 0, fC = NY, fF = fC + D * C, fG = fF + D * D, fH = fG + NY, NX = fH + D * C;
  static constexpr uint32_t ES = sizeof(TS);
  static constexpr uint32_t kDead = 0x80000000u;

  struct Tile {
    TS x[B][C];
    uint32_t w[WB ? 1 : B];
    uint32_t wm;
    TS lam[B];
    TS z[B][C];
  };
  struct Spike {
    double v[D + 1][D];  // v[j][c]: column c at row t - j
  };

  // wave-uniform
  __amdgpu_buffer_rsrc_t rx, rw, rl, rz, ro, rg, rck;
  int T, tps;
  uint32_t Rx;  // bytes per row of x, all bands (a constant for one band alone)
  // blocks of 64 series: bytes between two bands of a row, and per row of
  // lambda, of w and of one checkpoint field
  static constexpr uint32_t Sb = 64u * ES, Rl = Sb, Rw = WB ? 8u : 64u, ckrow = NT * 8u;
  // per lane
  uint32_t lx, ll, lw, lc, bit;
  int r0;               // first row of the segment
  bool hasR;            // a separator follows
  double lam_scalar;
  bool accum;

  static __device__ __forceinline__ int tri2(int r, int q) { return r * (r + 1) / 2 + q; }

  static __device__ __forceinline__ bool wt(const Tile& tl, int s) {
    if constexpr (WB) return (tl.wm >> s) & 1u;
    else return tl.w[s] != 0u;
  }

  template <bool SWEEP2>
  __device__ __forceinline__ void load_tile(Tile& tl, int j) const {
    constexpr int POL = SWEEP2 ? kStream : kKeep;
    const uint32_t t0 = (uint32_t)(r0 + j * B);
    const uint32_t ox = lx + t0 * Rx, ow = lw + t0 * Rw, ol = ll + t0 * Rl;
#pragma unroll
    for (int s = 0; s < B; ++s) {
#pragma unroll
      for (int c = 0; c < C; ++c) tl.x[s][c] = bload<TS, POL>(rx, ox + (uint32_t)s * Rx + (uint32_t)c * Sb);
      if constexpr (WB) {
        if (s == 0) tl.wm = 0u;
        tl.wm |= ((__builtin_amdgcn_raw_buffer_load_b32(rw, ow + (uint32_t)s * Rw, 0, POL) >> bit) & 1u) << s;
      } else {
        tl.w[s] = __builtin_amdgcn_raw_buffer_load_b8(rw, ow + (uint32_t)s * Rw, 0, POL);
      }
    }
    if constexpr (PERDIFF) {
#pragma unroll
      for (int s = 0; s < B; ++s) tl.lam[s] = bload<TS, POL>(rl, ol + (uint32_t)s * Rl);
    }
    if constexpr (BWD && SWEEP2) {
#pragma unroll
      for (int s = 0; s < B; ++s)
#pragma unroll
        for (int c = 0; c < C; ++c) tl.z[s][c] = bload<TS, POL>(rz, ox + (uint32_t)s * Rx + (uint32_t)c * Sb);
    }
  }

  // lambda of the D rows before row t0
  __device__ __forceinline__ void load_window(int t0, double (&lwin)[D + 1]) const {
    lwin[0] = 0.0;
#pragma unroll
    for (int m = 1; m <= D; ++m) {
      const int k = t0 - m;
      if constexpr (PERDIFF) {
        lwin[m] = to_f64(bload<TS>(rl, k >= 0 ? ll + (uint32_t)k * Rl : kDead));
      } else {
        lwin[m] = (k >= 0 && k < T - D) ? lam_scalar : 0.0;
      }
    }
  }

  __device__ __forceinline__ void store_ck(const State<D, C>& st, const Spike& sp, int j) const {
    const uint32_t base = lc + (uint32_t)((j - 1) * NF) * ckrow;
    int f = 0;
#pragma unroll
    for (int jj = 1; jj <= D; ++jj) bstore<double, kStream>(rck, base + (uint32_t)(f++) * ckrow, st.invD[jj]);
#pragma unroll
    for (int jj = 1; jj < D; ++jj)
#pragma unroll
      for (int k = 1; k <= D - jj; ++k) bstore<double, kStream>(rck, base + (uint32_t)(f++) * ckrow, st.R[jj][k]);
#pragma unroll
    for (int jj = 1; jj <= D; ++jj) {
#pragma unroll
      for (int c = 0; c < C; ++c) bstore<double, kStream>(rck, base + (uint32_t)(f++) * ckrow, st.y[jj][c]);
#pragma unroll
      for (int q = 0; q < D; ++q) bstore<double, kStream>(rck, base + (uint32_t)(f++) * ckrow, sp.v[jj][q]);
    }
  }

  // checkpoint of tile j >= 1; the segment's first tile starts from the zero state
  __device__ __forceinline__ void load_ck(int j, double (&ckv)[NF], double (&lwin)[D + 1]) const {
    const uint32_t base = j >= 1 ? lc + (uint32_t)((j - 1) * NF) * ckrow : kDead;
#pragma unroll
    for (int f = 0; f < NF; ++f) ckv[f] = bload<double, kStream>(rck, base + (uint32_t)f * ckrow);
    load_window(r0 + j * B, lwin);
  }

  // the checkpointed state with y - v zL in place of y
  __device__ __forceinline__ void restore(State<D, C>& st, const double (&ckv)[NF], const double (&lwin)[D + 1],
                                          const double (&zL)[D][C]) const {
    int f = 0;
#pragma unroll
    for (int jj = 1; jj <= D; ++jj) st.invD[jj] = ckv[f++];
#pragma unroll
    for (int jj = 1; jj < D; ++jj)
#pragma unroll
      for (int k = 1; k <= D - jj; ++k) st.R[jj][k] = ckv[f++];
#pragma unroll
    for (int jj = 1; jj <= D; ++jj) {
#pragma unroll
      for (int c = 0; c < C; ++c) st.y[jj][c] = ckv[f++];
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const double v = ckv[f++];
#pragma unroll
        for (int c = 0; c < C; ++c) st.y[jj][c] = __builtin_fma(-v, zL[q][c], st.y[jj][c]);
      }
    }
#pragma unroll
    for (int m = 0; m <= D; ++m) st.lw[m] = lwin[m];
  }

  // row t: factor and forward-substitution step; om: row t of Omega
  template <bool FULL>
  __device__ __forceinline__ void factor_row(State<D, C>& st, const Tile& tl, int s, int t, double (&om)[D + 1],
                                             double (&l)[D + 1], double& dt, double& invdt, double (&b)[C]) const {
    const bool obs = wt(tl, s);
    double lt;
    if constexpr (PERDIFF) lt = to_f64(tl.lam[s]);
    else lt = (FULL || t < T - D) ? lam_scalar : 0.0;
    double lwv[D + 1];
    lwv[0] = lt;
#pragma unroll
    for (int m = 1; m <= D; ++m) lwv[m] = st.lw[m];
    omega_row<D>(lwv, obs ? 1.0 : 0.0, om);
    ldl_step<D, C>(st, om, l, dt, invdt);
#pragma unroll
    for (int m = D; m >= 2; --m) st.lw[m] = st.lw[m - 1];
    st.lw[1] = lt;
#pragma unroll
    for (int c = 0; c < C; ++c) b[c] = to_f64((BWD || obs) ? tl.x[s][c] : TS(0));
  }

  // sweep 1 over one tile; first: the segment's first tile, sepR: its last D
  // rows are the separator that follows
  template <bool FULL>
  __device__ __forceinline__ bool fwd_tile(State<D, C>& st, Spike& sp, double (&G)[NY], double (&h)[D][C],
                                           const Tile& tl, int t0, bool first, bool sepR, int& nobs) const {
    bool ok = true;
#pragma unroll
    for (int s = 0; s < B; ++s) {
      const int t = t0 + s;
      double om[D + 1], l[D + 1], dt, invdt, b[C], yt[C], vt[D];
      factor_row<FULL>(st, tl, s, t, om, l, dt, invdt, b);
      fwd_step<D, C>(st, l, b, yt);
#pragma unroll
      for (int q = 0; q < D; ++q) {
        double a = 0.0;
        if (s < D && q >= s) a = first ? om[s + D - q < D ? s + D - q : D] : 0.0;
#pragma unroll
        for (int j = 1; j <= D; ++j) a = __builtin_fma(-l[j], sp.v[j][q], a);
        vt[q] = a;
      }
#pragma unroll
      for (int j = D; j >= 2; --j)
#pragma unroll
        for (int q = 0; q < D; ++q) sp.v[j][q] = sp.v[j - 1][q];
#pragma unroll
      for (int q = 0; q < D; ++q) sp.v[1][q] = vt[q];
      const bool in = FULL || t < T;
      // rows past the series (their values are not finite) and the separator's
      // own rows stay out of the interior's sums
      const double iv = (in && !(s >= B - D && sepR)) ? invdt : 0.0;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const double vq = in ? vt[q] : 0.0;
        const double pq = vq * iv;
#pragma unroll
        for (int q2 = 0; q2 <= q; ++q2)
          G[tri2(q, q2)] = __builtin_fma(pq, in ? vt[q2] : 0.0, G[tri2(q, q2)]);
#pragma unroll
        for (int c = 0; c < C; ++c) h[q][c] = __builtin_fma(pq, in ? yt[c] : 0.0, h[q][c]);
      }
      nobs += wt(tl, s) ? 1 : 0;
      ok = ok & (pivot_good(dt) | !in);
    }
    return ok;
  }

  // Schur term, right-hand side and coupling of this segment on the separator
  // that follows, and its interior sums, into LDS
  __device__ __forceinline__ void publish(const State<D, C>& st, const Spike& sp, const double (&G)[NY],
                                          const double (&h)[D][C], double* xs) const {
    double L[D][D], Dp[D];
#pragma unroll
    for (int u = 0; u < D; ++u) {
#pragma unroll
      for (int q = 0; q < D; ++q) L[u][q] = q == u ? 1.0 : 0.0;
      Dp[u] = 1.0 / st.invD[D - u];
    }
#pragma unroll
    for (int jj = 1; jj < D; ++jj)
#pragma unroll
      for (int k = 1; k <= D - jj; ++k) L[D - jj][D - jj - k] = st.R[jj][k];
#pragma unroll
    for (int u = 0; u < D; ++u) {
#pragma unroll
      for (int u2 = 0; u2 <= u; ++u2) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q <= u2; ++q) a = __builtin_fma(L[u][q] * Dp[q], L[u2][q], a);
        xs[(fY + tri2(u, u2)) * NT] = a;
      }
#pragma unroll
      for (int c = 0; c < C; ++c) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q <= u; ++q) a = __builtin_fma(L[u][q], st.y[D - q][c], a);
        xs[(fC + u * C + c) * NT] = a;
      }
#pragma unroll
      for (int w2 = 0; w2 < D; ++w2) {
        double a = 0.0;
#pragma unroll
        for (int q = 0; q <= u; ++q) a = __builtin_fma(L[u][q], sp.v[D - q][w2], a);
        xs[(fF + u * D + w2) * NT] = a;
      }
    }
#pragma unroll
    for (int i = 0; i < NY; ++i) xs[(fG + i) * NT] = G[i];
#pragma unroll
    for (int q = 0; q < D; ++q)
#pragma unroll
      for (int c = 0; c < C; ++c) xs[(fH + q * C + c) * NT] = h[q][c];
  }

  // Block-tridiagonal solve over the separators of one series (block LDL').
  // xs: the series' LDS column; sw: lanes between two segments.  Leaves z of
  // separator s in the c fields of segment s; false if a pivot fails.
  __device__ __forceinline__ bool interface_solve(double* xs, int sw, int ne) const {
    bool ok = true;
    double Lp[D][D], Di[D], q[D][C];  // unit factor, inverse pivots and L^-1 r of the separator before
    for (int s = 0; s + 1 < ne; ++s) {
      double* x0 = xs + s * sw;
      const double* x1 = x0 + sw;
      double A[NY], r[D][C];
#pragma unroll
      for (int i = 0; i < NY; ++i) A[i] = x0[(fY + i) * NT] - x1[(fG + i) * NT];
#pragma unroll
      for (int u = 0; u < D; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c)
          r[u][c] = x0[(fC + u * C + c) * NT] - x1[(fH + u * C + c) * NT];
      if (s > 0) {
        double U[D][D];  // rows of F Lp^-T
#pragma unroll
        for (int u = 0; u < D; ++u)
#pragma unroll
          for (int k = 0; k < D; ++k) {
            double a = x0[(fF + u * D + k) * NT];
#pragma unroll
            for (int m = 0; m < k; ++m) a = __builtin_fma(-U[u][m], Lp[k][m], a);
            U[u][k] = a;
          }
#pragma unroll
        for (int u = 0; u < D; ++u)
#pragma unroll
          for (int k = 0; k < D; ++k) {
            const double ud = U[u][k] * Di[k];
#pragma unroll
            for (int u2 = 0; u2 <= u; ++u2) A[tri2(u, u2)] = __builtin_fma(-ud, U[u2][k], A[tri2(u, u2)]);
#pragma unroll
            for (int c = 0; c < C; ++c) r[u][c] = __builtin_fma(-ud, q[k][c], r[u][c]);
          }
      }
#pragma unroll
      for (int u = 0; u < D; ++u) {
#pragma unroll
        for (int k = 0; k < u; ++k) {
          double a = A[tri2(u, k)];
#pragma unroll
          for (int m = 0; m < k; ++m) a = __builtin_fma(-Lp[u][m] * A[tri2(m, m)], Lp[k][m], a);
          Lp[u][k] = a * Di[k];
        }
        double dd = A[tri2(u, u)];
#pragma unroll
        for (int m = 0; m < u; ++m) dd = __builtin_fma(-Lp[u][m] * A[tri2(m, m)], Lp[u][m], dd);
        A[tri2(u, u)] = dd;  // the pivot
        ok = ok & pivot_good(dd);
        Di[u] = rcp64(dd);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          double a = r[u][c];
#pragma unroll
          for (int m = 0; m < u; ++m) a = __builtin_fma(-Lp[u][m], q[m][c], a);
          q[u][c] = a;
        }
      }
#pragma unroll
      for (int u = 0; u < D; ++u) {
#pragma unroll
        for (int k = 0; k < u; ++k) x0[(fY + tri2(u, k)) * NT] = Lp[u][k];
        x0[(fY + tri2(u, u)) * NT] = Di[u];
#pragma unroll
        for (int c = 0; c < C; ++c) x0[(fC + u * C + c) * NT] = q[u][c];
      }
    }
    double z[D][C];
#pragma unroll
    for (int u = 0; u < D; ++u)
#pragma unroll
      for (int c = 0; c < C; ++c) z[u][c] = 0.0;
    for (int s = ne - 2; s >= 0; --s) {
      double* x0 = xs + s * sw;
      const double* x1 = x0 + sw;
      double Lc[D][D], p[D][C];
#pragma unroll
      for (int u = 0; u < D; ++u)
#pragma unroll
        for (int k = 0; k < u; ++k) Lc[u][k] = x0[(fY + tri2(u, k)) * NT];
      // p = L^-1 (r - F' z) = q - L^-1 F' z
#pragma unroll
      for (int c = 0; c < C; ++c) {
        double fz[D];
#pragma unroll
        for (int u = 0; u < D; ++u) {
          double a = 0.0;
          if (s + 2 < ne) {
#pragma unroll
            for (int k = 0; k < D; ++k) a = __builtin_fma(x1[(fF + k * D + u) * NT], z[k][c], a);
          }
#pragma unroll
          for (int m = 0; m < u; ++m) a = __builtin_fma(-Lc[u][m], fz[m], a);
          fz[u] = a;
          p[u][c] = (x0[(fC + u * C + c) * NT] - a) * x0[(fY + tri2(u, u)) * NT];
        }
#pragma unroll
        for (int u = D - 1; u >= 0; --u) {
          double a = p[u][c];
#pragma unroll
          for (int m = u + 1; m < D; ++m) a = __builtin_fma(-Lc[m][u], z[m][c], a);
          z[u][c] = a;
        }
      }
#pragma unroll
      for (int u = 0; u < D; ++u)
#pragma unroll
        for (int c = 0; c < C; ++c) x0[(fC + u * C + c) * NT] = z[u][c];
    }
    return ok;
  }

  // -(D u)_t . (D z)_t from row t's values and the windows of the rows after it
  __device__ __forceinline__ double grad_row(const double (&zt)[C], const double (&zin)[C],
                                             const double (&zn)[D + 1][C], const double (&xn)[D + 1][C]) const {
    double gt = 0.0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      double du = cdiff<D>(0) * zt[c];
      double dz = cdiff<D>(0) * zin[c];
#pragma unroll
      for (int i = 1; i <= D; ++i) {
        du = __builtin_fma(cdiff<D>(i), zn[i][c], du);
        dz = __builtin_fma(cdiff<D>(i), xn[i][c], dz);
      }
      gt = __builtin_fma(-du, dz, gt);
    }
    return gt;
  }

  static __device__ __forceinline__ void shift_in(double (&win)[D + 1][C], const double (&v)[C]) {
#pragma unroll
    for (int i = D; i >= 2; --i)
#pragma unroll
      for (int c = 0; c < C; ++c) win[i][c] = win[i - 1][c];
#pragma unroll
    for (int c = 0; c < C; ++c) win[1][c] = v[c];
  }

  __device__ __forceinline__ void store_grad(int t, bool skip, bool failed, double gt, double& gsum) const {
    if constexpr (PERDIFF) {
      const uint32_t o = skip ? kDead : ll + (uint32_t)t * Rl;
      const double prev = accum ? to_f64(bload<TS>(rg, o)) : 0.0;
      bstore<TS, kStream>(rg, o, from_f64<TS>(failed ? __builtin_nan("") : prev + gt));
    } else {
      gsum += (!skip && t < T - D) ? gt : 0.0;
    }
  }

  template <bool FULL>
  __device__ __forceinline__ void rev_tile(State<D, C>& st, const Tile& tl, int t0, bool first, bool sepR,
                                           const double (&zL)[D][C], const double (&zR)[D][C], double (&zn)[D + 1][C], double (&xn)[D + 1][C],
                                           double (&lc_)[D + 1][D + 1], bool failed, bool out, bool grad,
                                           double& gsum) const {
    double lt[B][D + 1];
    double yd[B][C];
#pragma unroll
    for (int s = 0; s < B; ++s) {
      const int t = t0 + s;
      double om[D + 1], l[D + 1], dt, invdt, b[C], yt[C];
      factor_row<FULL>(st, tl, s, t, om, l, dt, invdt, b);
      if (s < D) {  // the segment's first rows see the separator before it
#pragma unroll
        for (int q = s; q < D; ++q) {
          const double e = first ? om[s + D - q < D ? s + D - q : D] : 0.0;
#pragma unroll
          for (int c = 0; c < C; ++c) b[c] = __builtin_fma(-e, zL[q][c], b[c]);
        }
      }
      fwd_step<D, C>(st, l, b, yt);
      const bool v = FULL || t < T;
#pragma unroll
      for (int i = 1; i <= D; ++i) lt[s][i] = v ? l[i] : 0.0;
#pragma unroll
      for (int c = 0; c < C; ++c) yd[s][c] = v ? yt[c] * invdt : 0.0;
    }
    const double qnan = __builtin_nan("");
    const uint32_t ox = lx + (uint32_t)t0 * Rx;
#pragma unroll
    for (int s = B - 1; s >= 0; --s) {
      const int t = t0 + s;
      const bool in = FULL || t < T;
      double zt[C];
#pragma unroll
      for (int c = 0; c < C; ++c) {
        double acc = yd[s][c];
#pragma unroll
        for (int i = 1; i <= D; ++i) {
          const double li = (s + i < B) ? lt[s + i < B ? s + i : 0][i] : lc_[s + i - B < 0 ? 0 : s + i - B][i];
          acc = __builtin_fma(-li, zn[i][c], acc);
        }
        if (s >= B - D) acc = sepR ? zR[s - (B - D) < 0 ? 0 : s - (B - D)][c] : acc;
        zt[c] = acc;
      }
      if constexpr (!BWD) {
#pragma unroll
        for (int c = 0; c < C; ++c)
          bstore<TS, kStream>(ro, ox + (uint32_t)s * Rx + (uint32_t)c * Sb, from_f64<TS>(failed ? qnan : zt[c]));
      } else {
        if (out) {
          const bool obs = wt(tl, s);
#pragma unroll
          for (int c = 0; c < C; ++c)
            bstore<TS, kStream>(ro, ox + (uint32_t)s * Rx + (uint32_t)c * Sb,
                                from_f64<TS>(failed ? qnan : (obs ? zt[c] : 0.0)));
        }
        if (grad) {
          double zin[C];
#pragma unroll
          for (int c = 0; c < C; ++c) zin[c] = to_f64(tl.z[s][c]);
          // the separator's rows need rows of the next segment: its lane has them
          store_grad(t, s >= B - D && sepR, failed, grad_row(zt, zin, zn, xn), gsum);
          if (in) shift_in(xn, zin);
        }
      }
      if (in) shift_in(zn, zt);
    }
#pragma unroll
    for (int r = 0; r < D; ++r)
#pragma unroll
      for (int i = 0; i <= D; ++i) lc_[r][i] = lt[r][i];
  }

  // exact index of the first failing pivot of the whole series, time order (rare)
  __device__ int first_bad_pivot() const {
    State<D, C> st;
    st.zero();
    for (int t = 0; t < T; ++t) {
      bool obs;
      if constexpr (WB) obs = (__builtin_amdgcn_raw_buffer_load_b32(rw, lw + (uint32_t)t * Rw, 0, 0) >> bit) & 1u;
      else obs = __builtin_amdgcn_raw_buffer_load_b8(rw, lw + (uint32_t)t * Rw, 0, 0) != 0;
      const double ltv = PERDIFF ? to_f64(bload<TS>(rl, ll + (uint32_t)t * Rl)) : (t < T - D ? lam_scalar : 0.0);
      double lwv[D + 1];
      lwv[0] = ltv;
      for (int q = 1; q <= D; ++q) lwv[q] = st.lw[q];
      double om[D + 1], l[D + 1], dt, invdt;
      omega_row<D>(lwv, obs ? 1.0 : 0.0, om);
      ldl_step<D, C>(st, om, l, dt, invdt);
      for (int q = D; q >= 2; --q) st.lw[q] = st.lw[q - 1];
      st.lw[1] = ltv;
      if (!pivot_good(dt)) return t + 1;
    }
    return 0;
  }

  __device__ __forceinline__ void run(const SegArgs& g, double* xs_all, int* nobs_all, int* flag_all) {
    const FastArgs& a = g.f;
    const int tid = threadIdx.x;
    const int SW = 1 << g.sw_log2;
    const int s_wg = tid & (SW - 1), seg = tid >> g.sw_log2;
    // workgroups that share 64-series rows run on one XCD (dispatch is round-robin over 8)
    int wg = blockIdx.x;
    if (g.sw_log2 < 6 && gridDim.x % 8 == 0) wg = (wg & 7) * (gridDim.x >> 3) + (wg >> 3);
    const int64_t p0 = (int64_t)wg << g.sw_log2;
    const int64_t bidx = p0 >> 6;
    const int s_in = (int)(p0 & 63) + s_wg;
    const int64_t p = p0 + s_wg;
    T = a.T;
    tps = g.tps;
    const int ctot = C == 1 && !MB ? 1 : a.Ctot;
    Rx = C == 1 && !MB ? Sb : (uint32_t)a.Ctot * Sb;
    accum = a.glam_accum != 0;
    const uint32_t xbytes = (uint32_t)T * Rx, lbytes = (uint32_t)(T - D) * Rl;
    rx = make_rsrc(static_cast<const TS*>(a.rhs) + bidx * T * ctot * 64, xbytes);
    rw = make_rsrc(a.w + bidx * T * (int64_t)Rw, (uint32_t)T * Rw);
    rl = make_rsrc(PERDIFF ? (const void*)(static_cast<const TS*>(a.lam) + bidx * (T - D) * 64) : (const void*)a.w,
                   PERDIFF ? lbytes : 0u);
    const bool out = a.out != nullptr, grad = BWD && a.glam != nullptr;
    ro = make_rsrc(out ? (const void*)(static_cast<TS*>(a.out) + bidx * T * ctot * 64) : (const void*)a.w,
                   out ? xbytes : 0u);
    if constexpr (BWD) {
      rz = make_rsrc(static_cast<const TS*>(a.zin) + bidx * T * ctot * 64, grad ? xbytes : 0u);
      rg = make_rsrc(grad && PERDIFF ? (const void*)(static_cast<TS*>(a.glam) + bidx * (T - D) * 64) : (const void*)a.w,
                     grad && PERDIFF ? lbytes : 0u);
    }
    const uint32_t ckbytes = (uint32_t)(tps - 1) * NF * ckrow;
    rck = make_rsrc(a.ck + (int64_t)wg * (ckbytes / 8), ckbytes);
    const bool live = p < a.P && seg < g.ne;
    const uint32_t l0 = (uint32_t)s_in * ES;
    lx = live ? l0 + (MB ? (uint32_t)a.c0 * Sb : 0u) : kDead;
    ll = live ? l0 : kDead;
    lw = live ? (WB ? ((uint32_t)s_in >> 5) << 2 : (uint32_t)s_in) : kDead;
    bit = (uint32_t)s_in & 31u;
    lc = (uint32_t)tid * 8u;
    r0 = live ? seg * tps * B : 0;
    hasR = live && seg + 1 < g.ne;
    lam_scalar = (!PERDIFF && p < a.P) ? to_f64(static_cast<const TS*>(a.lam)[p]) : 0.0;

    // every lane's rows of tile j lie inside [0, T - D): no masks
    const int seg_hi = __builtin_amdgcn_readfirstlane((tid | 63) >> g.sw_log2);  // last segment of this wavefront
    const int full_to = seg_hi < g.ne ? (T - D - seg_hi * tps * B) / B : 0;      // tiles j < full_to are full

    // ---------------- sweep 1 ----------------
    State<D, C> st;
    Spike sp;
    double G[NY], h[D][C];
    st.zero();
    load_window(r0, st.lw);
#pragma unroll
    for (int j = 0; j <= D; ++j)
#pragma unroll
      for (int q = 0; q < D; ++q) sp.v[j][q] = 0.0;
#pragma unroll
    for (int i = 0; i < NY; ++i) G[i] = 0.0;
#pragma unroll
    for (int q = 0; q < D; ++q)
#pragma unroll
      for (int c = 0; c < C; ++c) h[q][c] = 0.0;
    int nobs = 0;
    bool ok = true;
    Tile A, Bt;
    load_tile<false>(A, 0);
    for (int j = 0; j < tps; j += 2) {
      if (j + 1 < tps) load_tile<false>(Bt, j + 1);
      if (j > 0) store_ck(st, sp, j);
      ok &= j < full_to ? fwd_tile<true>(st, sp, G, h, A, r0 + j * B, j == 0, hasR && j == tps - 1, nobs)
                        : fwd_tile<false>(st, sp, G, h, A, r0 + j * B, j == 0, hasR && j == tps - 1, nobs);
      if (j + 1 < tps) {
        if (j + 2 < tps) load_tile<false>(A, j + 2);
        store_ck(st, sp, j + 1);
        ok &= j + 1 < full_to ? fwd_tile<true>(st, sp, G, h, Bt, r0 + (j + 1) * B, false, hasR && j + 1 == tps - 1, nobs)
                              : fwd_tile<false>(st, sp, G, h, Bt, r0 + (j + 1) * B, false, hasR && j + 1 == tps - 1,
                                                nobs);
      }
    }

    // ---------------- interface ----------------
    publish(st, sp, G, h, xs_all + tid);
    nobs_all[tid] = nobs;
    flag_all[tid] = (ok || !live) ? 0 : 1;
    int j = tps - 1;
    load_tile<true>(A, j);  // in flight across the interface
    __syncthreads();
    if (seg == 0) {
      bool good = interface_solve(xs_all + tid, SW, g.ne);
      int n = 0;
      for (int k = 0; k < g.ne; ++k) {
        n += nobs_all[tid + k * SW];
        good &= flag_all[tid + k * SW] == 0;
      }
      good &= n >= D;
      int info = 0;
      if (!good && p < a.P) {
        info = first_bad_pivot();
        if (info == 0) info = T;  // too few observations, or an interface pivot lost to rounding
      }
      if (p < a.P && a.info && a.write_info) a.info[p] = info;
      flag_all[tid] = info != 0;
    }
    __syncthreads();
    const bool failed = flag_all[s_wg] != 0;
    double zL[D][C], zR[D][C];
#pragma unroll
    for (int u = 0; u < D; ++u)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        zL[u][c] = seg > 0 && live ? xs_all[(fC + u * C + c) * NT + tid - SW] : 0.0;
        zR[u][c] = hasR ? xs_all[(fC + u * C + c) * NT + tid] : 0.0;
      }

    // ---------------- sweep 2 ----------------
    double zn[D + 1][C], xn[D + 1][C], lcr[D + 1][D + 1];
#pragma unroll
    for (int i = 0; i <= D; ++i) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        zn[i][c] = 0.0;
        xn[i][c] = 0.0;
      }
#pragma unroll
      for (int k = 0; k <= D; ++k) lcr[i][k] = 0.0;
    }
    double gsum = 0.0;
    double ck[NF], lwin[D + 1];
    load_ck(j, ck, lwin);
    for (; j >= 0; j -= 2) {
      if (j >= 1) load_tile<true>(Bt, j - 1);
      restore(st, ck, lwin, zL);
      if (j >= 1) load_ck(j - 1, ck, lwin);
      if (j < full_to)
        rev_tile<true>(st, A, r0 + j * B, j == 0, hasR && j == tps - 1, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
      else
        rev_tile<false>(st, A, r0 + j * B, j == 0, hasR && j == tps - 1, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
      if (j >= 1) {
        if (j >= 2) load_tile<true>(A, j - 2);
        restore(st, ck, lwin, zL);
        if (j >= 2) load_ck(j - 2, ck, lwin);
        if (j - 1 < full_to)
          rev_tile<true>(st, Bt, r0 + (j - 1) * B, j == 1, false, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        else
          rev_tile<false>(st, Bt, r0 + (j - 1) * B, j == 1, false, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
      }
    }
    if constexpr (BWD) {
      if (grad) {
        // grad_lambda of the separator before this segment
        const bool skip = !live || seg == 0;
#pragma unroll
        for (int u = D - 1; u >= 0; --u) {
          const int t = r0 - D + u;
          double zin[C], zt[C];
#pragma unroll
          for (int c = 0; c < C; ++c) {
            zin[c] = to_f64(bload<TS>(rz, skip ? kDead : lx + (uint32_t)t * Rx + (uint32_t)c * Sb));
            zt[c] = zL[u][c];
          }
          store_grad(t, skip, failed, grad_row(zt, zin, zn, xn), gsum);
          shift_in(zn, zt);
          shift_in(xn, zin);
        }
        if constexpr (!PERDIFF) {
          // the segments' sums, added in segment order
          __syncthreads();
          xs_all[tid] = gsum;
          __syncthreads();
          if (seg == 0 && p < a.P) {
            double sum = 0.0;
            for (int k = 0; k < g.ne; ++k) sum += xs_all[tid + k * SW];
            TS* gp = static_cast<TS*>(a.glam) + p;
            const double prev = accum ? to_f64(*gp) : 0.0;
            *gp = from_f64<TS>(failed ? __builtin_nan("") : prev + sum);
          }
        }
      }
    }
  }
};

template <int D, int C, int B, typename TS, bool BWD, bool PERDIFF, bool WB, int NT, bool MB = false>
__global__ __launch_bounds__(NT, 1) void k_seg(SegArgs g) {
  using K = Seg<D, C, B, TS, BWD, PERDIFF, WB, NT, MB>;
  __shared__ double xs[K::NX * NT];
  __shared__ int nobs[NT];
  __shared__ int flag[NT];
  K k;
  k.run(g, xs, nobs, flag);
}

}  // namespace whs
