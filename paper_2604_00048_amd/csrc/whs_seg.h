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

template <int D, int C, int B, typename TS, bool BWD, bool PERDIFF, bool WB, int NT, bool MB = false, bool CT = false>
struct Seg {
  static constexpr int NF = seg_fields<D, C>();
  static constexpr int NY = D * (D + 1) / 2;
  // LDS fields of one lane: Y, c, F, G, h
  static constexpr int fY = 0, fC = NY, fF = fC + D * C, fG = fF + D * D, fH = fG + NY, NX = fH + D * C;
  static constexpr uint32_t ES = sizeof(TS);
  static constexpr uint32_t kDead = 0x80000000u;

  static constexpr bool BITS = WB || CT;  // a tile's weights as the bits of one register

  struct Tile {
    TS x[B][C];
    uint32_t w[BITS ? 1 : B];
    uint32_t wm;
    TS lam[B];
  };
  struct Spike {
    double v[D + 1][D];  // v[j][c]: column c at row t - j
  };

  // wave-uniform
  __amdgpu_buffer_rsrc_t rx, rw, rl, rz, ro, rg, rck, rwm;
  int T, tps;
  uint32_t Rx;  // bytes per row of x, all bands (a constant for one band alone)
  // blocks of 64 series (CT: one series): bytes between two bands of a row, and
  // per row of lambda, of w and of one checkpoint field
  static constexpr uint32_t Sb = CT ? ES : 64u * ES, Rl = Sb, Rw = CT ? 1u : WB ? 8u : 64u, ckrow = NT * 8u;
  static_assert(!CT || (C == 1 && !MB && !WB && ES == 4 && (B + 3) / 4 == 6), "series-contiguous: one band, 6 quads");
  // per lane
  uint32_t lx, ll, lw, lc, bit;
  int r0;               // first row of the segment
  bool hasR;            // a separator follows
  double lam_scalar;
  bool accum;

  static __device__ __forceinline__ int tri2(int r, int q) { return r * (r + 1) / 2 + q; }

  static __device__ __forceinline__ bool wt(const Tile& tl, int s) {
    if constexpr (BITS) return (tl.wm >> s) & 1u;
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
  }

  // ---- series-contiguous arrays (CT) ----
  // A lane's tile is B consecutive values of its own row, so a wavefront reads
  // it as 64 row pieces of 6 quads: 16 bytes per lane, 6 lanes to a piece (96
  // contiguous bytes), into registers a tile ahead; on use the quads go through
  // LDS (36-word pitch: both sides without bank conflicts) and each lane takes
  // its piece.  w arrives as the aligned dwords that hold the piece, shifted to
  // its first byte and reduced to one bit per row.  Results leave the same way.
  // Tiles that are not full, the last D rows of the adjoint's separator
  // (stored by the next segment's lane) and the windows of lambda are read and
  // written row by row.
  typedef uint32_t quad __attribute__((ext_vector_type(4)));
  static constexpr int kPitch = 36;  // words
  struct Raw {
    quad x[6], lam[PERDIFF ? 6 : 1];
    uint32_t w[8];  // sweep 2: w[0], the tile's bits as sweep 1 stored them
  };
  uint32_t xo[3], lo[3], so[3];      // byte offsets of this lane's quads of pieces 0..31, and its LDS words
  uint32_t dx, dl;                   // bytes from piece n to n + 32
  uint32_t wo, wmis;                 // byte offset of this lane's w dwords of pieces 0..7; misalignment of the base
  int sw_log2;
  uint32_t* stage;                   // this wavefront's LDS: input, out, grad

  __device__ __forceinline__ uint32_t w_step(int i) const {  // bytes of w from piece n to n + 8 i
    return ((8 * i) >> sw_log2) * (uint32_t)(tps * B) + ((8 * i) & ((1 << sw_log2) - 1)) * (uint32_t)T;
  }
  template <bool SWEEP2>
  __device__ __forceinline__ void load_raw(Raw& r, int j) const {
    constexpr int POL = kKeep;
    const uint32_t o = (uint32_t)(j * B) * ES;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      r.x[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, xo[i % 3] + (i < 3 ? 0u : dx) + o, 0, POL);
      if constexpr (PERDIFF)
        r.lam[i] = __builtin_amdgcn_raw_buffer_load_b128(rl, lo[i % 3] + (i < 3 ? 0u : dl) + o, 0, POL);
    }
    if constexpr (SWEEP2) return;
    const uint32_t k = (threadIdx.x & 7u) * 4u;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      r.w[i] = __builtin_amdgcn_raw_buffer_load_b32(rw, ((wo + w_step(i) + (uint32_t)(j * B)) & ~3u) + k, 0, POL);
  }
  static __device__ __forceinline__ void lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
  }
  template <int N>
  __device__ __forceinline__ void turn(const quad (&q)[6], TS (&out)[N][1]) const {
    const int lane = threadIdx.x & 63;
    lds_order();
#pragma unroll
    for (int i = 0; i < 6; ++i) *(quad*)(stage + so[i % 3] + (i < 3 ? 0 : 32 * kPitch)) = q[i];
    lds_order();
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const quad v = *(const quad*)(stage + lane * kPitch + 4 * k);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * k + e < N) out[4 * k + e < N ? 4 * k + e : 0][0] = __builtin_bit_cast(TS, (uint32_t)v[e]);
    }
  }
  // four bytes of w as four bits
  static __device__ __forceinline__ uint32_t byte_bits(uint32_t v) {
    const uint32_t t = (((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) & 0x80808080u;  // bit 7 of every byte that is not 0
    return ((t >> 7) * 0x10204080u) >> 28;
  }
  // the bits of w of every tile, kept between the sweeps: 4 bytes per tile of
  // whole lines instead of 24 bytes of one line per lane
  __device__ __forceinline__ uint32_t load_bits(int j) const {
    return __builtin_amdgcn_raw_buffer_load_b32(rwm, (uint32_t)(j * NT + threadIdx.x) * 4u, 0, kStream);
  }
  __device__ __forceinline__ void store_bits(int j, uint32_t wm) const {
    __builtin_amdgcn_raw_buffer_store_b32(wm, rwm, (uint32_t)(j * NT + threadIdx.x) * 4u, 0, kStream);
  }
  template <bool SWEEP2>
  __device__ __forceinline__ void settle(const Raw& r, Tile& tl, int j, bool full) const {
    const int lane = threadIdx.x & 63;
    const int t0 = r0 + j * B;
    if (full) {
      turn(r.x, tl.x);
      if constexpr (PERDIFF) {
        TS v[B][1];
        turn(r.lam, v);
#pragma unroll
        for (int s = 0; s < B; ++s) tl.lam[s] = v[s][0];
      }
      if constexpr (SWEEP2) return;
      lds_order();
#pragma unroll
      for (int i = 0; i < 8; ++i) stage[(i * 8 + (lane >> 3)) * 9 + (lane & 7)] = r.w[i];
      lds_order();
      const uint32_t sh = ((lw + wmis + (uint32_t)t0) & 3u) * 8u;
      uint32_t d[7];
#pragma unroll
      for (int k = 0; k < 7; ++k) d[k] = stage[lane * 9 + k];
      tl.wm = 0u;
#pragma unroll
      for (int k = 0; k < 6; ++k) tl.wm |= byte_bits(__builtin_amdgcn_alignbit(d[k + 1], d[k], sh)) << (4 * k);
    } else {
      if constexpr (!SWEEP2) tl.wm = 0u;
#pragma unroll
      for (int s = 0; s < B; ++s) {
        const int t = t0 + s;
        const bool in = t < T && lx != kDead;
        tl.x[s][0] = bload<TS>(rx, in ? lx + (uint32_t)t * Rx : kDead);
        if constexpr (PERDIFF) tl.lam[s] = bload<TS>(rl, in && t < T - D ? ll + (uint32_t)t * Rl : kDead);
        if constexpr (!SWEEP2) {
          const uint32_t b = __builtin_amdgcn_raw_buffer_load_b8(rw, in ? lw + wmis + (uint32_t)t : kDead, 0, 0);
          tl.wm |= (b != 0u ? 1u : 0u) << s;
        }
      }
    }
  }
  // result of row s of the current tile into the wavefront's LDS: which = 1 out, 2 grad
  __device__ __forceinline__ void put(int which, int s, TS v) const {
    stage[which * 64 * kPitch + (threadIdx.x & 63) * kPitch + s] = __builtin_bit_cast(uint32_t, v);
  }
  // the tile's results from LDS to memory; rows: of the array, skip: last rows of a separator stored elsewhere
  __device__ __forceinline__ void flush(int which, __amdgpu_buffer_rsrc_t r, const uint32_t (&off)[3], uint32_t d32,
                                        uint32_t own, int j, bool whole, int rows, int skip) const {
    const uint32_t* st = stage + which * 64 * kPitch;
    const int lane = threadIdx.x & 63;
    lds_order();
    if (whole) {
      const uint32_t o = (uint32_t)(j * B) * ES;
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        const uint32_t a = off[i % 3] + (i < 3 ? 0u : d32) + o;
        const quad v = *(const quad*)(st + so[i % 3] + (i < 3 ? 0 : 32 * kPitch));
        if constexpr (B == 24) {
          __builtin_amdgcn_raw_buffer_store_b128(v, r, a, 0, kKeep);
        } else {  // B = 22: the last quad of a piece holds two rows
          static_assert(!CT || B == 24 || B == 22, "tail quad");
          typedef uint32_t pair2 __attribute__((ext_vector_type(2)));
          const bool tail = (uint32_t)(i % 3 * 64 + lane) % 6u == 5u;
          __builtin_amdgcn_raw_buffer_store_b128(v, r, tail ? kDead : a, 0, kKeep);
          __builtin_amdgcn_raw_buffer_store_b64(pair2{v[0], v[1]}, r, tail ? a : kDead, 0, kKeep);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < B; ++s) {
        const int t = r0 + j * B + s;
        const bool ok = t < rows && own != kDead && s < B - skip;
        __builtin_amdgcn_raw_buffer_store_b32(st[lane * kPitch + s], r, ok ? own + (uint32_t)t * ES : kDead, 0, kKeep);
      }
    }
    lds_order();
  }

  // lambda of the D rows before row t0
  __device__ __forceinline__ void load_window(int t0, double (&lwin)[D + 1]) const {
    lwin[0] = 0.0;
#pragma unroll
    for (int m = 1; m <= D; ++m) {
      const int k = t0 - m;
      if constexpr (PERDIFF) {
        lwin[m] = to_f64(bload<TS>(rl, k >= 0 && (!CT || (k < T - D && ll != kDead)) ? ll + (uint32_t)k * Rl : kDead));
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
  __device__ __forceinline__ void factor_row(State<D, C>& st, const Tile& tl, bool obs, int s, int t,
                                             double (&om)[D + 1], double (&l)[D + 1], double& dt, double& invdt,
                                             double (&b)[C]) const {
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
      factor_row<FULL>(st, tl, wt(tl, s), s, t, om, l, dt, invdt, b);
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
      const uint32_t o = skip || (CT && t >= T - D) ? kDead : ll + (uint32_t)t * Rl;
      const double prev = accum ? to_f64(bload<TS>(rg, o)) : 0.0;
      bstore<TS, kStream>(rg, o, from_f64<TS>(failed ? __builtin_nan("") : prev + gt));
    } else {
      gsum += (!skip && t < T - D) ? gt : 0.0;
    }
  }

  template <bool FULL>
  __device__ __forceinline__ void rev_tile(State<D, C>& st, const Tile& tl, int j, bool first, bool sepR,
                                           const double (&zL)[D][C], const double (&zR)[D][C], double (&zn)[D + 1][C], double (&xn)[D + 1][C],
                                           double (&lc_)[D + 1][D + 1], bool failed, bool out, bool grad,
                                           double& gsum) const {
    const int t0 = r0 + j * B;
    const uint32_t ox = lx + (uint32_t)t0 * Rx;
    // z is used from the back substitution on: its loads (dropped by an empty
    // range where no grad_lambda is wanted) return during the factorisation
    TS tz[BWD ? B : 1][C];
    quad rq[6];
    if constexpr (BWD) {
      if constexpr (CT && FULL) {
#pragma unroll
        for (int i = 0; i < 6; ++i)
          rq[i] = __builtin_amdgcn_raw_buffer_load_b128(rz, xo[i % 3] + (i < 3 ? 0u : dx) + (uint32_t)(j * B) * ES, 0,
                                                        kKeep);
      } else {
#pragma unroll
        for (int s = 0; s < B; ++s)
#pragma unroll
          for (int c = 0; c < C; ++c)
            tz[s][c] = bload<TS, kStream>(rz, !CT || (t0 + s < T && lx != kDead)
                                                  ? ox + (uint32_t)s * Rx + (uint32_t)c * Sb : kDead);
      }
    }
    double lt[B][D + 1];
    double yd[B][C];
#pragma unroll
    for (int s = 0; s < B; ++s) {
      const int t = t0 + s;
      double om[D + 1], l[D + 1], dt, invdt, b[C], yt[C];
      factor_row<FULL>(st, tl, wt(tl, s), s, t, om, l, dt, invdt, b);
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
    if constexpr (BWD && CT && FULL) turn(rq, tz);
    const double qnan = __builtin_nan("");
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
        for (int c = 0; c < C; ++c) {
          const TS v = from_f64<TS>(failed ? qnan : zt[c]);
          if constexpr (CT) put(1, s, v);
          else bstore<TS, kStream>(ro, ox + (uint32_t)s * Rx + (uint32_t)c * Sb, v);
        }
      } else {
        if (out) {
          const bool obs = wt(tl, s);
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const TS v = from_f64<TS>(failed ? qnan : (obs ? zt[c] : 0.0));
            if constexpr (CT) put(1, s, v);
            else bstore<TS, kStream>(ro, ox + (uint32_t)s * Rx + (uint32_t)c * Sb, v);
          }
        }
        if (grad) {
          double zin[C];
#pragma unroll
          for (int c = 0; c < C; ++c) zin[c] = to_f64(tz[s][c]);
          // the separator's rows need rows of the next segment: its lane has them
          const double gt = grad_row(zt, zin, zn, xn);
          if constexpr (CT && PERDIFF) put(2, s, from_f64<TS>(failed ? qnan : gt));
          else store_grad(t, s >= B - D && sepR, failed, gt, gsum);
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
      else obs = __builtin_amdgcn_raw_buffer_load_b8(rw, lw + (CT ? wmis : 0u) + (uint32_t)t * Rw, 0, 0) != 0;
      const double ltv = PERDIFF ? to_f64(bload<TS>(rl, !CT || t < T - D ? ll + (uint32_t)t * Rl : kDead))
                                 : (t < T - D ? lam_scalar : 0.0);
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

  __device__ __forceinline__ void run(const SegArgs& g, double* xs_all, int* nobs_all, int* flag_all,
                                      uint32_t* stage_all) {
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
    // the arrays of this workgroup's block of 64 series (CT: of its own series)
    const int64_t b0 = CT ? p0 : bidx;
    const int64_t rows = CT ? (a.P - p0 < SW ? a.P - p0 : (int64_t)SW) : 1;
    const int64_t xn_ = (int64_t)T * ctot * (CT ? 1 : 64), ln_ = (int64_t)(T - D) * (CT ? 1 : 64);
    const uint32_t xbytes = (uint32_t)(rows * T) * Rx, lbytes = (uint32_t)(rows * (T - D)) * Rl;
    rx = make_rsrc(static_cast<const TS*>(a.rhs) + b0 * xn_, xbytes);
    if constexpr (CT) {
      const uintptr_t wa = reinterpret_cast<uintptr_t>(a.w + b0 * T);
      wmis = (uint32_t)(wa & 3u);
      rw = make_rsrc(reinterpret_cast<const void*>(wa & ~(uintptr_t)3), wmis + (uint32_t)(rows * T));
    } else {
      rw = make_rsrc(a.w + b0 * T * (int64_t)Rw, (uint32_t)T * Rw);
    }
    rl = make_rsrc(PERDIFF ? (const void*)(static_cast<const TS*>(a.lam) + b0 * ln_) : (const void*)a.w,
                   PERDIFF ? lbytes : 0u);
    const bool out = a.out != nullptr, grad = BWD && a.glam != nullptr;
    ro = make_rsrc(out ? (const void*)(static_cast<TS*>(a.out) + b0 * xn_) : (const void*)a.w, out ? xbytes : 0u);
    if constexpr (BWD) {
      rz = make_rsrc(static_cast<const TS*>(a.zin) + b0 * xn_, grad ? xbytes : 0u);
      rg = make_rsrc(grad && PERDIFF ? (const void*)(static_cast<TS*>(a.glam) + b0 * ln_) : (const void*)a.w,
                     grad && PERDIFF ? lbytes : 0u);
    }
    const uint32_t ckbytes = (uint32_t)(tps - 1) * NF * ckrow;
    rck = make_rsrc(a.ck + (int64_t)wg * (ckbytes / 8), ckbytes);
    if constexpr (CT)
      rwm = make_rsrc(a.ck + (int64_t)gridDim.x * (ckbytes / 8) + (int64_t)wg * (tps * NT / 2), (uint32_t)tps * NT * 4u);
    const bool live = p < a.P && seg < g.ne;
    if constexpr (CT) {
      lx = live ? (uint32_t)(s_wg * T) * ES : kDead;
      ll = live ? (uint32_t)(s_wg * (T - D)) * ES : kDead;
      lw = live ? (uint32_t)(s_wg * T) : kDead;
    } else {
      const uint32_t l0 = (uint32_t)s_in * ES;
      lx = live ? l0 + (MB ? (uint32_t)a.c0 * Sb : 0u) : kDead;
      ll = live ? l0 : kDead;
      lw = live ? (WB ? ((uint32_t)s_in >> 5) << 2 : (uint32_t)s_in) : kDead;
    }
    bit = (uint32_t)s_in & 31u;
    lc = (uint32_t)tid * 8u;
    r0 = live ? seg * tps * B : 0;
    hasR = live && seg + 1 < g.ne;
    lam_scalar = (!PERDIFF && p < a.P) ? to_f64(static_cast<const TS*>(a.lam)[p]) : 0.0;

    if constexpr (CT) {
      sw_log2 = g.sw_log2;
      stage = stage_all + (tid >> 6) * ((BWD ? 3 : 2) * 64 * kPitch);
      const int seg0 = (tid & ~63) >> sw_log2, lane = tid & 63;  // the wavefront's first segment
      const uint32_t span = (uint32_t)(tps * B);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const uint32_t n = (uint32_t)(i * 64 + lane) / 6u, q = (uint32_t)(i * 64 + lane) % 6u;
        const uint32_t sn = n & (SW - 1), row = (seg0 + (n >> sw_log2)) * span + 4u * q;
        xo[i] = (sn * (uint32_t)T + row) * ES;
        lo[i] = (sn * (uint32_t)(T - D) + row) * ES;
        so[i] = n * kPitch + 4u * q;
      }
      dx = (SW == 64 ? 32u * (uint32_t)T : (32u >> sw_log2) * span) * ES;
      dl = (SW == 64 ? 32u * (uint32_t)(T - D) : (32u >> sw_log2) * span) * ES;
      const uint32_t n = (uint32_t)lane >> 3;
      wo = wmis + (n & (SW - 1)) * (uint32_t)T + (seg0 + (n >> sw_log2)) * span;
    }
    // every lane's rows of tile j lie inside [0, T - D): no masks (CT: with room
    // for the 24 rows and the 7 dwords of w that a piece reads)
    constexpr int kRoom = CT ? 24 - B + 4 : 0;
    const int seg_hi = __builtin_amdgcn_readfirstlane((tid | 63) >> g.sw_log2);  // last segment of this wavefront
    const int full_to = seg_hi < g.ne ? (T - D - kRoom - seg_hi * tps * B) / B : 0;  // tiles j < full_to are full

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
    Raw R;
    if constexpr (CT) {
      if (0 < full_to) load_raw<false>(R, 0);
      for (int j = 0; j < tps; ++j) {
        settle<false>(R, A, j, j < full_to);
        if (j + 1 < tps && j + 1 < full_to) load_raw<false>(R, j + 1);
        store_bits(j, A.wm);
        if (j > 0) store_ck(st, sp, j);
        ok &= j < full_to ? fwd_tile<true>(st, sp, G, h, A, r0 + j * B, j == 0, hasR && j == tps - 1, nobs)
                          : fwd_tile<false>(st, sp, G, h, A, r0 + j * B, j == 0, hasR && j == tps - 1, nobs);
      }
    } else {
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
    }

    // ---------------- interface ----------------
    publish(st, sp, G, h, xs_all + tid);
    nobs_all[tid] = nobs;
    flag_all[tid] = (ok || !live) ? 0 : 1;
    int j = tps - 1;
    if constexpr (!CT) load_tile<true>(A, j);  // in flight across the interface
    else if (j < full_to) load_raw<true>(R, j);
    uint32_t wm = CT ? load_bits(j) : 0u;
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
    if constexpr (CT) {
      for (; j >= 0; --j) {
        const bool full = j < full_to;
        settle<true>(R, A, j, full);
        A.wm = wm;
        if (j >= 1) wm = load_bits(j - 1);
        if (j >= 1 && j - 1 < full_to) load_raw<true>(R, j - 1);
        restore(st, ck, lwin, zL);
        if (j >= 1) load_ck(j - 1, ck, lwin);
        const bool sepR = hasR && j == tps - 1;
        if (full) rev_tile<true>(st, A, j, j == 0, sepR, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        else rev_tile<false>(st, A, j, j == 0, sepR, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        if (out) flush(1, ro, xo, dx, lx, j, full, T, 0);
        if constexpr (BWD && PERDIFF) {
          if (grad) flush(2, rg, lo, dl, ll, j, full && j < tps - 1, T - D, sepR ? D : 0);
        }
      }
    } else {
      for (; j >= 0; j -= 2) {
        if (j >= 1) load_tile<true>(Bt, j - 1);
        restore(st, ck, lwin, zL);
        if (j >= 1) load_ck(j - 1, ck, lwin);
        if (j < full_to)
          rev_tile<true>(st, A, j, j == 0, hasR && j == tps - 1, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        else
          rev_tile<false>(st, A, j, j == 0, hasR && j == tps - 1, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        if (j >= 1) {
          if (j >= 2) load_tile<true>(A, j - 2);
          restore(st, ck, lwin, zL);
          if (j >= 2) load_ck(j - 2, ck, lwin);
          if (j - 1 < full_to)
            rev_tile<true>(st, Bt, j - 1, j == 1, false, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
          else
            rev_tile<false>(st, Bt, j - 1, j == 1, false, zL, zR, zn, xn, lcr, failed, out, grad, gsum);
        }
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

template <int D, int C, int B, typename TS, bool BWD, bool PERDIFF, bool WB, int NT, bool MB = false, bool CT = false>
__global__ __launch_bounds__(NT, 1) void k_seg(SegArgs g) {
  using K = Seg<D, C, B, TS, BWD, PERDIFF, WB, NT, MB, CT>;
  __shared__ double xs[K::NX * NT];
  __shared__ int nobs[NT];
  __shared__ int flag[NT];
  __shared__ __align__(16) uint32_t stage[CT ? (NT / 64) * (BWD ? 3 : 2) * 64 * K::kPitch : 4];
  K k;
  k.run(g, xs, nobs, flag, stage);
}

}  // namespace whs
