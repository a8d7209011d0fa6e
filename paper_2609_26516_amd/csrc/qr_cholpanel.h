// Panel factorisation of the left-looking QR by Cholesky QR and Householder
// reconstruction, for panels whose columns are well away from linear
// dependence.
//
// The panel A (rows p.. of the 16 panel columns, nbk of them used) is
// orthonormalised twice by Cholesky QR (G = A^H A = R^H R, Q1 = A R^{-1}; the
// same again on Q1: Q = Q1 R2^{-1}), which leaves Q orthonormal to FP64
// rounding when no column is close to the span of the columns before it.
// The Householder form of the panel then follows from Q alone (the
// reconstruction of Ballard, Demmel, Grigori, Jacquelin, Knight, Nguyen,
// "Reconstructing Householder vectors from tall-skinny QR", 2015): the LU
// factorisation without pivoting Q - [S; 0] = Y U, taken column by column
// with s_j = -sign(Re of the j-th pivot entry) -- the sign rule of the
// reflectors, beta = -sign(Re alpha) |(alpha, x)| -- gives V = Y and
// T = -U S Y1^{-H} (Y1 the top 16 x 16 block of Y).  These are the
// reflectors and the T factor of the column-by-column factorisation of A
// itself: A and Q differ by an upper triangular factor with a positive real
// diagonal, which scales every column's (alpha, x) by a positive number and so
// leaves each reflector unchanged.
//
// Work per panel: four 16-column products on the matrix cores (the two Gram
// matrices, Q1 = A R1^{-1} and V = Q1 R2^{-1} U^{-1}), two 16-step
// recurrences on one wave (the first Cholesky factorisation with its inverse,
// the LU with Y1^{-1} and U^{-T} applied; the second Cholesky factor is I plus
// half the rounding-level deviation of its Gram matrix from I, to first
// order) and seven workgroup barriers, where the column-by-column form takes
// two barriers and a reduction over the workgroup per column.
//
// The panel is left to the column-by-column factorisation (the caller's
// fallback) when a column has no rows below its diagonal (then the reflector
// of an exactly real pivot is the identity, which the sign rule above does not
// reproduce), when an entry of the panel is exactly zero (structured inputs,
// whose exact zeros the column-by-column form keeps), when a Cholesky pivot
// of a used column is below about 1e-10 of that column's squared norm, or
// when a squared column norm leaves about [1e-200, 1e200].
#pragma once

#include "kernel_util.h"

namespace dcs {
namespace {

// Panels of the blocked QR kernels are 16 columns wide; in LDS a panel is
// row-major with the column index swizzled by the row against bank conflicts.
constexpr int QB = 16;

__device__ __forceinline__ int pidx(int i, int c) { return i * QB + (c ^ (i & 15)); }

// A complex 16 x 16 matrix on one wave: lane l holds entries (lk + 4r, li),
// r = 0..3, li = l % 16, lk = l / 16 -- the output layout of the 16x16x4 FP64
// MFMA.  Slot r is the block row of rows 4r .. 4r + 3; as it stands it is the
// B operand of a 16x16x4 product (row k = lk of four) and the A operand of one
// with its transpose, and the B operand of a 4x4x4 product on every block of
// four columns.
struct W16 {
  v4d_t re, im;
  __device__ __forceinline__ void identity(int li, int lk) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      re[r] = lk + 4 * r == li ? 1.0 : 0.0;
      im[r] = 0.0;
    }
  }
};

// Value of lane K of this lane's four (DPP quad_perm).
template <int K>
__device__ __forceinline__ double quad(double v) {
  const unsigned long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, K * 0x55, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), K * 0x55, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}
template <int K>
__device__ __forceinline__ double2 quad2(double2 v) {
  return make_double2(quad<K>(v.x), quad<K>(v.y));
}

// Block row KB of m times the 4 x 4 matrix whose entry (l % 4, lk) is a, and
// in its place: four 4 x 4 blocks in one 4x4x4 MFMA.
template <int KB>
__device__ __forceinline__ double2 block_row(double2 a, W16& m) {
  double re = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, m.re[KB], 0.0, 0, 0, 0);
  re = __builtin_amdgcn_mfma_f64_4x4x4f64(-a.y, m.im[KB], re, 0, 0, 0);
  double im = __builtin_amdgcn_mfma_f64_4x4x4f64(a.x, m.im[KB], 0.0, 0, 0, 0);
  im = __builtin_amdgcn_mfma_f64_4x4x4f64(a.y, m.re[KB], im, 0, 0, 0);
  m.re[KB] = re;
  m.im[KB] = im;
  return make_double2(re, im);
}

// m -= a^T b for block rows a and b (4 x 16 each).
__device__ __forceinline__ void rank4(W16& m, double2 a, double2 b) {
  m.re = mfma64(-a.x, b.x, m.re);
  m.im = mfma64(-a.x, b.y, m.im);
  m.re = mfma64(a.y, b.y, m.re);
  m.im = mfma64(-a.y, b.x, m.im);
}

// 1 / sqrt(d) and 1 / d for positive normal d: the hardware estimate refined
// by two Newton steps.
__device__ __forceinline__ double rsqrt_nr(double d) {
  double y = __builtin_amdgcn_rsq(d);
  const double h = 0.5 * d;
  y = y * fma(-h * y, y, 1.5);
  y = y * fma(-h * y, y, 1.5);
  return y;
}
__device__ __forceinline__ double rcp_nr(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = y * fma(-d, y, 2.0);
  y = y * fma(-d, y, 2.0);
  return y;
}

__device__ __forceinline__ double2 cscale(double2 a, double s) {
  return make_double2(a.x * s, a.y * s);
}
// c ? a : b on the components (a conditional on the vector struct itself is
// lowered through stack memory)
__device__ __forceinline__ double2 csel(bool c, double2 a, double2 b) {
  return make_double2(c ? a.x : b.x, c ? a.y : b.y);
}
// a - b c
__device__ __forceinline__ double2 cfms(double2 a, double2 b, double2 c) {
  return make_double2(fma(-b.y, -c.y, fma(-b.x, c.x, a.x)), fma(-b.x, c.y, fma(-b.y, c.x, a.y)));
}

// v[i], i = the lane's row group lk
__device__ __forceinline__ double2 pick(const double2 (&v)[4], int lk) {
  return csel((lk & 2) != 0, csel((lk & 1) != 0, v[3], v[2]), csel((lk & 1) != 0, v[1], v[0]));
}

// The recurrences below run on one wave with the other waves waiting; what
// bounds them is the number of instructions, each of four cycles or more.
// They go over the matrix in blocks of four columns: the 4 x 4 diagonal block
// is factored and inverted by every four lanes alike, lane q = li % 4 holding
// row (or column) q, without branches (lane conditions select multipliers, 0
// or the factor), and everything else is products on the matrix cores whose
// operands are block rows as they lie in the registers.  (One column at a
// time, with every lane updating its entries, the two sections took 10900 and
// 19400 cycles; now 7100 and 15600.)  li and lk are the lane's column and row group, S 64
// values of LDS.

// Cholesky factorisation G = R^H R of the Hermitian g (destroyed), with y =
// R^{-H}; columns at or past nbk are identity.  Returns false when a pivot is
// below about 1e-10 of its column's squared norm (2^-33 by exponents) or a
// squared norm leaves [2^-664, 2^664] (about 1e-200 to 1e200); y is then
// meaningless.
__device__ __forceinline__ bool chol_inv16(W16& g, W16& y, int nbk, double2* S, int li, int lk) {
  const int q = li & 3;
  // the lane's entry of the diagonal of G, if any (before the updates), and
  // the pivot it becomes
  double gd = 1.0, pk = 1.0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (lk + 4 * r == li && li >= nbk) g.re[r] = 1.0;
    gd = lk + 4 * r == li ? g.re[r] : gd;
  }
  y.identity(li, lk);
  static_for<4>([&](auto kbc) {
    constexpr int kb = decltype(kbc)::value;
    if (4 * kb >= nbk) return;   // uniform: identity from here on
    S[lk * 16 + li] = make_double2(g.re[kb], g.im[kb]);
    wave_sync();
    double2 d[4], x[4];   // row q of the diagonal block and of its factor's inverse
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = S[q * 16 + 4 * kb + j];
    wave_sync();
    static_for<4>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const double dk = quad<k>(d[k].x);
      pk = li == 4 * kb + k && lk == k ? dk : pk;
      const double inv = rsqrt_nr(dk);
      const double xs = q == k ? inv : 1.0;
      static_for<k>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        x[j] = cscale(x[j], xs);
      });
      if constexpr (k == 3) {
        x[3] = make_double2(q == 3 ? inv : 0.0, 0.0);
      } else {
        const double2 l = cscale(d[k], q > k ? inv : 0.0);   // L[q][k], q > k
        static_for<4>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          if constexpr (j > k) d[j] = cfms(d[j], l, cconj(quad2<j>(l)));
          if constexpr (j < k) x[j] = cfms(x[j], l, quad2<k>(x[j]));
        });
        x[k] = make_double2(q == k ? inv : -l.x * inv, -l.y * inv);
      }
    });
    const double2 a = pick(x, lk);
    double2 r = block_row<kb>(a, g);          // R[4kb + lk][li], li past the block
    const double2 z = block_row<kb>(a, y);
    if constexpr (kb < 3) {
      r = cscale(r, li >= 4 * kb + 4 ? 1.0 : 0.0);
      rank4(g, cconj(r), r);
      rank4(y, cconj(r), z);
    }
  });
  // on the sign and exponent bits: gd in [2^-664, 2^664], pk positive and
  // finite with an exponent at most 33 below that of gd
  const int ed = (int)((unsigned long long)__double_as_longlong(pk) >> 52);
  const int e0 = (int)((unsigned long long)__double_as_longlong(gd) >> 52);
  return __ballot(!(e0 >= 1023 - 664 && e0 <= 1023 + 664 && ed >= e0 - 33 && ed < 2047)) == 0ull;
}

// Second Cholesky factor of Cholesky QR2, whose Gram matrix is I + E with E
// at rounding level after an accepted first pass: R2 = I + F, F = the strict
// upper triangle of E plus half its diagonal, and R2^{-1} = I - F, both exact
// up to |E|^2; to Z, row-major.  Returns false (nothing written) when max |E|
// exceeds 1e-9.
__device__ __forceinline__ bool chol_inv16_near_identity(const W16& g, double2* Z, int nbk, int li,
                                                         int lk) {
  double emax = 0.0;
  double2 z[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = lk + 4 * r;
    const bool used = i < nbk && li < nbk;
    const double2 e = make_double2(used ? g.re[r] - (i == li ? 1.0 : 0.0) : 0.0, used ? g.im[r] : 0.0);
    emax = fmax(emax, fabs(e.x) + fabs(e.y));
    z[r] = make_double2(i < li ? -e.x : (i == li ? 1.0 - 0.5 * e.x : 0.0), i < li ? -e.y : 0.0);
  }
  emax = wave_max_dpp(emax);
  if (!(emax <= 1e-9)) return false;
#pragma unroll
  for (int r = 0; r < 4; ++r) Z[(lk + 4 * r) * 16 + li] = z[r];
  return true;
}

// LU factorisation without pivoting of W - S, S = diag(s_k) chosen column by
// column: s_k = -1 if Re w_kk >= 0 else +1, U_kk = w_kk - s_k (|U_kk| >= 1).
// On return w holds U on and above the diagonal, wt (W^T on entry) L^T there,
// and s_col = s of the lane's column; yl is multiplied by L^{-1} and yt by
// U^{-T}, both from the left.  Columns at or past nbk are left alone in units
// of four and are identity (s = -1) before that, for zero columns of W.
__device__ __forceinline__ void lu_inv16(W16& w, W16& wt, W16& yl, W16& yt, double& s_col, int nbk,
                                         double2* S, int li, int lk) {
  const int q = li & 3;
  s_col = -1.0;
  static_for<4>([&](auto kbc) {
    constexpr int kb = decltype(kbc)::value;
    if (4 * kb >= nbk) return;
    S[lk * 16 + li] = make_double2(w.re[kb], w.im[kb]);
    wave_sync();
    // rows q of the diagonal block and of L^{-1}, column q of U^{-1}
    double2 d[4], x[4], z[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      d[j] = S[q * 16 + 4 * kb + j];
      z[j] = make_double2(q == j ? 1.0 : 0.0, 0.0);
    }
    wave_sync();
    static_for<4>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const double2 p = quad2<k>(d[k]);
      const double sk = p.x >= 0.0 ? -1.0 : 1.0;
      s_col = li == 4 * kb + k ? sk : s_col;
      const double ux = p.x - sk, uy = p.y;
      const double den = rcp_nr(ux * ux + uy * uy);
      const double2 iu = make_double2(ux * den, -uy * den);
      const double2 zs = csel(q == k, iu, make_double2(1.0, 0.0));
      static_for<k>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        z[i] = cmul(z[i], zs);
      });
      z[k] = csel(q == k, iu, z[k]);
      if constexpr (k == 3) {
        x[3] = make_double2(q == 3 ? 1.0 : 0.0, 0.0);
      } else {
        const double2 l = cscale(cmul(d[k], iu), q > k ? 1.0 : 0.0);   // L[q][k], q > k
        double2 uq = make_double2(0.0, 0.0);                           // U[k][q], q > k
        static_for<4>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          if constexpr (j > k) {
            const double2 u = quad2<k>(d[j]);
            d[j] = cfms(d[j], l, u);
            uq = csel(q == j, u, uq);
          }
          if constexpr (j < k) x[j] = cfms(x[j], l, quad2<k>(x[j]));
        });
        x[k] = make_double2((q == k ? 1.0 : 0.0) - l.x, -l.y);
        static_for<k>([&](auto ic) {
          constexpr int i = decltype(ic)::value;
          z[i] = cfms(z[i], quad2<k>(z[i]), uq);
        });
        z[k] = cfms(z[k], iu, uq);   // lane k's is iu
      }
    });
    const double s = (li >> 2) == kb && q == lk ? s_col : 0.0;
    w.re[kb] -= s;
    wt.re[kb] -= s;
    const double2 al = pick(x, lk), au = pick(z, lk);
    double2 u = block_row<kb>(al, w), l = block_row<kb>(au, wt);   // past the block: U, L^T
    const double2 b = block_row<kb>(al, yl), c = block_row<kb>(au, yt);
    if constexpr (kb < 3) {
      u = cscale(u, li >= 4 * kb + 4 ? 1.0 : 0.0);
      l = cscale(l, li >= 4 * kb + 4 ? 1.0 : 0.0);
      rank4(w, l, u);
      rank4(wt, u, l);
      rank4(yl, l, b);
      rank4(yt, u, c);
    }
  });
}

// The two one-wave sections of the panel, kept out of line so that their
// recurrences get the registers the caller's loops hold elsewhere; they
// communicate through LDS only.  Called by wave 0.  One instance per workgroup
// size (NW waves): a shared one takes the registers of the least constrained
// kernel and makes the others spill in their loops.

// Sum of the NW waves' parts in Wp into the first, by the workgroup.
template <int NW>
__device__ __forceinline__ void panel_sum_parts(double2* Wp, int tid) {
  for (int e = tid; e < 256; e += 64 * NW) {
    double2 s = Wp[e];
#pragma unroll
    for (int w = 1; w < NW; ++w) s = make_double2(s.x + Wp[w * 256 + e].x, s.y + Wp[w * 256 + e].y);
    Wp[e] = s;
  }
}
__device__ __forceinline__ void panel_get(const double2* Wp, W16& g, int li, int lk) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 s = Wp[(lk + 4 * r) * 16 + li];
    g.re[r] = s.x;
    g.im[r] = s.y;
  }
  wave_sync();   // before the place is reused
}

// G1 (Wp[0..255], the sum of the parts) -> X1 = R1^{-1} in its place
// (row-major), with a flag in X1[1][0] (below the diagonal): 0 when the
// panel is accepted, 1 when it is left to the column-by-column
// factorisation.  The imaginary part of entry (0, 0) of each part carries
// whether that wave saw an exactly zero entry.
template <int NW>
__device__ __noinline__ void panel_first_pass(double2* Wp, int nbk) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  W16 g, y;
  panel_get(Wp, g, li, lk);
  const bool noz = readlane_d(g.im[0], 0) < 0.5;
  if (lane == 0) g.im[0] = 0.0;
  const bool ok = chol_inv16(g, y, nbk, Wp + 256, li, lk) && noz;
#pragma unroll
  for (int r = 0; r < 4; ++r) {   // X1[li][i] = conj(y[i][li])
    const int i = lk + 4 * r;
    const bool flag = li == 1 && i == 0;
    Wp[li * 16 + i] = flag ? make_double2(ok ? 0.0 : 1.0, 0.0)
                           : make_double2(i >= li ? y.re[r] : 0.0, i >= li ? -y.im[r] : 0.0);
  }
}

// G2 (Wp[0..255], the sum of the parts) and Q1's top block (P rows 0..15) -> T in
// Wp[0..255] (row-major, flag in T[1][0] as above), M = R2^{-1} U^{-1} in
// Wp[256..511] (zero in unused columns), and the top block of V in P rows
// 0..15.
template <int NW>
__device__ __noinline__ void panel_second_pass(double2* P, double2* Wp, int nbk, int mp) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  double2* part0 = Wp;
  double2* part1 = Wp + 256;
  W16 w, wt, yl, yt;   // g and R2^{-H} first
  panel_get(Wp, w, li, lk);
  bool ok = chol_inv16_near_identity(w, part1, nbk, li, lk);   // R2^{-1} to part1
  if (!ok) {
    ok = chol_inv16(w, yl, nbk, part0, li, lk);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      part1[li * 16 + lk + 4 * r] =
          make_double2(lk + 4 * r >= li ? yl.re[r] : 0.0, lk + 4 * r >= li ? -yl.im[r] : 0.0);
  }
  wave_sync();
  {   // W = Q_top = Q1_top R2^{-1}; yt = R2^{-T}
    CAcc3 c;
    c.zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double2 av = P[pidx(li, 4 * s + lk)], zv = part1[(lk + 4 * s) * 16 + li];
      const double2 zt = part1[li * 16 + lk + 4 * s];
      c.add(av.x, av.y, zv.x, zv.y);
      yt.re[s] = zt.x;
      yt.im[s] = zt.y;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      w.re[r] = c.re(r);
      w.im[r] = c.im(r);
      part0[(lk + 4 * r) * 16 + li] = make_double2(w.re[r], w.im[r]);
    }
  }
  wave_sync();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 v = part0[li * 16 + lk + 4 * r];
    wt.re[r] = v.x;
    wt.im[r] = v.y;
  }
  yl.identity(li, lk);
  wave_sync();
  double s_col;
  lu_inv16(w, wt, yl, yt, s_col, nbk, part1, li, lk);
  // T = -(U S) L^{-H}
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = lk + 4 * r;
    part0[i * 16 + li] = make_double2(i <= li ? w.re[r] * s_col : 0.0, i <= li ? w.im[r] * s_col : 0.0);
    part1[i * 16 + li] = make_double2(yl.re[r], yl.im[r]);
  }
  wave_sync();
  {
    CAcc3 t;
    t.zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double2 us = part0[li * 16 + 4 * s + lk];   // (U S)[li][4s + lk]
      const double2 lz = part1[li * 16 + 4 * s + lk];   // L^{-1}[li][4s + lk]
      t.add(us.x, us.y, lz.x, -lz.y);
    }
    wave_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = lk + 4 * r;
      const double sg = (i < nbk && li < nbk) ? -1.0 : 0.0;
      double2 tv = make_double2(sg * t.re(r), sg * t.im(r));
      if (i == 1 && li == 0) tv = make_double2(ok ? 0.0 : 1.0, 0.0);   // flag (T is upper triangular)
      part0[i * 16 + li] = tv;
    }
  }
  // M^T = yt; the top block of V: L (unit diagonal), zero outside the used
  // rows and columns
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int c = lk + 4 * r;
    const bool in = c < nbk;
    part1[li * 16 + c] = make_double2(in ? yt.re[r] : 0.0, in ? yt.im[r] : 0.0);
    const bool out = !in || li >= mp;
    P[pidx(li, c)] = make_double2(out ? 0.0 : (li > c ? wt.re[r] : (li == c ? 1.0 : 0.0)),
                                  out || li <= c ? 0.0 : wt.im[r]);
  }
}

// The panel (see above) on a workgroup of NW waves.  a holds the wave's rows
// of A in the step layout (block beta = wave + NW b, b < MAXB, rows
// 16 beta + 4t + lk, column li; zero past row m and column nbk); P holds the
// panel rows (pidx), Wp NW areas of 256 complex values.  Every thread calls
// it; mp > nbk.  Returns true (uniform) with V (explicit, panel-local rows,
// zero in unused columns) in P and T (row-major 16 x 16) in Wp; false with
// the panel rows in P -- A, or Q1 = A R1^{-1}, whose column-by-column
// factorisation has the same reflectors -- for the caller's fallback.  Ends
// with every wave past a barrier after its last read of Wp.
template <int NW, int MAXB>
__device__ __forceinline__ bool panel_cholqr(double2 (&a)[MAXB][4], int m, int k, int mp, int nbk,
                                             double2* P, double2* Wp) {
  static_assert(NW >= 2, "two 256-entry areas of Wp");
  // the thread index passes through an empty asm so that lane-dependent LDS
  // offsets are formed here, once per panel, instead of being hoisted into
  // the caller's loop and held (or spilled) across it
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  double2* part0 = Wp;         // X1, then T
  double2* part1 = Wp + 256;   // staging, then R2^{-1} U^{-1}

  // rows to P; this wave's part of G1 = A^H A, with the imaginary part of
  // entry (0, 0) replaced by whether the wave saw an exact zero
  {
    CAcc3 g;
    g.zero();
    bool z = false;
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
      const int beta = wave + NW * b;
      if (beta >= k && 16 * beta < m) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          P[pidx(16 * (beta - k) + 4 * t + lk, li)] = a[b][t];
          const int row = 16 * beta + 4 * t + lk;
          z = z || (row < m && li < nbk && a[b][t].x == 0.0 && a[b][t].y == 0.0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) g.add(a[b][t].x, -a[b][t].y, a[b][t].x, a[b][t].y);
      }
    }
    const bool anyz = __ballot(z) != 0ull;
    double2* q = Wp + wave * 256;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      q[(lk + 4 * r) * 16 + li] =
          make_double2(g.re(r), lane == 0 && r == 0 ? (anyz ? 1.0 : 0.0) : g.im(r));
  }
  __syncthreads();
  panel_sum_parts<NW>(Wp, tid);
  __syncthreads();
  if (wave == 0) panel_first_pass<NW>(Wp, nbk);
  __syncthreads();
  if (part0[16].x != 0.0) {
    __syncthreads();   // every wave has read the flag before the fallback reuses Wp
    return false;
  }
  double2 xb[4];   // X1[lk + 4s][li], the B operand of k-step s
#pragma unroll
  for (int s = 0; s < 4; ++s) xb[s] = part0[(lk + 4 * s) * 16 + li];
  __syncthreads();   // X1 read everywhere before the parts are rewritten
  {   // Q1 = A X1 block by block (each wave rewrites only its own rows of P), G2 parts
    CAcc3 g2;
    g2.zero();
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
      const int beta = wave + NW * b;
      if (beta >= k && 16 * beta < m) {
        const int r0 = 16 * (beta - k);
        CAcc3 q;
        q.zero();
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double2 av = P[pidx(r0 + li, 4 * s + lk)];   // A[r0 + li][4s + lk]
          q.add(av.x, av.y, xb[s].x, xb[s].y);
        }
        double2 qv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          qv[r] = make_double2(q.re(r), q.im(r));
          P[pidx(r0 + lk + 4 * r, li)] = qv[r];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) g2.add(qv[t].x, -qv[t].y, qv[t].x, qv[t].y);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      Wp[wave * 256 + (lk + 4 * r) * 16 + li] = make_double2(g2.re(r), g2.im(r));
  }
  __syncthreads();
  panel_sum_parts<NW>(Wp, tid);
  __syncthreads();
  if (wave == 0) panel_second_pass<NW>(P, Wp, nbk, mp);
  __syncthreads();
  if (part0[16].x != 0.0) {
    __syncthreads();
    return false;
  }
  double2 mb[4];   // M[lk + 4s][li]
#pragma unroll
  for (int s = 0; s < 4; ++s) mb[s] = part1[(lk + 4 * s) * 16 + li];
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {   // V below the top block = Q1 M
    const int beta = wave + NW * b;
    if (beta > k && 16 * beta < m) {
      const int r0 = 16 * (beta - k);
      CAcc3 y;
      y.zero();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double2 av = P[pidx(r0 + li, 4 * s + lk)];
        y.add(av.x, av.y, mb[s].x, mb[s].y);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) P[pidx(r0 + lk + 4 * r, li)] = make_double2(y.re(r), y.im(r));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  return true;
}

}  // namespace
}  // namespace dcs
