// Householder QR of one small matrix by one 256-thread workgroup, column by
// column in registers.
#pragma once

#include "wg_tile.h"

namespace dcs {
namespace {

template <int K>
__device__ __forceinline__ double bcol64(double v) {   // lane K of this lane's row of 16
  return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + K, 0xF, 0xF, true);
}
// Sum over the four rows of 16 lanes; every lane gets its column's sum.
__device__ __forceinline__ double sum_rows(double v) {
  unsigned long long b = __double_as_longlong(v);
  {
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    v = __longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]) +
        __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]);
  }
  b = __double_as_longlong(v);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
  return __longlong_as_double(((unsigned long long)hi[0] << 32) | lo[0]) +
         __longlong_as_double(((unsigned long long)hi[1] << 32) | lo[1]);
}
// Value of row G of 16 lanes in every row.
template <int G>
__device__ __forceinline__ double row_of(double v) {
  auto pick = [](unsigned u) -> unsigned {
    const auto s1 = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned y = (G & 1) ? s1[1] : s1[0];
    const auto s2 = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    return (G & 2) ? s2[1] : s2[0];
  };
  const unsigned long long b = __double_as_longlong(v);
  return __longlong_as_double(((unsigned long long)pick((unsigned)(b >> 32)) << 32) |
                              pick((unsigned)b));
}

// LDS of the QR of matrices of up to 2 CD x CD.
template <int CD>
struct QrSmem {
  static constexpr int P = CD + 1;   // padded row
  double2 V[2 * CD * P];             // reflectors, explicit
  double2 S[1024 > CD * CD ? 1024 : CD * CD];   // S[k CD + j] = v_j^H v_k, j < k; then parts of V Z
  double2 Z[CD * P];                 // T V_top^H
  double2 ex[2][CNW][4][16];         // per buffer and wave: x_k^H a_j and row k of two column blocks
  double2 tau[CD];
  double mx[CNW];
};

// Householder reflector of (alpha = ar + i ai, x), |x|^2 = xn, after LAPACK's
// zlarfg: tau and inv = 1 / (alpha - beta), so v = [1; x inv]; the identity
// (tau = inv = 0) where x has no non-zero entry (`some` false) and alpha is real,
// or the squared norm n2 is below 1e-200 (the caller has scaled what is not zero).
// I - tau v v^H is unitary to the accuracy of |(alpha, x)| and of the quotients,
// so each ends in a residual correction (Markstein's iterations: nrm ->
// sqrt(n2), h -> 1 / (2 sqrt(n2)), the residuals exact by FMA; the estimates are
// good to 2^-24, one step to 2^-47, the correction to the rounding), and Re tau =
// 1 - Re alpha / beta is rounded once.  The norms |q|^2 of random 32 x 16 columns
// are 2.5e-16 from 1 (rms; LAPACK's 2.6e-16, the blocked kernel's 2.7e-16);
// with plain Newton steps they were 3.2e-16 off, one-sided where the norm is a
// round number: F of the 13-qubit GHZ circuit 3.0e-14 from its value, 3.6e-15
// now.  The corrections cost nothing that shows in a step's time.
__device__ __forceinline__ void reflector(double ar, double ai, double xn, double n2, bool some,
                                          double2& tau, double2& inv) {
  double rs = __builtin_amdgcn_rsq(n2);
  double nrm = n2 * rs, h = 0.5 * rs;
  const double r = fma(-nrm, h, 0.5);
  nrm = fma(nrm, r, nrm);
  h = fma(h, r, h);
  nrm = fma(fma(-nrm, nrm, n2), h, nrm);
  rs = h + h;
  rs = fma(fma(-nrm, rs, 1.0), rs, rs);   // 1 / |(alpha, x)|
  const bool pos = ar >= 0.0;
  const double beta = pos ? -nrm : nrm, rb = pos ? -rs : rs;
  const double dx = ar - beta, den = fma(dx, dx, ai * ai);
  double rd = __builtin_amdgcn_rcp(den);
  rd = fma(fma(-den, rd, 1.0), rd, rd);
  const bool id = !(n2 >= 1e-200 && (some || xn != 0.0 || ai != 0.0));
  double ix = dx * rd, iy = -ai * rd;
  ix = fma(fma(-ix, den, dx), rd, ix);
  iy = fma(fma(-iy, den, -ai), rd, iy);
  tau = make_double2(id ? 0.0 : fma(-ar, rb, 1.0), id ? 0.0 : -ai * rb);
  inv = make_double2(id ? 0.0 : ix, id ? 0.0 : iy);
}
// Whether column k needs the slow look: its squared norm leaves [1e-200,
// 1e200], or |x|^2 is zero and alpha real (x may still hold tiny entries).
// The arguments are the same in every lane; by exponents, on the scalar unit.
__device__ __forceinline__ bool odd_column(double ai, double xn, double n2) {
  auto hi = [](double v) {
    return __builtin_amdgcn_readfirstlane((int)((unsigned long long)__double_as_longlong(v) >> 32));
  };
  const int e = (hi(n2) >> 20) & 0x7ff;   // 1e-200 to 1e200: 2^-664 to 2^664
  return e < 1023 - 664 || e > 1023 + 664 || (xn == 0.0 && ai == 0.0);
}
__device__ __forceinline__ bool in_range(double n2) { return n2 >= 1e-200 && n2 <= 1e200; }
// Power of two (a normal number) that brings the largest entry ma near 1; 0 for a
// zero column (below 1e-280), 1 where it is infinite (Q comes out as NaN).
__device__ __forceinline__ double column_scale(double ma) {
  return ma < 1e-280 ? 0.0 : ma <= 1.7976931348623157e308 ? ldexp(1.0, -ilogb(ma)) : 1.0;
}

// The columns of a block are taken in groups of four; between groups the
// lanes of a row of 16 rotate by four (lane li then holds column (li + 4 g) mod
// 16) and the registers of the rows move up by one slot, so that the code of a
// group is the same for every group: column 4 g + q sits in lane q, row 4 g + q
// in slot 0 of lane group q.
__device__ __forceinline__ double lanes_on(double v) {   // lane i takes lane i + 4 of its row
  const unsigned long long b = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)b, 0x12C, 0xF, 0xF, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(b >> 32), 0x12C, 0xF, 0xF, true);
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double2 lanes_on(double2 v) {
  return make_double2(lanes_on(v.x), lanes_on(v.y));
}
template <int G>
__device__ __forceinline__ double2 row_of(double2 v) {
  return make_double2(row_of<G>(v.x), row_of<G>(v.y));
}
template <int K>
__device__ __forceinline__ double2 bcol64(double2 v) {
  return make_double2(bcol64<K>(v.x), bcol64<K>(v.y));
}
__device__ __forceinline__ double2 keep_if(bool c, double2 v) {
  return make_double2(c ? v.x : 0.0, c ? v.y : 0.0);
}

template <int SL>
__device__ __forceinline__ double2 column_dot(const double2 (&x)[SL], const double2 (&a)[SL]) {
  double2 d = make_double2(0.0, 0.0), e = d;   // two chains
#pragma unroll
  for (int t = 0; t < SL; t += 2) {
    d.x = fma(x[t].x, a[t].x, fma(x[t].y, a[t].y, d.x));
    d.y = fma(x[t].x, a[t].y, fma(-x[t].y, a[t].x, d.y));
    e.x = fma(x[t + 1].x, a[t + 1].x, fma(x[t + 1].y, a[t + 1].y, e.x));
    e.y = fma(x[t + 1].x, a[t + 1].y, fma(-x[t + 1].y, a[t + 1].x, e.y));
  }
  return make_double2(sum_rows(d.x + e.x), sum_rows(d.y + e.y));
}
template <int SL>
__device__ __forceinline__ void column_sub(double2 (&a)[SL], double2 e, const double2 (&x)[SL]) {
#pragma unroll
  for (int t = 0; t < SL; ++t) {
    a[t].x = fma(-e.x, x[t].x, fma(e.y, x[t].y, a[t].x));
    a[t].y = fma(-e.x, x[t].y, fma(-e.y, x[t].x, a[t].y));
  }
}

// Z = T V_top^H, columns c0 .. c0 + 15 on one wave, by back substitution on
// T^{-1} Z = V_top^H: T^{-1} = diag(1 / tau) + the strict upper triangle of V^H
// V.  Rows lk + 4 r in slot r, in groups of four from the last, whose rows are
// always in the last slot.
template <int CD>
__device__ __forceinline__ void back_substitute(QrSmem<CD>& sm, int n, int c0) {
  constexpr int NR = CD / 4, P = QrSmem<CD>::P;
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const int c = c0 + li, last = (n - 1) >> 2;
  double2 z[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = 4 * (r + last - (NR - 1)) + lk;
    const bool in = c < n && i >= 0 && i <= c;
    const double2 v = sm.V[in ? c * P + i : 0];
    z[r] = make_double2(in ? v.x : 0.0, in ? -v.y : 0.0);
  }
#pragma unroll 1
  for (int g = last; g >= 0; --g) {
    static_for<4>([&](auto qc) {
      constexpr int kr = 3 - decltype(qc)::value;
      const int k = 4 * g + kr;
      if (k >= n) return;   // uniform, in the first group taken
      double2 sv[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int i = 4 * (r + g - (NR - 1)) + lk;
        sv[r] = sm.S[i >= 0 ? k * CD + i : 0];
      }
      const double2 zk = cmul(sm.tau[k], row_of<kr>(z[NR - 1]));
      sv[NR - 1] = keep_if(lk < kr, sv[NR - 1]);
      z[NR - 1].x = lk == kr ? zk.x : z[NR - 1].x;
      z[NR - 1].y = lk == kr ? zk.y : z[NR - 1].y;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        z[r].x = fma(-sv[r].x, zk.x, fma(sv[r].y, zk.y, z[r].x));
        z[r].y = fma(-sv[r].x, zk.y, fma(-sv[r].y, zk.x, z[r].y));
      }
    });
    if (4 * g + lk < n && c < n) sm.Z[(4 * g + lk) * P + c] = z[NR - 1];
#pragma unroll
    for (int r = NR - 1; r > 0; --r) z[r] = z[r - 1];
  }
}

// QR of the m x n matrix f (m <= 2 CD, n <= CD <= 32, m >= n; row-major,
// leading dimension n, in the path precision), Q through put(row, col, re,
// im).
//
// Householder, column by column, with LAPACK's reflectors.  The rows are held
// in registers in the layout of the FP64 MFMA result (lane: rows 4 t + lk,
// column li of a 16-column block).  Column k takes one reduction: d_j =
// sum_{r > k} conj(a_rk) a_rj for every column j at once gives |x|^2 (j = k),
// the update coefficients (j > k) and the products of the reflectors (j < k,
// whose columns hold x_j); x_k stays unscaled (v_k = x_k inv_k).  A column
// whose squared norm leaves [1e-200, 1e200] is first scaled by a power of two,
// which leaves Q as it is.  Then Q = E - V Z with Z = T V_top^H by back
// substitution, and V Z on the matrix cores.  What bounds it is the chain of
// dependent FP64 operations of a column, so a matrix of up to 32 x 16 stays
// on one wave (no barrier in the chain); a larger one is spread over four
// waves of 16 rows, two column blocks each, with one barrier per column (the
// exchange areas alternate, so a column's readers are past when they are
// written again).
template <int CD, typename T, typename Put>
__device__ __forceinline__ void small_qr(const T* f, int m, int n, QrSmem<CD>& sm, Put&& put) {
  constexpr int P = QrSmem<CD>::P;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  if (CD == 16 || (m <= 32 && n <= 16)) {
    if (wave == 0) {
      constexpr int SL = 8;
      double2 a[SL], myinv = zero;
#pragma unroll
      for (int t = 0; t < SL; ++t) {
        const int r = 4 * t + lk;
        const bool in = r < m && li < n;
        const T v = f[in ? r * n + li : 0];
        a[t] = make_double2(in ? (double)v.x : 0.0, in ? (double)v.y : 0.0);
      }
      int g = 0, col = li;   // group, and the column in this lane
#pragma unroll 1
      for (;; ++g) {
        static_for<4>([&](auto qc) {
          constexpr int q = decltype(qc)::value;
          const int k = 4 * g + q;
          if (k >= n) return;   // uniform
          double2 x[SL], tau, inv;
          double2 row = row_of<q>(a[0]);
          a[0] = keep_if(lk != q, a[0]);
#pragma unroll
          for (int t = 0; t < SL; ++t) x[t] = bcol64<q>(a[t]);
          double2 d = column_dot<SL>(x, a);
          double xn = readlane_d(d.x, q), ar = readlane_d(row.x, q), ai = readlane_d(row.y, q);
          double n2 = fma(ar, ar, fma(ai, ai, xn));
          bool some = false;
          if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)odd_column(ai, xn, n2)), 0)) {
            double mx = 0.0;
#pragma unroll
            for (int t = 0; t < SL; ++t) mx = fmax(mx, fmax(fabs(x[t].x), fabs(x[t].y)));
            mx = wave_max_dpp(mx);
            const double ma = fmax(mx, fmax(fabs(ar), fabs(ai)));
            const double sc = in_range(n2) ? 1.0 : column_scale(ma);
            const double own = col == k ? sc : 1.0;
            some = mx > 0.0 && sc != 0.0;
#pragma unroll
            for (int t = 0; t < SL; ++t) {
              x[t] = make_double2(x[t].x * sc, x[t].y * sc);
              a[t] = make_double2(a[t].x * own, a[t].y * own);
            }
            row = make_double2(row.x * own, row.y * own);
            d = column_dot<SL>(x, a);
            xn = readlane_d(d.x, q);
            ar = readlane_d(row.x, q);
            ai = readlane_d(row.y, q);
            n2 = fma(ar, ar, fma(ai, ai, xn));
          }
          reflector(ar, ai, xn, n2, some, tau, inv);
          // w_j = v_k^H a_j: columns j > k are updated, j < k give v_k^H x_j
          const double2 w = make_double2(row.x + inv.x * d.x + inv.y * d.y,
                                         row.y + inv.x * d.y - inv.y * d.x);
          const double2 e = keep_if(col > k, cmul(cmul(cconj(tau), inv), w));
          column_sub<SL>(a, e, x);
          // row k of V (lanes lk = 0), of the products (lk = 1, conjugated) and
          // tau (lane 32) in one write
          const double2 u = cmul(make_double2(lk ? w.x : row.x, lk ? w.y : row.y), myinv);
          const bool below = col < k;
          double2* const to = lk == 0 ? sm.V + (k * P + col) : lk == 1 ? sm.S + (k * CD + col) : sm.tau + k;
          if (lk == 0 || (lk == 1 && below) || lane == 32)
            *to = make_double2(lk >= 2 ? tau.x : below ? u.x : (col == k ? 1.0 : 0.0),
                               lk >= 2 ? tau.y : below ? (lk ? -u.y : u.y) : 0.0);
          myinv.x = col == k ? inv.x : myinv.x;
          myinv.y = col == k ? inv.y : myinv.y;
        });
        if (4 * g + 4 >= n) break;
#pragma unroll
        for (int t = 0; t < SL - 1; ++t) a[t] = lanes_on(a[t + 1]);
        a[SL - 1] = zero;
        myinv = lanes_on(myinv);
        col = (col + 4) & 15;
      }
#pragma unroll
      for (int t = 0; t < SL; ++t) {   // rows from n on
        const int r = 4 * (t + g) + lk;
        if (r >= n && r < m && col < n) sm.V[r * P + col] = cmul(a[t], myinv);
      }
      wave_sync();
      back_substitute<CD>(sm, n, 0);
    }
  } else {
    constexpr int SL = 4;
    double2 a0[SL], a1[SL], inv0 = zero, inv1 = zero;
#pragma unroll
    for (int t = 0; t < SL; ++t) {
      const int r = 16 * wave + 4 * t + lk;
      const bool i0 = r < m && li < n, i1 = r < m && 16 + li < n;
      const T v0 = f[i0 ? r * n + li : 0], v1 = f[i1 ? r * n + 16 + li : 0];
      a0[t] = make_double2(i0 ? (double)v0.x : 0.0, i0 ? (double)v0.y : 0.0);
      a1[t] = make_double2(i1 ? (double)v1.x : 0.0, i1 ? (double)v1.y : 0.0);
    }
    // block p is factored in a0 (its columns rotating), the other one is in a1
    int g = 0, gw = 0, col = li, buf = 0;   // group; this wave's slot shifts
#pragma unroll 1
    for (;; ++g) {
      const int p = g >> 2;
      const bool holds = wave == p;   // the rows of this block's diagonal
      static_for<4>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const int k = 4 * g + q;
        if (k >= n) return;   // uniform
        double2 x[SL], d0, d1, row0, row1, tau, inv;
        double2 r0 = row_of<q>(a0[0]), r1 = row_of<q>(a1[0]);
        const bool keep = !holds || lk != q;
        a0[0] = keep_if(keep, a0[0]);
        a1[0] = keep_if(keep, a1[0]);
#pragma unroll
        for (int t = 0; t < SL; ++t) x[t] = bcol64<q>(a0[t]);
        double xn, ar, ai, n2;
        auto exchange = [&]() {
          d0 = column_dot<SL>(x, a0);
          d1 = column_dot<SL>(x, a1);
          const double2 lo = make_double2(lk & 1 ? d1.x : d0.x, lk & 1 ? d1.y : d0.y);
          const double2 hi = make_double2(lk & 1 ? r1.x : r0.x, lk & 1 ? r1.y : r0.y);
          sm.ex[buf][wave][lk][li] = make_double2(lk & 2 ? hi.x : lo.x, lk & 2 ? hi.y : lo.y);
          lds_sync();
          double2 u0[CNW], u1[CNW];
#pragma unroll
          for (int w = 0; w < CNW; ++w) {
            u0[w] = sm.ex[buf][w][0][li];
            u1[w] = sm.ex[buf][w][1][li];
          }
          row0 = sm.ex[buf][p][2][li];
          row1 = sm.ex[buf][p][3][li];
          d0 = make_double2((u0[0].x + u0[1].x) + (u0[2].x + u0[3].x),
                            (u0[0].y + u0[1].y) + (u0[2].y + u0[3].y));
          d1 = make_double2((u1[0].x + u1[1].x) + (u1[2].x + u1[3].x),
                            (u1[0].y + u1[1].y) + (u1[2].y + u1[3].y));
          buf ^= 1;
          xn = readlane_d(d0.x, q);
          ar = readlane_d(row0.x, q);
          ai = readlane_d(row0.y, q);
          n2 = fma(ar, ar, fma(ai, ai, xn));
        };
        exchange();
        bool some = false;
        // (the same on every wave)
        if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)odd_column(ai, xn, n2)), 0)) {
          double mx = 0.0;
#pragma unroll
          for (int t = 0; t < SL; ++t) mx = fmax(mx, fmax(fabs(x[t].x), fabs(x[t].y)));
          mx = wave_max_dpp(mx);
          lds_sync();   // readers of an earlier column's maxima are past
          if (lane == 0) sm.mx[wave] = mx;
          lds_sync();
          mx = fmax(fmax(sm.mx[0], sm.mx[1]), fmax(sm.mx[2], sm.mx[3]));
          const double ma = fmax(mx, fmax(fabs(ar), fabs(ai)));
          const double sc = in_range(n2) ? 1.0 : column_scale(ma);
          const double own = li == q ? sc : 1.0;
          some = mx > 0.0 && sc != 0.0;
#pragma unroll
          for (int t = 0; t < SL; ++t) {
            x[t] = make_double2(x[t].x * sc, x[t].y * sc);
            a0[t] = make_double2(a0[t].x * own, a0[t].y * own);
          }
          r0 = make_double2(r0.x * own, r0.y * own);
          exchange();
        }
        reflector(ar, ai, xn, n2, some, tau, inv);
        const double2 w0 = make_double2(row0.x + inv.x * d0.x + inv.y * d0.y,
                                        row0.y + inv.x * d0.y - inv.y * d0.x);
        const double2 w1 = make_double2(row1.x + inv.x * d1.x + inv.y * d1.y,
                                        row1.y + inv.x * d1.y - inv.y * d1.x);
        const double2 ct = cmul(cconj(tau), inv);
        column_sub<SL>(a0, keep_if(col > (k & 15), cmul(ct, w0)), x);
        if (p == 0) column_sub<SL>(a1, cmul(ct, w1), x);
        if (wave == CNW - 1) {   // row k of V and of the products
          // lk 0: V in the current block, 1: V in the other one, 2, 3: products
          const bool cur = !(lk & 1), vr = lk < 2;
          const double2 iv = make_double2(cur ? inv0.x : inv1.x, cur ? inv0.y : inv1.y);
          const double2 rv = make_double2(cur ? row0.x : row1.x, cur ? row0.y : row1.y);
          const double2 wv = make_double2(cur ? w0.x : w1.x, cur ? w0.y : w1.y);
          const double2 v = cmul(make_double2(vr ? rv.x : wv.x, vr ? rv.y : wv.y), iv);
          // block 1 is the current one from column 16 on
          const int cc = (cur == (p == 1) ? 16 : 0) + (cur ? col : li);
          const bool below = cc < k;
          if (vr)
            sm.V[k * P + cc] = make_double2(below ? v.x : (cc == k ? 1.0 : 0.0), below ? v.y : 0.0);
          else if (below)
            sm.S[k * CD + cc] = cconj(v);
          if (lane == 0) sm.tau[k] = tau;
        }
        inv0.x = li == q ? inv.x : inv0.x;
        inv0.y = li == q ? inv.y : inv0.y;
      });
      if (4 * g + 4 >= n) break;
      if (holds) {
        ++gw;
#pragma unroll
        for (int t = 0; t < SL - 1; ++t) {
          a0[t] = lanes_on(a0[t + 1]);
          a1[t] = a1[t + 1];
        }
        a0[SL - 1] = a1[SL - 1] = zero;
      } else {
#pragma unroll
        for (int t = 0; t < SL; ++t) a0[t] = lanes_on(a0[t]);
      }
      inv0 = lanes_on(inv0);
      col = (col + 4) & 15;
      if (g == 3) {   // on to the second block (the lanes are back in place)
#pragma unroll
        for (int t = 0; t < SL; ++t) {
          const double2 u = a0[t];
          a0[t] = a1[t];
          a1[t] = u;
        }
        const double2 u = inv0;
        inv0 = inv1;
        inv1 = u;
      }
    }
    // rows from n on
    const bool swapped = n > 16;
#pragma unroll
    for (int t = 0; t < SL; ++t) {
      const int r = 16 * wave + 4 * (t + gw) + lk;
      const double2 v0 = cmul(a0[t], inv0), v1 = cmul(a1[t], inv1);
      if (r >= n && r < m && r < 16 * wave + 16) {
        const int c0 = (swapped ? 16 : 0) + col;
        if (c0 < n) sm.V[r * P + c0] = v0;
        if (swapped) sm.V[r * P + li] = v1;
      }
    }
    lds_sync();
    if (wave < (n + 15) >> 4) back_substitute<CD>(sm, n, 16 * wave);
  }
  lds_sync();
  wg_gemm<CT_F64>(
      m, n, n, sm.S, [&](int i, int k) { return sm.V[i * P + k]; },
      [&](int k, int j) { return sm.Z[k * P + j]; },
      [&](int i, int j, double re, double im) { put(i, j, (i == j ? 1.0 : 0.0) - re, -im); });
}

}  // namespace
}  // namespace dcs
