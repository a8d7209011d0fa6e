// Whole compression steps of small branches in one launch.
//
// One workgroup of 4 waves carries one branch through the entire step: the
// right environments of the starting guess, then every visit of every sweep
// (site contraction, gate operator, FP64 QR gauge shift, next environment).
// At small bond dimensions a visit is a handful of 16 x 16 tiles, so a chain
// of separate launches spends its time on launch latency and on kernels that
// fill one or two CUs; here the stages of a visit are separated by workgroup
// barriers and the intermediates X, F, Q stay in LDS.
//
// Both directions run the same stages on mirrored indices.  Moving right at
// site j (moving left in brackets), with the environment E behind the front
// (L_j [R_{j+1}], rows (g, i)), the one ahead E' (R_{j+1} [L_j], rows h) and
// the ket site K:
//   A   Y[(g,i)][t,n] = E K, X[(g,s)][(o,n)] = sum_{i,t} W Y    (i, o: operator
//       bonds behind / ahead, n: ket bond ahead)
//   B   F[(g,s)][h] = sum_z X[(g,s)][z] E'[h][z]
//   QR  F = Q R in FP64 (rows ordered (s, g) and conjugated when moving left:
//       the LQ of the site tensor)
//   D   next environment[h][z] = sum_{(g,s)} conj(B[(g,s)][h]) X[(g,s)][z]
// Contractions accumulate in the path precision (FP32 / FP64 MFMA, three real
// products per complex one); the QR is FP64 in every form.
//
// What bounds it is the chain of one workgroup: at bond 16 a visit takes about
// 53 000 cycles, half of them in the QR (about 2000 per column, some 265
// instructions on one wave), 9000 in stage A, 5000 each in B and D.  16 qubits,
// bond 16, two sweeps, one complex128 branch: 0.71 ms, against 1.57 ms as a
// sequence of launches (15 environments and 31 visits of 4 to 5 launches); 64
// branches 0.74 against 1.93 ms; bond 4: 0.43 against 1.15 ms.
#include "kernel_util.h"

namespace dcs {
namespace {

constexpr int CNT = 256, CNW = CNT / 64;   // threads and waves of a workgroup

typedef float v4f_t __attribute__((ext_vector_type(4)));

template <int CT>
struct Path;
template <>
struct Path<CT_F32> {
  using T = float2;
  using R = float;
  using V = v4f_t;
  static __device__ __forceinline__ V mma(R a, R b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};
template <>
struct Path<CT_F64> {
  using T = double2;
  using R = double;
  using V = v4d_t;
  static __device__ __forceinline__ V mma(R a, R b, V c) { return mfma64(a, b, c); }
  static __device__ __forceinline__ int row(int lk, int r) { return lk + 4 * r; }
};

// Complex accumulator of one 16 x 16 block.
template <int CT>
struct CAcc {
  typename Path<CT>::V p1, p2, p3;
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p1[r] = 0;
      p2[r] = 0;
      p3[r] = 0;
    }
  }
  template <typename T>
  __device__ __forceinline__ void add(T a, T b) {
    p1 = Path<CT>::mma(a.x, b.x, p1);
    p2 = Path<CT>::mma(a.y, b.y, p2);
    p3 = Path<CT>::mma(a.x + a.y, b.x + b.y, p3);
  }
  __device__ __forceinline__ typename Path<CT>::R re(int r) const { return p1[r] - p2[r]; }
  __device__ __forceinline__ typename Path<CT>::R im(int r) const { return p3[r] - p1[r] - p2[r]; }
};

// Wave-level ordering of LDS traffic: what a wave has written, its own lanes
// may read (the LDS serves one wave's accesses in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier for LDS traffic alone: global stores stay in flight.
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// C (M x N) = A B over a workgroup: 16 x 16 tiles dealt to the waves, or, when
// there are fewer tiles than waves, the K range of each tile split over
// several waves whose parts meet in `part` (256 complex values per wave).
// fa(m, k), fb(k, n) give the operands at indices inside the matrix; fc(m, n,
// re, im) takes the results.  Ends with the results written but not fenced.
template <int CT, typename FA, typename FB, typename FC>
__device__ __forceinline__ void wg_gemm(int M, int N, int K, typename Path<CT>::T* part, FA&& fa,
                                        FB&& fb, FC&& fc) {
  using T = typename Path<CT>::T;
  using R = typename Path<CT>::R;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int tn = (N + 15) >> 4, tiles = ((M + 15) >> 4) * tn;
  int sh = 0;   // parts of a tile's K range: 1 << sh
  while ((2 << sh) * tiles <= CNW && (16 << sh) < K) ++sh;
  const int per = ((K + (4 << sh) - 1) >> (2 + sh)) * 4;   // K range of a part, whole k-steps
  int mt = 0, nt = wave >> sh;
  for (int u = wave; u < tiles << sh; u += CNW, nt += CNW >> sh) {
    while (nt >= tn) {
      nt -= tn;
      ++mt;
    }
    const int m0 = mt * 16, n0 = nt * 16, k0 = (u & ((1 << sh) - 1)) * per, k1 = min(K, k0 + per);
    const bool am = m0 + li < M, bn = n0 + li < N;
    const int mi = am ? m0 + li : 0, ni = bn ? n0 + li : 0;
    CAcc<CT> acc;
    acc.zero();
    auto load = [&](int k, T& a, T& b) {
      const bool in = k + lk < k1;
      const int kc = in ? k + lk : 0;
      a = fa(mi, kc);
      b = fb(kc, ni);
      // selects, not products: what lies outside may not be finite
      const bool ia = am && in, ib = bn && in;
      a.x = ia ? a.x : R(0);
      a.y = ia ? a.y : R(0);
      b.x = ib ? b.x : R(0);
      b.y = ib ? b.y : R(0);
    };
    for (int k = k0; k < k1; k += 16) {   // four k-steps in flight
      T a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) load(k + 4 * q, a[q], b[q]);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc.add(a[q], b[q]);
    }
    if (sh == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + Path<CT>::row(lk, r), n = n0 + li;
        if (m < M && n < N) fc(m, n, acc.re(r), acc.im(r));
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T v;
        v.x = acc.re(r);
        v.y = acc.im(r);
        part[u * 256 + Path<CT>::row(lk, r) * 16 + li] = v;
      }
    }
  }
  if (sh > 0) {   // parts added in order
    lds_sync();
    for (int e = threadIdx.x; e < tiles * 256; e += CNT) {   // at most CNW / 2 tiles
      int m1 = 0, n1 = e >> 8;
      while (n1 >= tn) {
        n1 -= tn;
        ++m1;
      }
      const int m = m1 * 16 + ((e >> 4) & 15), n = n1 * 16 + (e & 15);
      if (m >= M || n >= N) continue;
      const T* q = part + ((e >> 8) << sh) * 256 + (e & 255);
      R re = q[0].x, im = q[0].y;
      for (int p = 1; p < 1 << sh; ++p) {
        re += q[p * 256].x;
        im += q[p * 256].y;
      }
      fc(m, n, re, im);
    }
  }
}

// Stage A: Y = E K and the gate operator, one wave per block of rows (g, all
// i) and 16 values of n; the product passes through the wave's own LDS tile
// (four planes (t, component) of 16 x 17).  The operator runs as a real
// matrix: 4 wo x 4 wi entries, inputs (i, t, component), outputs (j,
// component) with j = (s, o); one MFMA step per value of i, four in flight.
// Groups of four i without a non-zero entry for the outputs at hand are left
// out (gates passing a site leave most of a wide operator zero).
template <int CT, bool LEFT, typename PE, typename PK, typename PX>
__device__ __forceinline__ void stage_a(PE E, PK Kt, const typename Path<CT>::T* sW, int ng, int wi, int wo, int kd,
                                        int nn, typename Path<CT>::R* tile, PX Xo) {
  using T = typename Path<CT>::T;
  using R = typename Path<CT>::R;
  using V = typename Path<CT>::V;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  // rows (g, i) of a block: 16 / wi values of g; at most two blocks of n
  const int gper = wi == 1 ? 16 : wi == 2 ? 8 : wi == 3 ? 5 : wi == 4 ? 4 : wi == 5 ? 3 : wi <= 8 ? 2 : 1;
  const int nsh = nn > 16 ? 1 : 0;
  R* my = tile + wave * (4 * 16 * 17);
  const int t = lk >> 1, c = lk & 1;   // this lane's input component of a k-step
  for (int u = wave; (u >> nsh) * gper < ng; u += CNW) {
    const int g0 = (u >> nsh) * gper, n0 = (u & nsh) * 16;
    const int gn = min(gper, ng - g0), rows = gn * wi;
    const bool am = li < rows, bn = n0 + li < nn;
    const int e0 = (g0 * wi + (am ? li : 0)) * kd, ni = bn ? n0 + li : 0;
    CAcc<CT> y0, y1;
    y0.zero();
    y1.zero();
    for (int k = 0; k < kd; k += 8) {
      T a[2], b0[2], b1[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int kk = k + 4 * q + lk;
        const bool in = kk < kd;
        const int kc = in ? kk : 0;
        a[q] = E[e0 + kc];
        // K[x][t][y]: k = x, n = y moving right; k = y, n = x moving left
        const int kb = LEFT ? 2 * ni * kd + kc : 2 * kc * nn + ni, ts = LEFT ? kd : nn;
        b0[q] = Kt[kb];
        b1[q] = Kt[kb + ts];
        const bool ia = am && in, ib = bn && in;
        a[q].x = ia ? a[q].x : R(0);
        a[q].y = ia ? a[q].y : R(0);
        b0[q].x = ib ? b0[q].x : R(0);
        b0[q].y = ib ? b0[q].y : R(0);
        b1[q].x = ib ? b1[q].x : R(0);
        b1[q].y = ib ? b1[q].y : R(0);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        y0.add(a[q], b0[q]);
        y1.add(a[q], b1[q]);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = Path<CT>::row(lk, r) * 17 + li;
      my[row] = y0.re(r);
      my[272 + row] = y0.im(r);
      my[544 + row] = y1.re(r);
      my[816 + row] = y1.im(r);
    }
    wave_sync();
    const R* sWr = reinterpret_cast<const R*>(sW);
    for (int ot = 0; ot < 2 * wo; ot += 8) {   // 8 complex outputs j = ot .. ot + 7 per tile
      // bit q: some W with i in 4 q .. 4 q + 3 is not zero (lane: output, t, i)
      unsigned nz = 1;
      if (wi > 4) {
        nz = 0;
        const int jz = ot + (lane & 7), sz = jz >= wo ? 1 : 0, oz = jz - sz * wo;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int iz = 4 * q + (lane >> 4), tz = (lane >> 3) & 1;
          const bool in = jz < 2 * wo && iz < wi;
          const T v = sW[!in ? 0 : LEFT ? ((oz * 2 + sz) * 2 + tz) * wi + iz
                                        : ((iz * 2 + sz) * 2 + tz) * wo + oz];
          if (__ballot(in && (v.x != R(0) || v.y != R(0)))) nz |= 1u << q;
        }
      }
      // output row li of the tile: (j, component), paired so that a lane of
      // the result holds whole complex values
      const int j = ot + (sizeof(R) == 4 ? li >> 1 : li & 7), cp = sizeof(R) == 4 ? li & 1 : li >> 3;
      const bool jv = j < 2 * wo;
      const int s = jv && j >= wo ? 1 : 0, o = jv ? j - s * wo : 0;
      // W[wl][s][t][wr]: i = wl, o = wr moving right; i = wr, o = wl moving left
      const int w0 = 2 * (LEFT ? ((o * 2 + s) * 2 + t) * wi : (s * 2 + t) * wo + o) + (cp != c ? 1 : 0);
      const int ws = LEFT ? 2 : 8 * wo;
      const R sg = !jv ? R(0) : (cp == 0 && c == 1) ? R(-1) : R(1);
      const R* in0 = my + lk * 272 + li;
      for (int gb = 0; gb < gn; gb += 4) {   // four values of g at a time
        V acc[4];
#pragma unroll
        for (int y = 0; y < 4; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[y][r] = 0;
        for (int i = 0; i < wi; i += 4) {
          if (!((nz >> (i >> 2)) & 1u)) continue;   // uniform
          R wv[4], xv[4][4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int ii = i + q < wi ? i + q : i;
            wv[q] = (i + q < wi ? sg : R(0)) * sWr[w0 + ii * ws];
#pragma unroll
            for (int y = 0; y < 4; ++y)
              xv[y][q] = in0[((gb + y < gn ? gb + y : gb) * wi + ii) * 17];
          }
#pragma unroll
          for (int y = 0; y < 4; ++y)
            if (gb + y < gn) {   // uniform
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (i + q < wi) acc[y] = Path<CT>::mma(wv[q], xv[y][q], acc[y]);
            }
        }
        if (bn) {
          T* xo = Xo + (g0 + gb) * 2 * wo * nn + n0 + li;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int jj = ot + (sizeof(R) == 4 ? 2 * lk + q : lk + 4 * q);
            if (jj < 2 * wo) {   // rows (g, s, o) of X
#pragma unroll
              for (int y = 0; y < 4; ++y)
                if (gb + y < gn) {
                  T v;
                  v.x = acc[y][sizeof(R) == 4 ? 2 * q : q];
                  v.y = acc[y][sizeof(R) == 4 ? 2 * q + 1 : q + 2];
                  xo[(2 * wo * y + jj) * nn] = v;
                }
            }
          }
        }
      }
    }
    wave_sync();   // the tile is read before the next block rewrites it
  }
}

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
__device__ __forceinline__ void reflector(double ar, double ai, double xn, double n2, bool some,
                                          double2& tau, double2& inv) {
  double rs = __builtin_amdgcn_rsq(n2);   // 1 / |(alpha, x)|, two Newton steps
  const double h = 0.5 * n2;
  rs = rs * fma(-h * rs, rs, 1.5);
  rs = rs * fma(-h * rs, rs, 1.5);
  const double nrm = n2 * rs;
  const bool pos = ar >= 0.0;
  const double beta = pos ? -nrm : nrm, rb = pos ? -rs : rs;
  const double dx = ar - beta, den = fma(dx, dx, ai * ai);
  double rd = __builtin_amdgcn_rcp(den);
  rd = rd * fma(-den, rd, 2.0);
  rd = rd * fma(-den, rd, 2.0);
  const bool id = !(n2 >= 1e-200 && (some || xn != 0.0 || ai != 0.0));
  tau = make_double2(id ? 0.0 : (beta - ar) * rb, id ? 0.0 : -ai * rb);
  inv = make_double2(id ? 0.0 : dx * rd, id ? 0.0 : -ai * rd);
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
// Power of two that brings the largest entry ma near 1; 0 for a zero column
// (below 1e-280).
__device__ __forceinline__ double column_scale(double ma) {
  return ma < 1e-280 ? 0.0 : ma < 1e300 ? ldexp(1.0, -ilogb(ma)) : 1.0;
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

// ---------------------------------------------------------------------------

// Up to N elements per thread of src[0 .. count), loaded ahead of the work that
// hides their latency and put into LDS after it (what exceeds N goes through
// at the end).
template <typename T, int N>
struct Ahead {
  decltype(T::x) x[N], y[N];
  const T* src;
  int count;
  __device__ __forceinline__ void load(const T* s, int c) {
    src = s;
    count = c;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int e = (int)threadIdx.x + q * CNT;
      const T v = s[e < c ? e : 0];
      x[q] = v.x;
      y[q] = v.y;
    }
  }
  __device__ __forceinline__ void put(T* dst) const {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int e = (int)threadIdx.x + q * CNT;
      if (e < count) {
        dst[e].x = x[q];
        dst[e].y = y[q];
      }
    }
    for (int e = (int)threadIdx.x + N * CNT; e < count; e += CNT) dst[e] = src[e];
  }
};

// Where the intermediates live: LDS_ALL X, both environments and the ket site
// in LDS; LDS_X only X; LDS_NONE X in the slot's own buffer.
enum { LDS_NONE = 0, LDS_X = 1, LDS_ALL = 2 };

template <int CT, int CD, int MODE>
__global__ __launch_bounds__(CNT) void chain_kernel(const ChainArgs A) {
  using T = typename Path<CT>::T;
  using R = typename Path<CT>::R;
  constexpr bool ALL = MODE == LDS_ALL;
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  T* sW = reinterpret_cast<T*>(dyn);
  T* sF = reinterpret_cast<T*>(dyn + A.lds_f);     // F, then Q (m x n); the guess's site
  char* scr = dyn + A.lds_scr;                     // stage tiles, K-split parts, QR
  R* sTile = reinterpret_cast<R*>(scr);
  T* sPart = reinterpret_cast<T*>(scr);
  QrSmem<CD>& qsm = *reinterpret_cast<QrSmem<CD>*>(scr);
  __shared__ double s_red[CNW];

  const int n = A.n, br = blockIdx.x, tid = threadIdx.x;
  // the table by scalar loads
  typedef const __attribute__((address_space(4))) int* ctab;
  const ctab hd = (ctab)A.tab, rec = hd + 2 * n + 1 + (long long)br * chain_rec_ints(n);
  auto o_site = [&](int j) { return (long long)hd[j] * 256; };
  auto o_env = [&](int b) { return (long long)hd[n + b] * 256; };
  auto Kd = [&](int b) { return rec[4 + b]; };
  auto Dd = [&](int b) { return rec[4 + (n + 1) + b]; };
  auto wd = [&](int b) { return rec[4 + 2 * (n + 1) + b]; };
  auto o_mpo = [&](int j) { return (long long)rec[4 + 3 * (n + 1) + j] * 256; };

  char* slot = A.slots + (long long)rec[0] * A.slot_stride;
  const int cur = rec[1];
  const char* init = A.init + (long long)rec[2] * A.mps_bytes;
  const char* ket = slot + A.o_mps[cur];
  char* bra = slot + A.o_mps[1 - cur];
  char* envb = slot + A.o_env;
  T* X = MODE == LDS_NONE ? reinterpret_cast<T*>(slot + A.o_x2) : reinterpret_cast<T*>(dyn + A.lds_x);
  T* sE = reinterpret_cast<T*>(dyn + A.lds_e);     // LDS_ALL: the environment behind the front,
  T* sEa = reinterpret_cast<T*>(dyn + A.lds_ea);   // the one ahead,
  T* sK = reinterpret_cast<T*>(dyn + A.lds_k);     // and the ket site

  // operator (and ket site) of the next visit, loaded during stage D
  Ahead<T, 4> aw;
  Ahead<T, ALL ? 2 : 1> ak;
  auto site_load = [&](int j) {
    aw.load(reinterpret_cast<const T*>(A.mpo + o_mpo(j)), wd(j) * 4 * wd(j + 1));
    if constexpr (ALL)
      ak.load(reinterpret_cast<const T*>(ket + o_site(j)), 2 * Kd(j) * Kd(j + 1));
  };
  auto site_put = [&]() {
    aw.put(sW);
    if constexpr (ALL) ak.put(sK);
    lds_sync();
  };

  // stage A of site j into X[(g, s)][(o, n)], with `ahead` on the way to LDS
  auto stage_x = [&](int j, bool left) {
    const int wl = wd(j), wr = wd(j + 1), kl = Kd(j), kr = Kd(j + 1), ng = Dd(left ? j + 1 : j);
    const T* Eg = reinterpret_cast<const T*>(envb + o_env(left ? j + 1 : j));
    const T* Kg = reinterpret_cast<const T*>(ket + o_site(j));
    if constexpr (ALL) {
      if (left)
        stage_a<CT, true>(sE, sK, sW, ng, wr, wl, kr, kl, sTile, X);
      else
        stage_a<CT, false>(sE, sK, sW, ng, wl, wr, kl, kr, sTile, X);
    } else {
      if (left)
        stage_a<CT, true>(Eg, Kg, sW, ng, wr, wl, kr, kl, sTile, X);
      else
        stage_a<CT, false>(Eg, Kg, sW, ng, wl, wr, kl, kr, sTile, X);
    }
  };
  // next environment E[h][z] = sum_k B[h][k] X[k][z] to slot b, the site of the
  // next visit (jn) loaded meanwhile; `same`: that visit goes on from E
  auto stage_d = [&](int nh, int z, int m, int b, int jn, bool same, auto&& fb) {
    T* E = reinterpret_cast<T*>(envb + o_env(b));
    site_load(jn);
    wg_gemm<CT>(nh, z, m, sPart, fb, [&](int k, int c) { return X[k * z + c]; },
                [&](int h, int c, R re, R im) {
                  T v;
                  v.x = re;
                  v.y = im;
                  E[h * z + c] = v;
                  if constexpr (ALL)
                    if (same) sE[h * z + c] = v;
                });
    if constexpr (ALL) {
      if (!same && tid == 0) {   // the boundary environment
        sE[0].x = 1;
        sE[0].y = 0;
      }
    }
    // (sW and sK are free since stage A)
    site_put();   // X and the scratch are free from here; E is in flight to memory
  };
  // the visit after (t, j): false after the last one
  auto advance = [&](int t, int j, int& tn, int& jn) -> bool {
    if (t & 1) {
      if (j + 1 < n) {
        tn = t;
        jn = j + 1;
        return true;
      }
      tn = t + 1;
      jn = n - 2;
      return t < A.sweeps && n >= 2;
    }
    if (j > 0) {
      tn = t;
      jn = j - 1;
      return true;
    }
    tn = t + 1;
    jn = 1;
    return t < A.sweeps;
  };
  // whether the visit (t, j) moves left
  auto goes_left = [&](int t, int j) {
    int tn, jn;
    return advance(t, j, tn, jn) && jn < j;
  };

  site_load(n - 1);
  if constexpr (ALL) {
    if (tid == 0) {
      sE[0].x = 1;
      sE[0].y = 0;
    }
  }
  site_put();
  // right environments of the starting guess
  for (int j = n - 1; j >= 1; --j) {
    const int dl = Dd(j), dr = Dd(j + 1), z = wd(j) * Kd(j);
    Ahead<T, 2 * CD * CD / CNT> ab;
    ab.load(reinterpret_cast<const T*>(init + o_site(j)), dl * 2 * dr);
    stage_x(j, true);
    ab.put(sF);
    __syncthreads();   // also: the stores of the last stage D have landed
    stage_d(dl, z, 2 * dr, j, j - 1, j > 1 || goes_left(1, 0), [&](int h, int k) {
      T v = sF[h * 2 * dr + (k & 1) * dr + (k >> 1)];   // k = (c, s): conj(B[h][s][c])
      v.y = -v.y;
      return v;
    });
  }

  int t = 1, j = 0;
  for (;;) {
    int tn, jn;
    const bool more = advance(t, j, tn, jn), left = more && jn < j;
    const int ng = Dd(left ? j + 1 : j), nh = Dd(left ? j : j + 1), m = 2 * ng;
    const int b = left ? j : j + 1;   // slot of the environment ahead, then of the next one
    const int z = wd(b) * Kd(b);
    const T* Eg = reinterpret_cast<const T*>(envb + o_env(b));
    Ahead<T, ALL ? 4 : 1> ae;
    if constexpr (ALL) ae.load(Eg, nh * z);
    stage_x(j, left);
    if constexpr (ALL) ae.put(sEa);
    __syncthreads();   // also: the stores of the last stage D have landed
    auto put_f = [&](int r, int h, R re, R im) {   // rows (g, s); moving left (s, g), conjugated
      T v;
      v.x = re;
      v.y = left ? -im : im;
      sF[(left ? (r & 1) * ng + (r >> 1) : r) * nh + h] = v;
    };
    if constexpr (ALL)
      wg_gemm<CT>(m, nh, z, sPart, [&](int r, int k) { return X[r * z + k]; },
                  [&](int k, int h) { return sEa[h * z + k]; }, put_f);
    else
      wg_gemm<CT>(m, nh, z, sPart, [&](int r, int k) { return X[r * z + k]; },
                  [&](int k, int h) { return Eg[h * z + k]; }, put_f);
    lds_sync();
    T* B = reinterpret_cast<T*>(bra + o_site(j));
    if (!more) {   // T = F / |F|, f = |F|^2
      double q = 0.0;
      for (int e = tid; e < m * nh; e += CNT) {
        const double2 u = to_d2(sF[e]);
        q += u.x * u.x + u.y * u.y;
      }
      q = block_sum(q, s_red);
      const double sc = q > 0 ? 1.0 / sqrt(q) : 0.0;
      for (int e = tid; e < m * nh; e += CNT) {
        const double2 u = to_d2(sF[e]);
        T v;
        v.x = u.x * sc;
        v.y = u.y * sc;
        B[e] = v;
      }
      if (tid == 0) A.nrm[br] = q;
      return;
    }
    // (F is in registers before the QR's first barrier, Q written after its last)
    small_qr<CD>(sF, m, nh, qsm, [&](int r, int h, double re, double im) {
      T v;
      v.x = re;
      v.y = im;
      sF[r * nh + h] = v;
      if (left) {
        v.y = -v.y;
        B[h * m + r] = v;
      } else {
        B[r * nh + h] = v;
      }
    });
    lds_sync();
    stage_d(nh, z, m, b, jn, goes_left(tn, jn) == left, [&](int h, int k) {
      T v = sF[(left ? (k & 1) * ng + (k >> 1) : k) * nh + h];   // conj of the site tensor
      if (!left) v.y = -v.y;
      return v;
    });
    t = tn;
    j = jn;
  }
}

// Outcome norms n_m = <psi|P_m|psi> (FP64) of small branches, one workgroup per
// branch: the left transfer from the last left-canonical site (or a cached
// one) and the right transfer from the first right-canonical site to the
// measured qubit q, then n_m = Re sum conj(A_q[.][m][.]) (E A_q G^T)[.][m][.].
// The transfers stay in LDS, each site is loaded while the one before it is
// contracted; the left transfer at bond q goes back to the slot (the cache).
// Latency bound like the step above: 9 us for 10 qubits at bond 16, where two
// launches per site and transfer took about 100 us (a run of 13 qubits with 128
// shots and 12 measurements 6.0 ms with them, 4.45 ms with this kernel; 10
// qubits, one shot, 10 measurements 3.5 and 3.1 ms).
template <int CT>
__global__ __launch_bounds__(CNT) void transfer_kernel(const TransferArgs A) {
  using T = typename Path<CT>::T;
  constexpr int D = TRANSFER_MAX_D;
  __shared__ double2 sE[D * D], sG[D * D], sT[2 * D * D], sPart[CNW * 256];
  __shared__ T sA[2][2 * D * D];
  __shared__ double s_red[CNW];
  const int n = A.n, br = blockIdx.x, tid = threadIdx.x;
  typedef const __attribute__((address_space(4))) int* ctab;
  const ctab hd = (ctab)A.tab, rec = hd + n + (long long)br * transfer_rec_ints(n);
  char* slot = A.slots + (long long)rec[0] * A.slot_stride;
  const char* mps = slot + A.o_mps[rec[1]];
  const int q = rec[2], e_from = rec[3], e_cached = rec[4], g_from = rec[5];
  auto dim = [&](int b) { return rec[6 + b]; };
  double2* gE = reinterpret_cast<double2*>(slot + A.o_e);
  Ahead<T, 2 * D * D / CNT> next;
  auto load = [&](int j) {
    next.load(reinterpret_cast<const T*>(mps + (long long)hd[j] * 256), 2 * dim(j) * dim(j + 1));
  };
  // sites in the order they are used: e_from .. q - 1, then g_from - 1 .. q + 1, q
  int buf = 0;
  load(e_from < q ? e_from : g_from - 1 > q ? g_from - 1 : q);
  next.put(sA[0]);
  bool e_on = e_cached != 0;
  if (e_on) {
    const int d = dim(e_from);
    for (int i = tid; i < d * d; i += CNT) sE[i] = gE[i];
  }
  __syncthreads();
  for (int j = e_from; j < q; ++j, buf ^= 1) {
    const int dl = dim(j), dr = dim(j + 1);
    const T* a = sA[buf];
    load(j + 1 < q ? j + 1 : g_from - 1 > q ? g_from - 1 : q);
    if (e_on) {   // (E A)[a][s b]
      wg_gemm<CT_F64>(dl, 2 * dr, dl, sPart, [&](int i, int k) { return sE[i * dl + k]; },
                      [&](int k, int c) { return to_d2(a[k * 2 * dr + c]); },
                      [&](int i, int c, double re, double im) {
                        sT[i * 2 * dr + c] = make_double2(re, im);
                      });
      lds_sync();
    }
    wg_gemm<CT_F64>(dr, dr, 2 * dl, sPart,
                    [&](int i, int k) { return cconj(to_d2(a[k * dr + i])); },
                    [&](int k, int c) { return e_on ? sT[k * dr + c] : to_d2(a[k * dr + c]); },
                    [&](int i, int c, double re, double im) {
                      sE[i * dr + c] = make_double2(re, im);
                    });
    next.put(sA[buf ^ 1]);
    lds_sync();
    e_on = true;
  }
  bool g_on = false;
  for (int j = g_from - 1; j > q; --j, buf ^= 1) {
    const int dl = dim(j), dr = dim(j + 1);
    const T* a = sA[buf];
    load(j - 1);
    if (g_on) {   // (A G^T)[a s][c]
      wg_gemm<CT_F64>(2 * dl, dr, dr, sPart, [&](int i, int k) { return to_d2(a[i * dr + k]); },
                      [&](int k, int c) { return sG[c * dr + k]; },
                      [&](int i, int c, double re, double im) {
                        sT[i * dr + c] = make_double2(re, im);
                      });
      lds_sync();
    }
    wg_gemm<CT_F64>(dl, dl, 2 * dr, sPart,
                    [&](int i, int k) { return cconj(to_d2(a[i * 2 * dr + k])); },
                    [&](int k, int c) { return g_on ? sT[c * 2 * dr + k] : to_d2(a[c * 2 * dr + k]); },
                    [&](int i, int c, double re, double im) {
                      sG[i * dl + c] = make_double2(re, im);
                    });
    next.put(sA[buf ^ 1]);
    lds_sync();
    g_on = true;
  }
  const int dl = dim(q), dr = dim(q + 1);
  const T* a = sA[buf];
  if (e_on) {
    for (int i = tid; i < dl * dl; i += CNT) gE[i] = sE[i];
    wg_gemm<CT_F64>(dl, 2 * dr, dl, sPart, [&](int i, int k) { return sE[i * dl + k]; },
                    [&](int k, int c) { return to_d2(a[k * 2 * dr + c]); },
                    [&](int i, int c, double re, double im) {
                      sT[i * 2 * dr + c] = make_double2(re, im);
                    });
    lds_sync();
  }
  // z[(a, s)][c]; only the real part of conj(A) z is wanted, element by element
  double p[2] = {0.0, 0.0};
  if (g_on) {
    wg_gemm<CT_F64>(2 * dl, dr, dr, sPart,
                    [&](int i, int k) { return e_on ? sT[i * dr + k] : to_d2(a[i * dr + k]); },
                    [&](int k, int c) { return sG[c * dr + k]; },
                    [&](int i, int c, double re, double im) {
                      const double2 u = to_d2(a[i * dr + c]);
                      const double v = u.x * re + u.y * im;
                      p[0] += i & 1 ? 0.0 : v;
                      p[1] += i & 1 ? v : 0.0;
                    });
  } else {
    for (int i = tid >> 4; i < 2 * dl; i += CNT >> 4) {   // 16 lanes per row
      const int c = tid & 15;
      if (c < dr) {
        const double2 u = to_d2(a[i * dr + c]), z = e_on ? sT[i * dr + c] : u;
        const double v = u.x * z.x + u.y * z.y;
        p[0] += i & 1 ? 0.0 : v;
        p[1] += i & 1 ? v : 0.0;
      }
    }
  }
  const double n0 = block_sum(p[0], s_red), n1 = block_sum(p[1], s_red);
  if (tid == 0) {
    A.out[2 * br] = n0;
    A.out[2 * br + 1] = n1;
  }
}

template <int CT, int CD>
size_t scratch_bytes() {
  const size_t rs = CT == CT_F32 ? 4 : 8;
  size_t s = (size_t)CNW * 4 * 16 * 17 * rs;                    // stage A tiles
  s = s > (size_t)CNW * 256 * 2 * rs ? s : (size_t)CNW * 256 * 2 * rs;   // K-split parts
  return s > sizeof(QrSmem<CD>) ? s : sizeof(QrSmem<CD>);
}

template <int CT, int CD, int MODE>
hipError_t start_chain(const ChainArgs& a, int branches, size_t lds, hipStream_t s) {
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(&chain_kernel<CT, CD, MODE>),
      hipFuncAttributeMaxDynamicSharedMemorySize, CHAIN_LDS);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((chain_kernel<CT, CD, MODE>), dim3(branches), dim3(CNT), lds, s, a);
  return hipGetLastError();
}

template <int CT, int CD>
hipError_t run_chain(ChainArgs a, int branches, const ChainDims& d, hipStream_t s) {
  const size_t cs = CT == CT_F32 ? sizeof(float2) : sizeof(double2);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) / 256 * 256;
    return (int)o;
  };
  take((size_t)d.op_elems * cs);
  a.lds_f = take(2 * (size_t)d.d_max * d.d_max * cs);
  a.lds_scr = take(scratch_bytes<CT, CD>());
  const size_t none = off;
  a.lds_x = take(d.x_elems * cs);
  const size_t with_x = off;
  a.lds_e = take(d.e_elems * cs);
  a.lds_ea = take(d.e_elems * cs);
  a.lds_k = take(d.k_elems * cs);
  // More branches than CUs: the largest form of which two fit a CU (two
  // workgroups hide each other's chains); else as much in LDS as fits.
  const size_t half = 80 * 1024;
  const size_t lim = branches > 256 && none <= half ? half : CHAIN_LDS;
  if constexpr (CD == 16) {
    if (off <= lim) return start_chain<CT, CD, LDS_ALL>(a, branches, off, s);
  }
  if (with_x <= lim) return start_chain<CT, CD, LDS_X>(a, branches, with_x, s);
  if (none <= lim) return start_chain<CT, CD, LDS_NONE>(a, branches, none, s);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_transfer(int ct, const TransferArgs& a, int branches, hipStream_t s) {
  if (branches <= 0) return hipSuccess;
  if (ct == CT_F32)
    hipLaunchKernelGGL((transfer_kernel<CT_F32>), dim3(branches), dim3(CNT), 0, s, a);
  else
    hipLaunchKernelGGL((transfer_kernel<CT_F64>), dim3(branches), dim3(CNT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_chain(int ct, const ChainArgs& a, int branches, const ChainDims& d,
                        hipStream_t s) {
  if (branches <= 0) return hipSuccess;
  if (d.d_max > CHAIN_MAX_D || d.w_max > CHAIN_MAX_W) return hipErrorInvalidValue;
  if (ct == CT_F32)
    return d.d_max <= 16 ? run_chain<CT_F32, 16>(a, branches, d, s)
                         : run_chain<CT_F32, 32>(a, branches, d, s);
  return d.d_max <= 16 ? run_chain<CT_F64, 16>(a, branches, d, s)
                       : run_chain<CT_F64, 32>(a, branches, d, s);
}

}  // namespace dcs
