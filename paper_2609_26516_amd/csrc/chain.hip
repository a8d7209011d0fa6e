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
// 53 000 cycles, three fifths of them in the QR (about 2000 per column, some 265
// instructions on one wave), 9000 in stage A, 5000 each in B and D.  16 qubits,
// bond 16, two sweeps, one complex128 branch: 0.71 ms, against 1.24 ms as a
// sequence of launches (15 environments and 31 visits of 4 to 5 launches); 64
// branches 0.73 against 1.70 ms; bond 4: 0.43 against 0.90 ms.
#include "qr_small.h"

namespace dcs {
namespace {

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
    __syncthreads();
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
    // (sW and sK are free since stage A.)  The barrier at its end orders global
    // memory too: the next visit's waves read E as the other waves stored it.
    // X and the scratch are free from here.
    site_put();
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
    __syncthreads();   // X may lie in global memory
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
    __syncthreads();   // X may lie in global memory
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
