// QR of small and medium matrices in one launch, one 256-thread workgroup per
// matrix: up to 64 x 32 by the register QR of qr_small.h, up to 128 x 64 in
// 16-column panels.
//
// Panels: rows 32 w .. 32 w + 31 live in the registers of wave w (eight slots of
// four rows in the layout of the FP64 MFMA result, up to four 16-column
// blocks).  A panel is factored column by column (one reduction and one barrier
// per column, as in small_qr), its V goes to LDS, T follows from the products
// of the reflectors by back substitution, and the later blocks are updated on
// the matrix cores straight from the registers: W = V^H A takes both operands in
// the layout they are held in, only A -= V (T^H W) reads V from LDS.  Q is formed
// by the same update, the panels applied backwards to the identity, so nothing
// goes through memory between reading F and writing Q.
//
// What bounds it is the chain of one matrix: about 2000 cycles per column, more
// than half of the time, then the updates' exchanges through LDS.  75 complex64
// matrices of 90 x 45: 80 us, where the factorisation and the Q launch of the
// blocked kernel took 46 us each and the gap between them; 64 x 32: 45 us, 32 x
// 16: 10 us (17 us a launch).
#include "qr_small.h"

namespace dcs {
namespace {

constexpr int MQB = 16, MSL = 8, MNB = 4;   // panel width, row slots, column blocks

__device__ __forceinline__ int mpx(int i, int c) { return i * MQB + (c ^ (i & 15)); }

// LDS: the exchanges, T of every panel, V of every panel (rows 16 p .. of mr
// rows, swizzled): sum of (mr - 16 p) 16 values.
inline int mid_v_elems(int mr, int npan) {
  return MQB * (npan * mr - MQB * (npan * (npan - 1) / 2));
}
constexpr int MID_FIXED = 256 + 2 * CNW * 2 * MQB + CNW * 256 + 256 + MQB + CNW;   // S, ex, W, W2, tau, mx
inline size_t mid_lds(int m, int n) {
  const int mr = (m + 15) / 16 * 16, npan = (n + 15) / 16;
  return sizeof(double2) * ((size_t)MID_FIXED + npan * 256 + mid_v_elems(mr, npan));
}

// T (16 x 16, zero below the diagonal and in unused columns) of a panel of nbk
// columns from T^{-1} = diag(1 / tau) + S^H-part: S[k 16 + j] = v_j^H v_k, j < k.
// One wave.
__device__ __forceinline__ void panel_t(const double2* S, const double2* tau, int nbk,
                                        double2* T) {
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  double2 z[4];   // rows 4 (r + g - 3) + lk, column li
  const int last = (nbk - 1) >> 2;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 4 * (r + last - 3) + lk;
    z[r] = make_double2(i == li && li < nbk ? 1.0 : 0.0, 0.0);
  }
#pragma unroll 1
  for (int g = last; g >= 0; --g) {
    static_for<4>([&](auto qc) {
      constexpr int kr = 3 - decltype(qc)::value;
      const int k = 4 * g + kr;
      if (k >= nbk) return;   // uniform
      double2 sv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 4 * (r + g - 3) + lk;
        sv[r] = S[i >= 0 ? k * MQB + i : 0];
      }
      const double2 zk = cmul(tau[k], row_of<kr>(z[3]));
      sv[3] = keep_if(lk < kr, sv[3]);
      z[3].x = lk == kr ? zk.x : z[3].x;
      z[3].y = lk == kr ? zk.y : z[3].y;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[r].x = fma(-sv[r].x, zk.x, fma(sv[r].y, zk.y, z[r].x));
        z[r].y = fma(-sv[r].x, zk.y, fma(-sv[r].y, zk.x, z[r].y));
      }
    });
    if (4 * g + lk < nbk) T[(4 * g + lk) * MQB + li] = z[3];
    z[3] = z[2];
    z[2] = z[1];
    z[1] = z[0];
  }
  for (int i = nbk + lk; i < MQB; i += 4) T[i * MQB + li] = make_double2(0.0, 0.0);
}

// blk (this wave's rows base + 4 t + lk of one column block) -= V (X (V^H blk)),
// X = T^H or T.  v: V in the layout of blk (zero outside the matrix and above
// the panel).  Vp: the panel's V in LDS, row 0 = matrix row p0.
template <bool TRANS>
__device__ __forceinline__ void apply_panel(double2 (&blk)[MSL], const double2 (&v)[MSL],
                                            const double2* Vp, int p0, int base, int mr,
                                            const double2* T, double2* W, double2* W2) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  CAcc3 w;
  w.zero();
#pragma unroll
  for (int t = 0; t < MSL; ++t) w.add(v[t].x, -v[t].y, blk[t].x, blk[t].y);
#pragma unroll
  for (int r = 0; r < 4; ++r)
    W[wave * 256 + (lk + 4 * r) * MQB + li] = make_double2(w.re(r), w.im(r));
  lds_sync();
  {   // each wave adds up 64 entries
    const int e = wave * 64 + lane;
    const double2 a = W[e], b = W[256 + e], c = W[512 + e], d = W[768 + e];
    W2[e] = make_double2((a.x + b.x) + (c.x + d.x), (a.y + b.y) + (c.y + d.y));
  }
  lds_sync();
  CAcc3 x2;
  x2.zero();
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 4 * s + lk;
    const double2 tv = TRANS ? cconj(T[k * MQB + li]) : T[li * MQB + k];
    const double2 wv = W2[k * MQB + li];
    x2.add(tv.x, tv.y, wv.x, wv.y);
  }
  double xr[4], xi[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    xr[s] = x2.re(s);
    xi[s] = x2.im(s);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u) {   // two tiles of 16 rows
    const int r0 = base + 16 * u;
    if (r0 + 16 <= p0 || r0 >= mr) continue;   // uniform (mr: end of this wave's rows)
    const int row = r0 + li - p0;
    const bool in = row >= 0 && r0 + li < mr;
    CAcc3 e;
    e.zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double2 q = Vp[in ? mpx(row, 4 * s + lk) : 0];
      e.add(in ? q.x : 0.0, in ? q.y : 0.0, xr[s], xi[s]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      blk[4 * u + r].x -= e.re(r);
      blk[4 * u + r].y -= e.im(r);
    }
  }
}

template <int CTI, int CTO>
__global__ __launch_bounds__(CNT, 1) void qr_mid_kernel(const QrArgs args) {
  using TI = typename St<CTI>::T;
  using TO = typename St<CTO>::T;
  extern __shared__ __attribute__((aligned(16))) double2 mid_dyn[];
  __shared__ double s_red[CNW];
  const int gi = find_group<QR_MAX_GROUPS>(args.g, args.ngroups, blockIdx.x);
  const QrGroup& G = args.g[gi];
  const int item = blockIdx.x - G.blk_begin, m = G.m, n = G.n, mode = G.mode;
  const TI* __restrict__ F = reinterpret_cast<const TI*>(item_ptr(G.f, G.ids, item));
  TO* __restrict__ Q = reinterpret_cast<TO*>(const_cast<char*>(item_ptr(G.q, G.ids, item)));
  double* nrm = reinterpret_cast<double*>(const_cast<char*>(item_ptr(G.nrm2, G.ids, item)));
  const int mr = (m + 15) & ~15, npan = (n + 15) >> 4;
  double2* S = mid_dyn;
  double2* ex = S + 256;
  double2* W = ex + 2 * CNW * 2 * MQB;
  double2* W2 = W + CNW * 256;
  double2* tau = W2 + 256;
  double* mx = reinterpret_cast<double*>(tau + MQB);
  double2* Ts = tau + MQB + CNW;
  double2* V = Ts + npan * 256;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);

  double2 a[MNB][MSL];
  double nsq = 0.0;
#pragma unroll
  for (int j = 0; j < MNB; ++j)
#pragma unroll
    for (int t = 0; t < MSL; ++t) {
      const int row = 32 * wave + 4 * t + lk, col = MQB * j + li;
      const bool in = row < m && col < n;
      const TI u = F[!in ? 0 : mode == 0 ? row * n + col : col * m + row];
      a[j][t].x = in ? (double)u.x : 0.0;
      a[j][t].y = in ? (mode == 0 ? (double)u.y : -(double)u.y) : 0.0;
      nsq = fma(a[j][t].x, a[j][t].x, fma(a[j][t].y, a[j][t].y, nsq));
    }

  // ------- factorisation: the panel is a[0], the later blocks a[1 ..] --------
  int sh = 0, buf = 0;   // 16-row groups that this wave's rows have moved up by
  double2* Vp = V;
#pragma unroll 1
  for (int p = 0; p < npan; ++p) {
    const int p0 = MQB * p, nbk = min(MQB, n - p0), base = 32 * wave + 16 * sh;
    const bool holds = wave == p0 >> 5;   // the rows of the panel's diagonal
    int col = li, g = 0;
    double2 myinv = zero;
#pragma unroll 1
    for (;; ++g) {
      static_for<4>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const int k = 4 * g + q;   // column of the panel
        if (k >= nbk) return;      // uniform
        double2 x[MSL], d, row, tk, inv;
        double2 r0 = row_of<q>(a[0][0]);
        a[0][0] = keep_if(!holds || lk != q, a[0][0]);
#pragma unroll
        for (int t = 0; t < MSL; ++t) x[t] = bcol64<q>(a[0][t]);
        double xn, ar, ai, n2;
        auto exchange = [&]() {
          d = column_dot<MSL>(x, a[0]);
          if (lk < 2)
            ex[((buf * CNW + wave) * 2 + lk) * MQB + li] =
                make_double2(lk ? r0.x : d.x, lk ? r0.y : d.y);
          lds_sync();
          double2 u[CNW];
#pragma unroll
          for (int w = 0; w < CNW; ++w) u[w] = ex[(buf * CNW + w) * 2 * MQB + li];
          row = ex[((buf * CNW + (p0 >> 5)) * 2 + 1) * MQB + li];
          d = make_double2((u[0].x + u[1].x) + (u[2].x + u[3].x),
                           (u[0].y + u[1].y) + (u[2].y + u[3].y));
          buf ^= 1;
          xn = readlane_d(d.x, q);
          ar = readlane_d(row.x, q);
          ai = readlane_d(row.y, q);
          n2 = fma(ar, ar, fma(ai, ai, xn));
        };
        exchange();
        bool some = false;
        // (the same on every wave)
        if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)odd_column(ai, xn, n2)), 0)) {
          double big = 0.0;
#pragma unroll
          for (int t = 0; t < MSL; ++t) big = fmax(big, fmax(fabs(x[t].x), fabs(x[t].y)));
          big = wave_max_dpp(big);
          lds_sync();   // readers of an earlier column's maxima are past
          if (lane == 0) mx[wave] = big;
          lds_sync();
          big = fmax(fmax(mx[0], mx[1]), fmax(mx[2], mx[3]));
          const double ma = fmax(big, fmax(fabs(ar), fabs(ai)));
          const double sc = in_range(n2) ? 1.0 : column_scale(ma);
          const double own = li == q ? sc : 1.0;
          some = big > 0.0 && sc != 0.0;
#pragma unroll
          for (int t = 0; t < MSL; ++t) {
            x[t] = make_double2(x[t].x * sc, x[t].y * sc);
            a[0][t] = make_double2(a[0][t].x * own, a[0][t].y * own);
          }
          r0 = make_double2(r0.x * own, r0.y * own);
          exchange();
        }
        reflector(ar, ai, xn, n2, some, tk, inv);
        const double2 w = make_double2(row.x + inv.x * d.x + inv.y * d.y,
                                       row.y + inv.x * d.y - inv.y * d.x);
        column_sub<MSL>(a[0], keep_if(col > k, cmul(cmul(cconj(tk), inv), w)), x);
        if (wave == CNW - 1) {   // row k of V (lk = 0) and of the products (lk = 1), tau
          const double2 u = cmul(make_double2(lk ? w.x : row.x, lk ? w.y : row.y), myinv);
          const bool below = col < k;
          double2* const to = lk == 0 ? Vp + mpx(k, col) : lk == 1 ? S + (k * MQB + col) : tau + k;
          if (lk == 0 || (lk == 1 && below) || lane == 32)
            *to = make_double2(lk >= 2 ? tk.x : below ? u.x : (col == k ? 1.0 : 0.0),
                               lk >= 2 ? tk.y : below ? (lk ? -u.y : u.y) : 0.0);
        }
        myinv.x = col == k ? inv.x : myinv.x;
        myinv.y = col == k ? inv.y : myinv.y;
      });
      if (4 * g + 4 >= nbk) break;
      if (holds) {
#pragma unroll
        for (int t = 0; t < MSL - 1; ++t) a[0][t] = lanes_on(a[0][t + 1]);
        a[0][MSL - 1] = zero;
      } else {
#pragma unroll
        for (int t = 0; t < MSL; ++t) a[0][t] = lanes_on(a[0][t]);
      }
      myinv = lanes_on(myinv);
      col = (col + 4) & 15;
    }
    // V below the panel's own rows, zero in unused columns
    const double2 vinv = keep_if(col < nbk, myinv);
#pragma unroll
    for (int t = 0; t < MSL; ++t) {
      const int row = base + 4 * (t + (holds ? g : 0)) + lk;
      const double2 v = cmul(a[0][t], vinv);
      if (row >= p0 + nbk && row < mr && row < 32 * wave + 32) Vp[mpx(row - p0, col)] = v;
    }
    lds_sync();
    if (wave == 0) panel_t(S, tau, nbk, Ts + 256 * p);
    if (p + 1 < npan) {
      double2 v[MSL];
#pragma unroll
      for (int t = 0; t < MSL; ++t) {
        const int row = base + 4 * t + lk;
        const bool in = row >= p0 && row < mr && row < 32 * wave + 32;
        v[t] = keep_if(in, Vp[in ? mpx(row - p0, li) : 0]);
      }
#pragma unroll
      for (int j = 1; j < MNB; ++j)
        if (p + j < npan)   // uniform; T is there after the first barrier inside
          apply_panel<true>(a[j], v, Vp, p0, base, min(mr, 32 * wave + 32), Ts + 256 * p, W, W2);
      // the blocks move on by one, the panel's rows leave the wave that held them
#pragma unroll
      for (int j = 0; j < MNB - 1; ++j)
#pragma unroll
        for (int t = 0; t < MSL; ++t) a[j][t] = a[j + 1][t];
      if (holds) {
        ++sh;
#pragma unroll
        for (int j = 0; j < MNB - 1; ++j)
#pragma unroll
          for (int t = 0; t < MSL; ++t) a[j][t] = t < MSL / 2 ? a[j][t + MSL / 2] : zero;
      }
    }
    Vp += MQB * (mr - p0);
  }
  lds_sync();

  // ------- Q: the panels applied backwards to the identity --------------------
#pragma unroll
  for (int j = 0; j < MNB; ++j)
#pragma unroll
    for (int t = 0; t < MSL; ++t) {
      const int row = 32 * wave + 4 * t + lk;
      a[j][t] = make_double2(row == MQB * j + li ? 1.0 : 0.0, 0.0);
    }
#pragma unroll 1
  for (int p = npan - 1; p >= 0; --p) {
    const int p0 = MQB * p, base = 32 * wave;
    Vp -= MQB * (mr - p0);
    double2 v[MSL];
#pragma unroll
    for (int t = 0; t < MSL; ++t) {
      const int row = base + 4 * t + lk;
      const bool in = row >= p0 && row < mr;
      v[t] = keep_if(in, Vp[in ? mpx(row - p0, li) : 0]);
    }
#pragma unroll
    for (int j = 0; j < MNB; ++j)
      if (j >= p && j < npan)   // uniform
        apply_panel<false>(a[j], v, Vp, p0, base, mr, Ts + 256 * p, W, W2);
  }
#pragma unroll
  for (int j = 0; j < MNB; ++j)
#pragma unroll
    for (int t = 0; t < MSL; ++t) {
      const int row = 32 * wave + 4 * t + lk, c = MQB * j + li;
      if (row < m && c < n) {
        TO o;
        o.x = a[j][t].x;
        o.y = mode == 0 ? a[j][t].y : -a[j][t].y;
        Q[mode == 0 ? row * n + c : c * m + row] = o;
      }
    }
  nsq = block_sum(nsq, s_red);
  if (threadIdx.x == 0) *nrm = nsq;
}

// Up to 2 CD x CD: the register QR, F read and Q written by the caller's layout.
template <int CTI, int CTO, int CD>
__global__ __launch_bounds__(CNT) void qr_small_kernel(const QrArgs args) {
  using TI = typename St<CTI>::T;
  using TO = typename St<CTO>::T;
  extern __shared__ __attribute__((aligned(16))) double2 mid_dyn[];
  __shared__ double s_red[CNW];
  QrSmem<CD>& sm = *reinterpret_cast<QrSmem<CD>*>(mid_dyn);
  double2* f = mid_dyn + (sizeof(QrSmem<CD>) + sizeof(double2) - 1) / sizeof(double2);
  const int gi = find_group<QR_MAX_GROUPS>(args.g, args.ngroups, blockIdx.x);
  const QrGroup& G = args.g[gi];
  const int item = blockIdx.x - G.blk_begin, m = G.m, n = G.n, mode = G.mode;
  const TI* __restrict__ F = reinterpret_cast<const TI*>(item_ptr(G.f, G.ids, item));
  TO* __restrict__ Q = reinterpret_cast<TO*>(const_cast<char*>(item_ptr(G.q, G.ids, item)));
  double* nrm = reinterpret_cast<double*>(const_cast<char*>(item_ptr(G.nrm2, G.ids, item)));
  double nsq = 0.0;
  for (int e = threadIdx.x; e < m * n; e += CNT) {   // in F's order
    const double2 u = to_d2(F[e]);
    nsq = fma(u.x, u.x, fma(u.y, u.y, nsq));
    if (mode == 0) {
      f[e] = u;
    } else {
      const int c = e / m, r = e - c * m;
      f[r * n + c] = cconj(u);
    }
  }
  nsq = block_sum(nsq, s_red);
  if (threadIdx.x == 0) *nrm = nsq;
  small_qr<CD>(f, m, n, sm, [&](int r, int c, double re, double im) {
    TO o;
    o.x = re;
    o.y = mode == 0 ? im : -im;
    Q[mode == 0 ? r * n + c : c * m + r] = o;
  });
}

template <int CTI, int CTO>
hipError_t run_mid(const QrArgs& args, int m_max, int n_max, size_t lds, hipStream_t s) {
  const dim3 grid(args.total_blocks), blk(CNT);
  if (m_max <= 32 && n_max <= 16) {
    const size_t b = sizeof(QrSmem<16>) + sizeof(double2) * (1 + (size_t)m_max * n_max);
    hipLaunchKernelGGL((qr_small_kernel<CTI, CTO, 16>), grid, blk, b, s, args);
  } else if (m_max <= 64 && n_max <= 32) {
    const size_t b = sizeof(QrSmem<32>) + sizeof(double2) * (1 + (size_t)m_max * n_max);
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&qr_small_kernel<CTI, CTO, 32>),
        hipFuncAttributeMaxDynamicSharedMemorySize, 112 * 1024);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((qr_small_kernel<CTI, CTO, 32>), grid, blk, b, s, args);
  } else {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&qr_mid_kernel<CTI, CTO>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)mid_lds(QR_MID_M, QR_MID_N));
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((qr_mid_kernel<CTI, CTO>), grid, blk, lds, s, args);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_qr_mid(int ct_in, int ct_out, const QrArgs& args, hipStream_t s) {
  if (args.total_blocks <= 0) return hipSuccess;
  int m_max = 0, n_max = 0;
  size_t lds = 0;
  for (int g = 0; g < args.ngroups; ++g) {
    const QrGroup& G = args.g[g];
    if (G.mode == 2 || G.m < G.n || G.n < 1 || G.m > QR_MID_M || G.n > QR_MID_N)
      return hipErrorInvalidValue;
    m_max = G.m > m_max ? G.m : m_max;
    n_max = G.n > n_max ? G.n : n_max;
    const size_t b = mid_lds(G.m, G.n);
    lds = b > lds ? b : lds;
  }
  if (ct_in == CT_F32 && ct_out == CT_F32) return run_mid<CT_F32, CT_F32>(args, m_max, n_max, lds, s);
  if (ct_in == CT_F64 && ct_out == CT_F64) return run_mid<CT_F64, CT_F64>(args, m_max, n_max, lds, s);
  if (ct_in == CT_F64 && ct_out == CT_F32) return run_mid<CT_F64, CT_F32>(args, m_max, n_max, lds, s);
  return hipErrorInvalidValue;
}

}  // namespace dcs
