// FP64 Householder QR with explicit thin Q for local matrices of more than
// 512 rows (bond caps above 256), where one workgroup per matrix would leave
// the chip idle and the panel no longer fits in LDS, and the spread path for
// small batches of smaller matrices.  Same reflectors as the other QR kernels
// (LAPACK convention: v_k = 1, beta = -sign(Re alpha) |x|,
// tau = ((beta - Re alpha) / beta, -Im alpha / beta), tau = 0 for a zero
// column), blocked in panels of 16 columns with the compact WY form
// H_p ... H_{p+15} = I - V T V^H:
//   qrl_load   F (mode 0) or F^H (mode 1) -> FP64 working matrix A (m x n,
//              row-major), |F|^2 partial sums per chunk
//   qrt_* (m > 512) / qrs_panel (m <= 512)
//              A[p:, p:p+16] factored by Cholesky QR and Householder
//              reconstruction (qr_cholpanel.h), or column by column where
//              the panel does not allow it, by one 512-thread workgroup per
//              256-row chunk (m > 512) or per matrix (m <= 512); writes the
//              explicit V (unit diagonal) and T
//   qrl_wpart  W = V^H A[p:, c:] in parts over (16-column strip, 256-row
//   qrl_update chunk) tiles on FP64 MFMA, then A[p:, c:] -= V T^H W, every
//              chunk summing its strip's parts in one order
// After the last panel A is reset to [I; 0] and the reflectors are applied in
// reverse order, four panels at a time, which leaves the thin Q = H_0 ...
// H_{n-1} [I; 0] in A:
//   qrq_merge  the T factors of each four panels joined to one of 64 x 64
//   qrq_wpart  W = V^H A[p:, p:] for the four panels' 64 columns of V, and
//   qrq_update A[p:, p:] -= V T W
// qrl_store writes Q (mode 0) or Q^H (mode 1) in the output precision.
#include "dcs_internal.h"
#include "kernel_util.h"
#include "qr_panel.h"
#include "qr_cholpanel.h"
#include "tile_load.h"

namespace dcs {
namespace {


constexpr int QRL_CHUNKS = 64;   // load / store / fill work units per matrix

struct QrlItem {
  const QrGroup* g;
  int item;
};

__device__ __forceinline__ QrlItem qrl_item(const QrArgs& args, int flat) {
  const int gi = find_group<QR_MAX_GROUPS>(args.g, args.ngroups, flat);
  return {&args.g[gi], flat - args.g[gi].blk_begin};
}

__device__ __forceinline__ double2* qrl_ws(const QrlItem& it) {
  return reinterpret_cast<double2*>(const_cast<char*>(item_ptr(it.g->ws, it.g->ids, it.item)));
}

// workspace: A (m n), V (m n), T factors (16 (n + 16)), |F|^2 chunk partials,
// then the W parts of the strip updates
__device__ __forceinline__ double* qrl_partials(double2* ws, int m, int n) {
  return reinterpret_cast<double*>(ws + 2LL * m * n + 16LL * (n + 16));
}

template <int CTI>
__global__ __launch_bounds__(256) void qrl_load_kernel(const QrArgs args) {
  using TI = typename St<CTI>::T;
  __shared__ double s_red[4];
  const QrlItem it = qrl_item(args, blockIdx.y);
  const int m = it.g->m, n = it.g->n, mode = it.g->mode;
  const TI* __restrict__ F = reinterpret_cast<const TI*>(item_ptr(it.g->f, it.g->ids, it.item));
  double2* A = qrl_ws(it);
  const long long mn = (long long)m * n;
  const long long per = (mn + QRL_CHUNKS - 1) / QRL_CHUNKS;
  const long long e0 = per * blockIdx.x, e1 = min(mn, e0 + per);
  double part = 0.0;
  for (long long idx = e0 + threadIdx.x; idx < e1; idx += 256) {
    double2 v;
    if (mode == 0) {
      v = to_d2(F[idx]);
    } else {   // A[i][j] = conj(F[j][i]), F stored n x m
      const long long i = idx / n, j = idx % n;
      v = cconj(to_d2(F[j * m + i]));
    }
    part += v.x * v.x + v.y * v.y;
    A[idx] = v;
  }
  part = block_sum(part, s_red);
  if (threadIdx.x == 0) qrl_partials(A, m, n)[blockIdx.x] = part;
}

// A[p:, c0:c0+16] -= V T^H (V^H A[p:, c0:c0+16]), in two launches over (16-column strip, QRL_CH-row chunk) tiles so the chip
// has many waves in flight: qrl_wpart writes each chunk's W = V^H A part,
// qrl_update sums the parts of its strip in chunk order (the same sum in
// every chunk of the strip), forms T^H W and updates its rows.
constexpr int QRL_CH = 256;   // rows per chunk (four waves of 64)

__device__ __forceinline__ double2* qrl_wparts(double2* ws, int m, int n) {
  return reinterpret_cast<double2*>(qrl_partials(ws, m, n) + QRL_CHUNKS);
}

// Scratch of the split panel factorisation (after the W parts): G1 and G2
// parts of up to QRT_MAXCH row chunks, a copy of Q1's top block, and the
// fallback flag (its real part).
constexpr int QRT_CH = 256;                          // rows per chunk workgroup
constexpr int QRT_MAXCH = 2048 / QRT_CH;
constexpr int QRT_SCRATCH = 2 * QRT_MAXCH * 256 + 256 + 16;
__device__ __forceinline__ double2* qrt_scratch(double2* ws, int m, int n) {
  const long long parts = (long long)((n + 15) / 16) * ((m + QRL_CH - 1) / QRL_CH) * 256;
  return qrl_wparts(ws, m, n) + parts;
}

template <int NB>
__global__ __launch_bounds__(256) void qrl_wpart_kernel(const QrArgs args, int p) {
  __shared__ double2 sW[4][256];
  const QrlItem it = qrl_item(args, blockIdx.z);
  const int m = it.g->m, n = it.g->n;
  const int c0 = p + NB + 16 * blockIdx.x;
  const int mp = m - p;
  if (p >= n || c0 >= n || (int)blockIdx.y * QRL_CH >= mp) return;
  double2* A = qrl_ws(it);
  const double2* V = A + (long long)m * n;
  const int nbk = min(NB, n - p);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int col = c0 + li;
  const bool col_ok = col < n;
  const int r0 = blockIdx.y * QRL_CH + wave * 64, r1 = min(mp, r0 + 64);
  const double2 zero = make_double2(0.0, 0.0);
  CAcc3 w;
  w.zero();
  double2 vv[16], bb[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int i = r0 + 4 * u + lk;
    const bool ok = i < r1;
    vv[u] = (ok && li < nbk) ? V[(long long)(p + i) * n + p + li] : zero;
    bb[u] = (ok && col_ok) ? A[(long long)(p + i) * n + col] : zero;
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) w.add(vv[u].x, -vv[u].y, bb[u].x, bb[u].y);
#pragma unroll
  for (int t = 0; t < 4; ++t) sW[wave][(lk + 4 * t) * 16 + li] = make_double2(w.re(t), w.im(t));
  __syncthreads();
  const int e = threadIdx.x;
  double2 sum = sW[0][e];
#pragma unroll
  for (int w = 1; w < 4; ++w) {
    sum.x += sW[w][e].x;
    sum.y += sW[w][e].y;
  }
  const int nchunk = (mp + QRL_CH - 1) / QRL_CH;
  qrl_wparts(A, m, n)[((long long)blockIdx.x * nchunk + blockIdx.y) * 256 + e] = sum;
}

// The strip-0 workgroups, which update the next panel's columns, also leave that panel's G1 part of their rows (those
// below the next panel's first row) in the split panel's scratch.
template <int NB>
__global__ __launch_bounds__(256) void qrl_update_kernel(const QrArgs args, int p) {
  __shared__ double2 sW[256];
  __shared__ double2 sG[4 * 256];
  const QrlItem it = qrl_item(args, blockIdx.z);
  const int m = it.g->m, n = it.g->n;
  const int c0 = p + NB + 16 * blockIdx.x;
  const int mp = m - p;
  if (p >= n || c0 >= n || (int)blockIdx.y * QRL_CH >= mp) return;
  double2* A = qrl_ws(it);
  const double2* V = A + (long long)m * n;
  const double2* T = V + (long long)m * n + (long long)(p / NB) * NB * NB;
  const int nbk = min(NB, n - p);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int li = lane & 15, lk = lane >> 4;
  const int col = c0 + li;
  const bool col_ok = col < n;
  const double2 zero = make_double2(0.0, 0.0);
  {
    const int nchunk = (mp + QRL_CH - 1) / QRL_CH;
    const double2* parts = qrl_wparts(A, m, n) + (long long)blockIdx.x * nchunk * 256;
    const int e = threadIdx.x;
    double2 sum = parts[e];
    for (int c = 1; c < nchunk; ++c) {
      sum.x += parts[c * 256 + e].x;
      sum.y += parts[c * 256 + e].y;
    }
    sW[e] = sum;
  }
  __syncthreads();
  v4d_t wr, wi;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double2 w = sW[(lk + 4 * t) * 16 + li];
    wr[t] = w.x;
    wi[t] = w.y;
  }
  // W2 = T^H W (result item t = row lk + 4t = the B operand of k-step t)
  CAcc3 x2;
  x2.zero();
#pragma unroll
  for (int t = 0; t < NB / 4; ++t) {
    const int s = 4 * t + lk;
    double2 x = zero;
    if (li < nbk && s < nbk) x = cconj(T[s * NB + li]);
    x2.add(x.x, x.y, wr[t], wi[t]);
  }
  double xr[4], xi[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    xr[t] = x2.re(t);
    xi[t] = x2.im(t);
  }
  // this wave's 64 rows: A -= V W2, four 16-row blocks
  const int r0 = blockIdx.y * QRL_CH + wave * 64, r1 = min(mp, r0 + 64);
  double2 av[4][4];
  double2 vv[4][NB / 4];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int rb = r0 + 16 * h;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = rb + lk + 4 * t;
      av[h][t] = (i < r1 && col_ok) ? A[(long long)(p + i) * n + col] : zero;
    }
#pragma unroll
    for (int t = 0; t < NB / 4; ++t) {
      const int i = rb + li, sref = 4 * t + lk;
      vv[h][t] = (i < r1 && sref < nbk) ? V[(long long)(p + i) * n + p + sref] : zero;
    }
  }
  const bool gram = blockIdx.x == 0;   // uniform
  CAcc3 g;
  g.zero();
  bool z = false;
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    CAcc3 e;   // V W2 for this block
    e.zero();
#pragma unroll
    for (int t = 0; t < NB / 4; ++t) e.add(vv[h][t].x, vv[h][t].y, xr[t], xi[t]);
    double2 nv[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = r0 + 16 * h + lk + 4 * t;
      nv[t] = make_double2(av[h][t].x - e.re(t), av[h][t].y - e.im(t));
      if (col_ok && i < r1) A[(long long)(p + i) * n + col] = nv[t];
    }
    if (gram) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = r0 + 16 * h + lk + 4 * t;
        const bool in = col_ok && i >= NB && i < r1;
        const double2 a = in ? nv[t] : zero;
        z = z || (in && a.x == 0.0 && a.y == 0.0);
        g.add(a.x, -a.y, a.x, a.y);
      }
    }
  }
  if (gram) {
    const bool anyz = __ballot(z) != 0ull;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sG[wave * 256 + (lk + 4 * r) * 16 + li] =
          make_double2(g.re(r), lane == 0 && r == 0 ? (anyz ? 1.0 : 0.0) : g.im(r));
    __syncthreads();
    const int e = threadIdx.x;
    double2 sum = sG[e];
#pragma unroll
    for (int w = 1; w < 4; ++w) sum = make_double2(sum.x + sG[w * 256 + e].x, sum.y + sG[w * 256 + e].y);
    qrt_scratch(A, m, n)[blockIdx.y * 256 + e] = sum;
  }
}

// Q formation, four panels (64 columns of V) at a time: the working matrix is
// read and written once per four panels instead of once per panel, which is
// what bounds it (2048 x 1024, the last step's 33 MB each way: 124 us for four
// panels one by one, 49 now; a round at bond 1024: 11 ms of these kernels
// before, 5.1 now with qrq_merge).  A superpanel is as many panels as the W
// parts of one row chunk fit into the workspace of the single panels' parts:
// three for matrices of at most 768 rows.  Matrices of at most 64 columns are
// taken panel by panel: with one superpanel little is saved on the working
// matrix, and its T is not worth joining (64 matrices of up to 2048 x 32, a
// tree network's pass: 4.8 ms joined, 2.3 panel by panel).
struct QrqShape {
  int np, nch;   // panels of a superpanel, row chunks of its W (np nch <= 256-row chunks)
};
__host__ __device__ __forceinline__ QrqShape qrq_shape(int m, int n) {
  const int c = (m + QRL_CH - 1) / QRL_CH;
  QrqShape q;
  q.np = n <= 4 * QB ? 1 : c < 4 ? c : 4;
  q.nch = c / (q.np == 1 ? 2 : 4);
  if (q.nch < 1) q.nch = 1;
  return q;
}

// V[row][col] of the m x n area behind w, zero where not ok
__device__ __forceinline__ double2 qrq_v(__amdgpu_buffer_rsrc_t w, int n, int row, int col, bool ok) {
  double2 v[1];
  tl_run<double2, 1>(v, w, (unsigned)(row * n + col) * 16u, ok ? 1 : 0, false);
  return v[0];
}

// Block (i, j), i <= j, of the superpanel's T, element (r, c): the diagonal
// blocks are the panels' own, the others lie in V above their panel's top,
// which holds no part of V (readers of V take it as zero).
__device__ __forceinline__ double2 qrq_t(const double2* V, const double2* Tg, int n, int P, int i,
                                         int j, int r, int c) {
  if (P + 16 * i + r >= n || P + 16 * j + c >= n) return make_double2(0.0, 0.0);
  return i == j ? Tg[(long long)(P / QB + i) * QB * QB + r * QB + c]
                : V[(long long)(P + 16 * i + r) * n + P + 16 * j + c];
}

// One 512-thread workgroup per superpanel: G_ij = V_i^H V_j over the rows
// below, then column block by column block T_ij = -sum_l T_il G_lj T_jj.
__global__ __launch_bounds__(512, 1) void qrq_merge_kernel(const QrArgs args) {
  __shared__ __attribute__((aligned(16))) double2 sP[8 * 256];   // the waves' parts, then G_lj T_jj
  __shared__ __attribute__((aligned(16))) double2 sG[6 * 256];   // G_ij, then T_ij, at j (j - 1) / 2 + i
  const QrlItem it = qrl_item(args, blockIdx.y);
  const int m = it.g->m, n = it.g->n;
  const QrqShape q = qrq_shape(m, n);
  const int P = 16 * q.np * blockIdx.x;
  const int nb = min(q.np, (n - P + 15) / 16);
  if (nb < 2) return;   // uniform over the workgroup
  double2* A = qrl_ws(it);
  double2* V = A + (long long)m * n;
  const double2* Tg = V + (long long)m * n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const __amdgpu_buffer_rsrc_t rV = tl_rsrc(V, (long long)m * n * 16);
  CAcc3 g[6];
#pragma unroll
  for (int e = 0; e < 6; ++e) g[e].zero();
  for (int rb = P + 16 + 16 * wave; rb < m; rb += 128) {
    double2 v[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = rb + 4 * t + lk, col = P + 16 * i + li;
        v[i][t] = qrq_v(rV, n, row, col, i < nb && rb >= P + 16 * i && row < m && col < n);
      }
    static_for<4>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      static_for<j>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int t = 0; t < 4; ++t)
          g[j * (j - 1) / 2 + i].add(v[i][t].x, -v[i][t].y, v[j][t].x, v[j][t].y);
      });
    });
  }
#pragma unroll
  for (int e = 0; e < 6; ++e) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sP[wave * 256 + (lk + 4 * r) * 16 + li] = make_double2(g[e].re(r), g[e].im(r));
    __syncthreads();
    if (tid < 256) {
      double2 s = sP[tid];
#pragma unroll
      for (int w = 1; w < 8; ++w) s = make_double2(s.x + sP[w * 256 + tid].x, s.y + sP[w * 256 + tid].y);
      sG[e * 256 + tid] = s;
    }
    __syncthreads();
  }
  for (int j = 1; j < nb; ++j) {
    if (wave < j) {   // X_l = G_lj T_jj, l = wave
      CAcc3 x;
      x.zero();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double2 a = sG[(j * (j - 1) / 2 + wave) * 256 + li * 16 + 4 * s + lk];
        const double2 b = qrq_t(V, Tg, n, P, j, j, 4 * s + lk, li);
        x.add(a.x, a.y, b.x, b.y);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        sP[wave * 256 + (lk + 4 * r) * 16 + li] = make_double2(x.re(r), x.im(r));
    }
    __syncthreads();
    if (wave < j) {   // T_ij, i = wave
      CAcc3 x;
      x.zero();
      for (int l = wave; l < j; ++l) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double2 a = l == wave ? qrq_t(V, Tg, n, P, l, l, li, 4 * s + lk)
                                      : sG[(l * (l - 1) / 2 + wave) * 256 + li * 16 + 4 * s + lk];
          const double2 b = sP[l * 256 + (4 * s + lk) * 16 + li];
          x.add(a.x, a.y, b.x, b.y);
        }
      }
      const int col = P + 16 * j + li;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 t = make_double2(-x.re(r), -x.im(r));
        sG[(j * (j - 1) / 2 + wave) * 256 + (lk + 4 * r) * 16 + li] = t;
        if (col < n) V[(long long)(P + 16 * wave + lk + 4 * r) * n + col] = t;
      }
    }
    __syncthreads();
  }
}

// W = V_b^H A[P:, c0:c0+16] for panel b of the superpanel over one row chunk,
// one 512-thread workgroup per (strip, chunk and panel).
__global__ __launch_bounds__(512, 1) void qrq_wpart_kernel(const QrArgs args, int step) {
  __shared__ __attribute__((aligned(16))) double2 sW[8 * 256];
  const QrlItem it = qrl_item(args, blockIdx.z);
  const int m = it.g->m, n = it.g->n;
  const QrqShape q = qrq_shape(m, n);
  const int P = 16 * q.np * step, mp = m - P;
  const int c0 = P + 16 * blockIdx.x, b = blockIdx.y % q.np, chunk = blockIdx.y / q.np;
  if (c0 >= n || P + 16 * b >= n || chunk >= q.nch) return;   // uniform
  double2* A = qrl_ws(it);
  const double2* V = A + (long long)m * n;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int col = c0 + li, vcol = P + 16 * b + li;
  const int rows = ((mp + q.nch - 1) / q.nch + 63) / 64 * 64;   // of a chunk
  const int end = min(mp, (chunk + 1) * rows);
  const double2 zero = make_double2(0.0, 0.0);
  CAcc3 w;
  w.zero();
  for (int r0 = chunk * rows + 64 * wave; r0 < end; r0 += 512) {
    double2 vv[16], bb[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int i = r0 + 4 * u + lk;
      vv[u] = (i < end && r0 + 4 * u >= 16 * b && vcol < n) ? V[(long long)(P + i) * n + vcol] : zero;
      bb[u] = (i < end && col < n) ? A[(long long)(P + i) * n + col] : zero;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) w.add(vv[u].x, -vv[u].y, bb[u].x, bb[u].y);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) sW[wave * 256 + (lk + 4 * t) * 16 + li] = make_double2(w.re(t), w.im(t));
  __syncthreads();
  if (tid < 256) {
    double2 sum = sW[tid];
#pragma unroll
    for (int u = 1; u < 8; ++u) sum = make_double2(sum.x + sW[u * 256 + tid].x, sum.y + sW[u * 256 + tid].y);
    qrl_wparts(A, m, n)[((long long)(blockIdx.x * q.nch + chunk) * q.np + b) * 256 + tid] = sum;
  }
}

// A[P:, c0:c0+16] -= V T W, one 256-thread workgroup per (strip, 256 rows):
// the parts of W summed in chunk order, wave i forms rows 16 i .. of T W, and
// every wave updates 64 rows.  NP: panels of the launch's superpanels, at most.
template <int NP>
__global__ __launch_bounds__(256) void qrq_update_kernel(const QrArgs args, int step) {
  __shared__ __attribute__((aligned(16))) double2 sW[NP * 256];
  __shared__ __attribute__((aligned(16))) double2 sX[NP * 256];
  const QrlItem it = qrl_item(args, blockIdx.z);
  const int m = it.g->m, n = it.g->n;
  const QrqShape q = qrq_shape(m, n);
  const int P = 16 * q.np * step, mp = m - P;
  const int c0 = P + 16 * blockIdx.x;
  if (c0 >= n || (int)blockIdx.y * QRL_CH >= mp) return;   // uniform
  double2* A = qrl_ws(it);
  const double2* V = A + (long long)m * n;
  const double2* Tg = V + (long long)m * n;
  const int nb = min(q.np, (n - P + 15) / 16);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int col = c0 + li;
  const bool col_ok = col < n;
  const double2 zero = make_double2(0.0, 0.0);
  const int r0 = blockIdx.y * QRL_CH + wave * 64, r1 = min(mp, r0 + 64);
  const __amdgpu_buffer_rsrc_t rV = tl_rsrc(V, (long long)m * n * 16);
  const __amdgpu_buffer_rsrc_t rA = tl_rsrc(A, (long long)m * n * 16);
  double2 av[4][4], vv[4 * NP];
#pragma unroll
  for (int h = 0; h < 4; ++h)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = r0 + 16 * h + lk + 4 * t;
      av[h][t] = qrq_v(rA, n, P + i, col, i < r1 && col_ok);
    }
  auto load_v = [&](int rb) {   // V's rows rb .. rb + 15, panel b in vv[4b ..]
#pragma unroll
    for (int u = 0; u < 4 * NP; ++u) {
      const int vcol = P + 4 * u + lk;
      vv[u] = qrq_v(rV, n, P + rb + li, vcol,
                    (u >> 2) < nb && rb >= 16 * (u >> 2) && rb + li < r1 && vcol < n);
    }
  };
  load_v(r0);
  {
    const double2* parts = qrl_wparts(A, m, n) + (long long)blockIdx.x * q.nch * q.np * 256;
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      double2 sum = zero;
      if (b < nb) {
        sum = parts[b * 256 + tid];
        for (int c = 1; c < q.nch; ++c) {
          const double2 x = parts[(c * q.np + b) * 256 + tid];
          sum = make_double2(sum.x + x.x, sum.y + x.y);
        }
      }
      sW[b * 256 + tid] = sum;
    }
  }
  __syncthreads();
  if (wave < NP) {
    CAcc3 x;
    x.zero();
    for (int j = wave; j < nb; ++j) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const double2 a = qrq_t(V, Tg, n, P, wave, j, li, 4 * s + lk);
        const double2 b = sW[j * 256 + (4 * s + lk) * 16 + li];
        x.add(a.x, a.y, b.x, b.y);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) sX[wave * 256 + (lk + 4 * r) * 16 + li] = make_double2(x.re(r), x.im(r));
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    const int rb = r0 + 16 * h;
    if (rb >= r1) break;   // uniform over the wave
    CAcc3 e;
    e.zero();
#pragma unroll
    for (int u = 0; u < 4 * NP; ++u) {
      const double2 x = sX[(u >> 2) * 256 + (lk + 4 * (u & 3)) * 16 + li];   // (zero past the last panel)
      e.add(vv[u].x, vv[u].y, x.x, x.y);
    }
    if (h < 3) load_v(rb + 16);
    if (col_ok) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int i = rb + lk + 4 * t;
        if (i < r1)
          A[(long long)(P + i) * n + col] = make_double2(av[h][t].x - e.re(t), av[h][t].y - e.im(t));
      }
    }
  }
}

__global__ __launch_bounds__(256) void qrl_fill_kernel(const QrArgs args) {
  const QrlItem it = qrl_item(args, blockIdx.y);
  const int m = it.g->m, n = it.g->n;
  double2* A = qrl_ws(it);
  const long long mn = (long long)m * n;
  const long long per = (mn + QRL_CHUNKS - 1) / QRL_CHUNKS;
  const long long e0 = per * blockIdx.x, e1 = min(mn, e0 + per);
  for (long long idx = e0 + threadIdx.x; idx < e1; idx += 256)
    A[idx] = make_double2((idx / n == idx % n) ? 1.0 : 0.0, 0.0);
}

template <int CTO>
__global__ __launch_bounds__(256) void qrl_store_kernel(const QrArgs args) {
  using TO = typename St<CTO>::T;
  const QrlItem it = qrl_item(args, blockIdx.y);
  const int m = it.g->m, n = it.g->n, mode = it.g->mode;
  const double2* A = qrl_ws(it);
  TO* Q = reinterpret_cast<TO*>(const_cast<char*>(item_ptr(it.g->q, it.g->ids, it.item)));
  const long long mn = (long long)m * n;
  const long long per = (mn + QRL_CHUNKS - 1) / QRL_CHUNKS;
  const long long e0 = per * blockIdx.x, e1 = min(mn, e0 + per);
  for (long long idx = e0 + threadIdx.x; idx < e1; idx += 256) {
    double2 v;
    if (mode == 0) {
      v = A[idx];
    } else {   // Q^H: out[j][i] = conj(A[i][j]), out stored n x m
      const long long j = idx / m, i = idx % m;
      v = cconj(A[i * n + j]);
    }
    TO o;
    o.x = v.x;
    o.y = v.y;
    Q[idx] = o;
  }
}


// Spread path for small batches of matrices of at most 512 rows: the panels
// are factored by one 512-thread workgroup per matrix (Cholesky QR and
// Householder reconstruction where the panel allows it, else column by
// column), the trailing updates run over 16-column strips with one workgroup
// per strip and matrix, and Q is formed by the blocked kernel's Q-block
// launch from the explicit V and T in the workspace.  The workspace is the
// large path's.
constexpr int QRS_NW = 8, QRS_MAXB = 4;   // 512 threads, rows in 16-row blocks
constexpr size_t QRS_LDS = (size_t)512 * QB * sizeof(double2) + (size_t)QRS_NW * 256 * sizeof(double2);

// The panel at column p of one matrix, by the whole 512-thread workgroup; P
// (512 x 16 panel rows) and Wp (8 areas of 256) in LDS.  a: the panel's
// columns, block beta = wave + 8 b of 16 rows in a[b], row 16 beta + 4t + lk,
// column p + li (zero past row m and column n; blocks above row p not read).
__device__ __forceinline__ void spread_panel(const QrlItem& it, int p, double2 (&a)[QRS_MAXB][4],
                                             double2* P, double2* Wp) {
  PanelSmem2<QRS_NW, QB>& psm = *reinterpret_cast<PanelSmem2<QRS_NW, QB>*>(P);
  const int m = it.g->m, n = it.g->n;
  double2* V = qrl_ws(it) + (long long)m * n;
  double2* Tg = V + (long long)m * n;
  const int mp = m - p, nbk = min(QB, n - p), k = p / QB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  bool chol = false;
  if (mp > nbk) {
    chol = panel_cholqr<QRS_NW, QRS_MAXB>(a, m, k, mp, nbk, P, Wp);
  } else {
#pragma unroll
    for (int b = 0; b < QRS_MAXB; ++b) {
      const int beta = wave + QRS_NW * b;
      if (beta >= k && 16 * beta < m) {
#pragma unroll
        for (int t = 0; t < 4; ++t) P[pidx(16 * (beta - k) + 4 * t + lk, li)] = a[b][t];
      }
    }
    __syncthreads();
  }
  if (!chol) {
    double2 ar[1][QB];
#pragma unroll
    for (int c = 0; c < QB; ++c) ar[0][c] = tid < mp ? P[pidx(tid, c)] : zero;
    factor_panel2<1, QB, 512>(ar, mp, nbk, psm, Wp);
#pragma unroll
    for (int c = 0; c < QB; ++c) {
      const bool in = tid < mp && c < nbk;
      P[pidx(tid, c)] = !in ? zero : (tid > c ? ar[0][c] : make_double2(tid == c ? 1.0 : 0.0, 0.0));
    }
  }
  __syncthreads();
  if (tid < mp) {
#pragma unroll
    for (int c = 0; c < QB; ++c)
      if (c < nbk) V[(long long)(p + tid) * n + p + c] = P[pidx(tid, c)];
  }
  if (tid < QB * QB) Tg[(long long)k * QB * QB + tid] = Wp[tid];
}

// The first panel, and |F|^2.
__global__ __launch_bounds__(512, 1) void qrs_panel_kernel(const QrArgs args) {
  extern __shared__ __attribute__((aligned(16))) double2 qrs_dyn[];
  const QrlItem it = qrl_item(args, blockIdx.x);
  const int m = it.g->m, n = it.g->n, tid = threadIdx.x;
  double2* A = qrl_ws(it);
  if (tid == 0) {   // |F|^2 from the chunk partials, in a fixed order
    const double* part = qrl_partials(A, m, n);
    double s = 0.0;
    for (int c = 0; c < QRL_CHUNKS; ++c) s += part[c];
    *reinterpret_cast<double*>(const_cast<char*>(item_ptr(it.g->nrm2, it.g->ids, it.item))) = s;
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int li = lane & 15, lk = lane >> 4;
  double2 a[QRS_MAXB][4];
#pragma unroll
  for (int b = 0; b < QRS_MAXB; ++b)
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = 16 * (wave + QRS_NW * b) + 4 * t + lk;
      a[b][t] = (row < m && li < n) ? A[(long long)row * n + li] : make_double2(0.0, 0.0);
    }
  spread_panel(it, 0, a, qrs_dyn, qrs_dyn + 512 * QB);
}

// Trailing update of the spread path, one 512-thread workgroup per (16-column
// strip, matrix): A[p:, c0:c0+16] -= V T^H (V^H A[p:, c0:c0+16]).  The waves
// take the 16-row blocks from row p on in turn, in the panel's register
// layout; their parts of W = V^H A are summed through LDS in a fixed order,
// and V is kept in LDS for the second product.
// The workgroup of strip 0, whose columns are the next panel's, then factors
// that panel from its registers (look-ahead): its latency overlaps the other
// strips' updates, and the next update launch finds V and T in place.  These
// workgroups take longest, so the matrices' first strips come first in the
// grid.  A launch is bounded by this chain: the update's loads and two
// reductions, then the panel's two one-wave recurrences.  Mean over the
// launches of a round of 48 states at bonds up to 256 (512 rows): 51.0 us with the next
// panel read back from memory, V read twice and the matrices' strips in
// order, 44.7 now.
__global__ __launch_bounds__(512, 1) void qrs_update_kernel(const QrArgs args, int p) {
  extern __shared__ __attribute__((aligned(16))) double2 qrs_dyn[];
  double2* sV = qrs_dyn;
  double2 (*sW)[256] = reinterpret_cast<double2 (*)[256]>(qrs_dyn + 512 * QB);
  const QrlItem it = qrl_item(args, blockIdx.x);
  const int strip = blockIdx.y;
  const int m = it.g->m, n = it.g->n;
  const int c0 = p + QB + 16 * strip;
  if (p >= n || c0 >= n) return;   // uniform over the workgroup
  double2* A = qrl_ws(it);
  const double2* V = A + (long long)m * n;
  const int k0 = p / QB;
  const double2* T = V + (long long)m * n + (long long)k0 * QB * QB;
  const int nbk = min(QB, n - p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lk = lane >> 4;
  const int col = c0 + li;
  const bool col_ok = col < n;
  const double2 zero = make_double2(0.0, 0.0);
  // this wave's rows of the strip (block beta = wave + 8 h, row 16 beta + 4t +
  // lk) and its part of W.  V's block beta goes to place beta - k0 - 1 (mod
  // 32) of the LDS rows: the next panel puts the same wave's rows there.
  double2 av[QRS_MAXB][4], tt[4];
  CAcc3 w;
  w.zero();
#pragma unroll
  for (int h = 0; h < QRS_MAXB; ++h) {
    const int beta = wave + QRS_NW * h;
    const bool on = beta >= k0 && 16 * beta < m;   // uniform over the wave
    double2 vw[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = 16 * beta + 4 * t + lk;
      av[h][t] = (on && row < m && col_ok) ? A[(long long)row * n + col] : zero;
      vw[t] = (on && row < m && li < nbk) ? V[(long long)row * n + p + li] : zero;
    }
    if (on) {
      const int b0 = 16 * ((beta - k0 - 1) & 31);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        sV[pidx(b0 + 4 * t + lk, li)] = vw[t];
        w.add(vw[t].x, -vw[t].y, av[h][t].x, av[h][t].y);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
    tt[t] = (li < nbk && 4 * t + lk < nbk) ? T[(4 * t + lk) * QB + li] : zero;
#pragma unroll
  for (int r = 0; r < 4; ++r) sW[wave][(lk + 4 * r) * 16 + li] = make_double2(w.re(r), w.im(r));
  __syncthreads();
  if (tid < 256) {
    double2 sum = sW[0][tid];
#pragma unroll
    for (int u = 1; u < QRS_NW; ++u) {
      sum.x += sW[u][tid].x;
      sum.y += sW[u][tid].y;
    }
    sW[0][tid] = sum;
  }
  __syncthreads();
  // W2 = T^H W (item t = row lk + 4t = the B operand of k-step t)
  CAcc3 x2;
  x2.zero();
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double2 x = sW[0][(lk + 4 * t) * 16 + li];
    x2.add(tt[t].x, -tt[t].y, x.x, x.y);
  }
  double x2r[4], x2i[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    x2r[t] = x2.re(t);
    x2i[t] = x2.im(t);
  }
  // A -= V W2, block by block
#pragma unroll
  for (int h = 0; h < QRS_MAXB; ++h) {
    const int beta = wave + QRS_NW * h;
    if (beta >= k0 && 16 * beta < m) {
      const int b0 = 16 * ((beta - k0 - 1) & 31);
      CAcc3 e;
      e.zero();
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double2 v = sV[pidx(b0 + li, 4 * t + lk)];
        e.add(v.x, v.y, x2r[t], x2i[t]);
      }
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        av[h][t] = make_double2(av[h][t].x - e.re(t), av[h][t].y - e.im(t));
        const int row = 16 * beta + 4 * t + lk;
        if (strip > 0 && col_ok && row < m) A[(long long)row * n + col] = av[h][t];
      }
    }
  }
  // the next panel: its columns stay in registers (nothing else reads them)
  if (strip == 0) {
    __syncthreads();   // W is read everywhere before its place is reused
    spread_panel(it, c0, av, qrs_dyn, qrs_dyn + 512 * QB);
  }
}

// Column-by-column factorisation of the panel rows of A (m <= 2048 rows, RP
// rows per thread of a 512-thread workgroup), for panels the Cholesky QR does
// not take: writes V (unit diagonal) and T.  sP (16 QB values) and sWp
// (8 x 256) are its LDS scratch.  The panel is held in registers, 4 RP NB of a
// thread's 256, so the sizes at hand choose RP and NB: 2048 x 16 spills, and
// with every panel in that form 64 matrices of 2048 x 8 took 380 us, 150 now.
template <int RP, int NB>
__device__ __noinline__ void tall_columns(const double2* A, double2* V, double2* Tg, int p, int n,
                                          int mp, int nbk, int k, double2* sP, double2* sWp) {
  static_assert(sizeof(PanelSmem2<QRS_NW, NB>) <= 16 * QB * sizeof(double2), "fallback scratch fits");
  PanelSmem2<QRS_NW, NB>& psm = *reinterpret_cast<PanelSmem2<QRS_NW, NB>*>(sP);
  const int tid = threadIdx.x;
  const double2 zero = make_double2(0.0, 0.0);
  double2 a[RP][NB];
#pragma unroll
  for (int r = 0; r < RP; ++r) {
    const int i = tid + r * 512;
#pragma unroll
    for (int c = 0; c < NB; ++c)
      a[r][c] = (i < mp && c < nbk) ? A[(long long)(p + i) * n + p + c] : zero;
  }
  factor_panel2<RP, NB, 512>(a, mp, nbk, psm, sWp);
#pragma unroll
  for (int r = 0; r < RP; ++r) {
    const int i = tid + r * 512;
    if (i < mp) {
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        if (c < nbk) {
          const double2 v = (i < c) ? zero : (i == c ? make_double2(1.0, 0.0) : a[r][c]);
          V[(long long)(p + i) * n + p + c] = v;
        }
      }
    }
  }
  if (tid < QB * QB) {
    const int r = tid / QB, c = tid % QB;
    Tg[(long long)k * QB * QB + tid] = r < NB && c < NB ? sWp[r * NB + c] : zero;
  }
}

__device__ __forceinline__ void tall_fallback(const double2* A, double2* V, double2* Tg, int p, int n,
                                              int mp, int nbk, int k, double2* sP, double2* sWp) {
  if (nbk <= 8)
    tall_columns<4, 8>(A, V, Tg, p, n, mp, nbk, k, sP, sWp);
  else if (mp <= 1024)
    tall_columns<2, QB>(A, V, Tg, p, n, mp, nbk, k, sP, sWp);
  else
    tall_columns<4, QB>(A, V, Tg, p, n, mp, nbk, k, sP, sWp);
}

// Panel factorisation for 512 < m <= 2048 rows: Cholesky QR twice and
// Householder reconstruction (qr_cholpanel.h) with the row work of each
// 16-column panel spread over one 512-thread workgroup per 256-row chunk
// (block c of the chunk to wave c mod 8):
//   G1 parts   one per row chunk (exact-zero flag in Im G[0][0]): for the
//              first panel from qrt_gram, for the others from the strip-0
//              workgroups of the previous panel's update, which have just
//              written those columns
//   qrt_q1     every workgroup sums the parts in chunk order and forms
//              R1^{-1} (identical in all of them); Q1 = A R1^{-1} into the V
//              area, its top block also to the scratch, G2 parts
//   qrt_v      every workgroup sums the G2 parts and runs the
//              reconstruction on the top block (identical in all of them);
//              V = Q1 M in place, V's top block and T from chunk 0
// A panel the Cholesky QR does not take (an exact zero, a small pivot, a
// squared norm out of range, no rows below the diagonal block) is factored
// column by column by the chunk-0 workgroup of qrt_v (tall_fallback); qrt_q1
// passes its decision on through the flag in the scratch.
struct QrtCtx {
  double2 *A, *V, *Tg, *sc;
  int m, n, mp, nbk, k, nblk, nch;
  bool live;   // this workgroup's chunk holds rows of the panel
};

__device__ __forceinline__ QrtCtx qrt_ctx(const QrArgs& args, int p) {
  const QrlItem it = qrl_item(args, blockIdx.y);
  QrtCtx c;
  c.m = it.g->m;
  c.n = it.g->n;
  c.A = qrl_ws(it);
  c.V = c.A + (long long)c.m * c.n;
  c.Tg = c.V + (long long)c.m * c.n;
  c.sc = qrt_scratch(c.A, c.m, c.n);
  c.mp = c.m - p;
  c.nbk = min(QB, c.n - p);
  c.k = p / QB;
  c.nblk = (c.mp + 15) / 16;
  c.nch = (c.mp + QRT_CH - 1) / QRT_CH;
  c.live = p < c.n && (int)blockIdx.x < c.nch;
  return c;
}

// Sums the waves' 16 x 16 parts in sWp (8 x 256) into part 0 of sWp, then
// writes it to dst (256 values).
__device__ __forceinline__ void qrt_reduce_store(double2* sWp, double2* dst, int tid) {
  __syncthreads();
  if (tid < 256) {
    double2 s = sWp[tid];
#pragma unroll
    for (int w = 1; w < 8; ++w) s = make_double2(s.x + sWp[w * 256 + tid].x, s.y + sWp[w * 256 + tid].y);
    dst[tid] = s;
  }
}

// Loads the chunk parts src[0 .. nch) into sWp as eight parts (zeros beyond
// nch).
__device__ __forceinline__ void qrt_load_parts(double2* sWp, const double2* src, int nch, int tid) {
  for (int e = tid; e < 8 * 256; e += 512)
    sWp[e] = (e >> 8) < nch ? src[e] : make_double2(0.0, 0.0);
}

__global__ __launch_bounds__(512, 1) void qrt_gram_kernel(const QrArgs args, int p) {
  __shared__ __attribute__((aligned(16))) double2 sWp[8 * 256];
  const QrtCtx c = qrt_ctx(args, p);
  if (!c.live) return;
  if (p == 0 && blockIdx.x == 0 && threadIdx.x == 0) {   // |F|^2 from the load's chunk sums
    const QrlItem it = qrl_item(args, blockIdx.y);
    const double* part = qrl_partials(c.A, c.m, c.n);
    double s = 0.0;
    for (int q = 0; q < QRL_CHUNKS; ++q) s += part[q];
    *reinterpret_cast<double*>(const_cast<char*>(item_ptr(it.g->nrm2, it.g->ids, it.item))) = s;
  }
  if (c.mp <= c.nbk) return;   // column by column
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  const int b0 = blockIdx.x * (QRT_CH / 16), b1 = min(c.nblk, b0 + QRT_CH / 16);
  CAcc3 g;
  g.zero();
  bool z = false;
  for (int b = b0 + wave; b < b1; b += 8) {
    double2 a4[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int i = 16 * b + 4 * t + lk;
      const bool in = i < c.mp && li < c.nbk;
      a4[t] = in ? c.A[(long long)(p + i) * c.n + p + li] : zero;
      z = z || (in && a4[t].x == 0.0 && a4[t].y == 0.0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) g.add(a4[t].x, -a4[t].y, a4[t].x, a4[t].y);
  }
  const bool anyz = __ballot(z) != 0ull;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    sWp[wave * 256 + (lk + 4 * r) * 16 + li] =
        make_double2(g.re(r), lane == 0 && r == 0 ? (anyz ? 1.0 : 0.0) : g.im(r));
  qrt_reduce_store(sWp, c.sc + blockIdx.x * 256, tid);
}

__global__ __launch_bounds__(512, 1) void qrt_q1_kernel(const QrArgs args, int p) {
  __shared__ __attribute__((aligned(16))) double2 sWp[8 * 256];
  const QrtCtx c = qrt_ctx(args, p);
  if (!c.live) return;
  double2* flag = c.sc + QRT_SCRATCH - 16;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  if (c.mp <= c.nbk) {   // no rows below the diagonal block: column by column
    if (blockIdx.x == 0 && tid == 0) *flag = make_double2(1.0, 0.0);
    return;
  }
  // G1 parts: one per chunk of qrt_gram (first panel) or of the previous
  // panel's update (its rows start 16 above)
  const int nparts = p == 0 ? c.nch : (c.mp + QB + QRL_CH - 1) / QRL_CH;
  qrt_load_parts(sWp, c.sc, nparts, tid);
  __syncthreads();
  if (wave == 0) panel_first_pass<8>(sWp, c.nbk);
  __syncthreads();
  const bool ok = sWp[16].x == 0.0;
  if (blockIdx.x == 0 && tid == 0) *flag = make_double2(ok ? 0.0 : 1.0, 0.0);
  if (!ok) return;
  double2 xb[4];   // X1[lk + 4s][li], the B operand of k-step s
#pragma unroll
  for (int s = 0; s < 4; ++s) xb[s] = sWp[(lk + 4 * s) * 16 + li];
  __syncthreads();   // X1 read everywhere before the parts are rewritten
  const int b0 = blockIdx.x * (QRT_CH / 16), b1 = min(c.nblk, b0 + QRT_CH / 16);
  double2* qtop = c.sc + 2 * QRT_MAXCH * 256;
  CAcc3 g2;
  g2.zero();
  for (int b = b0 + wave; b < b1; b += 8) {
    CAcc3 q;
    q.zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int i = 16 * b + li, col = 4 * s + lk;
      const double2 av = (i < c.mp && col < c.nbk) ? c.A[(long long)(p + i) * c.n + p + col] : zero;
      q.add(av.x, av.y, xb[s].x, xb[s].y);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * b + lk + 4 * r;
      const double2 qv = make_double2(q.re(r), q.im(r));
      if (i < c.mp && li < c.nbk) c.V[(long long)(p + i) * c.n + p + li] = qv;
      if (b == 0) qtop[pidx(lk + 4 * r, li)] = qv;
      g2.add(qv.x, -qv.y, qv.x, qv.y);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
    sWp[wave * 256 + (lk + 4 * r) * 16 + li] = make_double2(g2.re(r), g2.im(r));
  qrt_reduce_store(sWp, c.sc + (QRT_MAXCH + blockIdx.x) * 256, tid);
}

__global__ __launch_bounds__(512, 1) void qrt_v_kernel(const QrArgs args, int p) {
  __shared__ __attribute__((aligned(16))) double2 sP[16 * QB];
  __shared__ __attribute__((aligned(16))) double2 sWp[8 * 256];
  const QrtCtx c = qrt_ctx(args, p);
  if (!c.live) return;
  const double2* flag = c.sc + QRT_SCRATCH - 16;
  if (flag->x != 0.0) {   // the first pass did not take the panel
    if (blockIdx.x == 0) tall_fallback(c.A, c.V, c.Tg, p, c.n, c.mp, c.nbk, c.k, sP, sWp);
    return;
  }
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const double2 zero = make_double2(0.0, 0.0);
  qrt_load_parts(sWp, c.sc + QRT_MAXCH * 256, c.nch, tid);
  const double2* qtop = c.sc + 2 * QRT_MAXCH * 256;
  if (tid < 256) sP[tid] = qtop[tid];
  __syncthreads();
  if (wave == 0) panel_second_pass<8>(sP, sWp, c.nbk, c.mp);
  __syncthreads();
  if (sWp[16].x != 0.0) {   // identical in every workgroup
    if (blockIdx.x == 0) {
      __syncthreads();   // the flag read everywhere before the LDS is reused
      tall_fallback(c.A, c.V, c.Tg, p, c.n, c.mp, c.nbk, c.k, sP, sWp);
    }
    return;
  }
  double2 mb[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) mb[s] = sWp[256 + (lk + 4 * s) * 16 + li];
  const int b0 = blockIdx.x * (QRT_CH / 16), b1 = min(c.nblk, b0 + QRT_CH / 16);
  for (int b = b0 + wave; b < b1; b += 8) {
    if (b == 0) continue;
    CAcc3 y;
    y.zero();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int i = 16 * b + li, col = 4 * s + lk;
      const double2 av = (i < c.mp && col < c.nbk) ? c.V[(long long)(p + i) * c.n + p + col] : zero;
      y.add(av.x, av.y, mb[s].x, mb[s].y);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * b + lk + 4 * r;
      if (i < c.mp && li < c.nbk) c.V[(long long)(p + i) * c.n + p + li] = make_double2(y.re(r), y.im(r));
    }
  }
  if (blockIdx.x == 0) {
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = lk + 4 * r;
        if (i < c.mp && li < c.nbk) c.V[(long long)(p + i) * c.n + p + li] = sP[pidx(i, li)];
      }
    }
    if (tid < QB * QB) c.Tg[(long long)c.k * QB * QB + tid] = sWp[tid];
  }
}

template <int CTI, int CTO>
hipError_t run_tall(QrArgs args, int items, int m_max, int n_max, hipStream_t s) {
  const dim3 chunks(QRL_CHUNKS, items);
  hipLaunchKernelGGL((qrl_load_kernel<CTI>), chunks, dim3(256), 0, s, args);
  const dim3 pch((m_max + QRT_CH - 1) / QRT_CH, items);
  hipLaunchKernelGGL(qrt_gram_kernel, pch, dim3(512), 0, s, args, 0);
  for (int p = 0; p < n_max; p += QB) {
    hipLaunchKernelGGL(qrt_q1_kernel, pch, dim3(512), 0, s, args, p);
    hipLaunchKernelGGL(qrt_v_kernel, pch, dim3(512), 0, s, args, p);
    const int strips = (n_max - p - QB + 15) / 16;
    if (strips > 0) {
      const dim3 grid(strips, (m_max - p + QRL_CH - 1) / QRL_CH, items);
      hipLaunchKernelGGL((qrl_wpart_kernel<QB>), grid, dim3(256), 0, s, args, p);
      hipLaunchKernelGGL((qrl_update_kernel<QB>), grid, dim3(256), 0, s, args, p);
    }
  }
  hipLaunchKernelGGL(qrl_fill_kernel, chunks, dim3(256), 0, s, args);
  // Q: superpanels in reverse, at most `steps` of `width` columns or more each
  int width = 4 * QB, steps = 0;
  int chunks_w = 1;
  bool joined = false;
  for (int g = 0; g < args.ngroups; ++g) {
    const QrqShape q = qrq_shape(args.g[g].m, args.g[g].n);
    width = min(width, q.np * QB);
    steps = max(steps, (args.g[g].n + q.np * QB - 1) / (q.np * QB));
    chunks_w = max(chunks_w, q.nch);
    joined = joined || q.np > 1;
  }
  if (joined) hipLaunchKernelGGL(qrq_merge_kernel, dim3(steps, items), dim3(512), 0, s, args);
  for (int step = steps - 1; step >= 0; --step) {
    const int p = step * width;   // no superpanel of this step starts above
    const int strips = (n_max - p + 15) / 16;
    hipLaunchKernelGGL(qrq_wpart_kernel, dim3(strips, (joined ? 4 : 1) * chunks_w, items), dim3(512), 0,
                       s, args, step);
    const dim3 grid(strips, (m_max - p + QRL_CH - 1) / QRL_CH, items);
    if (joined)
      hipLaunchKernelGGL(qrq_update_kernel<4>, grid, dim3(256), 0, s, args, step);
    else
      hipLaunchKernelGGL(qrq_update_kernel<1>, grid, dim3(256), 0, s, args, step);
  }
  hipLaunchKernelGGL((qrl_store_kernel<CTO>), chunks, dim3(256), 0, s, args);
  return hipGetLastError();
}

template <int CTI>
hipError_t run_spread(QrArgs args, int items, int m_max, int n_max, hipStream_t s) {
  static hipError_t attr1 = hipFuncSetAttribute(reinterpret_cast<const void*>(&qrs_panel_kernel),
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)QRS_LDS);
  static hipError_t attr2 = hipFuncSetAttribute(reinterpret_cast<const void*>(&qrs_update_kernel),
                                                hipFuncAttributeMaxDynamicSharedMemorySize,
                                                (int)QRS_LDS);
  if (attr1 != hipSuccess) return attr1;
  if (attr2 != hipSuccess) return attr2;
  const dim3 chunks(QRL_CHUNKS, items);
  hipLaunchKernelGGL((qrl_load_kernel<CTI>), chunks, dim3(256), 0, s, args);
  hipLaunchKernelGGL(qrs_panel_kernel, dim3(items), dim3(512), QRS_LDS, s, args);
  for (int p = 0; p + QB < n_max; p += QB)   // update by panel p, factor panel p + 16
    hipLaunchKernelGGL(qrs_update_kernel, dim3(items, (n_max - p - QB + 15) / 16), dim3(512), QRS_LDS,
                       s, args, p);
  return hipGetLastError();
}

}  // namespace

int qr_large_max_rows() { return 2048; }

size_t qr_large_ws_elems(int m, int n) {
  const size_t parts = (((size_t)n + 15) / 16) * (((size_t)m + QRL_CH - 1) / QRL_CH) * 256;
  return 2 * (size_t)m * n + 16 * ((size_t)n + 16) + QRL_CHUNKS / 2 + parts + QRT_SCRATCH + 1;
}

hipError_t launch_qr_large(int ct_in, int ct_out, const QrArgs& args_in, hipStream_t s) {
  QrArgs args = args_in;
  int items = 0, m_max = 0, n_max = 0;
  for (int g = 0; g < args.ngroups; ++g) {
    if (args.g[g].mode == 2 || args.g[g].m < args.g[g].n) return hipErrorInvalidValue;
    args.g[g].blk_begin = items;
    items += args.g[g].batch;
    m_max = max(m_max, args.g[g].m);
    n_max = max(n_max, args.g[g].n);
  }
  if (items == 0) return hipSuccess;
  if (m_max > qr_large_max_rows()) return hipErrorInvalidValue;
#define DCS_QRL(I, O)            \
  if (ct_in == I && ct_out == O) \
    return run_tall<I, O>(args, items, m_max, n_max, s);
  DCS_QRL(CT_F32, CT_F32)
  DCS_QRL(CT_F64, CT_F64)
  DCS_QRL(CT_F64, CT_F32)
#undef DCS_QRL
  return hipErrorInvalidValue;
}

int qr_spread_max_rows() { return 512; }
int qr_spread_max_items() { return 96; }

hipError_t launch_qr_spread(int ct_in, int ct_out, const QrArgs& args_in, hipStream_t s) {
  QrArgs args = args_in;
  int items = 0, m_max = 0, n_max = 0;
  for (int g = 0; g < args.ngroups; ++g) {
    if (args.g[g].mode == 2 || args.g[g].m < args.g[g].n) return hipErrorInvalidValue;
    args.g[g].blk_begin = items;
    items += args.g[g].batch;
    m_max = max(m_max, args.g[g].m);
    n_max = max(n_max, args.g[g].n);
  }
  if (items == 0) return hipSuccess;
  if (m_max > qr_spread_max_rows()) return hipErrorInvalidValue;
  hipError_t e = ct_in == CT_F32   ? run_spread<CT_F32>(args, items, m_max, n_max, s)
                 : ct_in == CT_F64 ? run_spread<CT_F64>(args, items, m_max, n_max, s)
                                   : hipErrorInvalidValue;
  if (e != hipSuccess) return e;
  // Q from V and T: the blocked kernel's Q blocks read V at the workspace
  // start and T after it, so each group's workspace is taken m n further on
  QrArgs qa = args;
  for (int g = 0; g < qa.ngroups; ++g)
    qa.g[g].ws.base = static_cast<const char*>(qa.g[g].ws.base) +
                      (size_t)qa.g[g].m * qa.g[g].n * sizeof(double2);
  return launch_qr_qblocks(ct_in, ct_out, qa, m_max, s);
}

}  // namespace dcs
