// Work of one 256-thread workgroup on small matrices: 16 x 16 MFMA tiles in
// either precision, ordering of LDS traffic, and a product spread over the
// waves.
#pragma once

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

}  // namespace
}  // namespace dcs
