// Loads of matrix tiles into registers for the GEMM kernels, without branches.
//
// Every lane reads its run of elements through a raw buffer descriptor whose
// range ends with the operand; what lies outside the matrix is read at an
// offset past the range and comes back as zero.  Predicated loads instead
// (a branch around each load, or an element cleared before it is loaded) make
// the compiler wait for the loads already in flight, which leaves the memory
// latency of every K step exposed; so does touching the loaded values before
// they are stored to LDS, which is why conjugation is left to the store.
// (Reading a valid element in place of one outside and clearing it at the
// store costs registers: the 128 x 128 tiles of a 256-state, bond-256 round
// took 1.55 ms instead of 1.43.)
#pragma once

#include "dcs_internal.h"

namespace dcs {
namespace {

constexpr unsigned TL_OUT = 0xFFFFFFFFu;   // past every range

// Descriptor of `bytes` bytes from p (the same in every lane).  A window of the GEMM
// kernels is at most 128 lines of fewer than GEMM_FAR_LD elements: 4 GB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tl_rsrc(const void* p, long long bytes) {
  const unsigned long long a = reinterpret_cast<unsigned long long>(p);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  const unsigned n = __builtin_amdgcn_readfirstlane((unsigned)bytes);
  return __builtin_amdgcn_make_buffer_rsrc(
      reinterpret_cast<void*>(((unsigned long long)hi << 32) | lo), 0, (int)n, 0x00020000);
}

// r[u] = element u of the run at byte offset voff for u < left, else zero
// (left <= 0: all zero).  vec (uniform): the run starts on 16 bytes and `left`
// is even, so complex64 elements come in pairs.
template <typename T, int E>
__device__ __forceinline__ void tl_run(T (&r)[E], __amdgpu_buffer_rsrc_t rsrc, unsigned voff,
                                       int left, bool vec) {
  if constexpr (sizeof(T) == 8 && E % 2 == 0) {
    if (vec) {
#pragma unroll
      for (int u = 0; u < E; u += 2) {
        const unsigned o = u < left ? voff + u * 8u : TL_OUT;
        const float4 v = __builtin_bit_cast(
            float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, 0, 0));
        r[u].x = v.x;
        r[u].y = v.y;
        r[u + 1].x = v.z;
        r[u + 1].y = v.w;
      }
      return;
    }
  }
#pragma unroll
  for (int u = 0; u < E; ++u) {
    const unsigned o = u < left ? voff + u * (unsigned)sizeof(T) : TL_OUT;
    if constexpr (sizeof(T) == 8) {
      const float2 v =
          __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)o, 0, 0));
      r[u].x = v.x;
      r[u].y = v.y;
    } else {
      const double2 v =
          __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)o, 0, 0));
      r[u].x = v.x;
      r[u].y = v.y;
    }
  }
}

// The same for an operand that a window does not cover.
template <typename T, int E>
__device__ __forceinline__ void tl_run_far(T (&r)[E], const T* __restrict__ p, int left) {
#pragma unroll
  for (int u = 0; u < E; ++u) {
    r[u].x = 0;
    r[u].y = 0;
    if (u < left) r[u] = p[u];
  }
}

}  // namespace
}  // namespace dcs
