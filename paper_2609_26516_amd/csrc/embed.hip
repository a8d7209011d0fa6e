// Site tensor embedded in larger bond dims with an optional multiple of a
// second tensor added (the warm-start guess of a compression step), or a
// plain batched copy of site tensors between slot regions; copies of whole
// branches.
#include "dcs_internal.h"
#include "kernel_util.h"

namespace dcs {
namespace {

constexpr int NT = 256;

template <int CT>
__global__ __launch_bounds__(NT) void embed_kernel(const EmbedArgs a) {
  using T = typename St<CT>::T;
  const int item = blockIdx.y;
  const long long idx = (long long)blockIdx.x * NT + threadIdx.x;
  const long long tot = (long long)a.dl * 2 * a.dr;
  if (idx >= tot) return;
  const int b = (int)(idx % a.dr), sa = (int)(idx / a.dr);   // sa = 2 a + s
  const int al = sa >> 1, s = sa & 1;
  T* dst = reinterpret_cast<T*>(const_cast<char*>(item_ptr(a.dst, a.ids, item)));
  double re = 0.0, im = 0.0;
  if (al < a.kl && b < a.kr) {
    const T* src = reinterpret_cast<const T*>(item_ptr(a.src, a.ids, item));
    const T v = src[((long long)al * 2 + s) * a.kr + b];
    re = v.x;
    im = v.y;
  }
  if (a.init.base) {
    const T* ini = reinterpret_cast<const T*>(item_ptr(a.init, a.ids, item));
    const T u = ini[idx];
    re += a.eta * (double)u.x;
    im += a.eta * (double)u.y;
  }
  T o;
  o.x = re;
  o.y = im;
  dst[idx] = o;
}

// Copies of many segments in one launch (branches copied by a measurement):
// 16 KB per workgroup, 16 bytes per lane and access; bound by memory.  As one
// copy command per branch, 1024 branches of 24 qubits at bond 64 (0.86 MB each
// in complex64) cost 1.9 us each on the device and the gap to the next; a
// measurement round of them (collapse into new slots, compression, two more
// measurements) went from 34.4 to 28.4 ms.
constexpr int COPY_CHUNK = 16 * 1024;
__global__ __launch_bounds__(NT) void copy_segments_kernel(const CopySegment* segs) {
  const CopySegment sg = segs[blockIdx.y];
  const long long first = (long long)blockIdx.x * COPY_CHUNK;
  const long long count = min((long long)COPY_CHUNK, sg.bytes - first) / 16;
  const float4* __restrict__ src = reinterpret_cast<const float4*>(sg.src + first);
  float4* __restrict__ dst = reinterpret_cast<float4*>(sg.dst + first);
#pragma unroll
  for (int q = 0; q < COPY_CHUNK / 16 / NT; ++q) {
    const int i = (int)threadIdx.x + q * NT;
    if (i < count) dst[i] = src[i];
  }
}

}  // namespace

hipError_t launch_embed(int ct, const EmbedArgs& args, hipStream_t s) {
  const long long tot = (long long)args.dl * 2 * args.dr;
  if (args.batch <= 0 || tot <= 0) return hipSuccess;
  if (args.kl < 0 || args.kr < 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((tot + NT - 1) / NT), args.batch), blk(NT);
  if (ct == CT_F32)
    hipLaunchKernelGGL((embed_kernel<CT_F32>), grid, blk, 0, s, args);
  else
    hipLaunchKernelGGL((embed_kernel<CT_F64>), grid, blk, 0, s, args);
  return hipGetLastError();
}

hipError_t launch_copy_segments(const CopySegment* segs_dev, int count, long long max_bytes,
                                hipStream_t s) {
  if (count <= 0 || max_bytes <= 0) return hipSuccess;
  const dim3 grid((unsigned)((max_bytes + COPY_CHUNK - 1) / COPY_CHUNK), count), blk(NT);
  hipLaunchKernelGGL(copy_segments_kernel, grid, blk, 0, s, segs_dev);
  return hipGetLastError();
}

}  // namespace dcs
