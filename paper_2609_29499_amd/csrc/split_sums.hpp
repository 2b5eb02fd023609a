// Sums of a prefill projection's K splits, added up by whoever reads them next. (Apart from the common
// header: counter summaries are tied to a hash of that one and of their kernel's source.)
#pragma once

#include "device_common.hpp"

namespace tasp {
namespace {

// v[i] += four floats of the K splits z0 .. ks - 1 of a projection, in split order, split z of item i
// at byte offset off[i] + z stride. The loads of up to eight splits are in flight together (one load
// and one wait per split made the consumers of a short prompt's eight splits wait eight memory
// latencies); slots past ks load nothing and add zero.
template <int Z, int N>
__device__ __forceinline__ void add_split_batch(__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[N], uint32_t stride,
                                                int z0, int ks, float4 (&v)[N]) {
  int4 p[Z][N];
#pragma unroll
  for (int z = 0; z < Z; ++z)
#pragma unroll
    for (int i = 0; i < N; ++i)
      p[z][i] = buf_load16(r, z0 + z < ks ? off[i] + uint32_t(z0 + z) * stride : kOOB);
#pragma unroll
  for (int z = 0; z < Z; ++z)
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float4 q = __builtin_bit_cast(float4, p[z][i]);
      v[i].x += q.x; v[i].y += q.y; v[i].z += q.z; v[i].w += q.w;
    }
}
template <int N>
__device__ __forceinline__ void add_splits(__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[N], uint32_t stride,
                                           int z0, int ks, float4 (&v)[N]) {
  for (; z0 < ks; z0 += 8) {
    if (ks - z0 > 4) add_split_batch<8>(r, off, stride, z0, ks, v);
    else if (ks - z0 > 2) add_split_batch<4>(r, off, stride, z0, ks, v);
    else add_split_batch<2>(r, off, stride, z0, ks, v);
  }
}

}  // namespace
}  // namespace tasp
