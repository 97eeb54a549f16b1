// ctmhd_workgroup.h -- device functions in which the wavefronts of a workgroup
// exchange values through LDS.  They use the HIP builtins only and nothing of
// the rest of the library, so that a host build that supplies those builtins
// can run a workgroup in any order of its wavefronts.
#pragma once

namespace ctmhd {

constexpr int kBlock = 256;

// Block maximum of a non-negative (or NaN) double, as its bit pattern (a NaN
// has larger bits than +inf as an unsigned integer); valid in thread 0.  All
// threads must call; a workgroup may call it again and again, so the first
// barrier keeps a wavefront that runs ahead from overwriting `red` while
// thread 0 still reads it for the call before.
__device__ __forceinline__ unsigned long long block_max_bits(double s) {
  __shared__ unsigned long long red[kBlock / 64];
  unsigned long long bits = (unsigned long long)__double_as_longlong(s);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long ob = __shfl_xor(bits, o, 64);
    bits = ob > bits ? ob : bits;
  }
  int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[w] = bits;
  __syncthreads();
  unsigned long long m = 0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) m = red[q] > m ? red[q] : m;
  return m;
}

}  // namespace ctmhd
