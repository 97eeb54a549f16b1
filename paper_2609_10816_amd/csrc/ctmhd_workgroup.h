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

// dt of a batched step from the per-box CFL maxima (the fix-up maximum where
// a box's second stage was fixed up); resets the per-step counters.  All
// threads read the stop flag before any sets it: the boxes after a bad dt
// still get theirs.
static __global__ void __launch_bounds__(kBlock)
    k_bdt_final(int nbox, int nphase, int dt_per_box, int level, unsigned long long* slots, int* nflag,
                int* done, int* cursor, double cfl, const double* dt_fixed, double* dt,
                double* dt_out, int* stop, const int* err, long long* diag) {
  __shared__ unsigned long long red[kBlock];
  const int t = threadIdx.x;
  unsigned long long mx = 0;
  const bool stopped = *stop != 0;
  __syncthreads();
  for (int b = t; b < nbox; b += kBlock) {
    unsigned long long v = nflag[4 * (level ? 0 : b) + 2] ? slots[2 * b + 1] : slots[2 * b];
    mx = v > mx ? v : mx;
    if (dt_per_box) {
      double x = stopped ? 0.0 : (dt_fixed ? dt_fixed[b] : cfl / __longlong_as_double((long long)v));
      if (!stopped && (!(x > 0.0) || !__builtin_isfinite(x))) atomicExch(stop, 1);
      dt[b] = x;
      if (dt_out) dt_out[b] = x;
    }
  }
  red[t] = mx;
  __syncthreads();
  for (int o = kBlock / 2; o > 0; o >>= 1) {
    if (t < o) red[t] = red[t + o] > red[t] ? red[t + o] : red[t];
    __syncthreads();
  }
  if (t == 0 && !dt_per_box) {
    double x = stopped ? 0.0 : (dt_fixed ? dt_fixed[0] : cfl / __longlong_as_double((long long)red[0]));
    if (!stopped && (!(x > 0.0) || !__builtin_isfinite(x))) *stop = 1;
    dt[0] = x;
    if (dt_out) dt_out[0] = x;
  }
  for (int b = t; b < nbox; b += kBlock) {
    slots[2 * b] = slots[2 * b + 1] = 0ull;
    nflag[4 * b] = nflag[4 * b + 1] = nflag[4 * b + 2] = nflag[4 * b + 3] = 0;
  }
  for (int i = t; i < nphase * nbox; i += kBlock) done[i] = 0;
  if (t < 4) cursor[t] = 0;
  __syncthreads();
  if (t == 0 && diag) {
    diag[0] = diag[1] = diag[2] = 0;
    diag[3] = (*stop ? 1 : 0) | (*err << 1);
  }
}

}  // namespace ctmhd
