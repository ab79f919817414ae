// Small bandwidth-bound kernels around the contractions: control words, the returned states,
// fills.
#include "common.h"
#include "prep.h"

// Control words of a call without steps (the others: k_prep_fwd, k_prep_bwd).
__global__ void __launch_bounds__(256) k_ctl(uint32_t* ctl, int keep_errors, int bwd) {
  if (bwd) zero_ctl_bwd(ctl, keep_errors);
  else init_ctl(ctl, keep_errors);
}

// h_top and c_top (either may be null): row (t, b) is a copy of the row of the state on top after
// step t. Bound by its writes. 2^ll lanes per row (the smallest power of two from 4 to 64 that covers it,
// so short rows fill the wave too), eight rows per lane with all indices, then all source vectors,
// in flight. (One vector per thread, with the row found by two 64-bit divisions each, took 655 us
// for 262144 rows of 1024 floats and 67 us for 61440 of 512.) V = 4: H is a multiple of 4 and the
// arrays are 16-byte aligned.
template <int V>
__global__ void __launch_bounds__(256) k_gather_top(GatherArgs a) {
  constexpr int R = 8;
  typedef float fv __attribute__((ext_vector_type(V)));
  const int HV = a.H / V, n = a.T * a.B, lane = threadIdx.x & 63, lpr = 1 << a.ll, rpw = 64 >> a.ll;
  const int first = ((int)blockIdx.x * 4 + (int)(threadIdx.x >> 6)) * (R * rpw) + (lane >> a.ll);
  int row[R];
  size_t src[R];
  bool init[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    row[k] = first + k * rpw;
    src[k] = (size_t)(unsigned)a.top[min(row[k], n - 1)];
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int r = min(row[k], n - 1), t = r / a.B, b = r - t * a.B;
    const int s = checked_src((int)src[k], t, a.ctl);
    init[k] = s < 0;
    src[k] = (s < 0 ? (size_t)b : (size_t)s * a.B + b) * HV;
  }
  auto copy = [&](const float* cell, const float* st0, float* out) {
    for (int u = lane & (lpr - 1); u < HV; u += lpr) {
      fv v[R];
#pragma unroll
      for (int k = 0; k < R; ++k) v[k] = ((const fv*)(init[k] ? st0 : cell))[src[k] + u];
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (row[k] < n) ((fv*)out)[(size_t)row[k] * HV + u] = v[k];
    }
  };
  if (a.htop) copy(a.hcell, a.h0, a.htop);
  if (a.ctop) copy(a.ccell, a.c0, a.ctop);
}
template __global__ void k_gather_top<1>(GatherArgs);
template __global__ void k_gather_top<4>(GatherArgs);

__global__ void __launch_bounds__(256) k_fill_f32(float* __restrict__ p, size_t n, float v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}
