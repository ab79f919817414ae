// Small bandwidth-bound kernels around the contractions: control words, the returned states,
// zero fills.
#include "common.h"
#include "prep.h"

// Control words of a forward call at 0 (status: no error). With keep_errors (a deferred
// call) the error words keep what earlier calls on the work space set: the lowest failing
// element's op status, the time-out and the index flag.
__global__ void __launch_bounds__(256) k_init_ctl(uint32_t* ctl, int keep_errors) {
  for (int i = threadIdx.x; i < CTL_WORDS; i += blockDim.x) {
    const bool err = i == CTL_STATUS || i == CTL_TIMEOUT || i == CTL_BADIDX;
    if (keep_errors && err) continue;
    ctl[i] = (i == CTL_STATUS) ? kStatusOk : 0u;
  }
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

// Clears the backward's control words: slot counters, group barrier counters, the wait flags
// and the index flag (the op status of the forward stays: the backward reports only its own).
// (keep_errors: a deferred call; the error words stay as earlier calls left them)
__global__ void __launch_bounds__(256) k_zero_ctl_bwd(uint32_t* __restrict__ ctl, int keep_errors) {
  for (int i = threadIdx.x; i < 16; i += blockDim.x) ctl[CTL_XCC_SLOT_B + i] = 0u;
  for (int i = threadIdx.x; i < 16 * MAX_GROUPS; i += blockDim.x) ctl[CTL_BAR_B + i] = 0u;
  if (threadIdx.x == 0) {
    ctl[CTL_ABORT] = 0u;
    if (!keep_errors) {
      ctl[CTL_STATUS] = kStatusOk;
      ctl[CTL_TIMEOUT] = 0u;
      ctl[CTL_BADIDX] = 0u;
    }
  }
}

// Zeroes the rows of out [n][cols] whose op is not a push (dx is exactly 0 there).
__global__ void __launch_bounds__(256) k_zero_nonpush_rows(const int8_t* __restrict__ ops, float* __restrict__ out,
                                                           size_t n, int cols) {
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, nth = (size_t)gridDim.x * blockDim.x;
  if ((cols & 3) == 0 && ((uintptr_t)out & 15) == 0) {
    const int cv = cols >> 2;
    const size_t nv = n * cv;
    for (size_t i = tid; i < nv; i += nth)
      if (ops[i / cv] != 1) ((float4*)out)[i] = float4{0.f, 0.f, 0.f, 0.f};
    return;
  }
  for (size_t i = tid; i < n * cols; i += nth)
    if (ops[i / cols] != 1) out[i] = 0.f;
}
