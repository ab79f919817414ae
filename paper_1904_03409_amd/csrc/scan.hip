// Small bandwidth-bound kernels around the contractions: control words, the returned states,
// zero fills.
#include "common.h"

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

// h_top / c_top materialisation: the state returned at step t (Algorithm 1's return value)
// is the one produced at step top[t][b], or the initial state when top is -1.
__global__ void __launch_bounds__(256) k_gather_top(const int32_t* __restrict__ top, const float* __restrict__ cellv,
                                                    const float* __restrict__ init, float* __restrict__ out, int T,
                                                    int B, int H, uint32_t* ctl) {
  const size_t n = (size_t)T * B * H;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    size_t tb = i / H;
    int u = (int)(i - tb * H);
    int b = (int)(tb % B);
    int s = top[tb];
    int t = (int)(tb / B);
    s = checked_src(s, t, ctl);
    out[i] = (s < 0) ? init[(size_t)b * H + u] : cellv[((size_t)s * B + b) * H + u];
  }
}

// The same for h_top and c_top in one pass (either may be null), four units per thread: H must
// be a multiple of 4 and the arrays 16-byte aligned.
__global__ void __launch_bounds__(256) k_gather_top4(const int32_t* __restrict__ top, const float* __restrict__ hcell,
                                                     const float* __restrict__ h0, float* __restrict__ htop,
                                                     const float* __restrict__ ccell, const float* __restrict__ c0,
                                                     float* __restrict__ ctop, int T, int B, int H, uint32_t* ctl) {
  const int H4 = H / 4;
  const size_t n = (size_t)T * B * H4;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t tb = i / H4;
    const int u4 = (int)(i - tb * H4);
    const int b = (int)(tb % B), t = (int)(tb / B);
    const int s = checked_src(top[tb], t, ctl);
    const size_t src = s < 0 ? (size_t)b * H4 + u4 : ((size_t)s * B + b) * H4 + u4;
    if (htop) ((float4*)htop)[i] = s < 0 ? ((const float4*)h0)[src] : ((const float4*)hcell)[src];
    if (ctop) ((float4*)ctop)[i] = s < 0 ? ((const float4*)c0)[src] : ((const float4*)ccell)[src];
  }
}

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
