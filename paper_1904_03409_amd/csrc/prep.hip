// Operand preparation: bf16 planes (split.h) of x, W, U and the initial states in the layouts the
// contractions read, and the interval sums of the upstream gradient. Bandwidth bound at large sizes
// (256 x 240 steps, H = 512: planes of x 4.1 to 5.5 TB/s, interval sums 4.0 to 4.3, where a copy reaches 5.1).
#include "common.h"
#include "levels.h"
#include "prep.h"
#include "split.h"

// Largest finite magnitude so far and |v| (an infinity is one at any scale)
__device__ __forceinline__ float max_finite(float m, float v) { return __builtin_isfinite(v) ? fmaxf(m, fabsf(v)) : m; }

// Columns k0 .. k0 + Kc - 1 (multiples of 8) of rows lo .. hi-1 of the step list (push nodes, then leaves) of
// x as planes [S][hi - lo][Kc], zero past I.
template <int S>
__global__ void __launch_bounds__(256) k_split_x(const float* __restrict__ x, const int32_t* __restrict__ order, int lo,
                                                 int hi, int I, int k0, int Kc, int vec, bf16_t* __restrict__ out,
                                                 size_t plane) {
  const int gr = Kc / 8;
  const size_t n = (size_t)(hi - lo) * gr;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const size_t row = i / gr;
    const int kc = (int)(i - row * gr) * 8, k = k0 + kc;
    const float* src = x + (size_t)order[lo + row] * I + k;
    float v[8];
    if (vec && k + 8 <= I) {
      const float4 p = *(const float4*)src, q = *(const float4*)(src + 4);
      v[0] = p.x; v[1] = p.y; v[2] = p.z; v[3] = p.w; v[4] = q.x; v[5] = q.y; v[6] = q.z; v[7] = q.w;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = k + j < I ? src[j] : 0.f;
    }
    uint4 g[S];
    split_granule<S>(v, g);
#pragma unroll
    for (int s = 0; s < S; ++s) *(uint4*)(out + s * plane + row * Kc + kc) = g[s];
  }
}
template __global__ void k_split_x<1>(const float*, const int32_t*, int, int, int, int, int, int, bf16_t*, size_t);
template __global__ void k_split_x<3>(const float*, const int32_t*, int, int, int, int, int, int, bf16_t*, size_t);

// Forward operands, by block range:
//  * W tiles of 32 inputs x 32 units: wt [S][4H][Ip] (rows n = 4u + gate) and wp [S][I][H4s]
//    (columns n), through LDS so that both are written along their rows;
//  * U fragments (MFMA A operand) of the forward, per 8 units of a workgroup:
//    uf[w][wave][tile][chunk][plane][lane], wave = column pair + 4 K half, a lane's eight values
//    U[32 (half KS / 2 + chunk) + 8 lq + j][column of (unit 32 w + 8 pair + 4 tile + l16 / 4, gate
//    l16 % 4)]; fp32 mode: scaled per unit, odd chunks as mfma_rec takes them (split.h);
//  * the initial states as nodes (planes of h0 and a copy of c0), one wave per element.
// The first block also sets up the control words.
template <int S>
__global__ void __launch_bounds__(256) k_prep_fwd(PrepFwdArgs a) {
  __shared__ float tile[32][129];
  const int tid = threadIdx.x, H = a.H, I = a.I;
  int blk = blockIdx.x;
  if (blk == 0) init_ctl(a.ctl, a.keep_errors);
  if (blk < a.n_w) {
    const int ut = (H + 31) / 32, i0 = (blk / ut) * 32, u0 = (blk % ut) * 32;
    for (int e = tid; e < 32 * 128; e += 256) {
      const int i = e >> 7, k = (e >> 5) & 3, u = e & 31;
      tile[i][4 * u + k] = (i0 + i < I && u0 + u < H) ? a.W[(size_t)(i0 + i) * 4 * H + (size_t)k * H + u0 + u] : 0.f;
    }
    __syncthreads();
    for (int e = tid; e < 32 * 16; e += 256) {
      const int i = e >> 4, c = (e & 15) * 8, n = 4 * u0 + c;
      if (i0 + i >= I || n >= a.H4s) continue;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = tile[i][c + j];
      uint4 g[S];
      split_granule<S>(v, g);
#pragma unroll
      for (int s = 0; s < S; ++s) *(uint4*)(a.wp + (size_t)s * I * a.H4s + (size_t)(i0 + i) * a.H4s + n) = g[s];
    }
    for (int e = tid; e < 128 * 4; e += 256) {
      const int c = e >> 2, i = (e & 3) * 8, n = 4 * u0 + c;
      if (n >= 4 * H || i0 + i >= a.Ip) continue;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = tile[i + j][c];
      uint4 g[S];
      split_granule<S>(v, g);
#pragma unroll
      for (int s = 0; s < S; ++s) *(uint4*)(a.wt + ((size_t)s * 4 * H + n) * a.Ip + i0 + i) = g[s];
    }
    return;
  }
  blk -= a.n_w;
  constexpr int NP = S == 3 ? 2 : 1;
  const int lane = tid & 63;
  if (blk < a.n_u) {
    const int w = blk >> 2, pair = blk & 3, u0 = 32 * w + 8 * pair;
    __shared__ float s_max[256];
    float m = 0.f;
    if (S == 3) {
      const int unit = u0 + (tid & 7), gate = (tid >> 3) & 3;
      if (unit < H)
#pragma unroll 8
        for (int k = tid >> 5; k < H; k += 8) m = max_finite(m, a.U[(size_t)k * 4 * H + (size_t)gate * H + unit]);
      s_max[tid] = m;
      __syncthreads();
      for (int k = 8; k < 256; k += 8) m = fmaxf(m, s_max[(tid & 7) + k]);
      m = fmaxf(m, s_max[tid & 7]);
      __syncthreads();
      s_max[tid] = rec_scale(rec_exp(m));
      if (tid < 8) a.uexp[u0 + tid] = -rec_exp(m);
      __syncthreads();
    }
    const int KH = a.KS / 2;
    for (int f = tid; f < 4 * KH * 64; f += 256) {       // (half, tile, chunk, lane)
      const int c = (f >> 6) % KH, tile = (f >> 6) / KH & 1, half = (f >> 6) / KH >> 1;
      const int ul = 4 * tile + ((lane & 15) >> 2), unit = u0 + ul, gate = lane & 3, kc = half * KH + c;
      const float sc = S == 3 ? s_max[ul] : 1.f;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = 32 * kc + 8 * (lane >> 4) + j;
        v[j] = (k < H && unit < H) ? a.U[(size_t)k * 4 * H + (size_t)gate * H + unit] : 0.f;
      }
      uint4 g[NP];
      split_rec_granule<NP>(v, sc, g);
      if (S == 3 && (kc & 1)) g[0] = rec_negated(g[0]);
#pragma unroll
      for (int s = 0; s < NP; ++s)
        a.uf[((((size_t)(w * 8 + pair + 4 * half) * 2 + tile) * KH + c) * NP + s) * 64 + lane] = g[s];
    }
    return;
  }
  blk -= a.n_u;
  const int b = blk * 4 + (tid >> 6);
  if (b >= a.B) return;
  const int init = lev_goff(a.B, a.G, b % a.G) + b / a.G;
  const size_t node = (size_t)a.N0 + init;
  float sc = 1.f;
  if (S == 3) {
    float m = 0.f;
    for (int k = lane; k < H; k += 64) m = max_finite(m, a.h0[(size_t)b * H + k]);
#pragma unroll
    for (int d = 32; d; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    sc = rec_scale(rec_exp(m));
    if (lane == 0) a.rinit[init] = -rec_exp(m);
  }
  for (int k = lane; k < a.Hs; k += 64) {
    const float v = k < H ? a.h0[(size_t)b * H + k] : 0.f;
    if (k < H) a.cn[node * H + k] = a.c0[(size_t)b * H + k];
    uint16_t p[NP];
    split_rec<NP>(v, sc, p);
#pragma unroll
    for (int s = 0; s < NP; ++s) a.hq[s * a.hplane + node * a.Hs + k] = p[s];
    if (S == 3 && a.h3) {
      bf16_t q[3];
      split_bf16<3>(v, q);
#pragma unroll
      for (int s = 0; s < 3; ++s) a.h3[s * a.hplane + node * a.Hs + k] = q[s];
    }
  }
}
template __global__ void k_prep_fwd<1>(PrepFwdArgs);
template __global__ void k_prep_fwd<3>(PrepFwdArgs);

// Sums of an upstream gradient [T][B][H] over the intervals of steps during which one state stays
// on top: G[gslot][:] (slots: a push node's first interval; N0 + B + the popped node for the
// interval of its parent that follows; an initial state's first interval). An interval is a run
// of consecutive steps of one element. A wave takes 32 steps of an element and 64 V units and sums
// the intervals that begin in them, the last one to its end, wherever that is: every slot is
// written once, with no atomics, in the order of the steps. (One wave for all steps of an element
// left the chip without enough loads in flight: 328 us for 1024 steps of 128 elements at H = 512.)
template <int V>
__device__ __forceinline__ void interval_sums(int blk, const float* __restrict__ d, const int32_t* __restrict__ gslot, int T,
                                              int B, int H, int G, float* __restrict__ out) {
  constexpr int UN = 16;
  typedef float fv __attribute__((ext_vector_type(V)));
  const int lane = threadIdx.x & 63, parts = (H + 64 * V - 1) / (64 * V);
  const int wv = uni(blk * 4 + (int)(threadIdx.x >> 6));
  const int seg = wv / (B * parts), bp = wv - seg * (B * parts);
  if (seg * 32 >= T) return;
  const int b = bp / parts, u = (bp - b * parts) * 64 * V + lane * V;
  const bool on = u < H;
  const size_t rs = (size_t)B * H;
  const float* src = d + (size_t)b * H + u;
  const int own = min(32, T - 32 * seg);               // steps in which intervals of this wave begin
  int cur = seg ? gslot[(size_t)(32 * seg - 1) * B + b] : T * B + lev_goff(B, G, b % G) + b / G;
  cur = uni(cur);
  int k = 0;                                           // lane k: step t0 + k
  fv acc = 0.f;
  for (int t0 = 32 * seg; t0 < T; t0 += 64) {
    const bool head = t0 == 32 * seg;
    const int sl = t0 + lane < T ? gslot[(size_t)(t0 + lane) * B + b] : -1;
    if (head && seg) {                                 // the interval that is open belongs to a wave before
      const uint64_t m = __ballot(lane < own && sl != cur);
      if (!m) return;
      k = __builtin_ctzll(m);
      cur = __builtin_amdgcn_readlane(sl, k);
    }
    const int last = head ? __builtin_amdgcn_readlane(sl, own - 1) : cur;
    const uint64_t m = __ballot(sl != last) & (head ? ~0ull << own : ~0ull);
    const int kn = m ? __builtin_ctzll(m) : 64;
    for (; k < kn; k += UN) {
      fv v[UN];
#pragma unroll
      for (int q = 0; q < UN; ++q)
        if (on && k + q < kn) v[q] = __builtin_nontemporal_load((const fv*)(src + (size_t)(t0 + k + q) * rs));
        else v[q] = 0.f;
#pragma unroll
      for (int q = 0; q < UN; ++q) {
        if (k + q < kn) {
          const int s = __builtin_amdgcn_readlane(sl, k + q);
          if (s != cur) {
            if (on) *(fv*)(out + (size_t)cur * H + u) = acc;
            cur = s;
            acc = v[q];
          } else {
            acc += v[q];
          }
        }
      }
    }
    if (m) break;
    k = 0;
  }
  if (on) *(fv*)(out + (size_t)cur * H + u) = acc;
}

// Backward operands, by block range: the interval sums of an upstream gradient (interval_sums), and
// the U^T fragments (MFMA A operand) ub[w][wave][tile][chunk][plane][lane], a
// lane's eight values U[unit 32 w + 16 tile + l16][column of gate column 32 (wave KS / 2 + chunk) +
// 8 lq + j], in fp32 mode scaled per unit, odd chunks as mfma_rec takes them.
// One launch: the fragments' blocks are few and wait on their loads. The first block also clears
// the control words.
template <int S, int V>
__global__ void __launch_bounds__(256) k_prep_bwd(PrepBwdArgs a) {
  constexpr int NP = S == 3 ? 2 : 1;
  const int H = a.H, H4 = 4 * H, tid = threadIdx.x, lane = tid & 63;
  const bool ok = has_plan(a.ctl, a.key);
  if (blockIdx.x == 0 && a.clear) {
    zero_ctl_bwd(a.ctl, a.keep_errors);
    if (!ok && tid == 0) raise_badidx(a.ctl);
  }
  if (!ok) return;
  if (blockIdx.x < (unsigned)a.n_u) {
    const int blk = blockIdx.x, wave = blk & 7, tile = (blk >> 3) & 1, w = blk >> 4, u0 = 32 * w + 16 * tile, KH = a.KS / 2;
    __shared__ float s_sc[16];
    if (S == 3) {
      const int unit = u0 + (tid >> 4);
      float m = 0.f;
      if (unit < H)
#pragma unroll 8
        for (int n = tid & 15; n < H4; n += 16) m = max_finite(m, a.U[(size_t)unit * H4 + n]);
#pragma unroll
      for (int d = 8; d; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 16));
      if ((tid & 15) == 0) {
        s_sc[tid >> 4] = rec_scale(rec_exp(m));
        if (wave == 0) a.uinv[unit] = rec_ldexp(1.f, kDaExp - rec_exp(m));
      }
      __syncthreads();
    }
    const int unit = u0 + (lane & 15);
    for (int f = tid; f < KH * 64; f += 256) {           // (chunk, lane)
      const int c = f >> 6, kc = wave * KH + c;
      const float sc = S == 3 ? s_sc[lane & 15] : 1.f;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int np = 32 * kc + 8 * (lane >> 4) + j;
        v[j] = (unit < H && np < H4) ? a.U[(size_t)unit * H4 + perm_to_orig(np, H)] : 0.f;
      }
      uint4 g[NP];
      split_rec_granule<NP>(v, sc, g);
      if (S == 3 && (kc & 1)) g[0] = rec_negated(g[0]);
#pragma unroll
      for (int s = 0; s < NP; ++s)
        a.ub[((((size_t)(w * 8 + wave) * 2 + tile) * KH + c) * NP + s) * 64 + lane] = g[s];
    }
    return;
  }
  interval_sums<V>((int)blockIdx.x - a.n_u, a.d, a.gslot, a.T, a.B, H, a.G, a.sums);
}
template __global__ void k_prep_bwd<1, 1>(PrepBwdArgs);
template __global__ void k_prep_bwd<1, 4>(PrepBwdArgs);
template __global__ void k_prep_bwd<3, 1>(PrepBwdArgs);
template __global__ void k_prep_bwd<3, 4>(PrepBwdArgs);
