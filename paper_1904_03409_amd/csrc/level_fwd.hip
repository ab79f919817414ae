// Forward recurrence over the level schedule (levels.h). Persistent; one group of batch
// elements per set of NW = ceil(H / 32) workgroups of one XCD (one L2).
//
// Workgroup w owns units 32 w .. 32 w + 31 and keeps its 128 gate columns of U in registers for
// the whole kernel: four pairs of waves, a pair 32 columns, each wave of it one half of K (so that
// a state's row is read from LDS four times, not eight). Per level, for 16 RT states at a time:
// copy the states' rows into LDS (LDS DMA, the next rows in flight behind the products), h U on
// MFMA, the result to hu (for the leaves) and through LDS to the push children of those states,
// which are consecutive nodes: gates, cell, stores. One group barrier per level.
#include "common.h"
#include "levels.h"
#include "split.h"

// CLK: with the stamps of dims.step_clock.
template <int NP, int KS, bool CLK>
__global__ void __launch_bounds__(kLevThreads, 2) k_lev_fwd(LevFwdArgs a) {
  constexpr int RT = lev_fwd_rt(NP, KS), ROWS = 16 * RT, GRW = KS * 4;  // rows per pass, 16-byte granules per row
  constexpr int KH = KS / 2;
  constexpr int PLANE = ROWS * GRW * 16, BUF = PLANE * NP;
  constexpr int HULD = kLevHuLd, HUH = ROWS * HULD;         // one K half of h U
  extern __shared__ __align__(16) unsigned char lsm[];
  float* hu_s = reinterpret_cast<float*>(lsm + 2 * BUF);    // [2][2][ROWS][HULD] h U of the pass, by K half
  float* c_s = hu_s + 4 * HUH;                              // [2][ROWS][32] c of the parents
  __shared__ int s_g, s_w, s_flag;
  claim_group_slot(a.ctl + CTL_XCC_SLOT, a.G, a.NW, &s_g, &s_w);
  const int g = uni(s_g), w = uni(s_w);
  if (g < 0) return;
  const int T = a.T, B = a.B, H = a.H, Hs = a.Hs, H4 = 4 * H, N0 = a.N0;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  uint32_t* bar = a.ctl + CTL_BAR_F + 16 * g;
  const int n_init = N0 + lev_goff(B, a.G, g), Bg = lev_bg(B, a.G, g);
  const int32_t* loff = a.ix.loff + (size_t)g * (T + 4);
  const int D = uni(a.ix.gmax[g]);
  const bool solo = KS == 2 && a.NW == 1;                   // the group is this workgroup: no exchange with others

  uint4 uf[2][KH][NP];
  {
    const uint4* src = a.uf + (size_t)(w * 8 + wave) * 2 * KH * NP * 64 + lane;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < KH; ++c)
#pragma unroll
        for (int s = 0; s < NP; ++s) uf[t][c][s] = src[((t * KH + c) * NP + s) * 64];
  }
  int ui[2] = {0, 0};                                       // exponents of the inverse scales of this lane's units
  if constexpr (NP == 2) {
    ui[0] = a.uexp[32 * w + 8 * (wave & 3) + lq];
    ui[1] = a.uexp[32 * w + 8 * (wave & 3) + 4 + lq];
  }

  // rows [row0, q1) (at most ROWS) into buffer buf; granule gr of row r sits at slot gr ^ (r & 7).
  // (A DMA costs the same with and without live lanes: those of missing rows are left out, and what
  // the buffer held stays in result columns nobody reads.)
  auto issue = [&](int row0, int q1, int buf) {
    row0 = uni(row0);
    const int nr = uni(min(ROWS, q1 - row0));
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      const rsrc_t rs = make_rsrc(a.hq + s * a.hplane + (size_t)row0 * Hs, (size_t)nr * Hs * 2);
#pragma unroll
      for (int q0 = 0; q0 < RT * KS; q0 += 8) {
        const int q = q0 + wave;
        if (q < RT * KS && q * 64 / GRW < nr) {
          const int L = q * 64 + opaque(lane), row = L / GRW, gr = (L % GRW) ^ (row & 7);
          const uint32_t off = gr * 8 < Hs ? (uint32_t)((row * Hs + gr * 8) * 2) : kOOB;
          bdma16_sc1(rs, off, 0u, lds_addr(lsm + buf * BUF + s * PLANE + q * 1024));
        }
      }
    }
  };
  // this thread's operands of a pass: of its first 16 children (fixed before the kernel), and c of
  // the parents (made a level earlier)
  struct Pre { f32x4 xw; float cp[RT]; int c0, c1, par, row; };
  // (c0: where the previous pass's children end; c1 arrives with the operands; a thread past c1 reads
  // a later child's operands in vain)
  auto prefetch = [&](Pre& p, int row0, int q1, int c0, int cend) {
    const int ot = opaque(tid), ou = 32 * w + (ot & 31);
    p.c0 = c0;
    p.c1 = row0 + ROWS < q1 ? a.ix.cs[row0 + ROWS] : cend;
    const int c = c0 + (ot >> 5);
    p.par = p.row = 0;
    p.xw = f32x4{0.f, 0.f, 0.f, 0.f};
    if (c < cend && ou < H) {
      p.xw = __builtin_nontemporal_load((const f32x4*)(a.hu + (size_t)c * H4 + 4 * ou));
      p.par = *at32(a.ix.opar, 4u * c);
      p.row = *at32(a.ix.order, 4u * c);
    }
  };
  auto prefetch_c = [&](Pre& p, int row0, int q1) {
    const int ot = opaque(tid), ou = 32 * w + (ot & 31);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
      const int q = row0 + (ot >> 5) + 16 * r;
      p.cp[r] = q < q1 && ou < H ? a.cn[(size_t)q * H + ou] : 0.f;
    }
  };
  auto h_u = [&](const float* hs, int r, int uu) {           // h U of row r of the pass, this thread's unit
    const f32x4 x = *(const f32x4*)&hs[r * HULD + 4 * uu], y = *(const f32x4*)&hs[HUH + r * HULD + 4 * uu];
    return f32x4{x[0] + y[0], x[1] + y[1], x[2] + y[2], x[3] + y[3]};
  };
  struct Cell { f32x4 g; float h, cc, cp; };
  auto cell = [&](int c, int row0, const float* hs, const float* cs, const f32x4& xw, int par) {
    const int uu = opaque(tid) & 31, u = 32 * w + uu;
    const int r = par - row0;
    const f32x4 hu = h_u(hs, r, uu);
    Cell o;
    o.cp = cs[r * kLevUnits + uu];
    o.g = f32x4{sigmoidf_(hu[0] + xw[0]), sigmoidf_(hu[1] + xw[1]), tanhf_(hu[2] + xw[2]), sigmoidf_(hu[3] + xw[3])};
    o.cc = o.g[1] * o.cp + o.g[0] * o.g[2];
    o.h = canon_nan(o.g[3] * tanhf_(o.cc));
    uint16_t p[NP];
    split_rec<NP>(o.h, kHScale, p);
#pragma unroll
    for (int s = 0; s < NP; ++s) *at32(a.hq + s * a.hplane, 2u * (uint32_t)(c * Hs + u)) = p[s];
    return o;
  };
  auto keep = [&](int c, int row, const Cell& o) {
    const int u = 32 * w + (opaque(tid) & 31);
    const uint32_t oc = 4u * (uint32_t)(c * H + u), orow = 4u * (uint32_t)(row * H + u);
    *at32(a.cn, oc) = o.cc;
    *at32(a.hcell, orow) = o.h;
    *at32(a.ccell, orow) = o.cc;
    if (a.stash) {
      *(f32x4*)(a.stash + (size_t)c * H4 + 4 * u) = o.g;
      *at32(a.cpn, oc) = o.cp;
      if constexpr (NP == 2) {
        bf16_t p[3];
        split_bf16<3>(o.h, p);
#pragma unroll
        for (int s = 0; s < 3; ++s) *at32(a.h3 + s * a.hplane, 2u * (uint32_t)(c * Hs + u)) = p[s];
      }
    }
  };
  auto store_hu = [&](const float* hs, int row0, int nr) {
    const int ot = opaque(tid), ou = ot & 31;
    for (int r = ot >> 5; r < nr; r += 16)
      *(f32x4*)(a.hu + (size_t)(row0 + r) * H4 + 4 * (32 * w + ou)) = h_u(hs, r, ou);
  };
  auto pad = [&](int c) {                                   // zero padding of a state's rows
    const int u = 32 * w + (opaque(tid) & 31);
#pragma unroll
    for (int s = 0; s < NP; ++s) a.hq[s * a.hplane + (size_t)c * Hs + u] = 0;
    if (NP == 2 && a.h3) {
#pragma unroll
      for (int s = 0; s < 3; ++s) a.h3[s * a.hplane + (size_t)c * Hs + u] = 0;
    }
  };

  // wall-clock stamps: level top, first rows landed, products of the last pass done, end
  auto stamp = [&](int d, int k) {
    if (CLK && tid == 0 && d < T) a.clk[((size_t)blockIdx.x * T + d) * 4 + k] = wall_clock64();
  };
  int q0 = n_init, q1 = n_init + Bg;
  int c0 = uni(loff[1]), cend = uni(loff[2]);               // children of the level: nodes [c0, cend)
  Pre pre;
  prefetch(pre, q0, q1, c0, cend);
  prefetch_c(pre, q0, q1);
  int hb = 0;                                               // buffer of hu_s and c_s
  for (int d = 0;; ++d) {
    stamp(d, 0);
    issue(q0, q1, 0);
    wait_vm<0>();
    __syncthreads();                                        // the level's first rows landed
    stamp(d, 1);
    if (q0 + ROWS < q1) issue(q0 + ROWS, q1, 1);
    const int next_end = loff[min(d + 3, D + 2)];           // (in flight until the level is done)
    int buf = 0;
    for (int row0 = q0; row0 < q1; row0 += ROWS, buf ^= 1, hb ^= 1) {
      const int nr = min(ROWS, q1 - row0), kh = wave >> 2;
      const bool more = row0 + ROWS < q1;
      float* hs = hu_s + hb * (2 * HUH);
      float* cs = c_s + hb * (ROWS * kLevUnits);
      const unsigned char* bs = lsm + buf * BUF + l16 * (GRW * 16);
      f32x4 acc[RT][2], lo[RT][2];
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[r][t] = lo[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < KH; ++c) {
        const int kc = kh * KH + c;
        const unsigned char* bc = bs + ((4 * kc + lq) ^ (l16 & 7)) * 16;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          uint4 b[NP];
#pragma unroll
          for (int s = 0; s < NP; ++s) b[s] = *(const uint4*)(bc + s * PLANE + r * 16 * GRW * 16);
#pragma unroll
          for (int t = 0; t < 2; ++t) mfma_rec<NP>(c, uf[t][c], b, acc[r][t], lo[r][t]);
        }
        // (a few chunks' fragments at a time: more of them read ahead cost registers)
        if (NP * KS >= 32 && (c & 1)) __builtin_amdgcn_sched_barrier(0);
      }
      // (KS = 2: the one chunk of the second half is an odd one)
      const float sg = (KH & 1) && kh ? -1.f : 1.f;
      if constexpr (NP == 2) {
        bool bad = false;
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          const bool live = 16 * r + l16 < nr;
          int f = -kHExp;
          if (d == 0 && live) f = a.rinit[row0 + 16 * r + l16 - N0];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[r][t][q] = rec_ldexp(acc[r][t][q] * sg + lo[r][t][q], ui[t] + f);
            bad |= live && has_nan(acc[r][t]);
          }
        }
        if (__ballot(bad)) {
#pragma unroll
          for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int c = 0; c < KH; ++c) {
                const uint4 b = *(const uint4*)(bs + ((4 * (kh * KH + c) + lq) ^ (l16 & 7)) * 16 + r * 16 * GRW * 16);
                mfma_rec_first(c, uf[t][c][0], b, v);
              }
#pragma unroll
              for (int q = 0; q < 4; ++q)
                if (acc[r][t][q] != acc[r][t][q]) acc[r][t][q] = v[q] * sg;
            }
        }
      }
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int t = 0; t < 2; ++t)
          *(f32x4*)&hs[kh * HUH + (r * 16 + l16) * HULD + 32 * (wave & 3) + 16 * t + 4 * lq] = acc[r][t];
      // the next pass's rows and this pass's operands, issued a pass ago (one in-order counter: the
      // stores in between are waited for too)
      wait_vm<0>();
#pragma unroll
      for (int r = 0; r < RT; ++r) cs[(opaque(tid) >> 5) * kLevUnits + 16 * r * kLevUnits + (opaque(tid) & 31)] = pre.cp[r];
      __syncthreads();
      if (!more) stamp(d, 2);
      // in flight behind the cell and the next products: the rows after the next (this buffer is free)
      // and the operands of the next pass
      const Pre cur = pre;
      if (row0 + 2 * ROWS < q1) issue(row0 + 2 * ROWS, q1, buf);
      if (more) {
        prefetch(pre, row0 + ROWS, q1, uni(cur.c1), cend);
        prefetch_c(pre, row0 + ROWS, q1);
      }
      const int ok = opaque(tid) >> 5, ou = 32 * w + (opaque(tid) & 31);
      if (ou < H) {
        if (cur.c0 + ok < cur.c1) keep(cur.c0 + ok, cur.row, cell(cur.c0 + ok, row0, hs, cs, cur.xw, cur.par));
        for (int c = cur.c0 + ok + 16; c < cur.c1; c += 16)
          keep(c, a.ix.order[c], cell(c, row0, hs, cs, *(const f32x4*)(a.hu + (size_t)c * H4 + 4 * ou), a.ix.opar[c]));
        store_hu(hs, row0, nr);
      } else if (ou < Hs) {
        for (int c = cur.c0 + ok; c < cur.c1; c += 16) pad(c);
      }
    }
    stamp(d, 3);
    if (d >= D) break;
    group_arrive(bar, solo);
    const uint32_t seen = solo ? 0u : group_peek(bar);
    q0 = c0;
    q1 = c0 = cend;                                         // (levels follow each other)
    cend = uni(next_end);
    prefetch(pre, q0, q1, c0, cend);
    prefetch_c(pre, q0, q1);
    if (!solo && group_wait(bar, (uint32_t)(a.NW * (d + 1)), seen, a.ctl, a.spin_limit, &s_flag)) break;
  }
}

template <int NP, int KS, bool CLK>
static hipError_t launch_t(const LevFwdArgs& a, int grid, hipStream_t st) {
  auto kern = k_lev_fwd<NP, KS, CLK>;
  constexpr int shm = (int)lev_fwd_lds(NP, KS);
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, shm);
  if (e != hipSuccess) return e;
  LevFwdArgs args = a;
  void* kargs[] = {&args};
  return hipLaunchCooperativeKernel((const void*)kern, dim3(grid), dim3(kLevThreads), kargs, (unsigned)shm, st);
}
hipError_t launch_lev_fwd(const LevFwdArgs& a, int NP, int KS, int grid, hipStream_t st) {
#define CASE(N_, KS_) \
  if (NP == N_ && KS == KS_) return a.clk ? launch_t<N_, KS_, true>(a, grid, st) : launch_t<N_, KS_, false>(a, grid, st);
  LEV_CASES(CASE)
#undef CASE
  return hipErrorInvalidValue;
}
