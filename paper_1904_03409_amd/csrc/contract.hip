// The non-recurrent contractions of the step, on bf16 planes (split.h), 16x16x32 MFMA:
//   k_nt  x W + b of the push nodes, x W + b and the whole cell of the leaves, dx = dA W^T
//   k_tn  dW = x^T dA and dU = h_prev^T dA over the push nodes, split over K
// 512 threads (two waves per SIMD), one workgroup per CU; operand slices go from global memory
// into two LDS stages by LDS DMA, the next slice in flight behind the products of the current one.
// A DMA writes one contiguous kilobyte per wave instruction, so each lane fetches the 16-byte
// granule that a swizzled layout puts at its slot; fragment reads then spread over the banks.
// S = 3: 256 x 128 block (or fewer rows: k_nt), 64 x 64 per wave, K steps of 32: six MFMAs per pair of three-plane
// fragments, bound by the matrix units. S = 1: 256 x 256 block, 128 x 64 per wave, K steps of 64
// (a wave reads 12 KB of fragments per 32 MFMAs).
#include <algorithm>

#include "common.h"
#include "contract.h"
#include "split.h"

namespace {

// The products of one K step of 32 on MI x NJ tiles. C^T = B^T A^T: a lane holds row l16 and
// columns 4 lq .. 4 lq + 3 of a tile. between(i) runs after the products of row tile i: the next
// slice's DMAs are issued there, a few at a time, because a wave that issues them all at once
// stands still until the memory queue has taken them (dW | dU of 17 k nodes: DMAs alone 211 us,
// products alone 218, one after the other 378, this way 325).
template <int S, int MI, int NJ, typename F>
__device__ __forceinline__ void tile_step(const bf16x8 (&a)[MI][S], const bf16x8 (&b)[NJ][S], f32x4 (&acc)[MI][NJ],
                                          F between) {
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if constexpr (S == 1) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = mfma_bf16_16x16x32(b[j][0], a[i][0], acc[i][j]);
    } else {
      mfma_planes_add<NJ>(b, a[i], acc[i]);
    }
    between(i);
  }
}

// fp32 mode: an infinite operand has no second and third plane, and products of infinities with planes of
// both signs or with zero planes give NaN where the fp32 product is infinite. The sum of the first
// planes' products is infinite or NaN as the fp32 sum is. So a wave with NaN among its results
// takes those from another pass over K with the first planes, straight from memory: half the
// time of the tile again at most. (One lane through all of K for each NaN: large training step with a NaN
// in every gradient 236 ms instead of 2.7.) init(i, j): where the sums started; frag(k, a, b): the
// fragments of K step k.
__device__ __forceinline__ bool is_nan(float v) { return v != v; }
template <int MI, int NJ, typename I, typename F>
__device__ __forceinline__ void redo_nan(f32x4 (&acc)[MI][NJ], int kbeg, int kend, I init, F frag) {
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) bad |= is_nan(acc[i][j][q]);
  if (__builtin_expect(__ballot(bad) == 0, 1)) return;
  f32x4 v[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) v[i][j] = init(i, j);
#pragma unroll 1
  for (int k = kbeg; k < kend; k += 32) {
    bf16x8 a[MI], b[NJ];
    frag(k, a, b);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) v[i][j] = mfma_bf16_16x16x32(b[j], a[i], v[i][j]);
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (is_nan(acc[i][j][q]) && !__builtin_isfinite(v[i][j][q])) acc[i][j][q] = v[i][j][q];
}

}  // namespace

// One block tile of k_nt: 16 MI x (8 / WN) rows, K steps of BK. PRE: the sums go on from C.
template <int S, int EPI, int MI, bool PRE>
__device__ __forceinline__ void nt_tile(const NtArgs& g, int r_lo, int r_hi, int lid, unsigned char* sm, int* s_row,
                                        int* s_par) {
  constexpr int BM = nt_bm(S, MI), BN = nt_bn(S), BK = nt_bk(S, MI), GR = BK / 8;
  constexpr int NJ = 4, WN = BN / (16 * NJ);
  static_assert(BM == 16 * MI * (8 / WN), "eight waves cover the block tile");
  static_assert(nt_lds(S, MI) <= nt_lds(S, nt_mi(S)) && nt_leaf_lds(S, MI) <= nt_leaf_lds(S, nt_mi(S)) && 8 * 16 * 68 * 4 <= nt_lds(S, MI), "LDS");
  constexpr int APL = BM * GR * 16, BPL = BN * GR * 16, STAGE = S * (APL + BPL);
  constexpr int IA = (BM * GR + 511) / 512, IB = BN * GR / 512;    // DMAs per wave, plane and slice
  const int NTL = (g.N + BN - 1) / BN, MTL = (r_hi - r_lo + BM - 1) / BM, active = NTL * MTL;
  // the tiles are dealt so that each XCD (workgroups go to the 8 XCDs in turn) takes a contiguous
  // run, in groups of 4 row tiles per column tile
  {
    const int full = active & ~7;
    if (lid < full) lid = (lid & 7) * (full >> 3) + (lid >> 3);
  }
  constexpr int GM = 4;
  const int gi = lid / (GM * NTL), gm = min(GM, MTL - gi * GM), rem = lid - gi * GM * NTL;
  const int m0 = r_lo + (gi * GM + rem % gm) * BM, n0 = (rem / gm) * BN;
  const int nr = min(BM, r_hi - m0), nc = min(BN, g.N - n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm = wave / WN, wn = wave % WN, l16 = lane & 15, lq = lane >> 4;
  // steps and parents of the tile's rows, for the epilogue (read after the barriers of the K loop)
  if (EPI != NT_XW && tid < nr) {
    s_row[tid] = g.order[m0 + tid];
    if (EPI == NT_LEAF) s_par[tid] = g.opar[m0 + tid];
  }
  const uint16_t* A = g.A + (size_t)(m0 - g.lo) * g.lda;
  const uint16_t* Bp = g.B + (size_t)n0 * g.ldb;

  auto swz = [](int row) { return GR == 4 ? (row >> 1) & 3 : row & 7; };
  // the lane's row and granule are the same for every DMA of the block up to a row offset
  const int rl = lane / GR;
  // the DMAs of a slice with part = (index of the DMA) % parts
  auto issue = [&](int k0, int buf, int part, int parts) {
    unsigned char* st = sm + buf * STAGE;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const rsrc_t ra = make_rsrc(A + s * g.aplane, (size_t)nr * g.lda * 2);
      const rsrc_t rb = make_rsrc(Bp + s * g.bplane, (size_t)nc * g.ldb * 2);
#pragma unroll
      for (int i = 0; i < IA; ++i) {
        if ((s * (IA + IB) + i) % parts != part) continue;
        const int q = i * 8 + wave, row = q * (64 / GR) + rl, k = k0 + 8 * ((lane % GR) ^ swz(row));
        if (BM * GR % 512 != 0 && q * 64 >= BM * GR) continue;
        bdma16(ra, (row < nr && k < g.K) ? (uint32_t)(row * g.lda + k) * 2u : kOOB, 0u, lds_addr(st + s * APL + q * 1024));
      }
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        if ((s * (IA + IB) + IA + i) % parts != part) continue;
        const int q = i * 8 + wave, row = q * (64 / GR) + rl, k = k0 + 8 * ((lane % GR) ^ swz(row));
        bdma16(rb, (row < nc && k < g.K) ? (uint32_t)(row * g.ldb + k) * 2u : kOOB, 0u,
               lds_addr(st + S * APL + s * BPL + q * 1024));
      }
    }
  };

  // what the sums start from
  auto init = [&](int i, int j) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if constexpr (PRE) {
      const int m = 16 * (MI * wm + i) + l16, n = n0 + 16 * (NJ * wn + j) + 4 * lq;
      if (m < nr && n < g.N) v = *(const f32x4*)(g.C + (size_t)(m0 + m) * g.ldc + n);
    }
    return v;
  };
  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = init(i, j);
  if (!PRE || g.K > 0) issue(0, 0, 0, 1);
  int buf = 0;
  for (int k0 = 0; k0 < g.K; k0 += BK, buf ^= 1) {
    wait_vm<0>();
    __syncthreads();                                   // this slice landed, the other stage is free
    const bool more = k0 + BK < g.K;
    const unsigned char* st = sm + buf * STAGE;
#pragma unroll
    for (int kc = 0; kc < BK / 32; ++kc) {
      bf16x8 a[MI][S], b[NJ][S];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int r = 16 * (MI * wm + i) + l16;
#pragma unroll
        for (int s = 0; s < S; ++s) a[i][s] = *(const bf16x8*)(st + s * APL + (r * GR + ((4 * kc + lq) ^ swz(r))) * 16);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int r = 16 * (NJ * wn + j) + l16;
#pragma unroll
        for (int s = 0; s < S; ++s)
          b[j][s] = *(const bf16x8*)(st + S * APL + s * BPL + (r * GR + ((4 * kc + lq) ^ swz(r))) * 16);
      }
      tile_step<S, MI, NJ>(a, b, acc, [&](int i) {
        if (kc == 0 && more) issue(k0 + BK, buf ^ 1, i, MI);
      });
    }
  }
  __syncthreads();                                     // the stages are free

  float* ws = reinterpret_cast<float*>(sm) + wave * (16 * 68);   // 16 rows x 64 columns (+ 4) of this wave
  if constexpr (S == 3) {
    // (rows and columns past the tile's: the last ones', whose results nobody reads)
    redo_nan<MI, NJ>(acc, 0, g.K, init, [&](int k, bf16x8 (&a)[MI], bf16x8 (&b)[NJ]) {
      const int kl = min(k + 8 * lq, g.K - 8);
      const bool in = k + 8 * lq < g.K;
#pragma unroll
      for (int i = 0; i < MI; ++i) a[i] = *(const bf16x8*)(A + (size_t)min(16 * (MI * wm + i) + l16, nr - 1) * g.lda + kl);
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        b[j] = *(const bf16x8*)(Bp + (size_t)min(16 * (NJ * wn + j) + l16, nc - 1) * g.ldb + kl);
        if (!in) b[j] = bf16x8{};
      }
      if (!in)
#pragma unroll
        for (int i = 0; i < MI; ++i) a[i] = bf16x8{};
    });
  }

  float bias[NJ][4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + 16 * (NJ * wn + j) + 4 * lq + q;
      bias[j][q] = (EPI != NT_DX && g.bias && n < g.N) ? g.bias[perm_to_orig(n, g.H)] : 0.f;
    }

  if constexpr (EPI == NT_LEAF) {
    // a lane's four columns are the four gates of one unit: the cell runs on the accumulators,
    // h and c go through LDS and out as whole 4 BN / 4-byte row pieces
    // (row stride UN + 4 words: the 16 rows x 4 units that a wave writes at once fall into 64 banks)
    constexpr int UN = BN / 4, ULD = UN + 4;
    float* hs = reinterpret_cast<float*>(sm);
    float* cs = hs + BM * ULD;
    const int H = g.H;
    // h U and c of the parents: the loads of PD row tiles are in flight at a time (the compiler's own
    // order waited for a parent's index and then its rows, row tile by row tile)
    constexpr int PD = MI < 3 ? MI : 3;
    f32x4 hu[PD][NJ];
    float cp[PD][NJ];
    auto fetch = [&](int i) {
      const int par = s_par[min(16 * (MI * wm + i) + l16, nr - 1)];
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int u = min(n0 / 4 + 4 * (NJ * wn + j) + lq, H - 1);
        hu[i % PD][j] = *(const f32x4*)(g.hu + (size_t)par * (4 * H) + 4 * u);
        cp[i % PD][j] = g.cn[(size_t)par * H + u];
      }
    };
#pragma unroll
    for (int i = 0; i < PD; ++i) fetch(i);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int r = 16 * (MI * wm + i) + l16;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int ul = 4 * (NJ * wn + j) + lq;
        const f32x4 x = hu[i % PD][j];
        const float gi = sigmoidf_(acc[i][j][0] + bias[j][0] + x[0]);
        const float gf = sigmoidf_(acc[i][j][1] + bias[j][1] + x[1]);
        const float gg = tanhf_(acc[i][j][2] + bias[j][2] + x[2]);
        const float go = sigmoidf_(acc[i][j][3] + bias[j][3] + x[3]);
        const float c = gf * cp[i % PD][j] + gi * gg;
        hs[r * ULD + ul] = canon_nan(go * tanhf_(c));
        cs[r * ULD + ul] = c;
      }
      if (i + PD < MI) fetch(i + PD);
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    const int uw = min(UN, H - n0 / 4);                // units of this block
    const bool vec = (H & 3) == 0 && ((((uintptr_t)g.hcell) | ((uintptr_t)g.ccell)) & 15u) == 0;
    for (int e = tid; e < nr * (UN / 4); e += 512) {
      const int r = e / (UN / 4), v = (e % (UN / 4)) * 4;
      if (v >= uw) continue;
      const size_t o = (size_t)s_row[r] * H + n0 / 4 + v;
      const f32x4 h4 = *(const f32x4*)&hs[r * ULD + v], c4 = *(const f32x4*)&cs[r * ULD + v];
      if (vec) {
        __builtin_nontemporal_store(h4, (f32x4*)(g.hcell + o));
        __builtin_nontemporal_store(c4, (f32x4*)(g.ccell + o));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (v + q < uw) {
            g.hcell[o + q] = h4[q];
            g.ccell[o + q] = c4[q];
          }
      }
    }
  } else {
    // each wave turns 16 rows x 64 columns at a time into 256-byte row pieces through LDS
    const bool vec = (g.ldc & 3) == 0 && (((uintptr_t)g.C) & 15u) == 0;
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *(f32x4*)&ws[l16 * 68 + j * 16 + 4 * lq] =
            f32x4{acc[i][j][0] + bias[j][0], acc[i][j][1] + bias[j][1], acc[i][j][2] + bias[j][2],
                  acc[i][j][3] + bias[j][3]};
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * e + (lane >> 4), m = 16 * (MI * wm + i) + r, n = n0 + 64 * wn + 4 * l16;
        if (m >= nr) continue;
        const f32x4 v = *(const f32x4*)&ws[r * 68 + 4 * l16];
        float* dst = g.C + (size_t)(EPI == NT_DX ? s_row[m] : m0 + m) * g.ldc + n;
        if (vec && n + 3 < g.N) {
          *(f32x4*)dst = v;
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (n + q < g.N) dst[q] = v[q];
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

template <int S, int EPI, bool PRE>
__global__ void __launch_bounds__(512, 2) k_nt(NtArgs g) {
  extern __shared__ __align__(16) unsigned char sm[];
  __shared__ int s_row[256], s_par[256];
  constexpr int BN = nt_bn(S), Q = nt_mi(S) / 4;
  // rows in use (the number of push nodes is known on the device only) and the row tile: one
  // workgroup per CU, so the time is the rounds of 256 tiles times a tile's row tiles plus what a
  // K step costs besides its products (about three quarters of a quarter tile: slices in flight,
  // the barrier, B fragments).
  // With 256 rows alone the dx product of 18 k nodes x 256 inputs ran on 144 CUs (176 us, now 141),
  // that of 2.2 k nodes x 128 inputs on 9 (73 us, now 25).
  if (EPI == NT_DX && !has_plan(g.ctl, g.key)) return;
  const int P = (int)g.ctl[CTL_NPUSHF];
  const int r_lo = g.leaves ? max(g.lo, P) : g.lo, r_hi = g.leaves ? g.hi : min(g.hi, P);
  const int NTL = (g.N + BN - 1) / BN, R = max(r_hi - r_lo, 0);
  int sel = 4, best = 1 << 30, active = 0;
#pragma unroll
  for (int m = 4; m >= 1; --m) {
    const int bm = nt_bm(S, m * Q), tiles = NTL * ((R + bm - 1) / bm), cost = (tiles + 255) / 256 * (4 * m + 3);
    if ((m == 4 || tiles < (int)gridDim.x) && cost < best) {
      sel = m;
      best = cost;
      active = tiles;
    }
  }
  const int lid = (int)blockIdx.x;
  if (lid >= active) {
    // dx is exactly 0 on the leaves: the blocks without a tile clear those rows, 16 lanes a row
    // (behind the products, where the last tiles leave CUs idle)
    if constexpr (EPI == NT_DX) {
      const int per = ((int)gridDim.x - active) * 32;
      const bool vec = (g.N & 3) == 0 && (((uintptr_t)g.C) & 15u) == 0;
      for (int i = P + (lid - active) * 32 + (int)(threadIdx.x >> 4); i < g.N0; i += per) {
        float* dst = g.C + (size_t)g.order[i] * g.ldc;
        if (vec)
          for (int n = 4 * (threadIdx.x & 15); n < g.N; n += 64) *(f32x4*)(dst + n) = f32x4{0.f, 0.f, 0.f, 0.f};
        else
          for (int n = threadIdx.x & 15; n < g.N; n += 16) dst[n] = 0.f;
      }
    }
    return;
  }
  switch (sel) {
    case 1: nt_tile<S, EPI, Q, PRE>(g, r_lo, r_hi, lid, sm, s_row, s_par); break;
    case 2: nt_tile<S, EPI, 2 * Q, PRE>(g, r_lo, r_hi, lid, sm, s_row, s_par); break;
    case 3: nt_tile<S, EPI, 3 * Q, PRE>(g, r_lo, r_hi, lid, sm, s_row, s_par); break;
    default: nt_tile<S, EPI, 4 * Q, PRE>(g, r_lo, r_hi, lid, sm, s_row, s_par); break;
  }
}

// dW | dU. Both operands are stored with the contraction index as rows, so a fragment is read from
// LDS by transposing reads (four k of a column per lane and read). Rows of a stage are whole block
// widths; granule c of row k sits at c ^ 2 p(k), p = k & 3 with bit 3 of k above it, so that the eight
// rows that half a wave reads at once fall into different banks.
// FAR: the state rows take more than a descriptor's 4 GiB (H of 1 or 2, T*B near 2^28): they are loaded
// with 64-bit addresses and stored to LDS.
template <int S, bool FAR>
__global__ void __launch_bounds__(512, 2) k_tn(TnArgs g) {
  constexpr int MI = nt_mi(S), BM = nt_bm(S, MI), BN = nt_bn(S), BK = nt_bk(S, MI);
  constexpr int NJ = 4, WN = BN / (16 * NJ);
  constexpr int AG = BM / 8, BG = BN / 8;                          // granules per row
  constexpr int APL = BK * BM * 2, BPL = BK * BN * 2, STAGE = S * (APL + BPL);
  constexpr int IA = BK * AG / 512, IB = BK * BG / 512;
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char sm[];
  const int NTL = (g.H4 + BN - 1) / BN, MTL = g.xt + (g.H + BM - 1) / BM, per = NTL * MTL, nblk = per * g.splits;
  int lid = (int)blockIdx.x;
  {
    const int full = nblk & ~7;
    if (lid < full) lid = (lid & 7) * (full >> 3) + (lid >> 3);
  }
  const int z = lid / per, rem = lid % per, tm = rem % MTL, n0 = (rem / MTL) * BN;
  const bool is_x = tm < g.xt;
  const int m0 = (is_x ? tm : tm - g.xt) * BM, mlim = is_x ? g.I : g.H;   // columns of the operand array
  const int P = has_plan(g.ctl, g.key) ? (int)g.ctl[CTL_NPUSHF] : 0;
  const int chunk = ((P + g.splits - 1) / g.splits + BK - 1) / BK * BK;
  const int kbeg = min(P, z * chunk), kend = min(P, kbeg + chunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6);
  const int wm = wave / WN, wn = wave % WN, l16 = lane & 15, lq = lane >> 4;
  const uint16_t* A = is_x ? g.X : g.Hp;
  const size_t aplane = is_x ? g.xplane : g.hplane;
  const int lda = is_x ? g.ldx : g.ldh;

  auto sw2 = [](int k) { return 2 * ((k & 3) | (((k >> 3) & 1) << 2)); };
  // array row of each of this lane's A rows in a slice (h_prev: the parent, looked up a slice ahead)
  int arow[IA];
  auto rows = [&](int k0) {
#pragma unroll
    for (int i = 0; i < IA; ++i) {
      const int k = k0 + ((i * 8 + wave) * 64 + lane) / AG;
      int r = k;
      if (!is_x) {
        r = g.opar[min(k, P - 1)];
      }
      arow[i] = k < kend ? r : -1;
    }
  };
  auto issue = [&](int k0, int buf, int part, int parts) {
    unsigned char* st = sm + buf * STAGE;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      // x rows are consecutive: offsets from the slice's first row
      const uint16_t* ab = A + s * aplane + (is_x ? (size_t)k0 * lda : 0);
      const rsrc_t ra = make_rsrc(ab, (size_t)(is_x ? min(BK, kend - k0) : g.hrows) * lda * 2);
      const rsrc_t rb = make_rsrc(g.D + s * g.dplane + (size_t)k0 * g.ldd, (size_t)min(BK, kend - k0) * g.ldd * 2);
#pragma unroll
      for (int i = 0; i < IA; ++i) {
        if ((s * (IA + IB) + i) % parts != part) continue;
        const int L = (i * 8 + wave) * 64 + lane, kr = L / AG, col = m0 + 8 * ((L % AG) ^ sw2(kr));
        if constexpr (FAR) {
          if (!is_x) {
            uint4 v = {0u, 0u, 0u, 0u};
            if (arow[i] >= 0 && col < lda) v = *(const uint4*)(ab + (size_t)arow[i] * lda + col);
            *(uint4*)(st + s * APL + L * 16) = v;
            continue;
          }
        }
        const uint32_t row = (uint32_t)(is_x ? arow[i] - k0 : arow[i]);
        bdma16(ra, (arow[i] >= 0 && col < lda) ? (row * (uint32_t)lda + (uint32_t)col) * 2u : kOOB, 0u,
               lds_addr(st + s * APL + (i * 8 + wave) * 1024));
      }
#pragma unroll
      for (int i = 0; i < IB; ++i) {
        if ((s * (IA + IB) + IA + i) % parts != part) continue;
        const int L = (i * 8 + wave) * 64 + lane, kr = L / BG, col = n0 + 8 * ((L % BG) ^ sw2(kr));
        bdma16(rb, (k0 + kr < kend && col < g.ldd) ? (uint32_t)(kr * g.ldd + col) * 2u : kOOB, 0u,
               lds_addr(st + S * APL + s * BPL + (i * 8 + wave) * 1024));
      }
    }
  };

  f32x4 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // transposing reads: lane group lq holds k = 8 lq .. 8 lq + 7; a lane gives the address of row
  // 8 lq + l16 / 4, columns 4 (l16 % 4) of the tile, and gets column l16, four consecutive k
  const int kf = 8 * lq + (l16 >> 2), pf = sw2(kf);
  auto addr = [&](int tile, int G) { return kf * (G * 16) + (((2 * tile + ((l16 & 3) >> 1)) ^ pf) * 16) + (l16 & 1) * 8; };
  auto frag = [&](const unsigned char* p, int G) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * G * 16));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  if (kbeg < kend) {
    rows(kbeg);
    issue(kbeg, 0, 0, 1);
    rows(kbeg + BK);
  }
  int buf = 0;
  for (int k0 = kbeg; k0 < kend; k0 += BK, buf ^= 1) {
    wait_vm<0>();
    __syncthreads();
    const bool more = k0 + BK < kend;
    const unsigned char* st = sm + buf * STAGE;
#pragma unroll
    for (int kc = 0; kc < BK / 32; ++kc) {
      bf16x8 a[MI][S], b[NJ][S];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const unsigned char* p = st + kc * 32 * AG * 16 + addr(MI * wm + i, AG);
#pragma unroll
        for (int s = 0; s < S; ++s) a[i][s] = frag(p + s * APL, AG);
      }
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const unsigned char* p = st + S * APL + kc * 32 * BG * 16 + addr(NJ * wn + j, BG);
#pragma unroll
        for (int s = 0; s < S; ++s) b[j][s] = frag(p + s * BPL, BG);
      }
      tile_step<S, MI, NJ>(a, b, acc, [&](int i) {
        if (kc == 0 && more) issue(k0 + BK, buf ^ 1, i, MI);
      });
    }
    if (more) rows(k0 + 2 * BK);
  }
  if constexpr (S == 3) {
    redo_nan<MI, NJ>(acc, kbeg, kend, [](int, int) { return f32x4{0.f, 0.f, 0.f, 0.f}; }, [&](int k0, bf16x8 (&a)[MI], bf16x8 (&b)[NJ]) {
      uint16_t va[MI][8], vb[NJ][8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = min(k0 + 8 * lq + e, kend - 1);
        const bool in = k0 + 8 * lq + e < kend;
        const uint16_t* ar = A + (size_t)(is_x ? k : g.opar[k]) * lda;
        const uint16_t* dr = g.D + (size_t)k * g.ldd;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const uint16_t v = ar[min(m0 + 16 * (MI * wm + i) + l16, mlim - 1)];
          va[i][e] = in ? v : (uint16_t)0;
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const uint16_t v = dr[min(n0 + 16 * (NJ * wn + j) + l16, g.H4 - 1)];
          vb[j][e] = in ? v : (uint16_t)0;
        }
      }
#pragma unroll
      for (int i = 0; i < MI; ++i) __builtin_memcpy(&a[i], va[i], 16);
#pragma unroll
      for (int j = 0; j < NJ; ++j) __builtin_memcpy(&b[j], vb[j], 16);
    });
  }
  __syncthreads();
  float* ws = reinterpret_cast<float*>(sm) + wave * (16 * 68);
  float* out = g.part + (size_t)z * g.split_stride + (size_t)(is_x ? 0 : g.I) * g.H4;
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) *(f32x4*)&ws[l16 * 68 + j * 16 + 4 * lq] = acc[i][j];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = 4 * e + (lane >> 4), m = m0 + 16 * (MI * wm + i) + r, n = n0 + 64 * wn + 4 * l16;
      if (m < mlim && n < g.H4) *(f32x4*)(out + (size_t)m * g.H4 + n) = *(const f32x4*)&ws[r * 68 + 4 * l16];
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// dW [I][4H], dU [H][4H] and db [4H] in the caller's column order: the partials of k_tn, and of the
// groups for db, added in order. The blocks past n_red check the caller's top and ops: a producer
// index outside [-1, t], or an op that is a push where the forward's was not (or the reverse),
// raises CTL_BADIDX (no kernel of the backward takes an address from either).
__global__ void __launch_bounds__(256) k_reduce_grads(ReduceArgs a) {
  const int H = a.H, H4 = 4 * H, I = a.I;
  if ((int)blockIdx.x >= a.n_red) {
    if (!has_plan(a.ctl, a.key)) return;
    const size_t P = a.ctl[CTL_NPUSHF], n = (size_t)a.T * a.B, step = (size_t)(gridDim.x - a.n_red) * 256;
    bool bad = false;
    for (size_t i = (size_t)(blockIdx.x - a.n_red) * 256 + threadIdx.x; i < n; i += step) {
      const int s = a.top[i];
      bad |= s < -1 || s > (int)(i / a.B);
      bad |= (a.ops[a.order[i]] == 1) != (i < P);
    }
    if (bad) raise_badidx(a.ctl);
    return;
  }
  const size_t n_w = (size_t)I * H, n = n_w + (size_t)H * H + H;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)a.n_red * 256) {
    const size_t row = i / H;
    const int u = (int)(i - row * H);
    const bool bias = row == (size_t)(I + H);
    const float* src = bias ? a.db_part : a.part + row * H4;
    const size_t st = bias ? (size_t)H4 : a.stride;
    const int cnt = bias ? a.groups : a.splits;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (bias) {                                        // (up to 128 groups: compensated)
      f32x4 e = {0.f, 0.f, 0.f, 0.f};
      for (int z = 0; z < cnt; ++z) {
        const f32x4 v = *(const f32x4*)(src + (size_t)z * st + 4 * u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          float t = s[k], r = e[k];
          comp_add(t, r, v[k]);
          s[k] = t;
          e[k] = r;
        }
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = comp_sum(s[k], e[k]);
    } else {
      for (int z = 0; z < cnt; ++z) s += *(const f32x4*)(src + (size_t)z * st + 4 * u);
    }
    float* dst = bias ? a.db : (row < (size_t)I ? a.dW + row * H4 : a.dU + (row - I) * H4);
#pragma unroll
    for (int k = 0; k < 4; ++k) dst[(size_t)k * H + u] = s[k];
  }
}

template <int S, int EPI, bool PRE>
static hipError_t launch_nt_t(const NtArgs& g, hipStream_t st) {
  auto kern = k_nt<S, EPI, PRE>;
  constexpr size_t stages = nt_lds(S, nt_mi(S)), leaf = EPI == NT_LEAF ? nt_leaf_lds(S, nt_mi(S)) : 0;
  constexpr int shm = (int)(leaf > stages ? leaf : stages);
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, shm);
  if (e != hipSuccess) return e;
  // the grid covers the static range in the largest tiles, or in the smallest up to two rounds of the
  // chip; blocks past the rows in use leave at once (NT_DX: clear the leaves' rows; one row tile
  // more, so that some block does where the push nodes fill every tile)
  auto count = [&](int bm) { return ((g.N + nt_bn(S) - 1) / nt_bn(S)) * ((g.hi - g.lo + bm - 1) / bm + (EPI == NT_DX ? 1 : 0)); };
  const int tiles = std::max(count(nt_bm(S, nt_mi(S))), std::min(count(nt_bm(S, nt_mi(S) / 4)) + 1, 513));
  hipLaunchKernelGGL(kern, dim3(tiles), dim3(512), shm, st, g);
  return hipGetLastError();
}
hipError_t launch_nt(const NtArgs& g, int S, int epi, hipStream_t st) {
  if (g.hi <= g.lo) return hipSuccess;
#define CASE(S_, E_, P_) \
  if (S == S_ && epi == E_ && (g.pre != 0) == P_) return launch_nt_t<S_, E_, P_>(g, st);
  CASE(1, NT_XW, false) CASE(1, NT_LEAF, false) CASE(1, NT_DX, false) CASE(1, NT_XW, true) CASE(1, NT_LEAF, true)
  CASE(3, NT_XW, false) CASE(3, NT_LEAF, false) CASE(3, NT_DX, false) CASE(3, NT_XW, true) CASE(3, NT_LEAF, true)
#undef CASE
  return hipErrorInvalidValue;
}
template <int S, bool FAR>
static hipError_t launch_tn_t(const TnArgs& g, hipStream_t st) {
  auto kern = k_tn<S, FAR>;
  constexpr int shm = (int)nt_lds(S, nt_mi(S));
  const hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, shm);
  if (e != hipSuccess) return e;
  const int tiles = ((g.H4 + nt_bn(S) - 1) / nt_bn(S)) * (g.xt + (g.H + nt_bm(S, nt_mi(S)) - 1) / nt_bm(S, nt_mi(S)));
  hipLaunchKernelGGL(kern, dim3(tiles * g.splits), dim3(512), shm, st, g);
  return hipGetLastError();
}
hipError_t launch_tn(const TnArgs& g, int S, hipStream_t st) {
  const bool far = tn_far(g.hrows, g.ldh);
  if (S == 3) return far ? launch_tn_t<3, true>(g, st) : launch_tn_t<3, false>(g, st);
  return far ? launch_tn_t<1, true>(g, st) : launch_tn_t<1, false>(g, st);
}
