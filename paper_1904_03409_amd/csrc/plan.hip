// Op validation, pointer scan, producer trace and the level schedule (levels.h) of the stack
// recurrence, in one launch. One workgroup per group; a wave walks one batch element, 64 steps
// at a time:
//  * the pointer is a scan: a valid op maps p to max(p + op, 0) (a pop at p = 0 is reported and
//    walked as a hold, an op outside {-1, 0, 1} too), and such maps compose to p -> max(p + A, M);
//  * the step that made the state at the pointer is the last push at that depth: among the 64
//    steps by comparing every step's depth with the pushes' (a loop over the pushes), before
//    them from the element's stack of producers.
// Walking 64 steps together costs about as much as walking two one after the other.
// Phases: (1) trace and pushes per depth, (2) a scan over (depth, element) for the first node id of
// each, (3) the walk again, now writing node ids, (4) for a backward, the numbers of the nodes with
// children.
#include "common.h"
#include "levels.h"

namespace {

// Exclusive scan over the workgroup of one value per thread; returns the total in *total.
__device__ __forceinline__ int block_excl(int v, int* s_w, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d, 64);
    if (lane >= d) incl += o;
  }
  __syncthreads();
  if (lane == 63) s_w[wave] = incl;
  __syncthreads();
  int base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) base += s_w[w];
    tot += s_w[w];
  }
  *total = tot;
  return base + incl - v;
}

struct Chunk {
  int op, pa, pb, jl, rank, rankc;   // op, depth after / before, last push lane <= this one at depth pa,
  bool push, later, valid;           // pushes before this lane at depth pa / pa + 1, a later push at pa
  uint64_t m_push;
};

// 64 steps from t0 of element b: p0 = the depth before them.
__device__ __forceinline__ Chunk walk_chunk(const int8_t* __restrict__ ops, int T, int B, int b, int t0, int p0) {
  const int lane = threadIdx.x & 63, t = t0 + lane;
  Chunk c;
  c.valid = t < T;
  c.op = c.valid ? (int)ops[(size_t)t * B + b] : 0;
  const int a = (c.op < -1 || c.op > 1) ? 0 : c.op;
  int A = a, M = 0;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int A2 = __shfl_up(A, d, 64), M2 = __shfl_up(M, d, 64);
    if (lane >= d) {
      M = max(M2 + A, M);
      A += A2;
    }
  }
  c.pa = max(p0 + A, M);
  const int prev = __shfl_up(c.pa, 1, 64);
  c.pb = lane ? prev : p0;
  c.push = a == 1;
  c.m_push = __ballot(c.push);
  c.jl = -1;
  c.rank = c.rankc = 0;
  c.later = false;
  for (uint64_t m = c.m_push; m; m &= m - 1) {
    const int j = __builtin_ctzll(m);
    const int dj = __builtin_amdgcn_readlane(c.pa, j);
    if (dj == c.pa) {
      if (lane >= j) c.jl = j;
      c.rank += j < lane ? 1 : 0;
      c.later |= j > lane;
    }
    c.rankc += (dj == c.pa + 1 && j < lane) ? 1 : 0;
  }
  return c;
}

}  // namespace

template <bool LDS>
__global__ void __launch_bounds__(1024) k_plan(PlanArgs a) {
  extern __shared__ int s_dyn[];
  __shared__ int s_w[16], s_max, s_before, s_total;
  const int T = a.T, B = a.B, G = a.G, cap = a.cap, N0 = T * B;
  const int g = blockIdx.x, Bg = lev_bg(B, G, g), goff = lev_goff(B, G, g);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwv = blockDim.x >> 6;
  int* base = LDS ? s_dyn + (size_t)wave * 2 * cap : a.walk + ((size_t)g * nwv + wave) * 2 * cap;
  int* stk = base;                                   // producer (phase 1: step, phase 3: node) by depth
  int* num = base + cap;                             // phase 1: pushes by depth; phase 3: next node id by depth
  int32_t* e_max = a.elem;
  int32_t* e_push = a.elem + B;
  int32_t* e_leaf = a.elem + 2 * (size_t)B;
  if (tid == 0) s_max = s_before = s_total = 0;
  __syncthreads();

  // pushes of the groups before this one, and all pushes (a push is always valid)
  {
    int before = 0, total = 0;
    const size_t n = (size_t)N0;
    if ((B & 3) == 0 && ((uintptr_t)a.ops & 3u) == 0) {
      const uint32_t* o4 = (const uint32_t*)a.ops;
      const int step = (int)(((size_t)blockDim.x * 4) % B);
      int b = (int)(((size_t)tid * 4) % B);
#pragma unroll 8
      for (size_t i = tid; i < n / 4; i += blockDim.x) {
        const uint32_t v = o4[i];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const int is = ((v >> (8 * k)) & 0xffu) == 1u ? 1 : 0;
          total += is;
          before += is && (b + k) % G < g ? 1 : 0;
        }
        b += step;
        if (b >= B) b -= B;
      }
    } else {
      const int step = (int)(blockDim.x % B);
      int b = tid % B;
#pragma unroll 8
      for (size_t i = tid; i < n; i += blockDim.x) {
        const int is = a.ops[i] == 1 ? 1 : 0;
        total += is;
        before += is && b % G < g ? 1 : 0;
        b += step;
        if (b >= B) b -= B;
      }
    }
#pragma unroll
    for (int d = 32; d; d >>= 1) {
      before += __shfl_down(before, d, 64);
      total += __shfl_down(total, d, 64);
    }
    if (lane == 0) {
      atomicAdd(&s_before, before);
      atomicAdd(&s_total, total);
    }
  }

  // phase 1
  for (int i = wave; i < Bg; i += nwv) {
    const int b = g + G * i;
    for (int d = lane; d < cap; d += 64) num[d] = 0;
    if (lane == 0) {
      stk[0] = -1;
      a.ptr[b] = 0;
    }
    __threadfence_block();
    int p0 = 0, maxd = 0, npush = 0, first_bad = 0x7fffffff, first_uf = 0x7fffffff;
    for (int t0 = 0; t0 < T; t0 += 64) {
      const Chunk c = walk_chunk(a.ops, T, B, b, t0, p0);
      const int t = t0 + lane;
      const int tp = c.jl >= 0 ? t0 + c.jl : stk[c.pa];
      __threadfence_block();
      if (c.push && !c.later) stk[c.pa] = t;
      if (c.push) atomicAdd(&num[c.pa], 1);
      __threadfence_block();
      if (c.valid) {
        a.ptr[(size_t)(t + 1) * B + b] = c.pa;
        a.top[(size_t)t * B + b] = tp;
      }
      const uint64_t mb = __ballot(c.valid && (c.op < -1 || c.op > 1)), mu = __ballot(c.valid && c.op == -1 && c.pb == 0);
      if (mb && first_bad == 0x7fffffff) first_bad = t0 + __builtin_ctzll(mb);
      if (mu && first_uf == 0x7fffffff) first_uf = t0 + __builtin_ctzll(mu);
      npush += __popcll(c.m_push);
      maxd = max(maxd, c.push ? c.pa : 0);
      p0 = __builtin_amdgcn_readlane(c.pa, 63);
    }
#pragma unroll
    for (int d = 32; d; d >>= 1) maxd = max(maxd, __shfl_xor(maxd, d, 64));
    for (int d = 1 + lane; d <= maxd; d += 64) a.cnt[(size_t)b * cap + d] = num[d];
    if (lane == 0) {
      e_max[b] = maxd;
      e_push[b] = npush;
      atomicMax(&s_max, maxd);
      if (first_bad != 0x7fffffff || first_uf != 0x7fffffff)
        atomicMin((int*)&a.ctl[CTL_STATUS], b * 8 + (first_uf < first_bad ? ST_EUNDERFLOW : ST_EOPS));
    }
  }
  __syncthreads();
  const int D = s_max, P = s_total;
  if (tid == 0) {
    a.ix.gmax[g] = D;
    if (g == 0) {
      a.ctl[CTL_NPUSHF] = (uint32_t)P;
      a.ctl[CTL_KEY] = (uint32_t)a.key;
      a.ctl[CTL_KEY + 1] = (uint32_t)(a.key >> 32);
    }
  }

  // phase 2: first node id of (depth, element), depth-major; leaf offset of each element
  {
    const size_t n = (size_t)D * Bg, per = (n + blockDim.x - 1) / blockDim.x;
    const size_t f0 = (size_t)tid * per, f1 = f0 + per < n ? f0 + per : n;
    int sum = 0;
    for (size_t f = f0; f < f1; ++f) {
      const int d = 1 + (int)(f / Bg), b = g + G * (int)(f % Bg);
      sum += d <= e_max[b] ? a.cnt[(size_t)b * cap + d] : 0;
    }
    int total;
    int off = s_before + block_excl(sum, s_w, &total);
    int32_t* loff = a.ix.loff + (size_t)g * (T + 4);
    for (size_t f = f0; f < f1; ++f) {
      const int d = 1 + (int)(f / Bg), i = (int)(f % Bg), b = g + G * i;
      const int v = d <= e_max[b] ? a.cnt[(size_t)b * cap + d] : 0;
      a.cnt[(size_t)b * cap + d] = off;
      if (i == 0) loff[d] = off;
      off += v;
    }
    const int end = s_before + total;
    for (int i = tid; i < Bg; i += blockDim.x) a.cnt[(size_t)(g + G * i) * cap + D + 1] = end;
    if (tid == 0) loff[D + 1] = loff[D + 2] = end;
  }
  {
    const int per = (Bg + (int)blockDim.x - 1) / (int)blockDim.x;
    const int i0 = tid * per, i1 = min(i0 + per, Bg);
    int sum = 0, total;
    for (int i = i0; i < i1; ++i) sum += T - e_push[g + G * i];
    int off = P + T * goff - s_before + block_excl(sum, s_w, &total);
    for (int i = i0; i < i1; ++i) {
      e_leaf[g + G * i] = off;
      off += T - e_push[g + G * i];
    }
  }
  __threadfence_block();
  __syncthreads();

  // phase 3
  for (int i = wave; i < Bg; i += nwv) {
    const int b = g + G * i, init = N0 + goff + i;
    for (int d = 1 + lane; d <= D + 1; d += 64) num[d] = a.cnt[(size_t)b * cap + d];
    if (lane == 0) {
      stk[0] = init;
      a.ix.cs[init] = a.cnt[(size_t)b * cap + 1];
    }
    __threadfence_block();
    int p0 = 0, cur = init, slot = init, leaf = e_leaf[b];
    const uint64_t below = (1ull << lane) - 1ull;
    for (int t0 = 0; t0 < T; t0 += 64) {
      const Chunk c = walk_chunk(a.ops, T, B, b, t0, p0);
      const int r = (t0 + lane) * B + b;
      const int id = c.push ? num[c.pa] + c.rank : 0;
      const int kids = c.push ? num[c.pa + 1] + c.rankc : 0;
      const int old = stk[c.pa], mine = __shfl(id, max(c.jl, 0), 64);
      const int topid = c.jl >= 0 ? mine : old;
      __threadfence_block();
      if (c.push && !c.later) stk[c.pa] = id;
      if (c.push) atomicAdd(&num[c.pa], 1);
      __threadfence_block();
      const int up = __shfl_up(topid, 1, 64), par = lane ? up : cur;
      const uint64_t m_leaf = __ballot(c.valid && !c.push);
      // the slot of a step's upstream gradient: a push opens its node's first interval, a pop the
      // interval of the parent that follows the popped node; other steps continue the last one
      const bool pop = c.valid && c.op == -1 && c.pb > 0;
      const uint64_t m_open = __ballot(c.push || pop) & (below | (1ull << lane));
      const int open = c.push ? id : N0 + B + par;
      const int from = __shfl(open, m_open ? 63 - __builtin_clzll(m_open) : 0, 64);
      const int sl = m_open ? from : slot;
      if (c.push) {
        a.ix.order[id] = r;
        a.ix.opar[id] = par;
        a.ix.cs[id] = kids;
      } else if (c.valid) {
        const int pos = leaf + __popcll(m_leaf & below);
        a.ix.order[pos] = r;
        a.ix.opar[pos] = par;
      }
      if (c.valid && a.key) a.ix.gslot[r] = sl;
      leaf += __popcll(m_leaf);
      p0 = __builtin_amdgcn_readlane(c.pa, 63);
      cur = __builtin_amdgcn_readlane(topid, 63);
      slot = __builtin_amdgcn_readlane(sl, 63);
    }
    if (!a.key) continue;
    // nodes still on the stack were never popped (marked here, resolved in phase 4)
    __threadfence_block();
    for (int d = 1 + lane; d <= p0; d += 64) a.ix.opar[stk[d]] = ~stk[d - 1];
  }
  if (!a.key) return;
  __threadfence_block();
  __syncthreads();

  // phase 4: internal numbers, in node order (initial states first)
  const int32_t* loff = a.ix.loff + (size_t)g * (T + 4);
  const int first = s_before, end = loff[D + 1], n = Bg + end - first, ibase = first + goff;
  auto node = [&](int q) { return q < Bg ? N0 + goff + q : first + q - Bg; };
  int run = ibase;
  for (int q0 = 0; q0 < n; q0 += blockDim.x) {
    const int q = q0 + tid;
    int flag = 0, c0 = 0;
    if (q < n) {
      c0 = a.ix.cs[node(q)];
      const int c1 = q + 1 == Bg ? loff[2] : (q + 1 == n ? end : a.ix.cs[node(q + 1)]);
      flag = c1 > c0 ? 1 : 0;
    }
    int total;
    const int idx = run + block_excl(flag, s_w, &total);
    if (q < n) a.ix.cidx[node(q)] = flag ? idx : ~idx;
    if (flag) a.ix.ics[idx] = c0;
    run += total;
  }
  if (tid == 0) a.ix.ics[run] = end;
  __threadfence_block();
  __syncthreads();
  int32_t* ioff = a.ix.ioff + (size_t)g * (T + 4);
  for (int d = tid; d <= D + 1; d += blockDim.x) {
    const int q = d == 0 ? 0 : Bg + loff[d] - first;
    const int v = q < n ? a.ix.cidx[node(q)] : run;
    ioff[d] = q < n && v < 0 ? ~v : v;
  }
  for (int c = first + tid; c < end; c += blockDim.x) {
    const int po = a.ix.opar[c], k = a.ix.cidx[c];
    if (po < 0) a.ix.opar[c] = ~po;
    a.ix.kin[c] = 2 * (k < 0 ? -1 : k) + (po < 0 ? 0 : 1);
  }
}
template __global__ void k_plan<true>(PlanArgs);
template __global__ void k_plan<false>(PlanArgs);
