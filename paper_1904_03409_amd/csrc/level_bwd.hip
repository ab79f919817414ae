// Backward recurrence over the level schedule (levels.h), from the deepest level up. Persistent,
// groups and unit ownership as in the forward.
//
// A node's gradient is complete when its children are done: dh = its interval sums (k_prep_bwd) + what
// its children send, dc likewise; the cell backward then gives its gate gradient dA (a push only;
// every other step's is 0) and dc f for its parent. The parent needs (sum of the children's dA) U^T:
// the sum first, so one product per node with children. Per level:
//  1. the cell of every node (64 at a time through LDS, the next ones' operands in flight), the
//     sums of dA, dc f and the interval gradients per parent, in node order; the dA sums go to
//     the exchange rows sx as recurrent planes (split.h);
//  2. a group barrier;
//  3. the parents' rows, 16 at a time: each wave copies its eighth of the 4H columns into LDS (LDS
//     DMA, the next rows in flight behind the products) and contracts it with its slice of U^T
//     (registers) for the workgroup's 32 units; the eight waves' partials are added in LDS in
//     wave order.
// Against exchanging partial sums (each workgroup contracting its own 128 columns for all units)
// this writes 1 / NW of the bytes, so the exchange stays in the XCD's L2: 5.2 ms that way at
// B = 1024, H = 1024 (bf16).
#include "common.h"
#include "levels.h"
#include "split.h"

// CLK: with the stamps of dims.step_clock. (A kernel of its own: the scalar registers spill, and every
// argument kept for later costs reads back on the chain of a level. deep, H = 512: 4266 us with
// the stamps' branches, 4064 without.)
template <int NP, int KS, bool CLK>
__global__ void __launch_bounds__(kLevThreads, 2) k_lev_bwd(LevBwdArgs a) {
  constexpr int S = NP == 2 ? 3 : 1;
  constexpr int KH = KS / 2, SG = KH * 4;                   // K chunks and 16-byte granules of a wave's row slice
  constexpr int WREG = NP * KH * 1024;                      // bytes of a wave's 16 row slices
  constexpr int kids = lev_bwd_kids(NP, KS), NI = kids / 16, NQ = kLevPars / 16;
  constexpr int RLD = 36;
  constexpr bool kDefer = NP == 1 && KS >= 24;              // (put_da)
  // the next level's first operands are fetched behind the first rows of the exchange (in one queue
  // with them, the rows would wait for HBM); with the most registers in use, ahead of the barrier
  constexpr bool kLate = NP * KS < 32 || NP == 1;
  extern __shared__ __align__(16) unsigned char lsm[];
  f32x4* ch_a = reinterpret_cast<f32x4*>(lsm);                                // [kids][32] dA of a child
  float2* ch_c = reinterpret_cast<float2*>(lsm + kids * kLevUnits * 16);      // [kids][32] dc f, interval gradient
  float* red = reinterpret_cast<float*>(lsm + lev_bwd_region(NP, KS));        // [8][16][RLD] partials of the waves
  float* keep = red + 8 * 16 * RLD;                         // [2][2][kLevKeep][32] eg and dcs of a level's first nodes
  __shared__ int s_g, s_w, s_flag, s_ics[kLevPars + 1];
  if (!has_plan(a.ctl, a.key)) return;
  claim_group_slot(a.ctl + CTL_XCC_SLOT_B, a.G, a.NW, &s_g, &s_w);
  const int g = uni(s_g), w = uni(s_w);
  if (g < 0) return;
  const int T = a.T, B = a.B, H = a.H, H4 = 4 * H, H4s = a.H4s, N0 = a.N0, NW = a.NW;
  const int tid = threadIdx.x, lane = tid & 63, wave = uni(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int uu = tid & 31, u = 32 * w + uu, kk = tid >> 5;
  const bool u_ok = u < H;
  const bool solo = KS == 2 && NW == 1;                     // the group is this workgroup: no exchange with others
  uint32_t* bar = a.ctl + CTL_BAR_B + 16 * g;
  const int n_init = N0 + lev_goff(B, a.G, g), Bg = lev_bg(B, a.G, g);
  const int32_t* ioff = a.ix.ioff + (size_t)g * (T + 4);
  const int D = uni(a.ix.gmax[g]);

  uint4 ub[2][KH][NP];
  {
    const uint4* src = a.ub + (size_t)(w * 8 + wave) * 2 * KH * NP * 64 + lane;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int c = 0; c < KH; ++c)
#pragma unroll
        for (int s = 0; s < NP; ++s) ub[t][c][s] = src[((t * KH + c) * NP + s) * 64];
  }
  const float ui = NP == 2 ? a.uinv[u] : 1.f;               // inverse scale of this thread's unit

  // sums over this thread's nodes for the bias gradient (comp_add)
  float db[4] = {0.f, 0.f, 0.f, 0.f}, dbe[4] = {0.f, 0.f, 0.f, 0.f};
  // operands of a pass of children that do not depend on other levels
  struct Pre { f32x4 ga; float cp, gf, ih; int kin; };
  Pre it[NI];
  const float* gi = a.gf + (size_t)(N0 + B) * H;            // interval sums after a popped node
  auto prefetch = [&](int cb, int c1) {
    const int ot = opaque(tid), ou = 32 * w + (ot & 31);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int c = cb + (ot >> 5) + 16 * j;
      if (c < c1 && ou < H) {
        const uint32_t o = 4u * (uint32_t)(c * H + ou);
        it[j].ga = __builtin_nontemporal_load((const f32x4*)(a.stash + (size_t)c * H4 + 4 * ou));
        it[j].cp = *at32(a.cpn, o);
        it[j].gf = *at32(a.gf, o);
        it[j].ih = *at32(gi, o);
        it[j].kin = *at32(a.ix.kin, 4u * c);
      }
    }
  };
  // wall-clock stamps of a level: top, sums stored, all sums there, gradients of the parents done
  auto stamp = [&](int d, int k) {
    if (CLK && tid == 0) a.clk[((size_t)blockIdx.x * T + d - 1) * 4 + k] = wall_clock64();
  };
  // dA of a child: the planes that dW, dU and dx read, and the bias gradient. Nobody waits for these
  // stores. H > 512: a pass that is not the level's last leaves it to the next one, which does it from
  // LDS while its own operands are on their way (H = 1024, levels of 170 nodes: 50.0 -> 46.7 us a
  // level by the step clock). The last pass does it in place (from LDS it costs 0.2 us a level, and after the barrier's
  // arrival 0.4: the next rows queue behind the stores); so do the others, whose levels gained 1% at
  // most from it (H = 512) or lost up to 4% (H = 300).
  auto put_da = [&](int c, int ou, const f32x4& da) {
    bf16_t p[4][S];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      comp_add(db[q], dbe[q], da[q]);
      split_bf16<S>(da[q], p[q]);
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      bf16_t* dst = (bf16_t*)((char*)(a.dap + s * a.dplane) + lev_da_off<NP>(c, H4s, ou));
      *(uint2*)dst = uint2{(uint32_t)p[0][s] | ((uint32_t)p[1][s] << 16), (uint32_t)p[2][s] | ((uint32_t)p[3][s] << 16)};
      if (ou == H - 1 && (H & 1)) *(uint2*)(dst + 4) = uint2{0u, 0u};   // row padding
    }
  };
  auto flush = [&](int cb, int ce) {
    const int ot = opaque(tid);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int k = (ot >> 5) + 16 * j;
      if (cb + k < ce && 32 * w + (ot & 31) < H) put_da(cb + k, 32 * w + (ot & 31), ch_a[k * 32 + (ot & 31)]);
    }
  };
  bool stop = false;
  // Level d: parents are the internal nodes [i0, i1) of level d - 1, whose children are the nodes
  // [c0, cend) of level d, whose own internal numbers start at i1. The first pass's operands and
  // the first parents' child ranges (s_ics) are fetched a level ahead, i0 two levels ahead.
  int i0 = 0, i1 = 0, c0 = 0, cend = 0, ics_r = 0, i0_next = 0;
  auto prefetch_ics = [&](int ib, int i1) { return ib + min((int)opaque(tid), kLevPars) <= i1 ? a.ix.ics[ib + min((int)opaque(tid), kLevPars)] : 0; };
  if (D > 0) {
    i0 = uni(ioff[D - 1]);
    i1 = uni(ioff[D]);
    c0 = uni(a.ix.ics[i0]);
    cend = uni(a.ix.ics[i1]);
    i0_next = D > 1 ? ioff[D - 2] : 0;
    ics_r = prefetch_ics(i0, i1);
    prefetch(c0, cend);
  }
  for (int d = D; d >= 1; --d) {
    stamp(d, 0);
    float* eg_in = keep + (d & 1) * (2 * kLevKeep * 32);
    float* eg_out = keep + (~d & 1) * (2 * kLevKeep * 32);
    int cs = c0, fb = 0, fe = 0;                            // children whose dA waits in LDS
    for (int ib = i0; ib < i1; ib += kLevPars) {
      const int ni = min(kLevPars, i1 - ib);
      if (ib > i0) {
        __syncthreads();                                    // (the last sums have read s_ics)
        ics_r = prefetch_ics(ib, i1);
      }
      if (tid <= kLevPars) s_ics[tid] = ics_r;
      const int c0 = cs, c1 = ib + kLevPars < i1 ? uni(a.ix.ics[ib + ni]) : cend;
      cs = c1;
      float sA[NQ][4], sc[NQ], sg[NQ];
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        sc[k] = sg[k] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) sA[k][q] = 0.f;
      }
      for (int cb = c0; cb < c1; cb += kids) {
        const bool defer = kDefer && cb + kids < cend;
        if constexpr (kDefer) flush(fb, fe);
        fb = cb;
        fe = defer ? min(cb + kids, c1) : cb;
        // cell backward of up to 64 (32) children
        {
          const int ot = opaque(tid), uu = ot & 31, u = 32 * w + uu;
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const int k = (ot >> 5) + 16 * j, c = cb + k;
            if (c < c1 && u < H) {
              const f32x4 ga = it[j].ga;
              const uint32_t o = 4u * (uint32_t)(c * H + u);
              float dh = it[j].gf, dc = 0.f, ih = 0.f, ic = 0.f;
              const int ci = it[j].kin >> 1;                // internal number
              const bool popped = it[j].kin & 1;            // (else no interval of the parent follows it)
              if (popped) ih = it[j].ih;
              if (a.gc) {
                dc = *at32(a.gc, o);
                if (popped) ic = *at32(a.gc + (size_t)(N0 + B) * H, o);
              }
              if (ci >= 0) {
                const int x = ci - i1;
                const bool near = x < kLevKeep;
                dh += near ? eg_in[x * 32 + uu] : a.eg[(size_t)ci * H + u];
                dc += near ? eg_in[(kLevKeep + x) * 32 + uu] : a.dcs[(size_t)ci * H + u];
              }
              const float tc = tanhf_(ga[1] * it[j].cp + ga[0] * ga[2]);   // (c as the forward computed it)
              const float dct = dc + dh * ga[3] * (1.f - tc * tc);
              const f32x4 da = {dct * ga[2] * ga[0] * (1.f - ga[0]), dct * it[j].cp * ga[1] * (1.f - ga[1]),
                                dct * ga[0] * (1.f - ga[2] * ga[2]), dh * tc * ga[3] * (1.f - ga[3])};
              ch_a[k * 32 + uu] = da;
              ch_c[k * 32 + uu] = float2{dct * ga[1] + ic, ih};
              if (!kDefer || !defer) put_da(c, u, da);
            }
            if (NP == 2 && KS > 8) __builtin_amdgcn_sched_barrier(0);   // (one node at a time: registers)
          }
        }
        // the next children of the level (passes end at a parent's last child)
        {
          const int nx = min(cb + kids, c1);
          if (nx < cend) prefetch(nx, nx < c1 ? c1 : cend);
        }
        __syncthreads();
        // sums per parent, children in node order
        {
          const int ot = opaque(tid), uu = ot & 31;
#pragma unroll
          for (int k = 0; k < NQ; ++k) {
            const int r = 32 * w + uu < H ? (ot >> 5) + 16 * k : kLevPars;   // (no sums past H)
            const int ka = r < ni ? s_ics[r] : 0, kb = r < ni ? s_ics[r + 1] : 0;
            for (int c = max(ka, cb); c < min(kb, cb + kids); ++c) {
              const f32x4 da = ch_a[(c - cb) * 32 + uu];
#pragma unroll
              for (int q = 0; q < 4; ++q) sA[k][q] += da[q];
              const float2 v = ch_c[(c - cb) * 32 + uu];
              sc[k] += v.x;
              sg[k] += v.y;
            }
          }
        }
        __syncthreads();
      }
      // the parents' sums: exchange rows (one scale per row and workgroup), dc, interval gradients
#pragma unroll
      for (int k = 0; k < NQ; ++k) {
        const int ot = opaque(tid), uu = ot & 31, u = 32 * w + uu, r = (ot >> 5) + 16 * k;
        float scale = 1.f;
        if constexpr (NP == 2) {
          float m = fmaxf(fmaxf(fabsf(sA[k][0]), fabsf(sA[k][1])), fmaxf(fabsf(sA[k][2]), fabsf(sA[k][3])));
          m = max16(m);
          m = fmaxf(m, __shfl_xor(m, 16, 32));
          const int e = rec_exp(m);
          scale = rec_scale(e);
          if (r < ni && uu == 0) a.sxs[(size_t)(ib + r) * NW + w] = rec_ldexp(1.f, -e - kDaExp);
        }
        if (r < ni && u < H) {
          uint16_t p[4][NP];
#pragma unroll
          for (int q = 0; q < 4; ++q) split_rec<NP>(sA[k][q], scale, p[q]);
#pragma unroll
          for (int s = 0; s < NP; ++s) {
            uint16_t* dst = a.sx + s * a.xplane + (size_t)(ib + r) * H4s + 4 * u;
            *(uint2*)dst = uint2{(uint32_t)p[0][s] | ((uint32_t)p[1][s] << 16), (uint32_t)p[2][s] | ((uint32_t)p[3][s] << 16)};
            if (u == H - 1 && (H & 1)) *(uint2*)(dst + 4) = uint2{0u, 0u};
          }
          const int x = ib + r - i0;
          if (x < kLevKeep) {
            eg_out[x * 32 + uu] = sg[k];
            eg_out[(kLevKeep + x) * 32 + uu] = sc[k];
          } else {
            a.eg[(size_t)(ib + r) * H + u] = sg[k];
            a.dcs[(size_t)(ib + r) * H + u] = sc[k];
          }
        }
      }
    }
    stamp(d, 1);
    group_arrive(bar, solo);
    int c0_next = 0, n0_next = 0;
    const uint32_t seen = solo ? 0u : group_peek(bar);
    {
      if (d > 1) {
        const int n0 = uni(i0_next);
        ics_r = prefetch_ics(n0, i0);
        i0_next = d > 2 ? ioff[d - 3] : 0;
        c0_next = uni(a.ix.ics[n0]);
        n0_next = n0;
        if constexpr (!kLate) prefetch(c0_next, c0);
      }
      if (!solo && group_wait(bar, (uint32_t)(NW * (D - d + 1)), seen, a.ctl, a.spin_limit, &s_flag)) {
        stop = true;
        break;
      }
    }
    stamp(d, 2);
    // (sum of dA) U^T for the parents, 16 rows at a time
    unsigned char* reg = lsm + wave * WREG;
    // granule gr of row r sits at slot gr ^ sw(r) of the wave's slice of the row
    auto sw = [](int r) { return SG >= 8 ? r & 7 : (r >> 1) & 3; };
    auto issue = [&](int row0) {
      row0 = uni(row0);
      const int nr = uni(min(16, i1 - row0));
#pragma unroll
      for (int s = 0; s < NP; ++s) {
        const rsrc_t rs = make_rsrc(a.sx + s * a.xplane + (size_t)row0 * H4s, (size_t)nr * H4s * 2);
#pragma unroll
        for (int q = 0; q < KH; ++q) {
          if (q * 64 / SG >= nr) continue;                  // (missing rows: columns nobody reads)
          const int L = q * 64 + opaque(lane), row = L / SG, col = 8 * (wave * SG + ((L % SG) ^ sw(row)));
          bdma16_sc1(rs, col < H4s ? (uint32_t)((row * H4s + col) * 2) : kOOB, 0u, lds_addr(reg + (s * KH + q) * 1024));
        }
      }
    };
    issue(i0);
    for (int row0 = i0; row0 < i1; row0 += 16) {
      const int nr = min(16, i1 - row0);
      // inverse scales of this lane's row in the wave's 128-column pieces
      constexpr int NS = NP == 2 ? (KH + 3) / 4 : 1;
      float xs[NS];
      if constexpr (NP == 2) {
        const rsrc_t rs = make_rsrc(a.sxs + (size_t)row0 * NW, (size_t)nr * NW * 4);
#pragma unroll
        for (int x = 0; x < NS; ++x) {
          const int piece = wave * KH / 4 + x;
          xs[x] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              rs, l16 < nr && piece < NW ? (uint32_t)((l16 * NW + piece) * 4) : kOOB, 0, kSc1));
        }
      }
      wait_vm<0>();
      hold(seen);
      if (kLate && row0 == i0 && d > 1) prefetch(c0_next, c0);
      f32x4 sum[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
      // (KS = 2: the one chunk of an odd wave is an odd one)
      const float sgn = (KH & 1) && (wave & 1) ? -1.f : 1.f;
#pragma unroll
      for (int x = 0; x < (KH + 3) / 4; ++x) {
        f32x4 acc[2], lo[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = lo[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 4 * x; c < 4 * x + 4 && c < KH; ++c) {
          uint4 b[NP];
#pragma unroll
          for (int s = 0; s < NP; ++s)
            b[s] = *(const uint4*)(reg + s * KH * 1024 + (l16 * SG + ((4 * c + lq) ^ sw(l16))) * 16);
#pragma unroll
          for (int t = 0; t < 2; ++t) mfma_rec<NP>(c, ub[t][c], b, NP == 2 ? acc[t] : sum[t], lo[t]);
          // (a few chunks' fragments at a time: more of them read ahead cost registers)
          if (NP * KS >= 32 && (c & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (NP == 2) {
#pragma unroll
          for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) sum[t][q] += (acc[t][q] * sgn + lo[t][q]) * xs[x];
        }
      }
      if constexpr (NP == 2) {
        // NaN results once more from the first planes (split.h: mfma_rec_first)
        if (__ballot(l16 < nr && (has_nan(sum[0]) || has_nan(sum[1])))) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < KH; ++c)
              mfma_rec_first(c, ub[t][c][0], *(const uint4*)(reg + (l16 * SG + ((4 * c + lq) ^ sw(l16))) * 16), v);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (sum[t][q] != sum[t][q] && !__builtin_isfinite(v[q])) sum[t][q] = v[q] * sgn;
          }
        }
      }
      if (row0 + 16 < i1) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the slices have been read
        issue(row0 + 16);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) *(f32x4*)&red[(wave * 16 + l16) * RLD + 16 * t + 4 * lq] = sum[t];
      __syncthreads();
      {
        const int ot = opaque(tid), uu = ot & 31, u = 32 * w + uu, r = ot >> 5;
        if (r < nr && u < H) {
          float v = 0.f;
#pragma unroll
          for (int x = 0; x < 8; ++x) v += red[(x * 16 + r) * RLD + uu];
          v *= ui;
          const int x = row0 + r - i0;
          if (x < kLevKeep) eg_out[x * 32 + uu] += v;
          else a.eg[(size_t)(row0 + r) * H + u] += v;
        }
      }
      __syncthreads();
    }
    stamp(d, 3);
    i1 = i0;
    i0 = n0_next;
    cend = c0;
    c0 = c0_next;
  }
  // bias gradient of the group: the 16 threads of a unit in order
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) db[q] = comp_sum(db[q], dbe[q]);
  ch_a[kk * 32 + uu] = f32x4{db[0], db[1], db[2], db[3]};
  __syncthreads();
  if (kk == 0 && u_ok) {
    f32x4 s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float t = ch_a[uu][q], e = 0.f;
      for (int k = 1; k < 16; ++k) comp_add(t, e, ch_a[k * 32 + uu][q]);
      s[q] = comp_sum(t, e);
    }
    *(f32x4*)(a.db_part + (size_t)g * H4 + 4 * u) = s;
  }
  // initial states (their gradients from children: the parity that level 1 wrote)
  if (u_ok && !stop) {
    const float* eg_in = keep;
    const int i0 = D > 0 ? ioff[0] : 0;
    for (int i = kk; i < Bg; i += 16) {
      const size_t o = (size_t)(n_init + i) * H + u, b = (size_t)(g + a.G * i) * H + u;
      float dh = a.gf[o], dc = a.gc ? a.gc[o] : 0.f;
      const int ci = a.ix.cidx[n_init + i];
      if (ci >= 0) {
        const int x = ci - i0;
        dh += x < kLevKeep ? eg_in[x * 32 + uu] : a.eg[(size_t)ci * H + u];
        dc += x < kLevKeep ? eg_in[(kLevKeep + x) * 32 + uu] : a.dcs[(size_t)ci * H + u];
      }
      a.dh0[b] = dh;
      a.dc0[b] = dc;
    }
  }
}

template <int NP, int KS, bool CLK>
static hipError_t launch_t(const LevBwdArgs& a, int grid, hipStream_t st) {
  auto kern = k_lev_bwd<NP, KS, CLK>;
  constexpr int shm = (int)lev_bwd_lds(NP, KS);
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, shm);
  if (e != hipSuccess) return e;
  LevBwdArgs args = a;
  void* kargs[] = {&args};
  return hipLaunchCooperativeKernel((const void*)kern, dim3(grid), dim3(kLevThreads), kargs, (unsigned)shm, st);
}
hipError_t launch_lev_bwd(const LevBwdArgs& a, int NP, int KS, int grid, hipStream_t st) {
#define CASE(N_, KS_) \
  if (NP == N_ && KS == KS_) return a.clk ? launch_t<N_, KS_, true>(a, grid, st) : launch_t<N_, KS_, false>(a, grid, st);
  LEV_CASES(CASE)
#undef CASE
  return hipErrorInvalidValue;
}
