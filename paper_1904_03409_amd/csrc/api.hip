// Host side of the StackLSTM library: argument checks, work-space layout, launch
// configuration and the launch order of the forward and backward passes.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <mutex>

#include "../../include/stacklstm.h"
#include "common.h"
#include "contract.h"
#include "levels.h"
#include "prep.h"

__global__ void k_ctl(uint32_t* ctl, int keep_errors, int bwd);
template <bool LDS> __global__ void k_plan(PlanArgs a);
template <int S>
__global__ void k_split_x(const float* x, const int32_t* order, int lo, int hi, int I, int k0, int Kc, int vec, bf16_t* out,
                          size_t plane);
template <int S> __global__ void k_prep_fwd(PrepFwdArgs a);
template <int S, int V> __global__ void k_prep_bwd(PrepBwdArgs a);
template <int V> __global__ void k_gather_top(GatherArgs a);
__global__ void k_fill_f32(float* p, size_t n, float v);
__global__ void k_reduce_grads(ReduceArgs a);

namespace {

constexpr int kDefaultSpin = 1 << 22;

struct DevInfo { int cus; bool ok; };

int device_cus() {
  static std::mutex mu;
  static DevInfo info[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  std::lock_guard<std::mutex> lk(mu);
  if (!info[dev].ok) {
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return 0;
    info[dev].cus = p.multiProcessorCount;
    info[dev].ok = true;
  }
  return info[dev].cus;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
bool al16(const void* q) { return ((uintptr_t)q & 15u) == 0; }

int planes_of(const slstm_dims* d) { return d->precision == SLSTM_BF16_GEMM ? 1 : 3; }
int rec_planes_of(const slstm_dims* d) { return d->precision == SLSTM_BF16_GEMM ? 1 : 2; }

bool dims_ok(const slstm_dims* d) {
  if (!d) return false;
  if (d->T < 0 || d->B < 1 || d->I < 1 || d->H < 1) return false;
  if (d->precision != SLSTM_FP32 && d->precision != SLSTM_BF16_GEMM) return false;
  if (d->H > (d->precision == SLSTM_FP32 ? 512 : 1024)) return false;
  if ((int64_t)d->T * d->B > ((int64_t)1 << 28)) return false;
  // sizes the kernels address with 32-bit byte offsets
  const int64_t esz = d->precision == SLSTM_FP32 ? 4 : 2;
  if ((int64_t)d->T * d->B * 4 * d->H * esz >= ((int64_t)1 << 32)) return false;
  if ((int64_t)d->T * d->B * d->H * 4 >= ((int64_t)1 << 32)) return false;
  return true;
}

// Workgroups per group, K chunks of 32 compiled into the recurrent kernels, and groups.
int groups_nw(int H) { return (H + kLevUnits - 1) / kLevUnits; }
// Largest number of groups on an XCD of `cus` CUs (one 512-thread workgroup per CU), times 8
int groups_max(int H, int cus) { return std::min(kLevMaxGroups, 8 * (cus / groups_nw(H))); }
// As many groups as there are elements and room for: a level's rows of a group are padded to 16
// and every row costs its group's workgroups a copy, so more groups mean shorter levels.
int groups_for(int B, int H, int cus) { return std::min(B, groups_max(H, cus)); }
// Largest batch: 128 elements for each set of ceil(H / 16) workgroup slots of an XCD's 32, at most 64 sets
int batch_max(int H) { return H > 512 ? 1024 : 128 * std::min(64, 8 * (32 / ((H + 15) / 16))); }

struct Plan {
  int prec, S, NP, KS, NW, G, xcc_cus;   // S: bf16 planes of an operand, NP: planes of the recurrent products
};

int make_plan(const slstm_dims* d, Plan* p) {
  if (!dims_ok(d)) return SLSTM_EINVAL;
  p->prec = d->precision;
  p->S = planes_of(d);
  p->NW = groups_nw(d->H);
  p->NP = rec_planes_of(d);
  p->KS = lev_ks(p->NP, p->NW);
  const int cus = device_cus();
  if (cus <= 0) return SLSTM_EDEVICE;
  p->xcc_cus = std::min(32, cus / 8);
  if (p->xcc_cus < p->NW || d->B > batch_max(d->H)) return SLSTM_ENORESIDENT;
  p->G = groups_for(d->B, d->H, p->xcc_cus);
  return SLSTM_OK;
}

// Split K of dW | dU: one workgroup per CU, K slices of at least one 64-row step.
int tn_tiles(const slstm_dims* d) {
  const int S = planes_of(d), bm = nt_bm(S, nt_mi(S)), bn = nt_bn(S);
  return ((4 * d->H + bn - 1) / bn) * ((d->I + bm - 1) / bm + (d->H + bm - 1) / bm);
}
int tn_splits(const slstm_dims* d) {
  const int64_t steps = ((int64_t)d->T * d->B + 63) / 64;
  return (int)std::max<int64_t>(1, std::min<int64_t>({256 / std::max(1, tn_tiles(d)), 64, steps}));
}

// Work-space layout. It does not depend on the device (group counts as for 32 CUs per XCD).
struct Layout {
  size_t ctl, order, opar, cs, loff, gmax, ics, ioff, cidx, kin, gslot, cnt, elem, walk;
  size_t wt, wp, uf, ufi, rin, hu, stash, cpn, hq, h3, cn, xs;
  size_t gf, gc, eg, dcs, dap, sxs, ub, ubi, part, dbp, total;
  int Ip, Hs, H4s, cap, G;
  int x_rows, x_cols;                // rows and columns of x whose planes fit (all, except in the static work space)
  size_t walk_lds;                   // bytes of a wave's walk arrays when they live in LDS, else 0
};

// keep: with the parts that only a backward needs; x_budget: bytes for the planes of x (0 = all rows)
Layout layout(const slstm_dims* d, bool keep, size_t x_budget) {
  const size_t T = d->T, B = d->B, I = d->I, H = d->H, S = planes_of(d), N0 = T * B, NN = N0 + B, NP = rec_planes_of(d);
  Layout L;
  L.Ip = (int)((I + 7) / 8 * 8);
  L.Hs = (int)((H + 7) / 8 * 8);
  L.H4s = (int)((4 * H + 7) / 8 * 8);
  L.cap = (int)T + 2;
  const int NW = groups_nw(d->H), KS = lev_ks((int)NP, NW);
  L.G = groups_for(d->B, d->H, 32);
  const size_t wave_walk = (size_t)2 * L.cap * 4;
  L.walk_lds = wave_walk <= 147456 ? wave_walk : 0;
  size_t o = 0;
  auto put = [&](size_t bytes) {
    const size_t at = o;
    o += align256(std::max<size_t>(bytes, 16));
    return at;
  };
  L.ctl = put(CTL_WORDS * 4);
  L.order = put(N0 * 4);
  L.opar = put(N0 * 4);
  L.cs = put(NN * 4);
  L.loff = put((size_t)L.G * (T + 4) * 4);
  L.gmax = put((size_t)kLevMaxGroups * 4);
  L.ics = put(keep ? NN * 4 : 0);
  L.ioff = put(keep ? (size_t)L.G * (T + 4) * 4 : 0);
  L.cidx = put(keep ? NN * 4 : 0);
  L.kin = put(keep ? N0 * 4 : 0);
  L.gslot = put(keep ? N0 * 4 : 0);
  L.elem = put(3 * B * 4);
  L.wt = put(S * 4 * H * L.Ip * 2);
  L.wp = put(keep ? S * I * L.H4s * 2 : 0);
  L.uf = put((size_t)NW * 8 * KS * 64 * NP * 16);
  L.ufi = put((size_t)NW * kLevUnits * 4);
  L.rin = put(B * 4);
  // k_plan's counts and walk arrays; then x W and h U of the nodes (forward); then the exchange rows of the
  // backward, in bf16 mode (rows half as long) with the interval sums of dc_top behind them
  const size_t walk = align256(B * L.cap * 4), sx = align256(NP * NN * L.H4s * 2), sums = 2 * NN * H * 4;
  L.hu = put(std::max({NN * 4 * H * 4, keep ? sx + (NP == 1 ? sums : 0) : 0,
                       walk + (L.walk_lds ? 0 : (size_t)L.G * 2 * L.cap * 4)}));
  L.cnt = L.hu;
  L.walk = L.hu + walk;
  L.stash = put(keep ? N0 * 4 * H * 4 : 0);
  L.cpn = put(keep ? N0 * H * 4 : 0);
  L.hq = put(NP * NN * L.Hs * 2);
  L.h3 = put(keep && S == 3 ? S * NN * L.Hs * 2 : 0);       // (bf16 mode: hq)
  L.cn = put(NN * H * 4);
  L.x_rows = (int)N0;
  L.x_cols = L.Ip;
  if (x_budget) {
    // all rows if 64 columns of them fit, and as many columns (64 at a time, two K steps) as do
    const size_t least = std::min(L.Ip, 64), a_col = S * 2;
    L.x_rows = (int)std::min<size_t>(N0, std::max<size_t>(x_budget / (least * a_col), 1));
    const size_t cols = x_budget / std::max<size_t>(L.x_rows * a_col, 1);
    if (cols < (size_t)L.Ip) L.x_cols = (int)std::max(cols / 64 * 64, least);
  }
  L.xs = put(S * (size_t)L.x_rows * L.x_cols * 2);
  if (!keep) {
    L.total = o;
    return L;
  }
  // a backward needs neither c of the nodes (it has the parents') nor, in fp32 mode, the recurrent planes of h
  L.gf = put(sums);
  L.gc = NP == 1 ? L.hu + sx : put(sums);
  L.eg = L.cn;
  L.dcs = NP == 2 ? L.hq : put(NN * H * 4);
  L.dap = put(S * N0 * L.H4s * 2);
  L.sxs = put(NP == 2 ? NN * NW * 4 : 0);
  L.ub = put((size_t)NW * 8 * KS * 64 * NP * 16);
  L.ubi = put((size_t)NW * kLevUnits * 4);
  L.part = put((size_t)tn_splits(d) * (I + H) * 4 * H * 4);
  L.dbp = put((size_t)kLevMaxGroups * 4 * H * 4);
  L.total = o;
  return L;
}
Layout layout(const slstm_dims* d) { return layout(d, true, 0); }

int hip_status(hipError_t e) {
  if (e == hipSuccess) return SLSTM_OK;
  if (e == hipErrorCooperativeLaunchTooLarge) return SLSTM_ENORESIDENT;
  return SLSTM_EDEVICE;
}

void mark(const slstm_dims* d, int i, hipStream_t st) {
  if (d->phase_events) (void)hipEventRecord(((hipEvent_t*)d->phase_events)[i], st);
}

int grid1d(size_t n) { return (int)std::min<size_t>((n + 255) / 256, 8192); }

// The call's one host synchronisation: reads the control words its kernels set and maps them
// to a status (op errors first, then a wait that gave up, then a producer index out of range).
int read_status(const uint32_t* ctl, hipStream_t st) {
  uint32_t v[CTL_BADIDX + 1] = {};
  if (hipMemcpyAsync(v, ctl, sizeof(v), hipMemcpyDeviceToHost, st) != hipSuccess) return SLSTM_EDEVICE;
  if (hipStreamSynchronize(st) != hipSuccess) return SLSTM_EDEVICE;
  if (v[CTL_STATUS] != kStatusOk) return (int)(v[CTL_STATUS] & 7u);
  if (v[CTL_TIMEOUT]) return SLSTM_ETIMEOUT;
  if (v[CTL_BADIDX]) return SLSTM_EINDEX;
  return SLSTM_OK;
}

// The status a call returns: its control words read back (one host synchronisation), or,
// for a deferred call, OK once its kernels are queued (sync_status reads the words later).
int call_status(const slstm_dims* d, const uint32_t* ctl, hipStream_t st) {
  if (hipGetLastError() != hipSuccess) return SLSTM_EDEVICE;
  return d->defer_status ? SLSTM_OK : read_status(ctl, st);
}

LevIdx idx_of(char* ws, const Layout& L) {
  LevIdx x;
  x.order = (int32_t*)(ws + L.order);
  x.opar = (int32_t*)(ws + L.opar);
  x.cs = (int32_t*)(ws + L.cs);
  x.loff = (int32_t*)(ws + L.loff);
  x.gmax = (int32_t*)(ws + L.gmax);
  x.ics = (int32_t*)(ws + L.ics);
  x.ioff = (int32_t*)(ws + L.ioff);
  x.cidx = (int32_t*)(ws + L.cidx);
  x.kin = (int32_t*)(ws + L.kin);
  x.gslot = (int32_t*)(ws + L.gslot);
  return x;
}
// Names the sizes of a schedule (FNV-1a); never 0.
uint64_t plan_key(const slstm_dims* d, int G) {
  uint64_t h = 1469598103934665603ull;
  for (int v : {d->T, d->B, d->I, d->H, d->precision, G}) h = (h ^ (uint32_t)v) * 1099511628211ull;
  return h | 1;
}
int spin_of(const slstm_dims* d) { return d->spin_limit > 0 ? d->spin_limit : kDefaultSpin; }
// workgroups of a recurrent kernel: every XCD takes the workgroups of its share of the groups
int lev_grid(const Plan& p) { return 8 * p.NW * ((p.G + 7) / 8); }

}  // namespace

extern "C" {

size_t stacklstm_workspace_bytes(const slstm_dims* d) {
  if (!dims_ok(d)) return 0;
  return layout(d).total;
}

const char* stacklstm_status_string(int s) {
  switch (s) {
    case SLSTM_OK: return "ok";
    case SLSTM_EINVAL: return "invalid argument (dims, null pointer or unsupported size)";
    case SLSTM_EOPS: return "op outside {-1, 0, 1}";
    case SLSTM_EUNDERFLOW: return "pop with only the initial state on the stack";
    case SLSTM_EWORKSPACE: return "work space too small";
    case SLSTM_ENORESIDENT: return "persistent kernels cannot be co-resident";
    case SLSTM_EDEVICE: return "HIP runtime error";
    case SLSTM_ETIMEOUT: return "a wait for another workgroup's data exceeded the spin limit";
    case SLSTM_EINDEX: return "a producer index or stack depth outside its valid range (top or ops not the forward's)";
    default: return "unknown status";
  }
}

int stacklstm_plan(const slstm_dims* d, slstm_plan* out) {
  Plan p;
  int rc = make_plan(d, &p);
  if (rc) return rc;
  if (!out) return SLSTM_EINVAL;
  memset(out, 0, sizeof(*out));
  out->groups = p.G;
  out->wg_per_group = p.NW;
  out->rows_per_group = (d->B + p.G - 1) / p.G;
  out->k_chunks = p.NW;
  out->fwd_tiles = lev_fwd_rt(p.NP, p.KS);
  out->k_chunk_cap = p.KS;
  out->occupancy = 2;
  out->bwd_groups = p.G;
  out->bwd_tiles = 1;
  return SLSTM_OK;
}

}  // extern "C"

namespace {

// The forward pass on a work space that the caller checked.
int fwd_impl(const slstm_dims* d, const Plan& p, const Layout& L, bool keep, const float* x, const int8_t* ops,
             const float* W, const float* U, const float* b, const float* h0, const float* c0, float* h_cell,
             float* c_cell, float* h_top, float* c_top, int32_t* ptr, int32_t* top, char* ws, hipStream_t st) {
  int rc = SLSTM_OK;
  uint32_t* ctl = (uint32_t*)(ws + L.ctl);
  const int T = d->T, B = d->B, I = d->I, H = d->H, S = p.S, N0 = T * B;
  const LevIdx ix = idx_of(ws, L);

  // control words; operand planes of W, U and the initial states
  mark(d, 0, st);
  float* hu = (float*)(ws + L.hu);
  uint16_t* hq = (uint16_t*)(ws + L.hq);
  uint16_t* h3 = keep && S == 3 ? (uint16_t*)(ws + L.h3) : nullptr;
  float* cn = (float*)(ws + L.cn);
  uint16_t* xs = (uint16_t*)(ws + L.xs);
  const size_t hplane = (size_t)(N0 + B) * L.Hs;
  if (T == 0) {
    hipLaunchKernelGGL(k_ctl, dim3(1), dim3(256), 0, st, ctl, d->defer_status ? 1 : 0, 0);
  } else {
    PrepFwdArgs a;
    a.I = I; a.Ip = L.Ip; a.H = H; a.Hs = L.Hs; a.H4s = keep ? L.H4s : 0; a.B = B; a.G = p.G; a.N0 = N0; a.NW = p.NW;
    a.KS = p.KS;
    a.n_w = ((I + 31) / 32) * ((H + 31) / 32);
    a.n_u = p.NW * 4;
    a.W = W; a.U = U; a.h0 = h0; a.c0 = c0;
    a.wt = (uint16_t*)(ws + L.wt); a.wp = (uint16_t*)(ws + L.wp); a.uf = (uint4*)(ws + L.uf);
    a.uexp = (int32_t*)(ws + L.ufi); a.rinit = (int32_t*)(ws + L.rin);
    a.hq = hq; a.hplane = hplane; a.h3 = h3; a.cn = cn;
    a.ctl = ctl; a.keep_errors = d->defer_status ? 1 : 0;
    const int grid = a.n_w + a.n_u + (B + 3) / 4;
    if (S == 3) hipLaunchKernelGGL(k_prep_fwd<3>, dim3(grid), dim3(256), 0, st, a);
    else        hipLaunchKernelGGL(k_prep_fwd<1>, dim3(grid), dim3(256), 0, st, a);
  }
  // op validation, pointer scan, producer trace and level schedule. One workgroup per group; as
  // many waves as have walk arrays in LDS (at most one per element of the group)
  {
    PlanArgs a;
    a.T = T; a.B = B; a.G = p.G; a.cap = L.cap;
    a.ops = ops; a.ptr = ptr; a.top = top; a.ix = ix;
    a.cnt = (int32_t*)(ws + L.cnt); a.elem = (int32_t*)(ws + L.elem); a.walk = (int32_t*)(ws + L.walk); a.ctl = ctl;
    a.key = keep ? plan_key(d, p.G) : 0;
    if (L.walk_lds) {
      const int waves = (int)std::min<size_t>(16, 147456 / L.walk_lds);
      const size_t shm = waves * L.walk_lds;
      if (hipFuncSetAttribute((const void*)k_plan<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) != hipSuccess)
        return SLSTM_EDEVICE;
      hipLaunchKernelGGL(k_plan<true>, dim3(p.G), dim3(64 * waves), shm, st, a);
    } else {
      hipLaunchKernelGGL(k_plan<false>, dim3(p.G), dim3(64), 0, st, a);
    }
  }
  if ((rc = hip_status(hipGetLastError()))) return rc;
  mark(d, 1, st);
  if (T == 0) return call_status(d, ctl, st);

  // planes of x, x W + b of the push nodes
  NtArgs g;
  memset(&g, 0, sizeof(g));
  g.N = 4 * H; g.N0 = N0;
  g.bplane = (size_t)4 * H * L.Ip; g.ldb = L.Ip;
  g.ctl = ctl; g.C = hu; g.ldc = 4 * H; g.H = H; g.order = ix.order;
  g.opar = ix.opar; g.hu = hu; g.cn = cn; g.hcell = h_cell; g.ccell = c_cell;
  // one contraction over columns k0 .. k0 + K - 1 of the rows lo .. hi - 1 whose planes are in xs
  auto x_w = [&](int epi, bool leaves, int lo, int hi, int k0, int K, const float* bias) {
    g.lo = lo; g.hi = hi; g.leaves = leaves; g.pre = k0 > 0; g.K = K; g.bias = bias;
    g.A = xs; g.lda = K; g.aplane = (size_t)(hi - lo) * K;
    g.B = (uint16_t*)(ws + L.wt) + k0;
    return hip_status(launch_nt(g, S, epi, st));
  };
  // (planes of all of x at once, or, where they have less room, of a range of its columns and if need be
  // rows at a time: the sums of both kinds of steps go on in hu, whose rows P .. N0 - 1 no node has, and the
  // leaves' cells start from theirs)
  const bool once = L.x_rows >= N0 && L.x_cols >= L.Ip;
  for (int lo = 0; lo < N0; lo += L.x_rows) {
    const int hi = std::min(N0, lo + L.x_rows);
    for (int k0 = 0; k0 < L.Ip; k0 += L.x_cols) {
      const int K = std::min(L.x_cols, L.Ip - k0), vec = I % 4 == 0 && al16(x);
      const int grid = grid1d((size_t)(hi - lo) * (K / 8));
      const size_t plane = (size_t)(hi - lo) * K;
      if (S == 3) hipLaunchKernelGGL(k_split_x<3>, dim3(grid), dim3(256), 0, st, x, ix.order, lo, hi, I, k0, K, vec, xs, plane);
      else        hipLaunchKernelGGL(k_split_x<1>, dim3(grid), dim3(256), 0, st, x, ix.order, lo, hi, I, k0, K, vec, xs, plane);
      if ((rc = x_w(NT_XW, false, lo, hi, k0, K, k0 + K >= L.Ip ? b : nullptr))) return rc;
      if (!once && (rc = x_w(NT_XW, true, lo, hi, k0, K, nullptr))) return rc;
    }
  }
  mark(d, 2, st);

  // the recurrence over the levels
  {
    LevFwdArgs a;
    memset(&a, 0, sizeof(a));
    a.T = T; a.B = B; a.H = H; a.Hs = L.Hs; a.G = p.G; a.NW = p.NW; a.N0 = N0; a.spin_limit = spin_of(d);
    a.ix = ix; a.hu = hu; a.hq = hq; a.hplane = hplane; a.cn = cn; a.hcell = h_cell; a.ccell = c_cell;
    a.stash = keep ? (float*)(ws + L.stash) : nullptr;
    a.cpn = (float*)(ws + L.cpn); a.h3 = h3;
    a.uf = (const uint4*)(ws + L.uf); a.uexp = (const int32_t*)(ws + L.ufi); a.rinit = (const int32_t*)(ws + L.rin);
    a.ctl = ctl;
    a.clk = (long long*)d->step_clock;
    if ((rc = hip_status(launch_lev_fwd(a, p.NP, p.KS, lev_grid(p), st)))) return rc;
  }
  mark(d, 3, st);

  // the leaves (pop and hold steps), then Algorithm 1's return values
  if ((rc = x_w(NT_LEAF, true, 0, N0, once ? 0 : L.Ip, once ? L.Ip : 0, b))) return rc;
  if (h_top || c_top) {
    GatherArgs a;
    a.top = top; a.ctl = ctl; a.hcell = h_cell; a.h0 = h0; a.ccell = c_cell; a.c0 = c0;
    a.htop = h_top; a.ctop = c_top; a.T = T; a.B = B; a.H = H;
    const bool vec = H % 4 == 0 && al16(h_cell) && al16(h0) && al16(h_top) && al16(c_cell) && al16(c0) && al16(c_top);
    for (a.ll = 2; a.ll < 6 && (1 << a.ll) < (vec ? H / 4 : H);) ++a.ll;
    const int rows = 4 * 8 * (64 >> a.ll);             // of a workgroup
    const dim3 grid(((size_t)N0 + rows - 1) / rows);
    if (vec) hipLaunchKernelGGL(k_gather_top<4>, grid, dim3(256), 0, st, a);
    else     hipLaunchKernelGGL(k_gather_top<1>, grid, dim3(256), 0, st, a);
  }
  if ((rc = hip_status(hipGetLastError()))) return rc;
  mark(d, 4, st);
  return call_status(d, ctl, st);
}

bool fwd_args_ok(const slstm_dims* d, const float* x, const int8_t* ops, const float* W, const float* U,
                 const float* b, const float* h0, const float* c0, const float* h_cell, const float* c_cell,
                 const int32_t* ptr, const int32_t* top) {
  return ptr && (d->T == 0 || (ops && x && W && U && b && h0 && c0 && h_cell && c_cell && top));
}

// Static work space of the allocation-free forward: one copy per GPU, held until the process
// ends. Host code uses the device address that hipGetSymbolAddress returns for the current
// device (kept per device), never the array's name. Of the dims that static_measure admits the one with the
// largest need beside the planes of x takes 242 MiB (3.7 M steps of one element at H = 1 in fp32 mode: state
// planes padded to 16 bytes).
constexpr size_t kScratchBytes = SLSTM_FWD_STATIC_BYTES;
__device__ __align__(256) unsigned char scratch[kScratchBytes];

// Bytes that decide whether dims are served from the static work space: the work space of a
// forward that keeps x W and the gate activations of every step.
size_t static_measure(const slstm_dims* d) {
  const size_t T = d->T, B = d->B, I = d->I, H = d->H;
  return align256((64 + 2 * 16 * 64) * 4) + align256(B * (T + 1) * 4) + align256(B * 4) + align256(I * 4 * H * 4) +
         2 * align256(std::max<size_t>(T * B * 4 * H * 4, 16)) +
         (d->precision == SLSTM_BF16_GEMM ? align256((T + 1) * B * H * 2) : 0);
}
// The forward's layout in the static work space: what is left beside the other parts holds the
// planes of x, a range of their columns (and rows) at a time if need be.
Layout static_layout(const slstm_dims* d) {
  const Layout L = layout(d, false, 1);
  return L.total >= kScratchBytes ? L : layout(d, false, std::max<size_t>(kScratchBytes - L.total, 1));
}

// Device address of `scratch` on the current device, looked up on the first call on that
// device; null if the lookup failed.
char* scratch_ptr() {
  static std::mutex mu;
  static void* addr[64] = {};
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  std::lock_guard<std::mutex> lk(mu);
  if (!done[dev]) {
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    addr[dev] = q;
    done[dev] = true;
  }
  return (char*)addr[dev];
}

}  // namespace

extern "C" {

int stacklstm_fwd(const slstm_dims* d, const float* x, const int8_t* ops, const float* W, const float* U,
                  const float* b, const float* h0, const float* c0, float* h_cell, float* c_cell, float* h_top,
                  float* c_top, int32_t* ptr, int32_t* top, void* workspace, size_t ws_bytes, void* stream) {
  if (!dims_ok(d)) return SLSTM_EINVAL;
  if (!workspace || !fwd_args_ok(d, x, ops, W, U, b, h0, c0, h_cell, c_cell, ptr, top)) return SLSTM_EINVAL;
  const Layout L = layout(d);
  if (ws_bytes < L.total) return SLSTM_EWORKSPACE;
  Plan p;
  int rc = make_plan(d, &p);
  if (rc) return rc;
  return fwd_impl(d, p, L, true, x, ops, W, U, b, h0, c0, h_cell, c_cell, h_top, c_top, ptr, top, (char*)workspace,
                  (hipStream_t)stream);
}

int stacklstm_fwd_static(const slstm_dims* d, const float* x, const int8_t* ops, const float* W, const float* U,
                         const float* b, const float* h0, const float* c0, float* h_cell, float* c_cell, float* h_top,
                         float* c_top, int32_t* ptr, int32_t* top, void* stream) {
  if (!dims_ok(d)) return SLSTM_EINVAL;
  if (!fwd_args_ok(d, x, ops, W, U, b, h0, c0, h_cell, c_cell, ptr, top)) return SLSTM_EINVAL;
  if (static_measure(d) > SLSTM_FWD_STATIC_MAX_BYTES) return SLSTM_EWORKSPACE;
  const Layout L = static_layout(d);
  if (L.total > kScratchBytes) return SLSTM_EWORKSPACE;
  Plan p;
  int rc = make_plan(d, &p);
  if (rc) return rc;
  char* ws = scratch_ptr();
  if (!ws) return SLSTM_EDEVICE;
  return fwd_impl(d, p, L, false, x, ops, W, U, b, h0, c0, h_cell, c_cell, h_top, c_top, ptr, top, ws,
                  (hipStream_t)stream);
}

int stacklstm_bwd(const slstm_dims* d, const float* x, const int8_t* ops, const float* W, const float* U,
                  const float* h0, const float* c0, const float* h_cell, const float* c_cell, const int32_t* top,
                  void* workspace, size_t ws_bytes, const float* dh_top, const float* dc_top, float* dx, float* dW,
                  float* dU, float* db, float* dh0, float* dc0, void* stream) {
  (void)W; (void)h0; (void)c0; (void)h_cell; (void)c_cell;
  if (!dims_ok(d)) return SLSTM_EINVAL;
  if (!workspace || !dW || !dU || !db || !dh0 || !dc0) return SLSTM_EINVAL;
  if (d->T > 0 && (!x || !ops || !U || !h0 || !c0 || !h_cell || !c_cell || !top || !dh_top || !dx))
    return SLSTM_EINVAL;
  const Layout L = layout(d);
  if (ws_bytes < L.total) return SLSTM_EWORKSPACE;
  Plan p;
  int rc = make_plan(d, &p);
  if (rc) return rc;
  hipStream_t st = (hipStream_t)stream;
  char* ws = (char*)workspace;
  uint32_t* ctl = (uint32_t*)(ws + L.ctl);
  const int T = d->T, B = d->B, I = d->I, H = d->H;
  const int keep_errors = d->defer_status ? 1 : 0;
  if (T == 0) {
    hipLaunchKernelGGL(k_ctl, dim3(1), dim3(256), 0, st, ctl, keep_errors, 1);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid1d((size_t)I * 4 * H)), dim3(256), 0, st, dW, (size_t)I * 4 * H, 0.f);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid1d((size_t)H * 4 * H)), dim3(256), 0, st, dU, (size_t)H * 4 * H, 0.f);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid1d((size_t)4 * H)), dim3(256), 0, st, db, (size_t)4 * H, 0.f);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid1d((size_t)B * H)), dim3(256), 0, st, dh0, (size_t)B * H, 0.f);
    hipLaunchKernelGGL(k_fill_f32, dim3(grid1d((size_t)B * H)), dim3(256), 0, st, dc0, (size_t)B * H, 0.f);
    if ((rc = hip_status(hipGetLastError()))) return rc;
    return call_status(d, ctl, st);
  }

  const int S = p.S, N0 = T * B;
  const uint64_t key = plan_key(d, p.G);
  const LevIdx ix = idx_of(ws, L);
  // control words, U^T fragments, interval sums of the upstream gradients
  float* gf = (float*)(ws + L.gf);
  float* gc = dc_top ? (float*)(ws + L.gc) : nullptr;
  {
    PrepBwdArgs a;
    a.T = T; a.B = B; a.H = H; a.G = p.G; a.NW = p.NW; a.KS = p.KS;
    a.U = U; a.ub = (uint4*)(ws + L.ub); a.uinv = (float*)(ws + L.ubi);
    a.gslot = ix.gslot; a.ctl = ctl; a.key = key; a.keep_errors = keep_errors;
    auto prep = [&](int n_u, const float* src, float* sums, int clear) {
      a.n_u = n_u; a.d = src; a.sums = sums; a.clear = clear;
      const bool vec = H % 4 == 0 && al16(src);
      const size_t parts = (H + (vec ? 255 : 63)) / (vec ? 256 : 64), segs = (T + 31) / 32;
      const dim3 grid(n_u + (B * parts * segs + 3) / 4);
      if (S == 3 && vec)  hipLaunchKernelGGL((k_prep_bwd<3, 4>), grid, dim3(256), 0, st, a);
      else if (S == 3)    hipLaunchKernelGGL((k_prep_bwd<3, 1>), grid, dim3(256), 0, st, a);
      else if (vec)       hipLaunchKernelGGL((k_prep_bwd<1, 4>), grid, dim3(256), 0, st, a);
      else                hipLaunchKernelGGL((k_prep_bwd<1, 1>), grid, dim3(256), 0, st, a);
    };
    prep(p.NW * 16, dh_top, gf, 1);
    if (gc) prep(0, dc_top, gc, 0);
  }
  uint16_t* dap = (uint16_t*)(ws + L.dap);
  const size_t dplane = (size_t)N0 * L.H4s;
  float* part = (float*)(ws + L.part);
  float* dbp = (float*)(ws + L.dbp);
  mark(d, 5, st);
  {
    LevBwdArgs a;
    memset(&a, 0, sizeof(a));
    a.T = T; a.B = B; a.H = H; a.H4s = L.H4s; a.G = p.G; a.NW = p.NW; a.N0 = N0; a.spin_limit = spin_of(d);
    a.ix = ix; a.cpn = (const float*)(ws + L.cpn);
    a.stash = (const float*)(ws + L.stash);
    a.gf = gf; a.gc = gc; a.eg = (float*)(ws + L.eg); a.dcs = (float*)(ws + L.dcs);
    a.dap = dap; a.dplane = dplane; a.sx = (uint16_t*)(ws + L.hu); a.xplane = (size_t)(N0 + B) * L.H4s;
    a.sxs = (float*)(ws + L.sxs); a.ub = (const uint4*)(ws + L.ub); a.uinv = (const float*)(ws + L.ubi);
    a.db_part = dbp; a.dh0 = dh0; a.dc0 = dc0; a.ctl = ctl; a.key = key;
    if (d->step_clock) a.clk = (long long*)d->step_clock + (size_t)512 * T * 4;
    if ((rc = hip_status(launch_lev_bwd(a, p.NP, p.KS, lev_grid(p), st)))) return rc;
  }
  mark(d, 6, st);

  // dW, dU over the push nodes (dA is exactly 0 on every other step), db from the groups' sums
  {
    TnArgs g;
    memset(&g, 0, sizeof(g));
    g.I = I; g.H = H; g.H4 = 4 * H; g.splits = tn_splits(d); g.xt = (I + nt_bm(S, nt_mi(S)) - 1) / nt_bm(S, nt_mi(S));
    g.X = (const uint16_t*)(ws + L.xs); g.xplane = (size_t)N0 * L.Ip; g.ldx = L.Ip;
    g.Hp = (const uint16_t*)(ws + (S == 3 ? L.h3 : L.hq)); g.hplane = (size_t)(N0 + B) * L.Hs; g.ldh = L.Hs; g.hrows = N0 + B;
    g.D = dap; g.dplane = dplane; g.ldd = L.H4s;
    g.opar = ix.opar; g.ctl = ctl; g.key = key; g.part = part; g.split_stride = (size_t)(I + H) * 4 * H;
    if ((rc = hip_status(launch_tn(g, S, st)))) return rc;
    ReduceArgs r;
    r.part = part; r.splits = g.splits; r.stride = g.split_stride; r.db_part = dbp; r.groups = p.G; r.I = I; r.H = H;
    r.dW = dW; r.dU = dU; r.db = db;
    r.T = T; r.B = B; r.n_red = grid1d((size_t)(I + H + 1) * H);
    r.ops = ops; r.top = top; r.order = ix.order; r.ctl = ctl; r.key = key;
    const int checks = (int)std::min<size_t>(((size_t)N0 + 1023) / 1024, 1024);
    hipLaunchKernelGGL(k_reduce_grads, dim3(r.n_red + checks), dim3(256), 0, st, r);
  }
  mark(d, 7, st);
  mark(d, 8, st);
  // dx = dA W^T on the push steps, 0 on the others (in the same launch)
  {
    NtArgs g;
    memset(&g, 0, sizeof(g));
    g.N = I; g.K = L.H4s; g.N0 = N0; g.lo = 0; g.hi = N0;
    g.A = dap; g.aplane = dplane; g.lda = L.H4s;
    g.B = (const uint16_t*)(ws + L.wp); g.bplane = (size_t)I * L.H4s; g.ldb = L.H4s;
    g.ctl = ctl; g.key = key; g.C = dx; g.ldc = I; g.order = ix.order; g.H = H;
    if ((rc = hip_status(launch_nt(g, S, NT_DX, st)))) return rc;
  }
  if ((rc = hip_status(hipGetLastError()))) return rc;
  mark(d, 9, st);
  return call_status(d, ctl, st);
}

int stacklstm_sync_status(const void* workspace, size_t ws_bytes, void* stream) {
  if (!workspace || ws_bytes < align256(CTL_WORDS * 4)) return SLSTM_EINVAL;
  return read_status((const uint32_t*)workspace, (hipStream_t)stream);
}

}  // extern "C"
