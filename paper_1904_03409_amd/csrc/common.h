// Shared device helpers for the StackLSTM HIP library (gfx950 / CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t bf16_t;  // raw bfloat16 bits in memory

// Status codes shared with the C-ABI (values fixed by include/stacklstm.h).
enum {
  ST_OK = 0, ST_EINVAL = 1, ST_EOPS = 2, ST_EUNDERFLOW = 3, ST_EWORKSPACE = 4,
  ST_ENORESIDENT = 5, ST_EDEVICE = 6, ST_ETIMEOUT = 7, ST_EINDEX = 8
};

// CTL_STATUS while every op is valid.
constexpr uint32_t kStatusOk = 0x7fffffffu;

// Work-space word offsets (uint32 units) of the control block at the start of the work space.
enum {
  CTL_STATUS = 0,        // lowest (element * 8 + code) of a failing element, or 0x7fffffff
  CTL_ABORT = 2,         // set when a wait ran out of spins: every workgroup leaves its loop
  CTL_TIMEOUT = 3,       // set when a wait ran out of spins (reported as SLSTM_ETIMEOUT)
  CTL_NPUSHF = 5,        // number of push steps (counted by k_plan in the forward)
  CTL_BADIDX = 6,        // set when a kernel read a producer index outside its valid range
  CTL_KEY = 8,           // 2 words: the sizes whose schedule the work space holds (k_plan), else 0
  CTL_XCC_SLOT = 16,     // 16 per-XCC slot counters (forward kernel)
  CTL_XCC_SLOT_B = 32,   // 16 per-XCC slot counters (backward kernel)
  CTL_BAR_F = 64,        // forward group barrier counters, one 64-byte line per group
  CTL_BAR_B = 64 + 16 * 128,  // backward group barrier counters
  CTL_WORDS = 64 + 2 * 16 * 128
};
#define MAX_GROUPS 128

// Control words of a forward call at 0 (status: no error), by one workgroup. With keep_errors (a
// deferred call) the error words keep what earlier calls on the work space set: the lowest failing
// element's op status, the time-out and the index flag.
__device__ __forceinline__ void init_ctl(uint32_t* ctl, int keep_errors) {
  for (int i = threadIdx.x; i < CTL_WORDS; i += blockDim.x) {
    const bool err = i == CTL_STATUS || i == CTL_TIMEOUT || i == CTL_BADIDX;
    if (keep_errors && err) continue;
    ctl[i] = (i == CTL_STATUS) ? kStatusOk : 0u;
  }
}
// Clears the backward's control words, by one workgroup: slot counters, group barrier counters, the
// wait flags and the index flag (the op status of the forward goes: the backward reports only its
// own). keep_errors: a deferred call; the error words stay as earlier calls left them.
__device__ __forceinline__ void zero_ctl_bwd(uint32_t* ctl, int keep_errors) {
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

// Whether the work space holds the schedule of a forward of these sizes. A backward takes its indices
// from there; in a work space that no such forward wrote they are anything, so its kernels leave
// without following one, and the call reports SLSTM_EINDEX.
__device__ __forceinline__ bool has_plan(const uint32_t* ctl, uint64_t key) {
  return ctl[CTL_KEY] == (uint32_t)key && ctl[CTL_KEY + 1] == (uint32_t)(key >> 32);
}

// Gate-interleaved ("permuted") column order used inside the library: column 4*u + k
// holds gate k (0=i, 1=f, 2=g, 3=o) of hidden unit u. The caller's order is k*H + u.
__device__ __forceinline__ int perm_to_orig(int np, int H) { return (np & 3) * H + (np >> 2); }

__device__ __forceinline__ float bf16_bits_to_f32(bf16_t v) {
  return __uint_as_float(((uint32_t)v) << 16);
}
// Round to bfloat16, nearest-even (the hardware conversion on gfx950).
__device__ __forceinline__ bf16_t f32_to_bf16_bits(float f) {
  __bf16 h = static_cast<__bf16>(f);
  return __builtin_bit_cast(bf16_t, h);
}

__device__ __forceinline__ f32x4 mfma_bf16_16x16x32(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Gate nonlinearities from the hardware base-2 exponential and reciprocal (about one ulp
// each): sigma(z) = 1 / (1 + 2^(-z log2 e)); tanh(x) = 2 sigma(2x) - 1. Absolute error is
// a few 1e-7 over the whole range; both saturate correctly (2^(+inf) = inf gives 0, 2^(-inf)
// = 0 gives 1) and need no branch.
__device__ __forceinline__ float sigmoidf_(float z) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
__device__ __forceinline__ float tanhf_(float x) {
  return 2.f * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-2.8853900817779268f * x)) - 1.f;
}

__device__ __forceinline__ unsigned xcc_id() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 0xf;
}

// Buffer descriptor of `bytes` bytes (an offset past them reads 0 instead of faulting; at most 4 GiB).
// Data that another CU wrote earlier in the same kernel is read with the sc1 cache policy, which
// bypasses this CU's L1 and reads the XCC's L2: a line that L1 cached before the other CU's write is
// never returned stale.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, size_t bytes) {
  uint32_t n = bytes > 0xffffffffu ? 0xffffffffu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n, 0x00020000);
}
constexpr int kSc1 = 16;  // cache-policy bit SC1 of gfx94x/gfx950 memory instructions
__device__ __forceinline__ float canon_nan(float h) { return h == h ? h : __builtin_nanf(""); }

// A producer index s read at step t must lie in [-1, t) (the state read at step t) or
// [-1, t] (the state at the top after step t). An index outside its range means that the
// producer table passed in was not the forward's, or that a read returned stale data: the
// kernel raises CTL_BADIDX (the call then reports SLSTM_EINDEX), and uses -1 so that every
// access stays inside the arrays.
__device__ __forceinline__ void raise_badidx(uint32_t* ctl) {
  __hip_atomic_store(&ctl[CTL_BADIDX], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int checked_src(int s, int hi, uint32_t* ctl) {
  if (s < -1 || s > hi) {
    raise_badidx(ctl);
    return -1;
  }
  return s;
}

// Group barrier for workgroups that all run on one XCC (one shared L2).
// Each wave waits until its own stores are acknowledged by L2, the workgroup meets at
// s_barrier, one lane adds to the group counter and polls it with L1-bypassing loads.
// Data written by other workgroups before the barrier must then be read past the L1 (sc1). Returns
// true when the spin limit ran out (or another group's did): the caller must then leave its loop so that every wave of the grid exits.
// Arrival half: stores acknowledged, workgroup met, the group counter incremented. The lane that
// polls is one of the last wave, whose threads have the fewest loads of their own in flight when
// the workgroup prefetches between the halves (loads return in order, a poll behind them).
__device__ __forceinline__ bool group_poller() { return threadIdx.x + 64 == blockDim.x; }
// (solo: the group is one workgroup and has then met; it neither counts nor polls. Training step of 599
// pushes at H = 32: 4348 -> 3573 us.)
__device__ __forceinline__ void group_arrive(uint32_t* ctr, bool solo) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (!solo && group_poller()) __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// First poll of a wait, issued before other loads: its value is looked at in group_wait.
__device__ __forceinline__ uint32_t group_peek(uint32_t* ctr) {
  return group_poller() ? __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
}
// Waiting half: the lane polls the counter up to target (seen: the value of the first poll);
// returns true when the spin limit ran out (spin_limit failed polls) or another workgroup gave
// up. Work that needs no other workgroup's data can run between the two halves.
__device__ __forceinline__ bool group_wait(uint32_t* ctr, uint32_t target, uint32_t seen, uint32_t* ctl, int spin_limit,
                                           int* s_flag) {
  if (group_poller()) {
    int spins = 0, bad = 0;
    while (seen < target) {
      ++spins;
      if ((spins & 255) == 0 && __hip_atomic_load(&ctl[CTL_ABORT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
        bad = 1;
        break;
      }
      if (spins >= spin_limit) {
        __hip_atomic_store(&ctl[CTL_ABORT], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl[CTL_TIMEOUT], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bad = 1;
        break;
      }
      seen = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    *s_flag = bad;
  }
  __syncthreads();
  return *s_flag != 0;
}

// Claims this workgroup's (group, member) slot from the XCC it runs on, so that every
// group's members share one XCC. Groups are dealt to XCCs round-robin (group g on XCC
// g % 8); a workgroup with nothing to do gets group -1 and must exit.
__device__ __forceinline__ void claim_group_slot(uint32_t* slot_ctrs, int G, int NW, int* s_g, int* s_w) {
  if (threadIdx.x == 0) {
    unsigned x = xcc_id();
    int g = -1, w = 0;
    if (x < 8) {
      unsigned slot = __hip_atomic_fetch_add(&slot_ctrs[x], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int per_xcc = NW * ((G + 7) / 8);
      if ((int)slot < per_xcc) {
        int lg = (int)slot / NW;
        w = (int)slot % NW;
        g = lg * 8 + (int)x;
        if (g >= G) g = -1;
      }
    }
    *s_g = g;
    *s_w = w;
  }
  __syncthreads();
}

// LDS DMA (global memory -> LDS, 16 bytes or 4 bytes per lane) written as inline assembly:
// the compiler then does not order every later LDS read behind it with a vmcnt(0) wait; a
// kernel that uses these counts its own waits. M0 holds the wave's LDS destination (lane i
// writes at M0 + i * size); writing M0 needs one wait state before the DMA. The buffer
// forms address descriptor base + soff (wave-uniform) + voff (the lane's offset, the only
// part the descriptor's range check covers).
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)p; }
// Buffer form: address = descriptor base + soff (wave-uniform) + voff (the lane's offset,
// the only part the descriptor's range check covers: a lane given kOOB reads no memory and
// writes zeros to its 16 LDS bytes). sc1 bypasses this CU's L1. An instruction immediate
// offset would move the LDS address as well (M0 + immediate + 16 * lane); these forms use none.
constexpr uint32_t kOOB = 0xffffffffu;
__device__ __forceinline__ void bdma16_sc1(rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lds) {
  lds = __builtin_amdgcn_readfirstlane(lds);   // wave-uniform by contract: kept in SGPRs
  soff = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen sc1 lds"
               ::"s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}
__device__ __forceinline__ void bdma16(rsrc_t r, uint32_t voff, uint32_t soff, uint32_t lds) {
  lds = __builtin_amdgcn_readfirstlane(lds);   // wave-uniform by contract: kept in SGPRs
  soff = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               ::"s"(lds), "v"(voff), "s"(r), "s"(soff) : "memory", "m0");
}
// Waits until at most N vector memory operations of this wave are outstanding (they
// complete in issue order).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N <= 63, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
  asm volatile("" ::: "memory");
}
// A sum with what its additions round off summed beside it, apart from the sum: where that is infinite the
// rest is NaN and is left out.
__device__ __forceinline__ void comp_add(float& s, float& e, float v) {
  const float z = s + v, w = z - s;
  e += (s - (z - w)) + (v - w);
  s = z;
}
__device__ __forceinline__ float comp_sum(float s, float e) { return __builtin_isfinite(e) ? s + e : s; }
// A copy of v the compiler cannot see through: what is computed from it is computed where it is
// used, instead of being kept in registers through a whole kernel.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
// Keeps v's register from being used again before this point. The compiler waits for all loads before it
// reuses the register of one that some path has not waited for (group_peek's value); between
// LDS DMAs that wait is for each DMA in turn.
__device__ __forceinline__ void hold(uint32_t v) { asm volatile("" ::"v"(v)); }
// Largest of 16 lanes (a DPP row), in every one of them.
__device__ __forceinline__ float max16(float m) {
  auto dpp = [](float v, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  m = fmaxf(m, dpp(m, std::integral_constant<int, 0xb1>()));    // quad_perm 1, 0, 3, 2
  m = fmaxf(m, dpp(m, std::integral_constant<int, 0x4e>()));    // quad_perm 2, 3, 0, 1
  m = fmaxf(m, dpp(m, std::integral_constant<int, 0x141>()));   // row_half_mirror
  return fmaxf(m, dpp(m, std::integral_constant<int, 0x140>()));  // row_mirror
}
// base + a 32-bit byte offset (scalar base, one offset register)
template <typename T>
__device__ __forceinline__ T* at32(T* base, uint32_t off) {
  return (T*)((uintptr_t)base + off);
}
// Wave-uniform value kept in a scalar register.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
