// Level schedule of the stack recurrence, shared by the host library and the kernels.
//
// A push step makes a state ("node"); its parent is the state at the stack pointer when the
// push ran. A node at depth d reads only its parent at depth d - 1, so all nodes of one depth
// (over every step and every batch element) can be computed together, and the serial chain is
// the stack depth instead of T. Pop and hold steps write states nobody reads: they are leaves,
// computed all at once after the last level. Every step that reads one state shares the
// product h U.
//
// Node ids: push nodes 0 .. P-1 (P = number of pushes), by group, then level, then element,
// then time, so that a level of a group is a contiguous range and the push children of
// consecutive nodes are consecutive nodes of the next level; the initial state of the i-th
// element of group g is node N0 + goff(g) + i with N0 = T*B. Element b belongs to group b % G.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

constexpr int kLevMaxGroups = 128;      // barrier counters, one 64-byte line per group
constexpr int kLevUnits = 32;           // hidden units per workgroup
constexpr int kLevThreads = 512;

// batch elements of group g and the index of its first one among the groups' elements
__host__ __device__ inline int lev_bg(int B, int G, int g) { return B / G + (g < B % G ? 1 : 0); }
__host__ __device__ inline int lev_goff(int B, int G, int g) { return g * (B / G) + (g < B % G ? g : B % G); }

// Byte offset of a push node's dA entries (unit u) in a plane. fp32 mode (NP = 2): 32 bits hold it, because T*B*16H
// bytes do (the entry points' limit) and a row has 8H, padded to 16 bytes. bf16 mode: the limit is T*B*8H,
// and the padding of an odd H (H = 3: 32 bytes a row instead of 24) takes a plane past 4 GiB.
template <int NP>
__host__ __device__ inline size_t lev_da_off(int c, int H4s, int u) {
  if (NP == 2) return 2u * ((uint32_t)c * (uint32_t)H4s + 4u * (uint32_t)u);
  return 2 * ((size_t)c * (size_t)H4s + 4 * (size_t)u);
}

// Index arrays written by k_plan.
struct LevIdx {
  int32_t* order;    // [N0]: step t*B + b of node i (i < P); of the leaves, by group, element and time (P <= i < N0)
  int32_t* opar;     // [N0]: parent node of entry i
  int32_t* cs;       // [N0 + B]: first push child of a node (its children end where the next node's begin)
  int32_t* loff;     // [G][T + 4]: first node of level d = 1 .. D + 1 of a group (level D + 1 and D + 2: the end)
  int32_t* gmax;     // [G]: deepest level D
  // For a backward. Internal nodes (with push children) are numbered by group, level and node: a group's
  // numbers start at the count of nodes of the groups before it.
  int32_t* ics;      // [N0 + B]: its first child (its children end where the next number's begin)
  int32_t* ioff;     // [G][T + 4]: first internal number of level d = 0 .. D + 1
  int32_t* cidx;     // [N0 + B]: internal number of a node; ~(the next internal number) if it has no children
  int32_t* kin;      // [N0]: of a push node, 2 * (its internal number, or -1) + (1 if it was popped)
  int32_t* gslot;    // [N0]: slot that the upstream gradient of step t*B + b is summed into (k_prep_bwd)
};

struct PlanArgs {
  int T, B, G, cap;             // cap = T + 2 slots per walk array
  const int8_t* ops;
  int32_t* ptr;                 // [T + 1][B]
  int32_t* top;                 // [T][B]
  LevIdx ix;
  int32_t* cnt;                 // [B][cap]: pushes of an element at a depth, then their first node id
  int32_t* elem;                // [3][B]: deepest level, pushes, leaf offset of an element
  int32_t* walk;                // [G][2][cap] when the walk arrays do not fit in LDS
  uint32_t* ctl;
  uint64_t key;                 // of the sizes (CTL_KEY); 0: no backward follows, nothing is written for one
};

struct LevFwdArgs {
  int T, B, H, Hs, G, NW, N0, spin_limit;
  LevIdx ix;
  float* hu;                    // [N0 + B][4H]: x W + b of a push node until its level has run, then h U of the node
  uint16_t* hq; size_t hplane;  // recurrent planes of h: [NP][N0 + B][Hs]
  float* cn;                    // [N0 + B][H]: c of a node
  float* hcell; float* ccell;   // [T][B][H]
  // for a backward (null: not kept): gate activations [P][4H] and the parent's c [P][H] of a push
  // node, fp32 mode also h as bf16 planes [3][N0 + B][Hs]
  float* stash; float* cpn; uint16_t* h3;
  const uint4* uf; const int32_t* uexp; // U fragments and the exponents of their units' inverse scales (k_prep_fwd)
  const int32_t* rinit;         // [B]: exponent of the inverse scale of an initial state's row, by node (fp32 mode)
  uint32_t* ctl;
  long long* clk;
};

struct LevBwdArgs {
  int T, B, H, H4s, G, NW, N0, spin_limit;
  LevIdx ix;
  const float* cpn; const float* stash;
  const float* gf;              // [2 (N0 + B)][H] interval sums of dh_top (k_prep_bwd)
  const float* gc;              // the same of dc_top, or null
  float* eg;                    // [N0 + B][H] gradient of h that reaches an internal node from its children
  float* dcs;                   // the same of c
  uint16_t* dap; size_t dplane; // bf16 planes of dA: [S][P][H4s]
  uint16_t* sx; size_t xplane;  // recurrent planes of the children's dA sums: [NP][N0 + B][H4s]
  float* sxs;                   // [N0 + B][NW]: inverse scale of a row's 128 columns of a workgroup (fp32 mode)
  const uint4* ub; const float* uinv;   // U^T fragments and the inverse scales of their units (k_prep_bwd); kDaExp
  float* db_part;               // [G][4H]
  float* dh0; float* dc0;
  uint32_t* ctl; uint64_t key;
  long long* clk;
};

// K chunks of 32 compiled into the recurrent kernels (NP planes), at least the NW workgroups of a
// group. fp32 mode: powers of two, so that a wave of the backward contracts whole or equal parts of
// the 128-column pieces that share a scale.
inline int lev_ks(int NP, int NW) {
  for (int ks : {2, 4, 8, 12, 16, 24, 32})
    if (ks >= NW && (NP == 1 || ks != 12)) return ks;
  return -1;
}
// Rows per pass of the forward: two row tiles while two buffers of them fit LDS
constexpr int lev_fwd_rt(int NP, int ks) { return ks * NP <= 16 ? 2 : 1; }
constexpr int kLevHuLd = kLevUnits * 4 + 4;
constexpr size_t lev_fwd_lds(int NP, int ks) {
  // two buffers each of the rows' planes, of h U (in two halves of K) and of the parents' c
  return (size_t)2 * lev_fwd_rt(NP, ks) * 16 * (ks * 64 * NP + 2 * kLevHuLd * 4 + kLevUnits * 4);
}
// Backward: children per pass of the cell and parents per pass of the sums; internal nodes of a
// level whose gradients stay in LDS; the exchange's row slices of the eight waves (or the cell's
// children: dA, dc f and the gradient of the interval after them, 6 floats per unit)
constexpr int kLevPars = 32, kLevKeep = 24;
constexpr int lev_bwd_kids(int NP, int ks) { return NP == 2 && ks > 8 ? 32 : 64; }   // (registers)
constexpr size_t lev_bwd_region(int NP, int ks) {
  const size_t x = (size_t)8 * NP * (ks / 2) * 1024, c = (size_t)lev_bwd_kids(NP, ks) * kLevUnits * 24;
  return x > c ? x : c;
}
constexpr size_t lev_bwd_lds(int NP, int ks) {
  return lev_bwd_region(NP, ks) + (size_t)8 * 16 * 36 * 4 + (size_t)2 * 2 * kLevKeep * kLevUnits * 4;
}

#define LEV_CASES(X) \
  X(2, 2) X(2, 4) X(2, 8) X(2, 16) \
  X(1, 2) X(1, 4) X(1, 8) X(1, 12) X(1, 16) X(1, 24) X(1, 32)

hipError_t launch_lev_fwd(const LevFwdArgs& a, int NP, int KS, int grid, hipStream_t st);
hipError_t launch_lev_bwd(const LevBwdArgs& a, int NP, int KS, int grid, hipStream_t st);
