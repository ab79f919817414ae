// Launch descriptions of the contractions over bf16 planes (contract.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

// C(i, n) = sum_k A(i, k) B(n, k) for a range of entries i of the step list (levels.h): the push
// nodes [0, P) or the leaves [P, N0), cut to [lo, hi); A row i is array row i - lo.
enum { NT_XW = 0, NT_LEAF = 1, NT_DX = 2 };
struct NtArgs {
  int N, K;                          // K: columns of A and B (a multiple of 8; NT_LEAF with pre: 0)
  int pre;                           // NT_XW, NT_LEAF: the sums go on from C[i][N] (K taken in parts)
  int lo, hi, leaves, N0;
  const uint16_t* A; size_t aplane; int lda;
  const uint16_t* B; size_t bplane; int ldb;
  const uint32_t* ctl; uint64_t key; // CTL_NPUSHF; NT_DX: CTL_KEY
  // NT_XW: C[i][N] + bias; NT_DX: C[order[i]][N], and 0 in the rows of the leaves
  float* C; int ldc;
  const float* bias; int H;          // caller's column order
  const int32_t* order;
  // NT_LEAF: the cell of a step whose state nobody reads: gates = x W + b + h U of the parent
  const int32_t* opar; const float* hu; const float* cn; float* hcell; float* ccell;
};

// dW | dU: C(m, n) = sum over push nodes k of X(k, m) dA(k, n); rows m < I of x (array row k), the
// others of the state the node read (array row parent(k)). Split over K into `splits` partials.
struct TnArgs {
  int I, H, H4, splits, xt;          // xt: row tiles that cover x
  const uint16_t* X; size_t xplane; int ldx;
  const uint16_t* Hp; size_t hplane; int ldh; int hrows;
  const uint16_t* D; size_t dplane; int ldd;
  const int32_t* opar;
  const uint32_t* ctl; uint64_t key;
  float* part; size_t split_stride;  // [splits][I + H][4H]
};

// Whether a plane of state rows is past the reach of a buffer descriptor and its 32-bit offsets
constexpr bool tn_far(int rows, int ld) { return (size_t)rows * (size_t)ld * 2 > 0xffffffffu; }

// Block tiles: rows x columns, K step, by the row tiles of 16 per wave (MI: nt_mi, or in k_nt one to
// three quarters of it; the smallest has room for K steps of 64 in fp32 mode too)
constexpr int nt_mi(int S) { return S == 3 ? 4 : 8; }
constexpr int nt_bm(int S, int MI) { return (S == 3 ? 64 : 32) * MI; }
constexpr int nt_bn(int S) { return S == 3 ? 128 : 256; }
constexpr int nt_bk(int S, int MI) { return S == 3 && MI > 1 ? 32 : 64; }
constexpr size_t nt_lds(int S, int MI) { return (size_t)2 * S * (nt_bm(S, MI) + nt_bn(S)) * nt_bk(S, MI) * 2; }
constexpr size_t nt_leaf_lds(int S, int MI) { return (size_t)2 * nt_bm(S, MI) * (nt_bn(S) / 4 + 4) * 4; }   // h and c of a tile

// dW, dU and db from the partials, and the check of the caller's top and ops (contract.hip)
struct ReduceArgs {
  const float* part; int splits; size_t stride;
  const float* db_part; int groups;
  int I, H;
  float* dW; float* dU; float* db;
  int T, B, n_red;                   // n_red: blocks of the sums; the rest check
  const int8_t* ops; const int32_t* top; const int32_t* order;
  uint32_t* ctl; uint64_t key;
};

hipError_t launch_nt(const NtArgs& g, int S, int epi, hipStream_t st);
hipError_t launch_tn(const TnArgs& g, int S, hipStream_t st);
