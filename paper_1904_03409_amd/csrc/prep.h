// Arguments of the operand preparation kernels (prep.hip).
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <hip/hip_runtime.h>

struct GatherArgs {
  const int32_t* top; uint32_t* ctl;
  const float *hcell, *h0, *ccell, *c0;
  float *htop, *ctop;              // [T][B][H], null: not wanted
  int T, B, H, ll;                 // 2^ll lanes per row
};

struct PrepFwdArgs {
  int I, Ip, H, Hs, H4s, B, G, N0, NW, KS;
  int n_w, n_u;                    // blocks of the W tiles and of the U fragments; the rest: initial states
  const float* W; const float* U; const float* h0; const float* c0;
  uint16_t* wt;                    // [S][4H][Ip]
  uint16_t* wp;                    // [S][I][H4s]
  uint4* uf; int32_t* uexp;
  uint16_t* hq; size_t hplane;
  uint16_t* h3;                    // fp32 mode with a backward: [3][N0 + B][Hs], else null
  int32_t* rinit;
  float* cn;
  uint32_t* ctl; int keep_errors;
};

struct PrepBwdArgs {
  int T, B, H, G, NW, KS;
  int n_u;                         // blocks of the U^T fragments; the rest: interval sums
  const float* U;
  uint4* ub; float* uinv;
  const float* d; const int32_t* gslot; float* sums;   // upstream gradient, its slots, the sums
  uint32_t* ctl; uint64_t key; int clear, keep_errors;   // clear: this launch clears the control words
};
