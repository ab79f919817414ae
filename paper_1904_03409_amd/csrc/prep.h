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
  uint4* uf; float* uinv;
  uint16_t* hq; size_t hplane;
  uint16_t* h3;                    // fp32 mode with a backward: [3][N0 + B][Hs], else null
  float* rinit;
  float* cn;
};

struct PrepBwdArgs {
  int T, B, H, NW, KS, n_u;
  const float* U; const int8_t* ops; const int32_t* top; const int32_t* order;
  uint4* ub; float* uinv;
  uint32_t* ctl;
};
