// Dense bf16 matrix products of linear layers (gemm_bf16.hip).  rows = tokens, K = input features,
// N = output features; x [rows][K], w [N][K], y / dy [rows][N], dw [N][K] float.
#pragma once
#include "common.h"

// K and N multiples of 8, every matrix below 2 GiB
bool gemm_bf16_supported(long long rows, int K, int N);
// y = x w^T + bias (bias may be null); with res (not with gelu): y = res + (x w^T + bias as stored);
// with gelu: u = x w^T + bias, y = gelu(u as stored)
int gemm_bf16_fwd(long long rows, int K, int N, const bf16_t* x, const bf16_t* w, const float* bias, const bf16_t* res, bool gelu,
                  bf16_t* u, bf16_t* y, hipStream_t st);
// dx = dy w
int gemm_bf16_dgrad(long long rows, int K, int N, const bf16_t* dy, const bf16_t* w, bf16_t* dx, hipStream_t st);
// dg = dy w, du = dg (as stored) * gelu'(u): the data gradient through the layer and the activation before it.
// sums: [gemm_bf16_dgrad_gelu_parts][K] partial column sums of du before it is rounded, 16-byte aligned.
int gemm_bf16_dgrad_gelu_parts(long long rows, int K, int N);
int gemm_bf16_dgrad_gelu(long long rows, int K, int N, const bf16_t* dy, const bf16_t* w, const bf16_t* u, bf16_t* dg, bf16_t* du,
                         float* sums, hipStream_t st);
// dw = dy^T x (fp32); ws: gemm_bf16_wgrad_ws bytes of partial sums
size_t gemm_bf16_wgrad_ws(long long rows, int K, int N);
int gemm_bf16_wgrad(long long rows, int K, int N, const bf16_t* x, const bf16_t* dy, float* dw, void* ws, hipStream_t st);
// The same for up to gemm_bf16_wgrad_group_max() layers in one launch, each with (db not null) the column sums of
// its dy.  K and N multiples of 8, 16-byte aligned pointers, every matrix below 2 GiB.
struct GemmWgrad {
  const bf16_t* dy;    // [rows][N]
  const bf16_t* x;     // [rows][K]
  float* dw;           // [N][K]
  float* db;           // [N], nullable
  long long rows;
  int K, N;
};
// splits: parts of the rows that are summed apart and then added; the sums depend on it and on nothing else of the group
// (gemm_bf16_wgrad_group_splits: what fills the device best for a group).
int gemm_bf16_wgrad_group_max();
int gemm_bf16_wgrad_tiles(int K, int N);      // workgroups of a large group that one layer stands for
int gemm_bf16_wgrad_group_splits(const GemmWgrad* p, int n);               // these two read rows, K, N only
size_t gemm_bf16_wgrad_group_ws(const GemmWgrad* p, int n, int splits);
int gemm_bf16_wgrad_group(const GemmWgrad* p, int n, int splits, void* ws, hipStream_t st);
