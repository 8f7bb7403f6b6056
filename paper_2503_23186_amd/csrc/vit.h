// Pieces of the Vision Transformer operators that the training step launches in its own grouping.
#pragma once
#include "common.h"
#include "../../include/cnnk_vit.h"

// whether the dense matrix-core kernels take a linear layer (vit_linear.hip)
bool linear_dense(long long rows, int K, int N, int dtype);

// cnnk_layernorm_bwd without its final sums: dx, and partial sums of dgamma and dbeta in `part`
// (cnnk_layernorm_workspace_bytes).  Arguments as checked by cnnk_layernorm_bwd.
int ln_bwd_rows_partial(const cnnk_ln_desc* d, const void* dy, const void* x, const float* gamma, const float* stats,
                        const void* dres, void* dx, float* part, hipStream_t st);
int ln_bwd_parts(const cnnk_ln_desc* d);       // rows of those partial sums

// The final sums of several tables of partial column sums [parts][2 * C] in one launch: out0 gets the first C columns,
// out1 the others.
constexpr int kColumnSumsMax = 32;
struct ColumnSums {
  int count;
  struct { const float* part; float *out0, *out1; int parts, C; } it[kColumnSumsMax];
};
int column_sums_group(const ColumnSums& t, hipStream_t st);

// cnnk_vit_embed_bwd on checked arguments; dbe null: the caller gets it elsewhere
int embed_bwd(const cnnk_embed_desc* d, const void* dtok, void* dz, float* dbe, float* dcls, float* dpos, hipStream_t st);
