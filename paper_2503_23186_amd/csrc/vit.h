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
// the final sums of several layer norms of one descriptor in one launch
constexpr int kLnGroupMax = 64;
struct LnFinalizeTable {
  int count;
  const float* part[kLnGroupMax];
  float* dgamma[kLnGroupMax];
  float* dbeta[kLnGroupMax];
};
int ln_bwd_finalize_group(const cnnk_ln_desc* d, const LnFinalizeTable& t, hipStream_t st);

// cnnk_vit_embed_bwd on checked arguments; dbe null: the caller gets it elsewhere
int embed_bwd(const cnnk_embed_desc* d, const void* dtok, void* dz, float* dbe, float* dcls, float* dpos, hipStream_t st);
