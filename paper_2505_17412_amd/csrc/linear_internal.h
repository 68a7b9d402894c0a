// Pieces of the linear-projection kernels that the layer composition calls directly (gfx950 only).
#pragma once

#include "ssa_internal.h"

struct GateJob;

// d_in, d_out multiples of 128 up to 16384; SSA_OK or the error the entry points report
int lin_check(int n_tokens, int d_in, int d_out);

// Y [M][O] (bf16) = sum over n_src <= 3 pairs of X_i [M][K_i] W_i[O][K_i]^T (+ bias [O]); every K_i a multiple of 128
int lin_nt_multi(int n_src, const void *const *X, const void *const *W, const int *K, const void *bias, int M, int O,
                 void *Y, hipStream_t s);

// Y_i [M][O_i] = X [M][K] W_i[O_i][K]^T (+ bias_i, may be null), i < n_dst <= 3, in one launch; checks and errors of
// ssa_linear_forward for each of them; gate: the gate predictor on the same X beside them, or null
int lin_forward_multi(int n_dst, int M, int K, const void *X, const void *const *W, const void *const *bias, const int *O,
                      void *const *Y, const GateJob *gate, hipStream_t s);

// wt_i [d_in][d_out_i] = w_i [d_out_i][d_in]^T, i < n, 1 or 3
void lin_transpose_w(int n, const void *const *w, const int *d_out, int d_in, void *const *wt, hipStream_t s);

// dw_i [d_out_i][d_in] (fp32) = dy_i^T x, dbias_i [d_out_i] (fp32, may be null) = column sums of dy_i, i < n, 1 or 3; ws: the
// sum of lin_dw_workspace() over them, 256-byte aligned
size_t lin_dw_workspace(int M, int d_in, int d_out);
void lin_dw(int n, int M, int d_in, const int *d_out, const void *x, const void *const *dy, float *const *dw,
            float *const *dbias, void *ws, hipStream_t s);
