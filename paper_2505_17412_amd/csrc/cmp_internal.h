// The learned compression module on one or two tensors at once (cmp_module.hip); the layer runs it on keys and values.
#pragma once
#include "ssa_internal.h"

struct CmpTensor {
  const void *x;               // [N][C] caller order
  const ssa_cmp_weights_t *w;
  void *xc;                    // forward: block tokens
  const float *dxc;            // backward: their gradient
  void *dx;                    //   added onto
  float *dpe, *dw, *dbias;
};

// Two regions: `in` (cmp_module_input_bytes) for the neighbour table and x + PE, which a backward pass can find there
// (prepared) from a forward pass on the same tensors, and `ws` (cmp_module_workspace) for the rest.
size_t cmp_module_input_bytes(const ssa_params_t *p, const ssa_blocks_t *b, int n);
size_t cmp_module_workspace(const ssa_params_t *p, const ssa_blocks_t *b, int n, bool backward);
int cmp_module_check(const CmpTensor &t, bool backward);
int cmp_module_forward(const ssa_params_t *p, const ssa_blocks_t *b, int n, const CmpTensor *t, void *in, void *ws, hipStream_t s);
int cmp_module_backward(const ssa_params_t *p, const ssa_blocks_t *b, int n, const CmpTensor *t, bool prepared, void *in, void *ws,
                        hipStream_t s);
