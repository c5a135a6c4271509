// The last layers of a small MLP, forward pass, loss and data gradients in one launch (chain_bf16.hip).
#pragma once
#include "kavg_internal.h"
#include "conv_pool.h"

namespace kavg {

constexpr int CHAIN_LAYERS = 6;              // layers a launch takes at most

// How many of the last layers of the MLP dims[0..L] one launch takes: 0, or n >= 1 for layers L-n+1 .. L, where that is
// faster than a launch each.  into_input: the gradient of the first layer's input is wanted (a convolution lies below).
int chain_layers(int P, int B, int L, const int* dims, bool into_input);

// calls[0..n-1]: those layers in ascending order.  Writes their activations (calls[].out), all dZ (calls[].dz) and, where
// calls[0].dz_prev is set, the gradient of the input rows; the loss of every sample into rowloss.  pool != null: the input rows are
// means that are formed here, and written to calls[0].in.
hipError_t bf16_chain(const LayerCall* calls, int n, const int32_t* y, const int32_t* idx, long idx_lstride, float* rowloss, const PoolSums* pool,
                      hipStream_t st);

}  // namespace kavg
