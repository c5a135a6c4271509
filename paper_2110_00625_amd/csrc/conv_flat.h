// 3x3 convolution, forward and data gradient, for images of any width (conv_flat.hip).
#pragma once
#include "kavg_internal.h"
#include "conv_pool.h"

namespace kavg {

// Positions with margins (conv_flat.hip): table[i] = pixel (n H + h) W + w of position i - (W+1) - 1, or -1 on a margin.
int conv_flat_table_len(int B, int H, int W);
hipError_t launch_flat_table(int32_t* table, int B, int H, int W, hipStream_t st);

// Weights in the order in which a wavefront of the kernels takes them as matrix operands, see conv_flat.hip.
struct FlatPlan {
    int CK, NB, PWAVES;          // channels per group; output blocks per wavefront; wavefronts side by side in positions
    int slabs, blocks;           // 16-channel slabs of the contraction; 32-channel blocks of the output (padded)
    size_t frag_elems() const { return (size_t)9 * slabs * blocks * 512; }
};
// workgroups of one direction of a layer with c_n channels out, as long as they are many (where they are few, twice as many)
int conv_flat_workgroups(int P, int B, int H, int W, int c_n);
// the plan of one direction of a layer: c_k channels contracted, c_n channels out; false: not covered
bool conv_flat_plan(int B, int H, int W, int c_k, int c_n, FlatPlan* plan);
bool conv_flat_plan_last(int B, int H, int W, int c_k, int c_n, FlatPlan* plan);      // data gradient of the last convolution, below the mean over the positions

// one layer of launch_pack_weights: W [c_out][9][c_in] (hi plane) into operand order, for the forward pass and,
// where bwd is not null, for the data gradient; lstride: elements between learners
struct PackLayer {
    const uint16_t* w;
    uint16_t* fwd; size_t fwd_lstride; FlatPlan fwd_plan;
    uint16_t* bwd; size_t bwd_lstride; FlatPlan bwd_plan;
    int c_in, c_out;
};
hipError_t launch_pack_weights(const PackLayer* layers, int n, size_t w_lstride, int P, hipStream_t st);

// Partial sums over the positions (ConvCall::pool_sums): places of images, of `channels` floats each, per wavefront;
// elements in all; 0: images too small.  pooled[P][B][c] = bf16(mean) out of them.
int conv_pool_slots(int P, int B, int H, int W, const FlatPlan& plan);
size_t conv_pool_elems(int P, int B, int H, int W, const FlatPlan& plan);
PoolSums conv_pool_sums(const float* sums, const FlatPlan& plan, int P, int B, int H, int W);
hipError_t launch_pool_finish(const PoolSums& q, void* pooled, int P, int B, int c, hipStream_t st);

// (These two compute their positions and read no table; the argument is the weight gradient's.  tests/test_boundary_cpu.py calls them so.)
// c.out = relu(conv(c.in, W) + b), or c.bits and c.pool_sums; gather != null: the images are rows gather[learner * gstride + n] of the data set X
hipError_t conv_flat_forward(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t* table, const void* X,
                             const int32_t* gather, long gstride, hipStream_t st);
// c.dz_in = [c.in > 0] * (transposed convolution of c.dz with W).  dpool != null (the last convolution, below the
// mean over the positions): c.dz is not read; the gradient images are formed while loading from c.bits and
// dpool [P][B][c_out], as pool_backward_kernel would.
hipError_t conv_flat_backward_data(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t* table, const void* dpool,
                                   hipStream_t st);

// Weight gradient (conv_flat_wgrad.hip): ranges of positions per learner, or 0 when the kernel does not cover the layer.
// first: the first convolution (gathered images of 8 channels).
int conv_flat_wgrad_splits(int P, int B, int H, int W, int c_in, int c_out, bool first);
// partial[learner * splits + range][c_out][9 c_in] (fp32) and the column sums of dZ in partial_bias; c.splits as above.
// gather (8 input channels) and dpool as in the functions above it.
hipError_t conv_flat_wgrad(const ConvCall& c, const int32_t* table, const void* X, const int32_t* gather, long gstride,
                           const void* dpool, hipStream_t st);


}  // namespace kavg
