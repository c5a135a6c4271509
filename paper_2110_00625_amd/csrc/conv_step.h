// SGD steps of convolutions from their partial weight gradients:
//
//     W[j][e] -= lr * sum_s partial[(j*S+s)][e]  and  b[j][r] -= lr * sum_s pbias[(j*S+s)][r]
//
// on the master's planes (split.h), for several layers: adds up the S partial gradients of four elements at a time in ascending order.
// Used by a launch of its own (conv.hip) and by spare workgroups of the MLP's updates (update_bf16.hip).
// The stepped bf16 values are also left in operand order for the next step's products (conv_flat.hip): a launch of its own for that was
// 4 - 5 us of a step (28x28 with channels 8-32-64, a round of four steps: 487 us with it, 479 without).
//
// What bounds it is latency, or with large layers the traffic of the partial sums (64 -> 128 channels, 16 learners of 16 ranges each: 75 MB in
// 19 us): sixteen of them on their way per lane, 16 bytes each.  As spare workgroups of the MLP's updates it adds 5 us to those of 28x28
// images with channels 8-32-64, 8 learners, where a launch of its own took 9.6 us.
#pragma once
#include "kavg_internal.h"
#include "fastdiv.h"
#include "split.h"

namespace kavg {

constexpr int STEP_GROUP = 8;
struct ConvSteps { ConvStep layer[STEP_GROUP]; uint32_t div_m[STEP_GROUP]; int div_s[STEP_GROUP]; int n, wgs; size_t lstride; float lr; };      // wgs: workgroups of 256 per learner

// element (output x, contraction k, tap) of a layer's weights in operand order (launch_pack_weights)
__device__ __forceinline__ uint16_t* frag_at(const FragPlace& f, int j, int x, int k, int tap) {
    const int slab = k >> 4, grp = slab / f.SL, it = grp * 9 * f.SL + tap * f.SL + slab - grp * f.SL;
    return f.frag + (size_t)j * f.lstride + ((size_t)(it * f.blocks + (x >> 5)) * 64 + (x & 31) + ((k >> 3) & 1) * 32) * 8 + (k & 7);
}

// workgroup b (of ConvSteps::wgs) of learner j.  (All counts are multiples of 8: four elements share an output and a tap.)
__device__ __forceinline__ void conv_step(const ConvSteps& a, int b, int j, int tid) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    int i0 = 0;
    while (i0 + 1 < a.n && b >= (a.layer[i0].n_w + a.layer[i0].n_b + 1023) / 1024) { b -= (a.layer[i0].n_w + a.layer[i0].n_b + 1023) / 1024; ++i0; }
    const ConvStep& q = a.layer[i0];
    const int e = (b * 256 + tid) * 4;
    if (e >= q.n_w + q.n_b) return;
    const bool is_w = e < q.n_w;
    const int i = is_w ? e : e - q.n_w, n = is_w ? q.n_w : q.n_b;
    const float* p = (is_w ? q.partial : q.pbias) + (size_t)j * q.S * n + i;
    uint16_t* const hi = (is_w ? q.whi : q.bhi) + (size_t)j * a.lstride + i;
    uint16_t* const lo = (is_w ? q.wlo : q.blo) + (size_t)j * a.lstride + i;
    const u32x2 h = *(const u32x2*)hi, l = *(const u32x2*)lo;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int r = 0; r < q.S; r += 16) {
        f32x4 t[16];                                          // (places beyond the last are read from there, and not used)
#pragma unroll
        for (int u = 0; u < 16; ++u) t[u] = *(const f32x4*)(p + (size_t)min(r + u, q.S - 1) * n);
#pragma unroll
        for (int u = 0; u < 16; ++u) if (r + u < q.S) s += t[u];
    }
    u32x2 oh, ol;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        uint32_t b0, b1, h2, l2;
        split_join2(h[c], l[c], b0, b1);
        const float w0 = __builtin_bit_cast(float, b0) - a.lr * s[2 * c], w1 = __builtin_bit_cast(float, b1) - a.lr * s[2 * c + 1];
        split_pack2(__builtin_bit_cast(uint32_t, w0), __builtin_bit_cast(uint32_t, w1), h2, l2);
        oh[c] = h2; ol[c] = l2;
    }
    *(u32x2*)hi = oh;
    *(u32x2*)lo = ol;
    if (is_w && (q.fwd.frag || q.bwd.frag)) {
        const int ot = (int)fastdiv((uint32_t)i, a.div_m[i0], a.div_s[i0]), c = i - ot * q.c_in, o = ot / 9, tap = ot - 9 * o;
        if (q.fwd.frag) *(u32x2*)frag_at(q.fwd, j, o, c, tap) = oh;
        if (q.bwd.frag) {
            uint16_t* to = frag_at(q.bwd, j, c, o, tap);      // (rows c .. c+3 of one block)
#pragma unroll
            for (int u = 0; u < 4; ++u) to[u * 8] = (uint16_t)(oh[u >> 1] >> (16 * (u & 1)));
        }
    }
}

// the first of n layers (at most STEP_GROUP) as arguments
inline ConvSteps conv_steps(const ConvStep* layers, int n, size_t lstride, float lr) {
    ConvSteps a = {};
    a.n = n < STEP_GROUP ? n : STEP_GROUP;
    a.lstride = lstride; a.lr = lr;
    for (int i = 0; i < a.n; ++i) {
        a.layer[i] = layers[i];
        fastdiv_make((uint32_t)layers[i].c_in, &a.div_m[i], &a.div_s[i]);
        a.wgs += (layers[i].n_w + layers[i].n_b + 1023) / 1024;
    }
    return a;
}

}  // namespace kavg
