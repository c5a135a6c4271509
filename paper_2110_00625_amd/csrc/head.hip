// Classifier head for small class counts (C <= 16), both precisions.
//
// With ten classes the last layer is a sliver: its forward product, the
// softmax cross-entropy, its data gradient and its weight update together
// move a few hundred KB per learner, and as four generic launches they cost
// four launch-plus-pipeline latencies.  Two kernels replace them:
//
//  head_forward_backward   one wavefront per sample row:
//        z = A_{L-1}[s] W_L^T + b_L                     (lanes split the contraction, butterfly sum)
//        loss_s = -log softmax(z)[y_s],  dZ_L[s] = (softmax(z) - onehot(y_s)) / B   (the 1/B_n of Algorithm 1)
//        dZ_{L-1}[s] = (dZ_L[s] W_L) * [A_{L-1}[s] > 0]
//  head_update             W_L <- W_L - lr * dZ_L^T A_{L-1},  b_L <- b_L - lr * colsum(dZ_L)
//        (the learner update of Algorithm 1 for the last layer; runs after the kernel above
//        because that one reads the weights of before the step; fp32: head_tile of gemm_f32.hip)
//
// Mixed precision follows the same rounding points as the generic kernels:
// products of bf16 operands accumulated in fp32, dZ_L and dZ_{L-1} rounded to
// bf16 (round to nearest even) before any use, logits / softmax / loss / bias
// / master update in fp32; the master is read and written as its two 16-bit
// planes (split.h), of which the bf16 one is the operand of the products.
#include "kavg_internal.h"
#include "head_update.h"
#include "split.h"
#include "wave_sum.h"

namespace kavg {

namespace {

constexpr int CMAX = 16;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    __bf16 h = (__bf16)x;                         // round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float bf16_round(float x) {
    return __builtin_bit_cast(float, (uint32_t)bf16_bits(x) << 16);
}

// A "piece" is what one lane loads at once: 8 bf16 or 1 float.  It is kept as loaded (r) and unpacked
// into floats (v) only where it is used, so that pieces can stay in registers cheaply.
template <bool BF16> struct Piece;
template <> struct Piece<true> {
    static constexpr int N = 8;
    u32x4 r;
    float v[8];
    __device__ __forceinline__ void fetch(const void* base, size_t elem) { r = *(const u32x4*)((const uint16_t*)base + elem); }
    __device__ __forceinline__ void clear() { r = (u32x4){0u, 0u, 0u, 0u}; }
    __device__ __forceinline__ void unpack() {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __builtin_bit_cast(float, r[i] << 16);
            v[2 * i + 1] = __builtin_bit_cast(float, r[i] & 0xFFFF0000u);
        }
    }
    __device__ __forceinline__ void load(const void* base, size_t elem) { fetch(base, elem); unpack(); }
};
template <> struct Piece<false> {
    static constexpr int N = 1;
    float r;
    float v[1];
    __device__ __forceinline__ void fetch(const void* base, size_t elem) { r = ((const float*)base)[elem]; }
    __device__ __forceinline__ void clear() { r = 0.f; }
    __device__ __forceinline__ void unpack() { v[0] = r; }
    __device__ __forceinline__ void load(const void* base, size_t elem) { fetch(base, elem); unpack(); }
};

struct HeadArgs {
    const void* act; int ld_act; size_t act_lstride;      // A_{L-1} [P][B][ld_act], or the data set when gather != null
    const int32_t* gather; long gather_lstride;           // row s of learner j is data row gather[j*gather_lstride + s]
    const void* wmul; size_t wmul_lstride;                // weights as multiplied: bf16 (hi) plane or fp32, [C][d]
    const float* bias; size_t w_lstride;                  // fp32 mode: the bias
    const uint16_t* bhi; const uint16_t* blo; size_t ws_lstride;     // bf16 mode: hi / lo planes of the bias (split.h)
    const int32_t* y;                                     // labels of the data set
    void* dz; int ldz; size_t dz_lstride;                 // dZ_L [P][B][ldz]
    void* dz_prev; size_t dz_prev_lstride;                // dZ_{L-1} [P][B][d], null for a single-layer model
    float* rowloss;                                       // [P][B]
    // fp32, FINISH > 0: A_{L-1} = relu(sum of the splits' partial products + bias of layer L-1), formed and written here
    const float* partial; size_t split_stride; int splits;
    const float* below_bias;                              // (stride w_lstride)
    int P, B, d, C;
};

// CT = compile-time bound on the class count (4, 8, 12 or 16): every loop over classes is fully
// unrolled and its loads are issued unconditionally (rows beyond C re-read row C-1 and are ignored),
// so that a lane's loads of a step go out together instead of one round trip per class.
// KEEP: the row has at most 128 pieces (two per lane); they are fetched once and stay in registers for
// the second pass (the data gradient) instead of being fetched again.
// FINISH: a row's activations are added up from the (at most FINISH) partial products of the layer below, in the order of
// finish_forward_kernel (gemm_f32.hip), whose launch this saves: every unit is read by one lane here anyway.
template <bool BF16, int CT, bool KEEP, int FINISH>
__global__ void __launch_bounds__(256) head_forward_backward_kernel(HeadArgs a) {
    constexpr int N = Piece<BF16>::N;
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);      // one wavefront per sample row
    const int learner = blockIdx.y;
    if (row >= a.B) return;                                   // whole wavefront leaves together
    const int32_t* g = a.gather + (long)learner * a.gather_lstride;
    const int sample = g[row];                                // data row of this sample (labels; inputs when L = 1)
    const size_t arow = a.act_lstride ? (size_t)learner * a.act_lstride + (size_t)row * a.ld_act
                                      : (size_t)sample * a.ld_act;
    const void* W = BF16 ? (const void*)((const uint16_t*)a.wmul + (size_t)learner * a.wmul_lstride)
                         : (const void*)((const float*)a.wmul + (size_t)learner * a.wmul_lstride);
    const int pieces = a.d / N;
    const int label_raw = a.y[sample];
    float bias_c[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int cc = c < a.C ? c : a.C - 1;
        if (BF16) {
            const size_t at = (size_t)learner * a.ws_lstride + cc;
            bias_c[c] = __builtin_bit_cast(float, split_join(a.bhi[at], a.blo[at]));
        } else {
            bias_c[c] = a.bias[(size_t)learner * a.w_lstride + cc];
        }
    }
    size_t wrow[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) wrow[c] = (size_t)(c < a.C ? c : a.C - 1) * a.d;

    // the partial products of a unit, requested together (those beyond the last re-read it and are not added)
    auto request = [&](float (&t)[FINISH + 1], size_t unit) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < FINISH; ++s) t[s] = a.partial[min(s, a.splits - 1) * a.split_stride + arow + unit];
        t[FINISH] = a.below_bias[(size_t)learner * a.w_lstride + unit];
    };
    auto finish = [&](const float (&t)[FINISH + 1]) __attribute__((always_inline)) {
        float z = 0.f;
#pragma unroll
        for (int s = 0; s < FINISH; ++s) if (s < a.splits) z += t[s];
        return fmaxf(z + t[FINISH], 0.f);
    };
    float* const act_out = FINISH ? (float*)const_cast<void*>(a.act) : nullptr;

    float acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = 0.f;
    Piece<BF16> xs[KEEP ? 2 : 1], ws[CT][KEEP ? 2 : 1];
    if constexpr (KEEP) {
        float parts[2][FINISH + 1];
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int q = lane + 64 * it;
            const size_t qq = (size_t)(q < pieces ? q : pieces - 1) * N;      // clamped: no predicated loads
            if constexpr (FINISH > 0) request(parts[it], qq); else xs[it].fetch(a.act, arow + qq);
#pragma unroll
            for (int c = 0; c < CT; ++c) ws[c][it].fetch(W, wrow[c] + qq);
        }
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            if constexpr (FINISH > 0) {
                xs[it].r = finish(parts[it]);
                if (lane + 64 * it < pieces) act_out[arow + lane + 64 * it] = xs[it].r;
            }
            if (lane + 64 * it >= pieces) xs[it].clear();                      // contributes nothing to either pass
            xs[it].unpack();
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                ws[c][it].unpack();
#pragma unroll
                for (int e = 0; e < N; ++e) acc[c] = fmaf(xs[it].v[e], ws[c][it].v[e], acc[c]);
            }
        }
    } else {
        for (int q = lane; q < pieces; q += 64) {
            Piece<BF16> x, w[CT];
            float parts[FINISH + 1];
            if constexpr (FINISH > 0) request(parts, q); else x.load(a.act, arow + (size_t)q * N);
#pragma unroll
            for (int c = 0; c < CT; ++c) w[c].load(W, wrow[c] + (size_t)q * N);
            if constexpr (FINISH > 0) { x.r = finish(parts); x.unpack(); act_out[arow + q] = x.r; }
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int e = 0; e < N; ++e) acc[c] = fmaf(x.v[e], w[c].v[e], acc[c]);
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        acc[c] = dpp_wave_sum(acc[c]) + bias_c[c];
        if (c < a.C) mx = fmaxf(mx, acc[c]);
    }
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CT; ++c) if (c < a.C) sum += expf(acc[c] - mx);
    const int label = label_raw < 0 ? 0 : (label_raw >= a.C ? a.C - 1 : label_raw);   // validated; never index outside
    const float invB = 1.0f / (float)a.B;
    float gz[CT];
    float zy = 0.f;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        gz[c] = 0.f;
        if (c < a.C) {
            const float p = expf(acc[c] - mx) / sum;
            gz[c] = (p - (c == label ? 1.0f : 0.0f)) * invB;
            if (BF16) gz[c] = bf16_round(gz[c]);
            if (c == label) zy = acc[c];
        }
    }
    if (lane == 0) a.rowloss[(size_t)learner * a.B + row] = -(zy - mx - logf(sum));
    if (lane < a.ldz) {                                       // dZ_L row, pad columns zero
        float mine = 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) if (c == lane) mine = gz[c];
        const size_t at = (size_t)learner * a.dz_lstride + (size_t)row * a.ldz + lane;
        if (BF16) ((uint16_t*)a.dz)[at] = bf16_bits(mine); else ((float*)a.dz)[at] = mine;
    }
    if (!a.dz_prev) return;

    // dZ_{L-1}[s][k] = (sum_c dZ_L[s][c] W_L[c][k]) * [A_{L-1}[s][k] > 0]      (gz[c] = 0 beyond C)
    auto data_gradient = [&](int q, Piece<BF16>& x, Piece<BF16> (&w)[CT]) {
        float da[N];
#pragma unroll
        for (int e = 0; e < N; ++e) da[e] = 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int e = 0; e < N; ++e) da[e] = fmaf(gz[c], w[c].v[e], da[e]);
#pragma unroll
        for (int e = 0; e < N; ++e) da[e] = x.v[e] > 0.f ? da[e] : 0.f;
        const size_t at = (size_t)learner * a.dz_prev_lstride + (size_t)row * a.d + (size_t)q * N;
        if (BF16) {
            u32x4 o;
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = (uint32_t)bf16_bits(da[(2 * i) % N]) | ((uint32_t)bf16_bits(da[(2 * i + 1) % N]) << 16);
            *(u32x4*)((uint16_t*)a.dz_prev + at) = o;
        } else {
            ((float*)a.dz_prev)[at] = da[0];
        }
    };
    if constexpr (KEEP) {
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int q = lane + 64 * it;
            if (q < pieces) {
                Piece<BF16> w[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) { w[c] = ws[c][it]; w[c].unpack(); }
                xs[it].unpack();
                data_gradient(q, xs[it], w);
            }
        }
    } else {
        for (int q = lane; q < pieces; q += 64) {
            Piece<BF16> x, w[CT];
            x.load(a.act, arow + (size_t)q * N);
#pragma unroll
            for (int c = 0; c < CT; ++c) w[c].load(W, wrow[c] + (size_t)q * N);
            data_gradient(q, x, w);
        }
    }
}

__global__ void __launch_bounds__(256) head_update_bf16_kernel(HeadStep a) {
    __shared__ __align__(16) float xch[HEAD_LDS / 4];
    head_step(a, blockIdx.x, gridDim.z > 1 ? (int)blockIdx.z : -1, blockIdx.y, xch);
}

HeadArgs make_args(const LayerCall& c, const int32_t* y, const int32_t* idx, long idx_lstride, float* rowloss, bool bf16) {
    HeadArgs a = {};
    a.act = c.in; a.ld_act = c.ld_in; a.act_lstride = c.gather ? 0 : c.in_stride;
    a.gather = idx; a.gather_lstride = idx_lstride;
    a.wmul = bf16 ? (const void*)c.ws : (const void*)c.w;
    a.wmul_lstride = bf16 ? c.ws_stride : c.w_stride;
    a.bias = c.b; a.w_lstride = c.w_stride;
    a.bhi = c.bhi; a.blo = c.blo; a.ws_lstride = c.ws_stride;
    a.y = y;
    a.dz = (void*)c.dz; a.ldz = c.ld_dz; a.dz_lstride = c.dz_stride;
    a.dz_prev = c.dz_prev; a.dz_prev_lstride = c.dz_prev_stride;
    a.rowloss = rowloss;
    a.P = c.P; a.B = c.B; a.d = c.d_in; a.C = c.d_out;
    return a;
}

}  // namespace

bool head_supported(int C) { return C <= CMAX; }

namespace {
template <bool BF16, bool KEEP, int FINISH>
void launch_fb2(const HeadArgs& a, dim3 grid, hipStream_t st) {
    if (a.C <= 4) hipLaunchKernelGGL((head_forward_backward_kernel<BF16, 4, KEEP, FINISH>), grid, dim3(256), 0, st, a);
    else if (a.C <= 8) hipLaunchKernelGGL((head_forward_backward_kernel<BF16, 8, KEEP, FINISH>), grid, dim3(256), 0, st, a);
    else if (a.C <= 12) hipLaunchKernelGGL((head_forward_backward_kernel<BF16, 12, KEEP, FINISH>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((head_forward_backward_kernel<BF16, 16, KEEP && !BF16, FINISH>), grid, dim3(256), 0, st, a);   // bf16 x 16 classes: too many registers to keep
}
template <bool BF16, int FINISH>
void launch_fb(const HeadArgs& a, dim3 grid, hipStream_t st) {
    const int pieces = a.d / Piece<BF16>::N;
    if (pieces <= 128) launch_fb2<BF16, true, FINISH>(a, grid, st); else launch_fb2<BF16, false, FINISH>(a, grid, st);
}
}  // namespace

hipError_t head_forward_backward(const LayerCall& c, const int32_t* y, const int32_t* idx, long idx_lstride,
                                 float* rowloss, int bf16, const LayerCall* below, hipStream_t st) {
    HeadArgs a = make_args(c, y, idx, idx_lstride, rowloss, bf16 != 0);
    dim3 grid((c.B + 3) / 4, c.P);
    if (below) {
        a.splits = f32_forward_plan(c.P, c.B, below->d_in, below->d_out, nullptr);
        if (bf16 || c.gather || c.in != below->out || !below->scratch || a.splits < 2 || a.splits > HEAD_SPLITS) return hipErrorInvalidValue;
        a.partial = (const float*)below->scratch; a.split_stride = (size_t)c.P * below->out_stride;
        a.below_bias = below->b;
        if (a.splits <= HEAD_SPLITS / 2) launch_fb<false, HEAD_SPLITS / 2>(a, grid, st); else launch_fb<false, HEAD_SPLITS>(a, grid, st);
    } else if (bf16) {
        launch_fb<true, 0>(a, grid, st);
    } else {
        launch_fb<false, 0>(a, grid, st);
    }
    return hipGetLastError();
}

hipError_t head_update(const LayerCall& c, const int32_t* idx, long idx_lstride, hipStream_t st) {
    hipLaunchKernelGGL(head_update_bf16_kernel, dim3(head_blocks(c.d_in), c.P, head_class_groups(c.P, c.d_in, c.d_out)), dim3(256), 0, st,
                       head_step_args(c, idx, idx_lstride));
    return hipGetLastError();
}

}  // namespace kavg
