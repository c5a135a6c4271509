// The SGD updates of several layers in one launch (KAVG_BF16), for models whose weights stay in the memory-side cache, and with
// learner momentum for those whose weights do not:
//
//     W_l <- W_l - lr * dZ_l^T A_{l-1};    b_l <- b_l - lr * colsum(dZ_l)       (with learner momentum: u <- beta u + gradient, W <- W - lr u)
//
// (the learner update of Algorithm 1 on the fp32 master, stored as two 16-bit planes, split.h).  The updates of a step
// depend on nothing but its backward pass, and on small models each launch is five microseconds of latency whatever it does.
//
// Workgroup = 64 output x 128 input units of one layer of one learner, four wavefronts of 32 x 64.  MFMA 32x32x16 bf16,
// rows = input units, columns = output units, k = samples, both operands by transpose reads out of LDS in slices of 64
// samples.  The master -- and the velocity -- are requested right after the first slice and arrive under the contraction;
// the gradient passes through LDS so that a thread then holds eight consecutive columns of a row.  A last layer of few
// classes is stepped by workgroups of head_update.h.  Every sum is taken in the order of the one-layer kernels (gemm_bf16.hip,
// head.hip): with the head as a matrix-core tile the same steps were up to 4 % faster and moved the results by half a per
// cent of the block momentum within a round.
//
// Measured, all updates of a step, us (one launch per layer, the velocity read after the contraction -> this kernel):
// 3072-1024-1024-10, 16 learners of 128 samples 79 + 31 + 9 -> 104 (5.3 TB/s); 3080-1032-520-24 with momentum, 5 learners of
// 70: 84 + 27 -> 58 (5.2 TB/s); models of a few hundred units: 4 - 6 per layer -> 5 - 8 in all.  What bounds
// it: the traffic of the planes on large models, latency on small ones.  Where the hi planes stream as well and there is no velocity, the
// one-layer kernel is as fast (4096 wide, 32 learners: 630 against 595 + 23) and stays.
#include "kavg_internal.h"
#include "column_sum.h"
#include "conv_step.h"
#include "head_update.h"
#include "loss_mean.h"
#include "split.h"

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 256;
constexpr int TR = 64, TC = 128, BK = 64;    // output units, input units, samples per slice
constexpr int ZP = TR + 32, XP = TC + 32;    // LDS rows of the operands: 64 bytes of padding (transpose reads)
constexpr int GP = TC + 4;                   // LDS rows of the gradient (fp32)
constexpr int ZN = BK * TR / 8 / NT, XN = BK * TC / 8 / NT, WN = TR * TC / 8 / NT;
constexpr int OPERANDS = BK * (ZP + XP) * 2, GRADIENT = TR * GP * 4;
constexpr int TILE_LDS = OPERANDS > GRADIENT ? OPERANDS : GRADIENT;    // (the gradient lies over the operands)
constexpr int SMEM = TILE_LDS > HEAD_LDS ? TILE_LDS : HEAD_LDS;
static_assert(HEAD_PIECES * 8 == TC, "a workgroup of the head takes as many input units as a tile");
constexpr int GROUP = 8;                     // layers per launch

struct Layer {
    const uint16_t* dz; size_t dz_lstride; int ld_dz;                // [learner][B][ld_dz]
    const uint16_t* in; size_t in_lstride; int ld_in;                // [learner][B][ld_in], or rows of a data set:
    const int32_t* gather; const int32_t* next_gather; long gather_lstride;       // (this step's and the next's)
    uint16_t* hi; uint16_t* lo; uint16_t* bhi; uint16_t* blo; float* u; float* ub;
    int d_out, d_in, tiles_r, tiles_c, total, padded;
    int head;                                // head_step (tiles_r: groups of classes)
};
struct Args {
    Layer layer[GROUP];
    int n_layers, B;
    int head_every;                          // > 0: layer 0 is the head, its workgroups (latency, hardly any traffic) are spread over the launch
    int by_rows;                             // the tiles of a row follow each other, not those of a column
    size_t lstride;                          // between learners, in planes and velocities
    float lr, beta;
    ConvSteps conv; int conv_wgs;            // conv_wgs > 0: steps of convolutions, by the workgroups behind those of the layers
    LossMeans losses;                        // n > 0: computed by the workgroups behind those, four each
};

// fragment of a [k][x] tile by transpose reads: lane l receives x0 + l%32 at k = k0 + 8 (l/32) .. +7
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* tile, int pitch, int k0, int x0, int lane) {
    const int t = lane & 15, grp = lane >> 4;
    const uint16_t* p = tile + (k0 + (grp >> 1) * 8 + (t >> 2)) * pitch + x0 + (grp & 1) * 16 + (t & 3) * 4;
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(p + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// STREAM: the lo planes (and velocities) of all learners do not stay in the memory-side cache; STREAM_HI: nor do the hi planes
template <bool MOMENTUM, bool STREAM, bool STREAM_HI>
__global__ void __launch_bounds__(NT, 2) update_group_kernel(Args a) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[SMEM];
    uint16_t* const Z = (uint16_t*)smem;                     // [BK][ZP] dZ
    uint16_t* const X = Z + BK * ZP;                         // [BK][XP] activations
    float* const G = (float*)smem;                           // [TR][GP] gradient
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int g = blockIdx.x, li = 0;
    bool head = false;
    if (a.head_every) {                                      // layer 0 is the head: one octet of workgroups in head_every
        const int octet = g >> 3, t = octet / a.head_every, heads = a.layer[0].padded >> 3;
        head = t < heads && octet - t * a.head_every == a.head_every - 1;
        g = head ? t * 8 + (g & 7) : g - min(t, heads) * 8;
        li = head ? 0 : 1;
    }
    while (!head && li + 1 < a.n_layers && g >= a.layer[li].padded) g -= a.layer[li++].padded;
    const Layer& q = a.layer[li];
    if (g >= q.padded) {
        g -= q.padded;
        if (g < a.conv_wgs) {
            const int learner = g / a.conv.wgs;
            conv_step(a.conv, g - learner * a.conv.wgs, learner, tid);
            return;
        }
        const int r = (g - a.conv_wgs) * 4 + wave;
        if (r < a.losses.n) loss_mean_wave(a.losses, r, lane);
        return;
    }
    // workgroup g runs on XCD g mod 8: each XCD gets one contiguous range of (learner, column tile, row tile), or row before column
    int at = (g & 7) * (q.padded >> 3) + (g >> 3);
    if (at >= q.total) return;
    const int inner = a.by_rows ? q.tiles_c : q.tiles_r, outer = a.by_rows ? q.tiles_r : q.tiles_c;
    const int ti = at % inner; at /= inner;
    const int to = at % outer, learner = at / outer, rt = a.by_rows ? to : ti, ct = a.by_rows ? ti : to;
    if (q.head) {
        HeadStep h = {};
        h.act = q.in; h.ld_act = q.ld_in; h.act_lstride = q.in_lstride; h.gather = q.gather; h.gather_lstride = q.gather_lstride;
        h.dz = q.dz; h.ldz = q.ld_dz; h.dz_lstride = q.dz_lstride;
        h.whi = q.hi; h.wlo = q.lo; h.bhi = q.bhi; h.blo = q.blo; h.lstride = a.lstride;
        if (MOMENTUM) { h.u = q.u; h.ub = q.ub; h.beta = a.beta; }
        h.B = a.B; h.d = q.d_in; h.C = q.d_out; h.lr = a.lr;
        head_step(h, ct, q.tiles_r > 1 ? rt : -1, learner, (float*)smem);
        return;
    }
    const int r0 = rt * TR, c0 = ct * TC, B = a.B;
    const uint16_t* dz = q.dz + (size_t)learner * q.dz_lstride;
    const uint16_t* in = q.in + (size_t)learner * q.in_lstride;
    // (without a gather the look-ups read, and ignore, words of dZ: no branch around a load)
    const int32_t* table = q.gather ? q.gather + (long)learner * q.gather_lstride : (const int32_t*)q.dz;
    const int take = q.gather ? -1 : 0;
    const size_t lat = (size_t)learner * a.lstride;

    // No load is predicated: places outside are read from clamped ones and dropped later.
    u32x4 zr[ZN], xr[XN];
    int row[XN];                                             // memory rows of the slice that is requested next
    auto look_up = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < XN; ++i) {
            const int s = min(k0 + (tid + NT * i) / (TC / 8), B - 1);
            row[i] = (table[s] & take) | (s & ~take);
        }
    };
    auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ZN; ++i) {
            const int e = tid + NT * i, s = min(k0 + e / (TR / 8), B - 1);
            zr[i] = *(const u32x4*)(dz + (size_t)s * q.ld_dz + min(r0 + (e % (TR / 8)) * 8, q.ld_dz - 8));
        }
#pragma unroll
        for (int i = 0; i < XN; ++i)
            xr[i] = *(const u32x4*)(in + (long)row[i] * q.ld_in + min(c0 + (tid + NT * i) % (TC / 8) * 8, q.d_in - 8));
    };
    const u32x4 zero = {0u, 0u, 0u, 0u};
    auto store = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ZN; ++i) {
            const int e = tid + NT * i, s = e / (TR / 8);
            *(u32x4*)(Z + s * ZP + (e % (TR / 8)) * 8) = k0 + s < B ? zr[i] : zero;
        }
#pragma unroll
        for (int i = 0; i < XN; ++i) {
            const int e = tid + NT * i, s = e / (TC / 8);
            *(u32x4*)(X + s * XP + (e % (TC / 8)) * 8) = k0 + s < B ? xr[i] : zero;
        }
    };
    look_up(0);
    load(0);
    look_up(BK);

    // piece i of this thread: row (tid + 256 i) / 16 of the tile, eight columns
    u32x4 hr[WN], lr_[WN];
    f32x4 ur[MOMENTUM ? WN : 1][2];
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int e = tid + NT * i;
        const size_t p = lat + (size_t)min(r0 + e / (TC / 8), q.d_out - 1) * q.d_in + min(c0 + e % (TC / 8) * 8, q.d_in - 8);
        hr[i] = plane_get<STREAM_HI>((const u32x4*)(q.hi + p));
        lr_[i] = plane_get<STREAM>((const u32x4*)(q.lo + p));
        if constexpr (MOMENTUM) { ur[i][0] = plane_get<STREAM>((const f32x4*)(q.u + p)); ur[i][1] = plane_get<STREAM>((const f32x4*)(q.u + p + 4)); }
    }

    const int rb = wave >> 1, cb = (wave & 1) * 2;           // 32 output units, two blocks of 32 input units
    const bool bias = ct == 0 && cb == 0;                    // (uniform) this wavefront sums dZ as well: unit rb*32 + lane%32
    float bsum = 0.f;
    f32x16 acc[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) { acc[0][e] = 0.f; acc[1][e] = 0.f; }
    auto contract = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < BK / 16; ++k) {
            const bf16x8 zf = frag_tr(Z, ZP, k * 16, rb * 32, lane);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag_tr(X, XP, k * 16, (cb + j) * 32, lane), zf, acc[j], 0, 0, 0);
        }
        if (bias) {
#pragma unroll
            for (int k = 0; k < BK / 16; ++k) bsum = column_sum16(frag_tr(Z, ZP, k * 16, rb * 32, lane), bsum);
        }
    };
    // the first slice outside the loop: its waits leave the master in flight
    store(0);
    __syncthreads();
    if (B > BK) load(BK);
    contract();
    for (int k0 = BK; k0 < B; k0 += BK) {
        __syncthreads();
        store(k0);
        __syncthreads();
        if (k0 + BK < B) { look_up(k0 + BK); load(k0 + BK); }
        contract();
    }
    __syncthreads();
    // accumulator e: input unit 8 (e/4) + 4 (lane/32) + e%4 of the block, output unit lane%32
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            *(f32x4*)(G + (rb * 32 + (lane & 31)) * GP + (cb + j) * 32 + 8 * t + 4 * (lane >> 5)) =
                (f32x4){acc[j][4 * t], acc[j][4 * t + 1], acc[j][4 * t + 2], acc[j][4 * t + 3]};
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WN; ++i) {
        const int e = tid + NT * i, r = r0 + e / (TC / 8), c = c0 + e % (TC / 8) * 8;
        f32x4 g0 = *(const f32x4*)(G + (e / (TC / 8)) * GP + e % (TC / 8) * 8), g1 = *(const f32x4*)(G + (e / (TC / 8)) * GP + e % (TC / 8) * 8 + 4);
        if constexpr (MOMENTUM) { g0 = a.beta * ur[i][0] + g0; g1 = a.beta * ur[i][1] + g1; }
        const float gs[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        u32x4 oh, ol;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t b0, b1, h2, l2;
            split_join2(hr[i][t], lr_[i][t], b0, b1);
            const float w0 = __builtin_bit_cast(float, b0) - a.lr * gs[2 * t], w1 = __builtin_bit_cast(float, b1) - a.lr * gs[2 * t + 1];
            split_pack2(__builtin_bit_cast(uint32_t, w0), __builtin_bit_cast(uint32_t, w1), h2, l2);
            oh[t] = h2; ol[t] = l2;
        }
        if (r < q.d_out && c < q.d_in) {
            const size_t p = lat + (size_t)r * q.d_in + c;
            plane_put<STREAM_HI>((u32x4*)(q.hi + p), oh);
            plane_put<STREAM>((u32x4*)(q.lo + p), ol);
            if constexpr (MOMENTUM) { plane_put<STREAM>((f32x4*)(q.u + p), g0); plane_put<STREAM>((f32x4*)(q.u + p + 4), g1); }
        }
    }
    if (bias && lane < 32 && r0 + rb * 32 + lane < q.d_out) {
        const size_t p = lat + r0 + rb * 32 + lane;
        if constexpr (MOMENTUM) { bsum = a.beta * q.ub[p] + bsum; q.ub[p] = bsum; }
        const float b = __builtin_bit_cast(float, split_join(q.bhi[p], q.blo[p])) - a.lr * bsum;
        q.bhi[p] = (uint16_t)split_hi(__builtin_bit_cast(uint32_t, b));
        q.blo[p] = (uint16_t)split_lo(__builtin_bit_cast(uint32_t, b));
    }
    if (rt == 0 && q.next_gather) {
        // the lines of the rows that the next step gathers, so that its forward pass finds them in the cache
        for (int e = tid; e < B * 2; e += NT) {
            const int c = c0 + (e & 1) * 64;
            if (c < q.d_in) {
                const uint32_t v = *(const uint32_t*)(in + (long)q.next_gather[(long)learner * q.gather_lstride + (e >> 1)] * q.ld_in + c);
                asm volatile("" ::"v"(v));
            }
        }
    }
}

}  // namespace

bool bf16_update_group_ok(const LayerCall& c) {
    // Planes that do not stay in the cache: with a velocity only, which is the larger part of the traffic and which the one-layer
    // kernel reads after the contraction; with long contractions that kernel's larger tiles outweigh it.  (us per round of two steps,
    // one-layer / this.  Rows of whole lines: 2048-2048-10, 24 learners of 16 and 250 rows 922 / 899 and 1118 / 1071, 4096-4096-10, 8 of 64
    // and 400 1202 / 1151 and 1750 / 1629, 4096-4096-1000, 9 of 400 2528 / 2496.  Ragged rows, both with ordinary accesses:
    // 1000-3000-1000-10, 20 of 64 and 400 1359 / 1253 and 2087 / 2007, 1544-2504-1320-10, 30 of 400 3626 / 3493; but 4088-4008-1000, 10 of
    // 400, 450 and 1024 3159 / 3162, 3233 / 3272 and 4442 / 4988, 1000-3000-1000-10, 20 of 768 2619 / 2710.)
    return (c.shadow_cached || (c.u && c.B <= 400)) && !c.rows && !c.partial && !c.skip_bias && c.d_in >= 8 && c.ld_dz >= 8;
}

hipError_t bf16_update_group(const LayerCall* calls, int n, const LossMeans* losses, const ConvStep* convs, int n_convs, hipStream_t st) {
    if (n_convs > STEP_GROUP) return hipErrorInvalidValue;
    for (int at = 0; at < n; at += GROUP) {
        Args a = {};
        a.n_layers = n - at < GROUP ? n - at : GROUP;
        a.B = calls[at].B; a.lstride = calls[at].ws_stride; a.lr = calls[at].lr; a.beta = calls[at].beta;
        int wgs = 0;
        for (int i = 0; i < a.n_layers; ++i) {
            const LayerCall& c = calls[at + i];
            Layer& q = a.layer[i];
            q.dz = (const uint16_t*)c.dz; q.dz_lstride = c.dz_stride; q.ld_dz = c.ld_dz;
            q.in = (const uint16_t*)c.in; q.in_lstride = c.gather ? 0 : c.in_stride; q.ld_in = c.ld_in;
            q.gather = c.gather; q.next_gather = c.gather ? c.next_gather : nullptr; q.gather_lstride = c.gather_stride;
            q.hi = c.ws; q.lo = c.wlo; q.bhi = c.bhi; q.blo = c.blo; q.u = c.u; q.ub = c.ub;
            q.d_out = c.d_out; q.d_in = c.d_in;
            q.head = c.head;
            q.tiles_r = c.head ? head_class_groups(c.P, c.d_in, c.d_out) : (c.d_out + TR - 1) / TR; q.tiles_c = (c.d_in + TC - 1) / TC;
            q.total = q.tiles_r * q.tiles_c * c.P;
            q.padded = (q.total + 7) / 8 * 8;
            wgs += q.padded;
        }
        // Long launches spread the head's workgroups, which fetch little and wait much (3072-1024-1024-10, 16 learners: a round 1.5 %
        // faster than with the head in front); in short ones the head would be the tail.
        if (a.n_layers > 1 && a.layer[0].head && wgs >= 9 * a.layer[0].padded) a.head_every = wgs / a.layer[0].padded;
        if (n_convs > 0 && at + a.n_layers == n) {
            a.conv = conv_steps(convs, n_convs, calls[at].ws_stride, calls[at].lr);
            a.conv_wgs = a.conv.wgs * calls[at].P;
            wgs += a.conv_wgs;
        }
        if (losses && at + a.n_layers == n) {
            a.losses = *losses;
            wgs += (losses->n + 3) / 4;
        }
        // (the memory-side cache holds 256 MB: read-modify-write at 6.9 TB/s inside it, and outside it 5.4 with ordinary and
        // 6.2 TB/s with streaming accesses)
        const bool momentum = calls[at].u != nullptr;
        const LayerCall* most = calls + at;                  // the layer with most weights
        for (int i = 1; i < a.n_layers; ++i)
            if ((size_t)calls[at + i].d_in * calls[at + i].d_out > (size_t)most->d_in * most->d_out) most = calls + at + i;
        const bool stream = (size_t)calls[at].P * a.lstride * (momentum ? 8 : 4) > ((size_t)224 << 20) && (calls[at].shadow_cached || whole_lines(*most, false));
        // Out of memory whole rows of tiles: a column of tiles is a stripe of the planes whose lines lie a row apart, on few of the memory's
        // channels where rows are powers of two long, and with as many learners as XCDs, or a multiple, every XCD is at the same stripe.
        // (us per round of two steps, column by column / so: 4096-4096-10, 8 learners of 16 rows 1271 / 1152, 16 of 64 2497 / 2262; 9 of 64
        // of 4096-4096-1000 1708 / 1682; 1000-3000-1000-10, 20 of 64 1341 / 1253.)
        a.by_rows = !calls[at].shadow_cached;
        if (stream && !calls[at].shadow_cached) hipLaunchKernelGGL((update_group_kernel<true, true, true>), dim3(wgs), dim3(NT), 0, st, a);
        else if (momentum && stream) hipLaunchKernelGGL((update_group_kernel<true, true, false>), dim3(wgs), dim3(NT), 0, st, a);
        else if (momentum) hipLaunchKernelGGL((update_group_kernel<true, false, false>), dim3(wgs), dim3(NT), 0, st, a);
        else if (stream) hipLaunchKernelGGL((update_group_kernel<false, true, false>), dim3(wgs), dim3(NT), 0, st, a);
        else hipLaunchKernelGGL((update_group_kernel<false, false, false>), dim3(wgs), dim3(NT), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kavg
