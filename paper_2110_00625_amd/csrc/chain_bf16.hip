// Forward pass, loss and data gradients of a small MLP in one launch (KAVG_BF16):
//
//     A_l = bf16(relu(A_{l-1} W_l^T + b_l));  loss and dZ_L (softmax cross-entropy, the 1/B of Algorithm 1);
//     dZ_{l-1} = bf16((dZ_l W_l) * [A_{l-1} > 0])
//
// Nothing here mixes samples, so a workgroup takes eight rows of a minibatch through all layers: activations and gradients
// stay in its LDS, the weights are read out of L2 once in either direction, each by the one wavefront that multiplies them.  Only
// the update contracts over the samples; it is the next launch (update_bf16.hip), and reads the activations and gradients that
// this one leaves in memory.  Why: on small models every launch of a step is four to six microseconds of latency whatever it
// does, and a step was L + 1 + (L - 1) of them before its update.
//
// What bounds it is a chain of latencies, and the vector units of one compute unit wherever a row is worked on lane by lane; so
// a workgroup takes few rows (the matrix instructions multiply 32 anyway), one per wavefront, and the code, which runs once from
// end to end, is kept short.
//
// Eight wavefronts; a wavefront owns blocks of 32 outputs times the rows (MFMA 32x32x16, rows of the instruction = outputs).
// Weights are requested in whole lines, four sets of 64 along the contraction ahead, and pass through a patch of LDS that belongs
// to the wavefront (requested in operand order, 32 rows per instruction, they arrived at a quarter of that rate); those of
// the next layer are requested before the barrier between two layers.
// Every sum is taken in the order of the one-layer kernels (gemm_bf16.hip with the contraction split over two groups of
// wavefronts; head.hip; softmax_ce_kernel): the results are theirs bit for bit.
//
// Measured inside a workgroup of 304-72-302 (us): rows and first weights 1.8, forward 2.3 and 2.9, softmax 2.2, data gradient
// 2.3, 12.4 in all; with its launch 14 against 22 for a launch each.  A step of 64-64-64-64-2 30 -> 22 with its update,
// 128-128-128-100 (16 learners of 128) 36 -> 27, three hidden layers of 256 39 -> 33; a net of 3x3 convolutions whose MLP is
// 16-72-82 92 -> 83.  Unrolled over rows and classes the code was 53 KB and took twice as long as the launches it replaces.
#include "kavg_internal.h"
#include "chain_bf16.h"
#include "split.h"
#include "wave_sum.h"
#include <algorithm>
#include <type_traits>

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int WAVES = 8, NT = 64 * WAVES, ROWS = WAVES;      // rows per workgroup, one per wavefront
constexpr int FP = 64 + 8;                   // LDS rows of a patch, forward: 64 inputs plus 16 bytes
constexpr int BP = 32 + 8;                   // ... and backward: 32 inputs plus 16 bytes
constexpr int PATCH = 32 * FP > 64 * BP ? 32 * FP : 64 * BP;         // of a wavefront: 32 outputs, or 64
constexpr int SHARED_BYTES = WAVES * PATCH * 2;
constexpr int SETS = 4;                      // sets of 64 inputs (forward) or outputs (backward) in flight

// LDS rows of d values: zeros up to whole sets, and 16 bytes
__host__ __device__ constexpr int lds_pitch(int d) { return (d + 63) / 64 * 64 + 8; }

struct Layer {
    const uint16_t* w; const uint16_t* bhi; const uint16_t* blo;     // learner 0
    uint16_t* act; uint16_t* dz;             // [P][B][d_out], [P][B][ld_dz]
    int d_in, d_out, ld_dz;
    int in_at, dz_at, bias_at;               // LDS: bytes of its input rows, its dZ rows, its bias
};
struct Args {
    Layer layer[CHAIN_LAYERS];
    int L, B, blocks;                        // workgroups per learner
    size_t lstride;                          // between learners, in the weights
    const uint16_t* in; int ld_in; size_t in_lstride;                // rows of the first layer, or (gather_in) of the data set
    int gather_in;
    PoolSums pool; uint16_t* pooled;         // POOL: the rows are means over positions, formed here and written there ([P][B][d_in])
    const int32_t* idx; long idx_lstride;    // samples of this step
    const int32_t* y;
    float* rowloss;                          // [P][B]
    uint16_t* dz0;                           // gradient of the rows, null: not wanted
    int dz0_at, logits_at, head_at;          // LDS (head_at: the weights of a last layer of few classes)
};

__device__ __forceinline__ uint16_t bf16_bits(float x) {
    __bf16 h = (__bf16)x;                    // round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ uint32_t pack2(float lo, float hi) { return (uint32_t)bf16_bits(lo) | ((uint32_t)bf16_bits(hi) << 16); }

// fragment of a [16][x] patch by transpose reads: lane l receives x = l%32 at k = 8 (l/32) .. +7
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* patch, int lane) {
    const int t = lane & 15, grp = lane >> 4;
    const uint16_t* p = patch + ((grp >> 1) * 8 + (t >> 2)) * BP + (grp & 1) * 16 + (t & 3) * 4;
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(p + 4 * BP));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ void unpack(const u32x4& p, float (&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __builtin_bit_cast(float, p[i] << 16);
        v[2 * i + 1] = __builtin_bit_cast(float, p[i] & 0xFFFF0000u);
    }
}

// HEAD: a last layer of few classes, which takes its sums in the order of head.hip
// POOL: the rows of the first layer are means over positions that are formed here.  (An instance of its own: as a branch it cost rounds
// without it 1 %, 4 learners of 94 rows of 264-128-10, six steps 114.9 -> 116.4 us, 10 of 21 of 152-120-696-10, eleven 363.9 -> 366.3.)
template <bool HEAD, bool POOL>
__global__ void __launch_bounds__(NT, 2) chain_kernel(Args a) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5;
    uint16_t* const patch = (uint16_t*)smem + wave * PATCH;
    const int learner = blockIdx.x / a.blocks, row0 = (blockIdx.x - learner * a.blocks) * ROWS;
    const size_t lat = (size_t)learner * a.lstride, lrow = (size_t)learner * a.B + row0;
    const int rows = min(ROWS, a.B - row0);                  // (those beyond the batch repeat its last one)
    const int my_row = lane & (ROWS - 1);                    // of the matrix instruction's 32
    const u32x4 zero = {0u, 0u, 0u, 0u};
    auto pitch = [](int d) { return lds_pitch(d); };
    constexpr std::integral_constant<bool, false> no;
    constexpr std::integral_constant<bool, true> yes;

    // A contraction is summed in two groups, forward of 64 inputs each in turn, backward of 32 outputs each, joined at the end.
    // Set q of a block's weights: inputs (backward: outputs) 64 q .. 64 q + 63.
    u32x4 w[SETS][4];
    // No request stands behind a branch, so that every wait is a counted one: sets beyond the last and places outside are read
    // from inside, and not used or replaced on their way to LDS.
    uint32_t at[4];                                          // forward: elements from the layer's weights to the rows of this lane's pieces
    auto place = [&](auto back, const Layer& l, int blk) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            at[s] = back ? (uint32_t)min(blk * 32 + (lane & 3) * 8, l.d_in - 8) : __umul24(min(blk * 32 + s * 8 + (lane >> 3), l.d_out - 1), l.d_in);
    };
    auto fetch = [&](auto back, u32x4 (&to)[4], const Layer& l, int q) __attribute__((always_inline)) {
        const uint16_t* p = l.w + lat;
        const uint32_t c = back ? 0 : (uint32_t)min(q * 64 + (lane & 7) * 8, l.d_in - 8);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t r = back ? __umul24(min(q * 64 + s * 16 + (lane >> 2), l.d_out - 1), l.d_in) : 0;
            to[s] = *(const u32x4*)(p + (at[s] + r + c));
        }
    };
    f32x16 acc[2];
    auto multiply = [&](auto back, auto odd, u32x4 (&from)[4], const Layer& l, const uint16_t* x, int q) __attribute__((always_inline)) {
        const int left = (back ? l.d_out : l.d_in) - q * 64;
        if (left < 64) {
#pragma unroll
            for (int s = 0; s < 4; ++s) if ((back ? s * 16 + (lane >> 2) : (lane & 7) * 8) >= left) from[s] = zero;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (back) *(u32x4*)(patch + (s * 16 + (lane >> 2)) * BP + (lane & 3) * 8) = from[s];
            else *(u32x4*)(patch + (s * 8 + (lane >> 3)) * FP + (lane & 7) * 8) = from[s];
        }
        bf16x8 wf[4], xf[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (back) wf[s] = frag_tr(patch + s * 16 * BP, lane);
            else wf[s] = *(const bf16x8*)(patch + (lane & 31) * FP + s * 16 + half * 8);
            xf[s] = *(const bf16x8*)(x + q * 64 + s * 16);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            f32x16& c = acc[back ? s >> 1 : (int)odd];
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[s], xf[s], c, 0, 0, 0);
        }
    };
    // The products of a layer in one direction (back: its outputs are the gradients of its inputs); x: the operand rows in
    // LDS.  out(block, sums) is called with a block's sums.  A wavefront's blocks (every eighth) follow each other without a
    // gap: the sets of the next one are requested while this one is multiplied.
    int next_blk, next_q;                                    // of the next request
    auto sets_of = [&](auto back, const Layer& l) { return ((back ? l.d_out : l.d_in) + 127) / 128 * 2; };      // (an even number: the groups alternate)
    auto request = [&](auto back, u32x4 (&to)[4], const Layer& l) __attribute__((always_inline)) {
        fetch(back, to, l, next_q);
        if (++next_q == sets_of(back, l)) { next_q = 0; next_blk += WAVES; place(back, l, next_blk); }
    };
    auto ahead = [&](auto back, const Layer& l) __attribute__((always_inline)) {
        next_blk = wave; next_q = 0;
        place(back, l, wave);
#pragma unroll
        for (int i = 0; i < SETS; ++i) request(back, w[i], l);
    };
    auto product = [&](auto back, const Layer& l, const uint16_t* x, auto out) __attribute__((always_inline)) {
        const int blocks = ((back ? l.d_in : l.d_out) + 31) / 32, n = sets_of(back, l), depth = back ? l.d_out : l.d_in;
        const uint16_t* const xr = x + my_row * pitch(back ? l.ld_dz : l.d_in) + half * 8;
        int blk = wave, q = 0;
        if (blk >= blocks) return;
#pragma unroll
        for (int e = 0; e < 16; ++e) { acc[0][e] = 0.f; acc[1][e] = 0.f; }
#pragma unroll 1
        for (;;) {
#pragma unroll
            for (int i = 0; i < SETS; ++i) {
                if (q * 64 < depth) { if (i & 1) multiply(back, yes, w[i], l, xr, q); else multiply(back, no, w[i], l, xr, q); }
                request(back, w[i], l);
                ++q;
                if ((i & 1) && q == n) {                     // (n is even)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[0][e] += acc[1][e];
                    if ((lane & 31) < ROWS) out(blk, acc[0]);
                    blk += WAVES; q = 0;
                    if (blk >= blocks) return;
#pragma unroll
                    for (int e = 0; e < 16; ++e) { acc[0][e] = 0.f; acc[1][e] = 0.f; }
                }
            }
        }
    };
    // zeros behind the LDS rows of a buffer
    auto pad = [&](uint16_t* rows_at, int d) __attribute__((always_inline)) {
        const int c = d + (tid & 7) * 8;
        if (tid < ROWS * 8 && c < pitch(d) - 8) *(u32x4*)(rows_at + (tid >> 3) * pitch(d) + c) = zero;
    };
    // LDS rows to memory (d: a multiple of 8)
    auto copy_out = [&](const uint16_t* from, int d, uint16_t* to) __attribute__((always_inline)) {
        if (wave < rows)
#pragma unroll 1
            for (int c = lane * 8; c < d; c += 512) *(u32x4*)(to + (lrow + wave) * d + c) = *(const u32x4*)(from + wave * pitch(d) + c);
    };

    // the rows and their labels, the first weights, the biases, the head's weights
    const int32_t* const idx = a.idx + (long)learner * a.idx_lstride + row0;
    const int C = a.layer[a.L - 1].d_out;
    const int my = min(wave, rows - 1), sample = idx[my];
    const int label = min(max(a.y[sample], 0), C - 1);       // (validated; never index outside)
    {
        const Layer l = a.layer[0];
        uint16_t* const x = (uint16_t*)(smem + l.in_at);
        const uint16_t* p = a.gather_in ? a.in + (size_t)sample * a.ld_in : a.in + (size_t)learner * a.in_lstride + (size_t)(row0 + my) * a.ld_in;
        if constexpr (POOL) {
#pragma unroll 1
            for (int c = lane; c < l.d_in; c += 64) {
                const uint16_t h = pool_mean(a.pool, learner, row0 + my, c);
                x[wave * pitch(l.d_in) + c] = h;
                if (wave < rows) a.pooled[(lrow + wave) * l.d_in + c] = h;
            }
        } else {
#pragma unroll 4
            for (int c = lane * 8; c < l.d_in; c += 512) *(u32x4*)(x + wave * pitch(l.d_in) + c) = *(const u32x4*)(p + c);
        }
        ahead(no, l);
        pad(x, l.d_in);
        for (int i = 0; i < a.L; ++i) {
            const Layer& b = a.layer[i];
            float* bias = (float*)(smem + b.bias_at);
            for (int c = tid; c < b.d_out; c += NT) bias[c] = __builtin_bit_cast(float, split_join(b.bhi[lat + c], b.blo[lat + c]));
        }
        if constexpr (HEAD) {
            const Layer& t = a.layer[a.L - 1];
            uint16_t* const hw = (uint16_t*)(smem + a.head_at);
#pragma unroll 1
            for (int c = wave; c < C; c += WAVES)
                for (int i = lane * 8; i < t.d_in; i += 512) *(u32x4*)(hw + c * pitch(t.d_in) + i) = *(const u32x4*)(t.w + lat + (uint32_t)(c * t.d_in + i));
        }
    }
    __syncthreads();

    // forward
    const int forward = HEAD ? a.L - 1 : a.L;
#pragma unroll 1
    for (int i = 0; i < forward; ++i) {
        const Layer l = a.layer[i];                          // (in scalar registers)
        const float* bias = (const float*)(smem + l.bias_at);
        const bool last = i == a.L - 1;
        uint16_t* const to = last ? nullptr : (uint16_t*)(smem + a.layer[i + 1].in_at);
        float* const logits = (float*)(smem + a.logits_at);
        product(no, l, (const uint16_t*)(smem + l.in_at), [&](int blk, const f32x16& v) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = blk * 32 + t * 8 + half * 4;
                if (c >= l.ld_dz) continue;                  // (ld_dz: d_out rounded up to whole eights; the biases end there, too)
                const f32x4 b = *(const f32x4*)(bias + c);
                const f32x4 o = {v[4 * t] + b.x, v[4 * t + 1] + b.y, v[4 * t + 2] + b.z, v[4 * t + 3] + b.w};
                if (last) *(f32x4*)(logits + my_row * (l.ld_dz + 4) + c) = o;
                else *(u32x2*)(to + my_row * pitch(l.d_out) + c) =
                         (u32x2){pack2(fmaxf(o.x, 0.f), fmaxf(o.y, 0.f)), pack2(fmaxf(o.z, 0.f), fmaxf(o.w, 0.f))};
            }
        });
        if (!last) pad(to, l.d_out);
        if (i + 1 < forward) ahead(no, a.layer[i + 1]);
        __syncthreads();
        if (!last) copy_out(to, l.d_out, l.act);
    }

    // loss and the gradients of the last layer's outputs, row by row
    const Layer& top = a.layer[a.L - 1];
    uint16_t* const ztop = (uint16_t*)(smem + top.dz_at);
    uint16_t* const zbelow = (uint16_t*)(smem + (a.L > 1 ? a.layer[a.L - 2].dz_at : a.dz0_at));
    uint16_t* const below = a.L > 1 ? a.layer[a.L - 2].dz : a.dz0;       // null: no gradient below the last layer
    const float invB = 1.0f / (float)a.B;
    const int ldz = top.ld_dz;
    const int downto = a.dz0 ? 0 : 1;                        // the last layer whose data gradient is formed
    if (HEAD ? a.L - 2 >= downto : a.L - 1 >= downto) ahead(yes, a.layer[HEAD ? a.L - 2 : a.L - 1]);
    pad(ztop, ldz);
    if (HEAD && below) pad(zbelow, top.d_in);
    auto larger = [](float p, float q) { return fmaxf(p, q); };
    auto plus = [](float p, float q) { return p + q; };
    if constexpr (!HEAD) {
        const float* z = (const float*)(smem + a.logits_at) + wave * (ldz + 4);
        float mx = -INFINITY;
#pragma unroll 1
        for (int c = lane; c < C; c += 64) mx = fmaxf(mx, z[c]);
        mx = butterfly(mx, larger);
        float sum = 0.f;
#pragma unroll 1
        for (int c = lane; c < C; c += 64) sum += expf(z[c] - mx);
        sum = butterfly(sum, plus);
#pragma unroll 1
        for (int c = lane; c < ldz; c += 64)
            ztop[wave * pitch(ldz) + c] = bf16_bits(c < C ? (expf(z[c] - mx) / sum - (c == label ? 1.0f : 0.0f)) * invB : 0.f);
        if (lane == 0 && wave < rows) a.rowloss[lrow + wave] = -(z[label] - mx - logf(sum));
    } else {
        // Logits: the lanes split the contraction, eight units at a time.  The sums over the lanes of up to sixteen classes
        // are taken together: at each step a lane hands on one half of its values and keeps the other, so that class c
        // ends up in the lanes c, 16 + c, ... (pairs, quads, eights, sixteens, then (r0 + r1) + (r2 + r3), as dpp_wave_sum).
        const uint16_t* x = (const uint16_t*)(smem + top.in_at) + wave * pitch(top.d_in);
        const uint16_t* hw = (const uint16_t*)(smem + a.head_at);
        const int d = top.d_in;
        float g[16];
#pragma unroll
        for (int c = 0; c < 16; ++c) g[c] = 0.f;
#pragma unroll 1
        for (int p = lane * 8; p < d; p += 512) {
            float xv[8];
            unpack(*(const u32x4*)(x + p), xv);
#pragma unroll
            for (int c0 = 0; c0 < 16; c0 += 4) {
                if (c0 >= C) break;
#pragma unroll
                for (int c = c0; c < c0 + 4; ++c) {
                    float wv[8];
                    unpack(*(const u32x4*)(hw + min(c, C - 1) * pitch(d) + p), wv);
#pragma unroll
                    for (int e = 0; e < 8; ++e) g[c] = fmaf(xv[e], wv[e], g[c]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int n = 8; n >= 1; n /= 2)
#pragma unroll
            for (int i = 0; i < n; ++i) {
                const int bit = n == 8 ? 1 : n == 4 ? 2 : n == 2 ? 4 : 8;
                const bool upper = lane & bit;
                const float keep = upper ? g[2 * i + 1] : g[2 * i], give = upper ? g[2 * i] : g[2 * i + 1];
                float got;
                if (bit == 1) got = dpp_move<0xB1>(give);            // quad_perm [1,0,3,2]
                else if (bit == 2) got = dpp_move<0x4E>(give);       // quad_perm [2,3,0,1]
                else if (bit == 8) got = dpp_move<0x128>(give);      // row_ror:8
                else {                                               // from lane + 4 (row_shl:4) and from lane - 4 (row_shr:4)
                    const int gi = __builtin_bit_cast(int, give);
                    const int up = __builtin_amdgcn_update_dpp(0, gi, 0x104, 0xF, 0x5, true);
                    got = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(up, gi, 0x114, 0xF, 0xA, false));
                }
                g[i] = keep + got;
            }
        const int c = lane & 15;
        const float z = rows_sum(g[0]) + ((const float*)(smem + top.bias_at))[min(c, C - 1)];
        float mx = c < C ? z : -INFINITY;
        mx = fmaxf(mx, dpp_move<0x128>(mx));
        mx = fmaxf(mx, dpp_move<0x124>(mx));
        mx = fmaxf(mx, dpp_move<0x4E>(mx));
        mx = fmaxf(mx, dpp_move<0xB1>(mx));
        const float e = expf(z - mx);
        float sum = 0.f;
#pragma unroll 1
        for (int i = 0; i < C; ++i) sum += __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, e), i));
        if (lane < ldz) ztop[wave * pitch(ldz) + lane] = c < C ? bf16_bits((e / sum - (c == label ? 1.0f : 0.0f)) * invB) : (uint16_t)0;
        if (lane == label && wave < rows) a.rowloss[lrow + wave] = -(z - mx - logf(sum));
        // the gradient of its inputs, eight units per lane (a wavefront's LDS accesses complete in order)
        if (below)
#pragma unroll 1
            for (int p = lane * 8; p < d; p += 512) {
                float da[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
                for (int k = 0; k < C; ++k) {
                    float wv[8];
                    unpack(*(const u32x4*)(hw + k * pitch(d) + p), wv);
                    const float gk = __builtin_bit_cast(float, (uint32_t)ztop[wave * pitch(ldz) + k] << 16);
#pragma unroll
                    for (int q = 0; q < 8; ++q) da[q] = fmaf(gk, wv[q], da[q]);
                }
                const u32x4 m = *(const u32x4*)(x + p);
                u32x4 o;
#pragma unroll
                for (int q = 0; q < 4; ++q) o[q] = pack2((m[q] & 0x7FFFu) ? da[2 * q] : 0.f, (m[q] & 0x7FFF0000u) ? da[2 * q + 1] : 0.f);
                *(u32x4*)(zbelow + wave * pitch(d) + p) = o;
            }
    }
    // These rows leave LDS before the barrier: with a head the first product below it writes to the place of the last layer's
    // gradients again.  A wavefront copies the row that it wrote itself, and its LDS accesses complete in order.
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    copy_out(ztop, ldz, top.dz);
    if (HEAD && below) copy_out(zbelow, top.d_in, below);
    __syncthreads();

    // Data gradients.  The two places take turns: a product reads one and writes the other, the copy out of the one written stands
    // between the barrier behind that product and the barrier behind the next, and only the product after that writes there again.
#pragma unroll 1
    for (int i = HEAD ? a.L - 2 : a.L - 1; i >= downto; --i) {
        const Layer l = a.layer[i];
        const uint16_t* act = (const uint16_t*)(smem + l.in_at) + my_row * pitch(l.d_in);
        uint16_t* const to = (uint16_t*)(smem + (i > 0 ? a.layer[i - 1].dz_at : a.dz0_at));
        product(yes, l, (const uint16_t*)(smem + l.dz_at), [&](int blk, const f32x16& v) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = blk * 32 + t * 8 + half * 4;
                if (c >= l.d_in) continue;
                // activations (and means of activations) are never negative: positive <=> non-zero magnitude
                const u32x2 m = *(const u32x2*)(act + c);
                *(u32x2*)(to + my_row * pitch(l.d_in) + c) =
                    (u32x2){pack2((m.x & 0x7FFFu) ? v[4 * t] : 0.f, (m.x & 0x7FFF0000u) ? v[4 * t + 1] : 0.f),
                            pack2((m.y & 0x7FFFu) ? v[4 * t + 2] : 0.f, (m.y & 0x7FFF0000u) ? v[4 * t + 3] : 0.f)};
            }
        });
        pad(to, l.d_in);
        if (i - 1 >= downto) ahead(yes, a.layer[i - 1]);
        __syncthreads();
        copy_out(to, l.d_in, i > 0 ? a.layer[i - 1].dz : a.dz0);
    }
}

int round8(int x) { return (x + 7) / 8 * 8; }
size_t row_bytes(int d) { return (size_t)ROWS * lds_pitch(d) * 2; }

// LDS of layers l0 .. L of dims: rows of every layer's input and bias, gradients in two places that take turns, logits
// (dead before the gradients below the last layer are written) in the second of them.  Fills in places where q is given.
size_t lds_plan(int L, const int* dims, Args* q) {
    size_t at = SHARED_BYTES;
    auto take = [&](size_t bytes) { const size_t p = at; at += (bytes + 15) / 16 * 16; return (int)p; };
    for (int l = 0; l < L; ++l) {
        const int in_at = take(row_bytes(dims[l])), bias_at = take((size_t)round8(dims[l + 1]) * 4);
        if (q) { q->layer[l].in_at = in_at; q->layer[l].bias_at = bias_at; }
    }
    const bool head = head_supported(dims[L]);
    size_t need[2] = {0, head ? 0 : (size_t)ROWS * (round8(dims[L]) + 4) * 4};
    for (int l = L; l >= 0; --l) need[(L - l) & 1] = std::max(need[(L - l) & 1], row_bytes(round8(dims[l])));
    if (head) {
        const int w_at = take((size_t)dims[L] * lds_pitch(dims[L - 1]) * 2);
        if (q) q->head_at = w_at;
    }
    const int place[2] = {take(need[0]), take(need[1])};
    if (q) {
        for (int l = 0; l < L; ++l) q->layer[l].dz_at = place[(L - 1 - l) & 1];
        q->dz0_at = place[L & 1];
        q->logits_at = place[1];
    }
    return at;
}

template <bool HEAD, bool POOL>
hipError_t launch(const Args& a, dim3 grid, size_t smem, hipStream_t st) {
    static const hipError_t raised = hipFuncSetAttribute((const void*)chain_kernel<HEAD, POOL>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (raised != hipSuccess) return raised;
    hipLaunchKernelGGL((chain_kernel<HEAD, POOL>), grid, dim3(NT), smem, st, a);
    return hipGetLastError();
}

}  // namespace

// Times in tenths of a microsecond, from the shapes alone.  One launch: 40 whatever it does, its loss, and a product 9, 4 per
// turn of eight blocks, 8 per 128 of a turn's contraction, and the traffic of all workgroups' weights out of L2 (25 TB/s).
// Separate launches: a product 43 and 3 (backward 2) per 64 of its contraction, a head 55 (up to four classes 35) and 1 per 64
// units, the softmax 40.
// One launch / a launch each, measured per step with its updates (us): 512-256-64, 4 learners of 32 samples 21.5 / 25.2; its
// last layer alone of 512-480-40 25 / 27.5, both 27.8; 128-128-128-100, 16 learners of 128 27 / 36; all of 3072-256-256-10,
// 16 of 64 72 / 62, and of 104-1000-100, 5 of 118 36 / 32: left apart.
int chain_layers(int P, int B, int L, const int* dims, bool into_input) {
    const long wgs = (long)P * ((B + ROWS - 1) / ROWS);
    if (wgs > 256) return 0;                                 // more than one workgroup per compute unit: two rounds of a long chain
    const bool head = head_supported(dims[L]);
    auto product = [&](int outputs, int depth) {
        return 9 + (outputs + 255) / 256 * (4 + 8 * ((depth + 127) / 128)) + (int)(wgs * outputs * depth / 1250000);
    };
    int best = 0, gain = 0;
    int one = 40 + (head ? 30 : 20), many = head ? (dims[L] <= 4 ? 35 : 55) + dims[L - 1] / 64 : 40;
    for (int n = 1; n <= L && n <= CHAIN_LAYERS; ++n) {
        const int l = L - n + 1, d_in = dims[l - 1], d_out = dims[l];        // the layer that comes in
        if (d_in >= 1 << 14 || d_out >= 1 << 14 || lds_plan(n, dims + l - 1, nullptr) > 160 * 1024) break;
        if (!(head && l == L)) {
            if (!bf16_forward_splits(P, B, d_in, d_out)) break;
            one += product(d_out, d_in); many += 43 + 3 * d_in / 64;
            if (l > 1 || into_input) {
                if (!bf16_backward_splits(P, B, d_in, d_out)) break;
                one += product(d_in, d_out); many += 43 + 2 * d_out / 64;
            }
        }
        if (many - one > gain && !(head && n == 1)) { best = n; gain = many - one; }     // (alone the head is one launch anyway)
    }
    return best;
}

hipError_t bf16_chain(const LayerCall* calls, int n, const int32_t* y, const int32_t* idx, long idx_lstride, float* rowloss, const PoolSums* pool,
                      hipStream_t st) {
    if (n < 1 || n > CHAIN_LAYERS) return hipErrorInvalidValue;
    Args a = {};
    int dims[CHAIN_LAYERS + 1];
    dims[0] = calls[0].d_in;
    for (int l = 0; l < n; ++l) {
        const LayerCall& c = calls[l];
        Layer& q = a.layer[l];
        dims[l + 1] = c.d_out;
        q.w = c.ws; q.bhi = c.bhi; q.blo = c.blo;
        q.act = (uint16_t*)c.out; q.dz = (uint16_t*)c.dz;
        q.d_in = c.d_in; q.d_out = c.d_out; q.ld_dz = c.ld_dz;
    }
    a.L = n; a.B = calls[0].B; a.blocks = (a.B + ROWS - 1) / ROWS;
    a.lstride = calls[0].ws_stride;
    a.in = (const uint16_t*)calls[0].in; a.ld_in = calls[0].ld_in; a.in_lstride = calls[0].in_stride;
    a.gather_in = calls[0].gather != nullptr;
    if (pool) { a.pool = *pool; a.pooled = (uint16_t*)calls[0].in; }
    a.idx = idx; a.idx_lstride = idx_lstride; a.y = y; a.rowloss = rowloss;
    a.dz0 = (uint16_t*)calls[0].dz_prev;
    const size_t smem = lds_plan(n, dims, &a);
    if (smem > 160 * 1024) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(calls[0].P * a.blocks));
    return head_supported(dims[n]) ? pool ? launch<true, true>(a, grid, smem, st) : launch<true, false>(a, grid, smem, st)
                                   : pool ? launch<false, true>(a, grid, smem, st) : launch<false, false>(a, grid, smem, st);
}

}  // namespace kavg
