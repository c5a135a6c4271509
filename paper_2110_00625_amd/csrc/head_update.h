// The SGD step of a last layer of few classes (KAVG_BF16), as device code of a workgroup: a kernel of its own (head.hip), or
// workgroups of the launch that updates all layers (update_bf16.hip).
//
//     W_L <- W_L - lr * dZ_L^T A_{L-1},  b_L <- b_L - lr * colsum(dZ_L)
#pragma once
#include "kavg_internal.h"
#include "split.h"

namespace kavg {

struct HeadStep {
    const uint16_t* act; int ld_act; size_t act_lstride;  // A_{L-1} [P][B][ld_act], or (act_lstride 0) the data set:
    const int32_t* gather; long gather_lstride;           // row s of learner j is data row gather[j*gather_lstride + s]
    const uint16_t* dz; int ldz; size_t dz_lstride;       // dZ_L [P][B][ldz]
    uint16_t* whi; uint16_t* wlo; uint16_t* bhi; uint16_t* blo;      // planes of weights and bias
    float* u; float* ub; float beta;                      // velocities, null: plain SGD
    size_t lstride;                                       // between learners, in planes and velocities
    int B, d, C;
    float lr;
};

// Sum over the 16 lanes that differ in bits 2..5 of the lane index (same low two bits), in every lane: data-parallel
// rotations by 4 and 8 inside a row of 16 lanes keep the low bits; the rows are joined by two shuffles.
template <int CTRL>
__device__ __forceinline__ float head_row_move(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float groups_sum(float x) {
    x += head_row_move<0x124>(x);       // row_ror:4
    x += head_row_move<0x128>(x);       // row_ror:8
    x += __shfl_xor(x, 16, 64);
    x += __shfl_xor(x, 32, 64);
    return x;
}

constexpr int HEAD_SPLITS = 16;           // partial tiles of the layer below that head_forward_backward adds up at most
constexpr int HEAD_CT = 4;                // classes at a time
constexpr int HEAD_PIECES = 16;           // pieces of 8 input units per workgroup
// floats between classes in a wavefront's exchange patch (36: classes fall on different banks); the patches of four wavefronts
constexpr int XCH_CS = 16 * 32 + 36;
constexpr int HEAD_LDS = 4 * HEAD_CT * XCH_CS * 4;

// 256 threads = 4 wavefronts.  Lane = 4*g + pl: sample group g (samples s = g mod 16) and piece 16 block + 4 wave + pl.  For
// four classes at a time every lane sums dZ_L[s][c] * A[s][piece] over its samples in ascending order, and the sixteen
// partial sums meet in the wavefront's LDS patch, where lane 4*g + pl adds those of class g mod 4, units 2 (g/4) and the next
// of the piece, in ascending order of the groups.  A wavefront's LDS accesses complete in order: no barrier.
// What waits here is a chain of latencies, so the master's words of all classes are requested first, and up to NB * 16 samples
// of activations stay in registers for all classes.  A workgroup takes all classes where there are workgroups enough, else four
// (head_class_groups).
__device__ __forceinline__ void head_step(const HeadStep& a, int block, int classes /*group of four, -1: all*/, int learner, float* lds) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int NB = 8;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane >> 2, pl = lane & 3;
    const int q = block * HEAD_PIECES + wave * 4 + pl, pieces = a.d / 8;
    const int qq = min(q, pieces - 1);                        // out-of-range lanes shadow the last piece, never store
    const int32_t* g = a.gather + (long)learner * a.gather_lstride;
    const uint16_t* dz = a.dz + (size_t)learner * a.dz_lstride;
    const size_t lat = (size_t)learner * a.lstride;
    const size_t unit = (size_t)qq * 8 + 2 * (grp >> 2);      // this lane's two units of a row of W_L
    const bool once = a.B <= 16 * NB;

    // (places outside are read from clamped ones and not used)
    uint32_t h[4], l[4];
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
        const size_t at = lat + (size_t)min(4 * cc + (grp & 3), a.C - 1) * a.d + unit;
        h[cc] = *(const uint32_t*)(a.whi + at);
        l[cc] = *(const uint32_t*)(a.wlo + at);
    }
    u32x4 x[NB];
    auto load_x = [&](int base) __attribute__((always_inline)) {
        size_t row[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int s = min(base + grp + 16 * i, a.B - 1);
            row[i] = a.act_lstride ? (size_t)learner * a.act_lstride + (size_t)s * a.ld_act : (size_t)g[s] * a.ld_act;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) x[i] = *(const u32x4*)(a.act + row[i] + (size_t)qq * 8);
    };
    load_x(0);
    float* patch = lds + wave * (HEAD_CT * XCH_CS);
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) {
        if (4 * cc >= a.C || (classes >= 0 && classes != cc)) continue;
        float acc[HEAD_CT][8], bsum[HEAD_CT];
#pragma unroll
        for (int c = 0; c < HEAD_CT; ++c) {
            bsum[c] = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[c][e] = 0.f;
        }
        for (int base = 0; base < a.B; base += 16 * NB) {
            u32x2 z[NB];
#pragma unroll
            for (int i = 0; i < NB; ++i) z[i] = *(const u32x2*)(dz + (size_t)min(base + grp + 16 * i, a.B - 1) * a.ldz + 4 * cc);      // (rows are padded with zeros to 8 or 16 classes)
            if (!once) load_x(base);
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                if (base + grp + 16 * i >= a.B) continue;
                const float gz[HEAD_CT] = {__builtin_bit_cast(float, z[i].x << 16), __builtin_bit_cast(float, z[i].x & 0xFFFF0000u),
                                           __builtin_bit_cast(float, z[i].y << 16), __builtin_bit_cast(float, z[i].y & 0xFFFF0000u)};
                float v[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[2 * e] = __builtin_bit_cast(float, x[i][e] << 16);
                    v[2 * e + 1] = __builtin_bit_cast(float, x[i][e] & 0xFFFF0000u);
                }
#pragma unroll
                for (int c = 0; c < HEAD_CT; ++c) {
                    bsum[c] += gz[c];                         // bias gradient: column sum of dZ_L
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[c][e] = fmaf(gz[c], v[e], acc[c][e]);
                }
            }
        }
#pragma unroll
        for (int c = 0; c < HEAD_CT; ++c) {
            *(f32x4*)(patch + c * XCH_CS + lane * 8) = (f32x4){acc[c][0], acc[c][1], acc[c][2], acc[c][3]};
            *(f32x4*)(patch + c * XCH_CS + lane * 8 + 4) = (f32x4){acc[c][4], acc[c][5], acc[c][6], acc[c][7]};
        }
        float m0 = 0.f, m1 = 0.f;
        const float* src = patch + (grp & 3) * XCH_CS + pl * 8 + 2 * (grp >> 2);
#pragma unroll
        for (int g2 = 0; g2 < 16; ++g2) {
            const f32x2 t = *(const f32x2*)(src + g2 * 32);
            m0 += t.x; m1 += t.y;
        }
        const int cls = 4 * cc + (grp & 3);
        if (q < pieces && cls < a.C) {
            const size_t at = lat + (size_t)cls * a.d + unit;
            if (a.u) {                                        // heavy ball inside the learner
                m0 = a.beta * a.u[at] + m0; m1 = a.beta * a.u[at + 1] + m1;
                a.u[at] = m0; a.u[at + 1] = m1;
            }
            // the master lives in two 16-bit planes; the hi plane is what the next products read
            uint32_t b0, b1, h2, l2;
            split_join2(h[cc], l[cc], b0, b1);
            const float w0 = __builtin_bit_cast(float, b0) - a.lr * m0, w1 = __builtin_bit_cast(float, b1) - a.lr * m1;
            split_pack2(__builtin_bit_cast(uint32_t, w0), __builtin_bit_cast(uint32_t, w1), h2, l2);
            *(uint32_t*)(a.whi + at) = h2;
            *(uint32_t*)(a.wlo + at) = l2;
        }
        if (block == 0 && wave == 0) {                        // the sums are the same in all lanes of a row of W_L
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < HEAD_CT; ++c) {
                const float t = groups_sum(bsum[c]);
                if (c == grp) sum = t;
            }
            if (pl == 0 && grp < HEAD_CT && cls < a.C) {
                const size_t at = lat + cls;
                if (a.ub) { sum = a.beta * a.ub[at] + sum; a.ub[at] = sum; }
                const float b = __builtin_bit_cast(float, split_join(a.bhi[at], a.blo[at])) - a.lr * sum;
                a.bhi[at] = (uint16_t)split_hi(__builtin_bit_cast(uint32_t, b));
                a.blo[at] = (uint16_t)split_lo(__builtin_bit_cast(uint32_t, b));
            }
        }
    }
}

inline int head_blocks(int d) { return (d / 8 + HEAD_PIECES - 1) / HEAD_PIECES; }
// Groups of classes that are workgroups of their own: below half a workgroup per compute unit the chain inside one counts,
// above it what all of them fetch.  (One group against one per four classes, us: rounds of eight steps on
// 512-12, 16 learners 146 / 121; the update launch of 256-1024 and 1024-10, 32 learners of 64 21.5 / 24.4.)
inline int head_class_groups(int P, int d, int C) { return P * head_blocks(d) >= 128 ? 1 : (C + HEAD_CT - 1) / HEAD_CT; }

inline HeadStep head_step_args(const LayerCall& c, const int32_t* idx, long idx_lstride) {
    HeadStep a = {};
    a.act = (const uint16_t*)c.in; a.ld_act = c.ld_in; a.act_lstride = c.gather ? 0 : c.in_stride;
    a.gather = idx; a.gather_lstride = idx_lstride;
    a.dz = (const uint16_t*)c.dz; a.ldz = c.ld_dz; a.dz_lstride = c.dz_stride;
    a.whi = c.ws; a.wlo = c.wlo; a.bhi = c.bhi; a.blo = c.blo;
    a.u = c.u; a.ub = c.ub; a.beta = c.beta; a.lstride = c.ws_stride;
    a.B = c.B; a.d = c.d_in; a.C = c.d_out; a.lr = c.lr;
    return a;
}

}  // namespace kavg
