// 3x3 convolution (stride 1, zero padding 1) on channels-last bf16 images of any size, forward and data gradient:
//
//   forward        out[p][o] = relu( b[o] + sum over (tap, c) of in[p + (dy, dx)][c] * W[o][tap][c] )
//   data gradient  din[p][c] = [act[p][c] > 0] * sum over (tap, o) of dz[p - (dy, dx)][o] * W[o][tap][c]
//
// (the learner's forward and backward pass of Algorithm 1 through a convolutional layer; tap = 3 (dy+1) + (dx+1)).
//
// Positions are numbered with one zero pixel behind every image row and one zero row behind every image:
// q = (n (H+1) + h) (W+1) + w.  The neighbour a tap points at is then q + dy (W+1) + dx everywhere -- the zero column
// serves as the right margin of its row and the left margin of the next, the zero row as the lower margin of its image
// and the upper one of the next -- so a tile is any range of q, whatever the image size, and a tap is a constant
// offset into it.  (The price is the margin positions: 7 % of the products at 28x28.)
//
// A workgroup of four wavefronts owns 512 (256 with more than 64 output channels; half of that in small launches) consecutive
// positions and all output channels; the pixels it needs, W+2 further ones on either side included, are brought to LDS once per group of
// CK channels.  A wavefront owns 128 positions times up to 64 channels: eight accumulator blocks of the 32x32x16
// matrix instruction, four pixel operands out of LDS and two weight operands per slab of 16 channels.
//
// Why this split: with the weights in LDS as well (one image row per wavefront, as an earlier version of these kernels
// had it) a slab of 64 -> 128 channels takes five LDS reads per four matrix instructions, 160 LDS cycles per 128
// matrix cycles, and every step waits at two barriers for its weights.  Here it is four reads per eight instructions,
// and the weights come straight from L2 in operand order (launch_pack_weights; 1 KB per operand, consecutive, requested
// slabs ahead), so nothing inside a channel group waits for anything but the matrix cores.
//
// Measured on 28x28 images, channels 8-32-64, 8 learners of 32 images (us per launch; before: the generic kernel on an
// implicit patch matrix, the first layer on a written one): forward 15 + 17 -> 9 (first layer) and 27 -> 16, data gradient
// 37 and a rotated weight copy -> 16, weight gradient 17 -> 12 and 49 -> 27 (conv_flat_wgrad.hip).
//
// What bounds it (64 -> 128 channels, 32x32 images, 960 TFLOP/s, a clock of 1.9 GHz): two workgroups share a compute unit, out of step,
// so one contracts (12.5 k cycles, 9.2 k of them matrix instructions) while the other looks up and brings in pixels (9.6 k) and
// writes outputs (9.2 k).  Beside a wavefront that feeds the matrix cores every other instruction takes seven or eight cycles
// instead of four, so what counts is their number: pixels are found by arithmetic and not in a table, distances are 32 bits
// wide, bits and masks are formed two values at a time, gradients of the mean are scaled once per tile.  Forward pass of that layer 177 -> 161 us,
// its data gradient 231 -> 158, 32 -> 64 channels forward 76 -> 61.
//
// The last convolution, below the mean over the positions, writes no activations: what is read of them afterwards is their
// ReLU mask, one bit each, and their sums.  The sums of an image are a product with ones out of the epilogue's patch, over
// the positions of a wavefront (128, 64 in small launches), joined in ascending order (pool_mean).  16 learners of 64 images of 32x32, channels
// 8-32-64-128: 268 MB of activations were written once and read three times; without them the mean takes 5 us instead of 47 and
// the data gradient 184 instead of 203, a round 6.92 -> 6.28 ms; one convolution on 60x32 images 141 -> 97 us, 28x28 536 -> 514.
#include "kavg_internal.h"
#include "conv_flat.h"
#include "conv_pool.h"
#include "fastdiv.h"
#include "split.h"
#include <algorithm>
#include <type_traits>

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NT = 256;
enum { FWD = 0, FWD_GATHER = 1, BWD = 2, BWD_POOL = 3 };

struct FlatArgs {
    const uint16_t* in; size_t in_lstride; int c_k;      // images of c_k contraction channels
    const int32_t* gather; long gather_lstride;          // FWD_GATHER: rows of `in`
    const uint16_t* frag; size_t frag_lstride; int slabs, blocks;
    const uint16_t* bhi; const uint16_t* blo; size_t b_lstride;      // forward: bias planes
    const uint16_t* act;                                 // data gradient: activations of the layer below (strides of out)
    uint16_t* out; size_t out_lstride; int c_n;
    int H, W, sign;                                      // sign: +1 forward, -1 data gradient
    int end, image;                                      // positions up to the last pixel of the last image; positions of an image
    uint32_t div_row_m; int div_row_s;                   // division by the positions of an image row, W + 1
    uint32_t div_img_m; int div_img_s;                   // division by the rows of an image, H + 1
    int PB, tiles, total, padded; uint32_t div_tiles_m; int div_tiles_s;      // tiles per learner; workgroups
    const uint16_t* dpool; size_t dpool_lstride; float inv; int images, places;      // BWD_POOL: gradients from the bits and these; images per learner, of a tile
    uint32_t* bits; int bits_pitch; size_t bits_lstride;             // words per pixel; LAST: written, BWD_POOL: read
    float* sums; int slots;                                          // LAST: places of images per wavefront
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));      // round to nearest even
}

constexpr float BF16_MAX = 0x1.FEp127f;

// Two bf16 numbers that are +-0 or positive and finite: bits 15 and 31, those that are positive.  (No half of the sum carries.)
__device__ __forceinline__ uint32_t positive2(uint32_t two) { return (two + 0x7FFF7FFFu) & ~two & 0x80008000u; }

// fragment of a [position][channel] patch by transpose reads: lane l receives channel x0 + l%32 at positions 8 (l/32) .. +7
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* patch, int pitch, int x0, int lane) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const int t = lane & 15, grp = lane >> 4;
    const uint16_t* p = patch + ((grp >> 1) * 8 + (t >> 2)) * pitch + x0 + (grp & 1) * 16 + (t & 3) * 4;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(p + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Pixel of position q, counted from an image's first one, -1 on a margin; image: its image, counted likewise.  (Counted from an
// image near by, pixels and what is at them are 32-bit distances from a pointer that the wavefront shares.)
__device__ __forceinline__ int pixel_at(const FlatArgs& a, int q, int end, int& image) {
    const int u = max(q, 0), row = (int)fastdiv((uint32_t)u, a.div_row_m, a.div_row_s), w = u - __mul24(row, a.W + 1);
    image = (int)fastdiv((uint32_t)row, a.div_img_m, a.div_img_s);
    const int h = row - __mul24(image, a.H + 1);
    return q >= 0 && q < end && w < a.W && h < a.H ? __mul24(__mul24(image, a.H) + h, a.W) + w : -1;
}

// LDS of a pixel: its channels plus 16 bytes, or (64 channels) the channels alone with their 16-byte pieces permuted by the
// pixel's number: either way eight pixels in a row lie on different banks.  Permuted, two workgroups with 512 positions of 64
// channels fit a compute unit.
__host__ __device__ constexpr bool permuted(int CK) { return CK == 64; }
__host__ __device__ constexpr int pixel_pitch(int CK) { return permuted(CK) ? CK : CK + 8; }
// bytes of the output patches of the four wavefronts (two each, in turn), and of the pixels of a tile, which those lie over;
// behind the patches a byte for each position of each wavefront (LAST)
__host__ __device__ constexpr int patch_area(int NB) { return 2 * 4 * 32 * (NB * 32 + 8) * 2; }
__host__ __device__ constexpr int tile_area(int n_px, int CK, int NB, int PB) {
    return n_px * pixel_pitch(CK) * 2 > patch_area(NB) + 4 * PB * 32 ? n_px * pixel_pitch(CK) * 2 : patch_area(NB) + 4 * PB * 32;
}

// PB: blocks of 32 positions per wavefront.  LAST (forward): the layer below the mean over the positions; bits and partial sums instead of activations
template <int CK, int NB, int PWAVES, int PB, int KIND, bool LAST>
__global__ void __launch_bounds__(NT, 2) conv_flat_kernel(FlatArgs a) {
    constexpr int IP = pixel_pitch(CK);
    constexpr int TP = PWAVES * PB * 32, SL = CK / 16, C8 = CK / 8;
    constexpr int AHEAD = PB < 4 ? 9 : SL == 4 ? 4 : SL == 2 ? 6 : 3;      // weight operands in flight, in slabs (divides the 9 SL slabs of a group)
    constexpr bool BACK = KIND == BWD || KIND == BWD_POOL;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* const IN = (uint16_t*)smem;
    const int n_px = TP + 2 * (a.W + 1) + 2;              // pixels q0 - W - 2 .. of the tile
    // where a pixel lies, counted from image n0 on, -1: margin.  FWD_GATHER: pixel of the data set; BWD_POOL: and its image
    typedef typename std::conditional<KIND == FWD_GATHER, int64_t, typename std::conditional<KIND == BWD_POOL, int2, int>::type>::type Source;
    Source* const SRC = (Source*)(smem + tile_area(n_px, CK, NB, PB));
    float* const BIAS = (float*)(smem + tile_area(n_px, CK, NB, PB) + (size_t)((n_px + 3) & ~3) * sizeof(Source));
    uint16_t* const DP = (uint16_t*)BIAS;                 // BWD_POOL: [place][channel], bf16(dpool / (H W))
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pw = wave % PWAVES, cw = wave / PWAVES;
    // workgroup g runs on XCD g mod 8: each XCD gets one contiguous range of (learner, tile)
    const int at = (blockIdx.x & 7) * (a.padded >> 3) + (blockIdx.x >> 3);
    if (at >= a.total) return;
    const int learner = (int)fastdiv((uint32_t)at, a.div_tiles_m, a.div_tiles_s), q0 = (at - learner * a.tiles) * TP;
    const int pitch = a.W + 1;
    // the image of the tile's first pixel; positions, pixels and images are counted from there
    const int n0 = (int)fastdiv(fastdiv((uint32_t)max(q0 - pitch - 1, 0), a.div_row_m, a.div_row_s), a.div_img_m, a.div_img_s);
    const int at0 = q0 - n0 * a.image, end = a.end - n0 * a.image, px0 = n0 * a.H * a.W;
    const uint16_t* in = a.in + (size_t)learner * a.in_lstride + (KIND == FWD_GATHER ? 0 : (size_t)px0 * a.c_k);

    uint16_t bias_hi = 0, bias_lo = 0;
    if constexpr (!BACK) {
        const size_t at_b = (size_t)learner * a.b_lstride + min(tid & 127, a.c_n - 1);
        bias_hi = a.bhi[at_b];
        bias_lo = a.blo[at_b];
    }
    const char* const frag = (const char*)(a.frag + (size_t)learner * a.frag_lstride + (size_t)cw * NB * 512);
    const int steps = 9 * a.slabs;
    bf16x8 wr[AHEAD][NB];
    auto wfetch = [&](int set, int it) __attribute__((always_inline)) {
        const char* p = frag + __builtin_amdgcn_readfirstlane(min(it, steps - 1) * a.blocks * 1024);
#pragma unroll
        for (int j = 0; j < NB; ++j) wr[set][j] = *(const bf16x8*)(p + (uint32_t)(lane * 16 + j * 1024));
    };

    // Where the pixels lie, computed: out of a table (an earlier version) every workgroup began with two or three dependent reads
    // from memory, 6.4 k of its 39 k cycles.
    constexpr int LOT = KIND == FWD_GATHER ? 3 : 1;           // rows of the data set that a thread looks up at once
    for (int i0 = tid; i0 < n_px; i0 += NT * LOT) {
        int px[LOT], n[LOT], row[LOT];
#pragma unroll
        for (int i = 0; i < LOT; ++i) {
            px[i] = pixel_at(a, at0 - pitch - 1 + i0 + NT * i, end, n[i]);
            if constexpr (KIND == FWD_GATHER) row[i] = a.gather[(long)learner * a.gather_lstride + (px[i] < 0 ? 0 : n0 + n[i])];
        }
#pragma unroll
        for (int i = 0; i < LOT; ++i) {
            if (i0 + NT * i >= n_px) break;
            if constexpr (KIND == FWD_GATHER) SRC[i0 + NT * i] = px[i] < 0 ? -1 : ((int64_t)row[i] - n[i]) * (a.H * a.W) + px[i];
            else if constexpr (KIND == BWD_POOL) SRC[i0] = make_int2(px[0], n[0]);
            else SRC[i0] = px[0];
        }
    }
    if constexpr (KIND == BWD_POOL) {
        const uint16_t* dpool = a.dpool + (size_t)learner * a.dpool_lstride;
        for (int e = tid * 8; e < a.places * a.c_k; e += NT * 8) {
            const size_t from = (size_t)n0 * a.c_k + e, all = (size_t)a.images * a.c_k;
            const u32x4 g = *(const u32x4*)(dpool + (from < all ? from : 0));
            *(u32x4*)(DP + e) = pool_scale(g, a.inv);
        }
    }
    __syncthreads();

    // all pixels of channel group g: the requests of a thread are in flight (two lots of them where they are many) before the first
    // is waited for
    const int pieces = n_px * C8;
    auto place = [&](int e) __attribute__((always_inline)) {      // of piece e, in LDS
        const int px = e / C8, c = e % C8;
        return px * IP + (permuted(CK) ? c ^ (px & 7) : c) * 8;
    };
    // BWD_POOL: a thread takes whole pixels, its bits of the group at once (three pixels' bits in flight), and writes every channel's
    // gradient where its bit is set
    auto form_tile = [&](int g) __attribute__((always_inline)) {
        constexpr int N = 3;
        const int word = g * CK / 32, shift = g * CK % 32, two = min(word + 1, a.bits_pitch - 1) - word;
        const uint32_t* const bits = a.bits + (size_t)learner * a.bits_lstride + (size_t)px0 * a.bits_pitch + word;
        for (int i0 = tid; i0 < n_px; i0 += NT * N) {
            int2 src[N];
            uint32_t b0[N], b1[N];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int2 s2 = *(const int2*)&SRC[min(i0 + NT * i, n_px - 1)];
                src[i] = s2;
                const uint32_t* p = bits + (uint32_t)(max(src[i].x, 0) * a.bits_pitch);
                b0[i] = p[0];
                b1[i] = CK > 32 || CK % 32 ? p[two] : 0u;
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int px = i0 + NT * i;
                if (px < n_px) {
                    uint64_t m = (((uint64_t)b1[i] << 32) | b0[i]) >> shift;
                    if (src[i].x < 0) m = 0;
                    const uint16_t* dp = DP + __mul24(src[i].y, a.c_k) + g * CK;
#pragma unroll
                    for (int c = 0; c < C8; ++c) {
                        u32x4 x = {0u, 0u, 0u, 0u};
                        if (g * CK + c * 8 < a.c_k) x = pool_mask((uint32_t)(m >> (8 * c)) & 0xFFu, *(const u32x4*)(dp + c * 8));
                        *(u32x4*)(IN + px * IP + (permuted(CK) ? c ^ (px & 7) : c) * 8) = x;
                    }
                }
            }
        }
    };
    auto load_tile = [&](int g) __attribute__((always_inline)) {
        constexpr int ALL = ((TP + 132) * C8 + NT - 1) / NT, N = ALL <= 11 ? ALL : ALL <= 13 ? 6 : ALL <= 16 ? 8 : 7;
        for (int e0 = tid; e0 < pieces; e0 += NT * N) {
            u32x4 v[N];
            unsigned ok = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int e = min(e0 + NT * i, pieces - 1);
                const int ch = g * CK + (e % C8) * 8;
                if constexpr (KIND == FWD_GATHER) {
                    const int64_t px = SRC[e / C8];
                    const bool in_ok = px >= 0 && ch < a.c_k;
                    if (in_ok) ok |= 1u << i;
                    v[i] = *(const u32x4*)(in + (in_ok ? px * a.c_k + ch : 0));
                } else if constexpr (KIND != BWD_POOL) {
                    const int px = SRC[e / C8];
                    const bool in_ok = px >= 0 && ch < a.c_k;
                    if (in_ok) ok |= 1u << i;
                    v[i] = *(const u32x4*)((const char*)in + (uint32_t)(in_ok ? (__mul24(px, a.c_k) + ch) * 2 : 0));
                }
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int e = e0 + NT * i;
                const u32x4 zero = {0u, 0u, 0u, 0u};
                if (e < pieces) *(u32x4*)(IN + place(e)) = (ok >> i) & 1u ? v[i] : zero;
            }
        }
    };

    f32x16 acc[NB][PB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][b][e] = 0.f;

    const int lane_px = pw * PB * 32 + (lane & 31) + pitch + 1, half = lane >> 5;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) wfetch(s, s);
    static_assert(9 * SL % AHEAD == 0, "a group leaves the weight registers where it found them");
    const int groups = a.slabs / SL;
    for (int g = 0; g < groups; ++g) {
        if (g) __syncthreads();                               // everyone is done with the previous group's pixels
        if constexpr (KIND == BWD_POOL) form_tile(g); else load_tile(g);
        if constexpr (!BACK) {                                // (here, and not before the tile's requests, which would wait with it)
            if (g == 0 && tid < 128) BIAS[tid] = __builtin_bit_cast(float, split_join(bias_hi, bias_lo));
        }
        __syncthreads();
        bf16x8 x[2][PB];                                      // pixel operands of this slab and the next
        auto xfetch = [&](int s) __attribute__((always_inline)) {
            const int tap = s / SL, px = lane_px + a.sign * ((tap / 3 - 1) * pitch + tap % 3 - 1);
            // (permuted: the pieces' numbers are the low bits of the place, so the slab is one more exclusive or)
            const uint16_t* p = IN + (permuted(CK) ? (px * IP + ((half ^ (px & 7)) * 8)) ^ ((s % SL) * 16) : px * IP + half * 8 + (s % SL) * 16);
#pragma unroll
            for (int b = 0; b < PB; ++b) x[s & 1][b] = *(const bf16x8*)(p + b * 32 * IP);
        };
        xfetch(0);
#pragma unroll
        for (int s = 0; s < 9 * SL; ++s) {
            if (s + 1 < 9 * SL) xfetch(s + 1);
            __builtin_amdgcn_sched_barrier(0);                // (left alone, the compiler moves every request to just before its use)
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int b = 0; b < PB; ++b)
                    acc[j][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[s % AHEAD][j], x[s & 1][b], acc[j][b], 0, 0, 0);
            wfetch(s % AHEAD, g * SL * 9 + s + AHEAD);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    __syncthreads();                                          // the tile is dead: output patches

    // accumulator e of block (j, b) = output channel 32 j + 8 (e/4) + 4 (lane/32) + e%4 at position 32 b + lane%32.
    // The outputs of 32 positions pass through a patch of LDS that belongs to the wavefront (its LDS accesses complete
    // in order) and leave as whole rows of its channels.  Nothing here waits for a load that was requested after a
    // store: the counter is in order, and such a wait is a wait for the stores.
    constexpr int OP = NB * 32 + 8, C16 = NB * 4;
    uint16_t* patch = (uint16_t*)smem + wave * 2 * 32 * OP;
    char* const out = (char*)(a.out + (size_t)learner * a.out_lstride + (LAST ? 0 : (size_t)px0 * a.c_n));
    auto position = [&](int b, int i) __attribute__((always_inline)) {     // pixel of position i of block b, -1: margin
        const int p = (pw * PB + b) * 32 + i;
        int n;
        if constexpr (KIND == FWD_GATHER) return pixel_at(a, at0 + p, end, n);
        else if constexpr (KIND == BWD_POOL) return SRC[p + pitch + 1].x;
        else return SRC[p + pitch + 1];
    };
    float4 bias[BACK ? 1 : NB][4];
    if constexpr (!BACK) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) bias[j][q] = *(const float4*)(BIAS + (cw * NB + j) * 32 + q * 8 + half * 4);
    }
    // LAST: an infinity would reach every sum of the product with ones (0 times infinity is NaN), so the largest finite bf16 number
    // stands for it.  A sum that holds such a number is at least as large, and infinite again in pool_mean.
    auto relu = [&](float v) __attribute__((always_inline)) {
        if constexpr (LAST) return __builtin_amdgcn_fmed3f(v, 0.f, BF16_MAX); else return fmaxf(v, 0.f);
    };
    // block (j, b), after bias and ReLU or as it is, as bf16 in the patch `to`
    auto leave = [&](int b, uint16_t* to, uint32_t (&signs)[NB]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            signs[j] = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v0 = acc[j][b][4 * q + 0], v1 = acc[j][b][4 * q + 1], v2 = acc[j][b][4 * q + 2], v3 = acc[j][b][4 * q + 3];
                if constexpr (!BACK) {
                    v0 = relu(v0 + bias[j][q].x);
                    v1 = relu(v1 + bias[j][q].y);
                    v2 = relu(v2 + bias[j][q].z);
                    v3 = relu(v3 + bias[j][q].w);
                }
                const uint32_t o0 = pack_bf16x2(v0, v1), o1 = pack_bf16x2(v2, v3);
                if constexpr (LAST) {
                    // bits 4 q + {0, 2} and 16 + 4 q + {0, 2}: the four values are not zero
                    signs[j] |= positive2(o0) >> (15 - 4 * q);
                    signs[j] |= positive2(o1) >> (13 - 4 * q);
                }
                *(u32x2*)(to + (lane & 31) * OP + j * 32 + q * 8 + half * 4) = (u32x2){o0, o1};
            }
        }
    };
    if constexpr (!LAST) {
        // data gradient: the mask is applied to whole rows of channels on their way out, from reads of the same shape (read as
        // the accumulators lie, 8 bytes of 32 rows each, the masks alone took the address unit 8 k cycles per two workgroups)
        u32x4 mask[BACK ? C16 / 2 : 1];
        int to[C16 / 2];
        auto fetch_mask = [&](int b) __attribute__((always_inline)) {
            const char* const act = (const char*)(a.act + (size_t)learner * a.out_lstride + (size_t)px0 * a.c_n);
#pragma unroll
            for (int pass = 0; pass < C16 / 2; ++pass) {
                const int id = pass * 64 + lane, ch = cw * NB * 32 + (id % C16) * 8;
                to[pass] = ch < a.c_n ? position(b, id / C16) : -1;
                if constexpr (BACK) mask[pass] = *(const u32x4*)(act + (uint32_t)(to[pass] >= 0 ? (__mul24(to[pass], a.c_n) + ch) * 2 : 0));
            }
        };
        fetch_mask(0);
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            uint32_t none[NB];
            leave(b, patch + (b & 1) * 32 * OP, none);
            __builtin_amdgcn_sched_barrier(0);
            u32x4 v[C16 / 2];
            int now[C16 / 2];
#pragma unroll
            for (int pass = 0; pass < C16 / 2; ++pass) {
                const int id = pass * 64 + lane;
                v[pass] = *(const u32x4*)(patch + (b & 1) * 32 * OP + (id / C16) * OP + (id % C16) * 8);
                if constexpr (BACK) {
                    // stored activations are ReLU outputs (never negative): positive <=> non-zero magnitude
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[pass][q] &= where_nonzero2(mask[pass][q]);
                }
                now[pass] = to[pass];
            }
            if (b + 1 < PB) fetch_mask(b + 1);               // (before the stores: the counter is in order)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int pass = 0; pass < C16 / 2; ++pass)
                if (now[pass] >= 0) *(u32x4*)(out + (uint32_t)((__mul24(now[pass], a.c_n) + cw * NB * 32 + ((pass * 64 + lane) % C16) * 8) * 2)) = v[pass];
        }
    } else {
        f32x16 sums[NB];                                      // [place of an image][channel] of the wavefront's positions
        uint8_t* const SLOT = (uint8_t*)smem + patch_area(NB) + wave * (PB * 32);      // place of a position's image among those of its wavefront; 255: margin
        const int group = q0 / (PB * 32) + pw, first = (q0 + pw * PB * 32) / a.image, last = (q0 + pw * PB * 32 + PB * 32 - 1) / a.image - first;
#pragma unroll
        for (int h = 0; h < PB / 2; ++h) {
            int n;
            const int px = pixel_at(a, at0 + (pw * PB + 2 * h) * 32 + lane, end, n);
            SLOT[h * 64 + lane] = px < 0 ? 255 : (uint8_t)(n0 + n - first);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) sums[j][e] = 0.f;
        // The sum over the positions of an image is a product with ones where a position is of that image (margins: of none).
        char* const bits = (char*)(a.bits + (size_t)learner * a.bits_lstride + (size_t)px0 * a.bits_pitch);
        auto add_up = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const u32x2 sl = *(const u32x2*)(SLOT + b * 32 + t * 16 + half * 8);
                u32x4 ones;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = i < 2 ? sl.x : sl.y;
                    ones[i] = (((w >> (i & 1) * 16) & 0xFFu) == (uint32_t)(lane & 31) ? 0x3F80u : 0u) |
                              (((w >> ((i & 1) * 16 + 8)) & 0xFFu) == (uint32_t)(lane & 31) ? 0x3F800000u : 0u);
                }
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    sums[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ones),
                                                                     frag_tr(patch + ((b & 1) * 32 + t * 16) * OP, OP, j * 32, lane), sums[j], 0, 0, 0);
            }
        };
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            uint32_t signs[NB];
            leave(b, patch + (b & 1) * 32 * OP, signs);
            const int to = position(b, lane & 31);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                uint32_t w = (signs[j] | signs[j] >> 15) & 0xFFFFu;      // four bits for each q: channels 8 q + 4 half ..
                w = (w | w << 8) & 0x00FF00FFu;
                w = ((w | w << 4) & 0x0F0F0F0Fu) << (half * 4);
                const auto h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
                if (lane < 32 && to >= 0 && cw * NB + j < a.bits_pitch)
                    *(uint32_t*)(bits + (uint32_t)((__mul24(to, a.bits_pitch) + cw * NB + j) * 4)) = (uint32_t)h[0] | (uint32_t)h[1];
            }
            __builtin_amdgcn_sched_barrier(0);
            if (b > 0) add_up(b - 1);                         // (the block before: its patch is written by now)
            __builtin_amdgcn_sched_barrier(0);
        }
        add_up(PB - 1);
        float* to = a.sums + ((size_t)learner * a.tiles * PWAVES + group) * a.slots * (a.blocks * 32) + cw * NB * 32 + (lane & 31);
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int slot = 8 * (e >> 2) + 4 * half + (e & 3);
                if (slot <= last) to[(size_t)slot * (a.blocks * 32) + j * 32] = sums[j][e];
            }
    }
}

// pooled[learner][image][channel] = bf16(mean), one lane per output.  (One row of the grid per learner: all learners' outputs together may be
// more than 2^31.)  Where one launch takes all layers of the MLP it forms its rows itself (chain_bf16.hip).
__global__ void __launch_bounds__(NT) pool_finish_kernel(PoolSums q, uint16_t* pooled, int c, int outputs) {
    const int e = blockIdx.x * NT + threadIdx.x, learner = blockIdx.y;
    if (e < outputs) pooled[(size_t)learner * outputs + e] = pool_mean(q, learner, e / c, e % c);
}

__global__ void __launch_bounds__(NT) flat_table_kernel(int32_t* table, int len, int end, int H, int W) {
    const int i = blockIdx.x * NT + threadIdx.x;
    if (i >= len) return;
    const int q = i - W - 2, row = q / (W + 1), w = q - row * (W + 1), n = row / (H + 1), h = row - n * (H + 1);
    table[i] = q >= 0 && q < end && w < W && h < H ? (n * H + h) * W + w : -1;
}

// ---- weights in operand order -------------------------------------------------------------------
// frag[(group * 9 * SL + tap * SL + slab in the group) * blocks + block][lane][8]: lane l of the matrix
// operand holds output channel 32 block + l%32, contraction channels 16 slab + 8 (l/32) .. +7; zero outside the layer.
struct PackDir { uint16_t* frag; size_t frag_lstride; const uint16_t* w; int c_in, c_out, back, SL, slabs, blocks, wgs; };
constexpr int PACK_MAX = 16;                 // directions per launch
struct PackArgs { PackDir d[PACK_MAX]; int n; size_t w_lstride; };

__global__ void __launch_bounds__(NT) pack_weights_kernel(PackArgs a) {
    int g = blockIdx.x, i = 0;
    while (i + 1 < a.n && g >= a.d[i].wgs) g -= a.d[i++].wgs;
    const PackDir& d = a.d[i];
    const int e = g * NT + threadIdx.x;
    if (e >= 9 * d.slabs * d.blocks * 64) return;
    const int lane = e & 63, block = (e >> 6) % d.blocks, it = (e >> 6) / d.blocks;
    const int grp = it / (9 * d.SL), rem = it - grp * 9 * d.SL;
    const int tap = rem / d.SL, slab = grp * d.SL + rem - tap * d.SL;
    const int x = block * 32 + (lane & 31), k = slab * 16 + (lane >> 5) * 8;
    const uint16_t* w = d.w + (size_t)blockIdx.y * a.w_lstride;
    u32x4 v = {0u, 0u, 0u, 0u};
    if (!d.back) {
        if (x < d.c_out && k < d.c_in)                        // (all channel counts are multiples of 8, so layers and rows start at 16 bytes)
            v = *(const u32x4*)(w + ((size_t)x * 9 + tap) * d.c_in + k);
    } else if (x < d.c_in && k < d.c_out) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint16_t* p = w + ((size_t)(k + 2 * q) * 9 + tap) * d.c_in + x;
            v[q] = (uint32_t)p[0] | ((uint32_t)p[(size_t)9 * d.c_in] << 16);
        }
    }
    *(u32x4*)(d.frag + (size_t)blockIdx.y * d.frag_lstride + (size_t)e * 8) = v;
}

// places for the images of a tile
int tile_images(int n_px, int H, int W) { return (n_px - 1) / ((H + 1) * (W + 1)) + 2; }

// the tile, where its pixels lie, the bias or (dpool_channels) the gradients of the means
size_t lds_bytes(const FlatPlan& p, int PB, int H, int W, int dpool_channels, int source) {
    const int n_px = p.PWAVES * PB * 32 + 2 * (W + 1) + 2;
    return (size_t)tile_area(n_px, p.CK, p.NB, PB) + (size_t)((n_px + 3) & ~3) * source +
           (dpool_channels ? (size_t)tile_images(n_px, H, W) * dpool_channels * 2 : 128 * 4);
}

// Blocks of 32 positions per wavefront: four, and half as many (with weights requested further ahead) where workgroups of four would
// not even be one for each of the 256 compute units.  us per round of two steps, half / whole: 2 learners of 32 images of 11x24,
// 8-32-128 (40 workgroups) 162 / 178, 4 of 60 of 14x14, 8-64-64-64 (106) 274 / 309, 10 of 6 of 45x35, 8-16-16 (200) 156 / 156; but
// 8 of 32 of 28x28, 8-32-64 (424) 233 / 224.
int blocks_per_wave(int P, int B, int H, int W, const FlatPlan& plan) { return conv_flat_workgroups(P, B, H, W, plan.PWAVES == 2 ? 128 : 64) <= 256 ? 2 : 4; }

FlatArgs make_args(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag) {
    FlatArgs a = {};
    a.frag = frag; a.frag_lstride = plan.frag_elems(); a.slabs = plan.slabs; a.blocks = plan.blocks;
    a.H = c.H; a.W = c.W;
    a.end = ((c.B - 1) * (c.H + 1) + c.H - 1) * (c.W + 1) + c.W;
    fastdiv_make((uint32_t)(c.W + 1), &a.div_row_m, &a.div_row_s);
    fastdiv_make((uint32_t)(c.H + 1), &a.div_img_m, &a.div_img_s);
    a.PB = blocks_per_wave(c.P, c.B, c.H, c.W, plan);
    const int TP = plan.PWAVES * a.PB * 32;
    a.tiles = (a.end + TP - 1) / TP;
    a.total = a.tiles * c.P;
    a.padded = (a.total + 7) / 8 * 8;
    a.image = (c.H + 1) * (c.W + 1);
    fastdiv_make((uint32_t)a.tiles, &a.div_tiles_m, &a.div_tiles_s);
    return a;
}

template <int CK, int NB, int PWAVES, int PB, int KIND, bool LAST>
hipError_t launch(const FlatArgs& a, size_t smem, hipStream_t st) {
    if (smem > 64 * 1024) {
        static hipError_t raised = hipFuncSetAttribute((const void*)conv_flat_kernel<CK, NB, PWAVES, PB, KIND, LAST>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (raised != hipSuccess) return raised;
    }
    hipLaunchKernelGGL((conv_flat_kernel<CK, NB, PWAVES, PB, KIND, LAST>), dim3(a.padded), dim3(NT), smem, st, a);
    return hipGetLastError();
}

template <int PB, int KIND, bool LAST>
hipError_t run_pb(const FlatArgs& a, const FlatPlan& p, hipStream_t st) {
    const int source = KIND == FWD_GATHER || KIND == BWD_POOL ? 8 : 4;
    const size_t smem = lds_bytes(p, PB, a.H, a.W, KIND == BWD_POOL ? a.c_k : 0, source);
    if (p.PWAVES == 2) {
        if (p.CK == 64) return launch<64, 2, 2, PB, KIND, LAST>(a, smem, st);
        if (p.CK == 48) return launch<48, 2, 2, PB, KIND, LAST>(a, smem, st);
        if (p.CK == 32) return launch<32, 2, 2, PB, KIND, LAST>(a, smem, st);
        return launch<16, 2, 2, PB, KIND, LAST>(a, smem, st);
    }
    if (p.NB == 2) {
        if (p.CK == 64) return launch<64, 2, 4, PB, KIND, LAST>(a, smem, st);
        if (p.CK == 48) return launch<48, 2, 4, PB, KIND, LAST>(a, smem, st);
        if (p.CK == 32) return launch<32, 2, 4, PB, KIND, LAST>(a, smem, st);
        return launch<16, 2, 4, PB, KIND, LAST>(a, smem, st);
    }
    if (p.CK == 64) return launch<64, 1, 4, PB, KIND, LAST>(a, smem, st);
    if (p.CK == 48) return launch<48, 1, 4, PB, KIND, LAST>(a, smem, st);
    if (p.CK == 32) return launch<32, 1, 4, PB, KIND, LAST>(a, smem, st);
    return launch<16, 1, 4, PB, KIND, LAST>(a, smem, st);
}

template <int KIND, bool LAST = false>
hipError_t run(const FlatArgs& a, const FlatPlan& p, hipStream_t st) {
    return a.PB == 2 ? run_pb<2, KIND, LAST>(a, p, st) : run_pb<4, KIND, LAST>(a, p, st);
}

}  // namespace

int conv_flat_table_len(int B, int H, int W) { return ((B - 1) * (H + 1) + H - 1) * (W + 1) + W + W + 3; }

hipError_t launch_flat_table(int32_t* table, int B, int H, int W, hipStream_t st) {
    const int len = conv_flat_table_len(B, H, W);
    hipLaunchKernelGGL(flat_table_kernel, dim3((len + NT - 1) / NT), dim3(NT), 0, st, table, len, len - W - 3, H, W);
    return hipGetLastError();
}

int conv_flat_workgroups(int P, int B, int H, int W, int c_n) {
    const long end = ((long)(B - 1) * (H + 1) + H - 1) * (W + 1) + W, tile = c_n <= 64 ? 512 : 256;
    return (int)std::min((end + tile - 1) / tile * P, (long)INT32_MAX);
}

namespace {

// dpool_channels: those of a data gradient below the mean over the positions, whose gradients lie in LDS as well
bool plan_of(int B, int H, int W, int c_k, int c_n, int dpool_channels, FlatPlan* plan) {
    FlatPlan p = {};
    if (c_n > 128 || (size_t)B * (H + 1) * (W + 1) >= ((size_t)1 << 30)) return false;
    p.NB = c_n <= 32 ? 1 : 2;
    p.PWAVES = c_n <= 64 ? 4 : 2;
    p.blocks = p.NB * (4 / p.PWAVES);
    // Slabs per group: the largest number whose tile leaves room for two workgroups per compute unit, among those that
    // pad the contraction least.  (More channels per group: fewer reloads, each of which the workgroup waits for.)
    const int slabs = (c_k + 15) / 16;
    int best = 0;
    for (int SL = 1; SL <= 4 && SL <= slabs; ++SL) {
        FlatPlan q = p;
        q.CK = SL * 16;
        q.slabs = (slabs + SL - 1) / SL * SL;
        if (lds_bytes(q, 4, H, W, dpool_channels, 8) > 80 * 1024 || (best && q.slabs > best)) continue;
        p.CK = q.CK; p.slabs = best = q.slabs;
    }
    if (!best) return false;
    *plan = p;
    return true;
}

}  // namespace

bool conv_flat_plan(int B, int H, int W, int c_k, int c_n, FlatPlan* plan) { return plan_of(B, H, W, c_k, c_n, 0, plan); }

// (Where the mean's gradients leave no room for a second workgroup, the plan without them: then there is one.)
bool conv_flat_plan_last(int B, int H, int W, int c_k, int c_n, FlatPlan* plan) {
    return plan_of(B, H, W, c_k, c_n, c_k, plan) || plan_of(B, H, W, c_k, c_n, 0, plan);
}

hipError_t launch_pack_weights(const PackLayer* layers, int n, size_t w_lstride, int P, hipStream_t st) {
    PackArgs a = {};
    a.w_lstride = w_lstride;
    int wgs = 0;
    auto flush = [&]() -> hipError_t {
        if (a.n == 0) return hipSuccess;
        hipLaunchKernelGGL(pack_weights_kernel, dim3(wgs, P), dim3(NT), 0, st, a);
        a.n = 0; wgs = 0;
        return hipGetLastError();
    };
    auto add = [&](const PackLayer& l, const FlatPlan& p, uint16_t* frag, size_t lstride, int back) {
        PackDir& d = a.d[a.n++];
        d.frag = frag; d.frag_lstride = lstride; d.w = l.w; d.c_in = l.c_in; d.c_out = l.c_out; d.back = back;
        d.SL = p.CK / 16; d.slabs = p.slabs; d.blocks = p.blocks;
        d.wgs = (9 * p.slabs * p.blocks * 64 + NT - 1) / NT;
        wgs += d.wgs;
    };
    for (int i = 0; i < n; ++i) {
        if (a.n + 2 > PACK_MAX) { const hipError_t e = flush(); if (e != hipSuccess) return e; }
        if (layers[i].fwd) add(layers[i], layers[i].fwd_plan, layers[i].fwd, layers[i].fwd_lstride, 0);
        if (layers[i].bwd) add(layers[i], layers[i].bwd_plan, layers[i].bwd, layers[i].bwd_lstride, 1);
    }
    return flush();
}

int conv_pool_slots(int P, int B, int H, int W, const FlatPlan& plan) {
    const int image = (H + 1) * (W + 1);
    return image < 5 ? 0 : blocks_per_wave(P, B, H, W, plan) * 32 / image + 2;          // (at most the 32 rows of a matrix instruction)
}

size_t conv_pool_elems(int P, int B, int H, int W, const FlatPlan& plan) {
    const int end = ((B - 1) * (H + 1) + H - 1) * (W + 1) + W, TP = plan.PWAVES * blocks_per_wave(P, B, H, W, plan) * 32;
    return (size_t)P * ((end + TP - 1) / TP) * plan.PWAVES * conv_pool_slots(P, B, H, W, plan) * plan.blocks * 32;
}

PoolSums conv_pool_sums(const float* sums, const FlatPlan& plan, int P, int B, int H, int W) {
    const int end = ((B - 1) * (H + 1) + H - 1) * (W + 1) + W, PB = blocks_per_wave(P, B, H, W, plan), TP = plan.PWAVES * PB * 32;
    return {sums, (H + 1) * (W + 1), (H - 1) * (W + 1) + W - 1, conv_pool_slots(P, B, H, W, plan), PB * 32, (end + TP - 1) / TP * plan.PWAVES, plan.blocks * 32,
            1.0f / (float)(H * W)};
}

hipError_t launch_pool_finish(const PoolSums& q, void* pooled, int P, int B, int c, hipStream_t st) {
    const int outputs = B * c;                                // (at most 2^16 images of 128 channels)
    hipLaunchKernelGGL(pool_finish_kernel, dim3((outputs + NT - 1) / NT, P), dim3(NT), 0, st, q, (uint16_t*)pooled, c, outputs);
    return hipGetLastError();
}

hipError_t conv_flat_forward(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t*, const void* X,
                             const int32_t* gather, long gstride, hipStream_t st) {
    if (!c.bits && !c.out) return hipErrorInvalidValue;
    FlatArgs a = make_args(c, plan, frag);
    const size_t rows = (size_t)c.B * c.H * c.W;
    a.in = (const uint16_t*)(gather ? X : c.in); a.in_lstride = gather ? 0 : rows * c.c_in; a.c_k = c.c_in;
    a.gather = gather; a.gather_lstride = gstride;
    a.bhi = c.bhi; a.blo = c.blo; a.b_lstride = c.ws_stride;
    a.out = (uint16_t*)c.out; a.out_lstride = rows * c.c_out; a.c_n = c.c_out;
    a.sign = 1;
    if (c.bits) {
        a.bits = c.bits; a.bits_pitch = conv_bits_pitch(c.c_out); a.bits_lstride = rows * a.bits_pitch;
        a.sums = c.pool_sums; a.slots = conv_pool_slots(c.P, c.B, c.H, c.W, plan);
        if (!a.sums || !a.slots) return hipErrorInvalidValue;
        return gather ? run<FWD_GATHER, true>(a, plan, st) : run<FWD, true>(a, plan, st);
    }
    return gather ? run<FWD_GATHER>(a, plan, st) : run<FWD>(a, plan, st);
}

hipError_t conv_flat_backward_data(const ConvCall& c, const FlatPlan& plan, const uint16_t* frag, const int32_t*, const void* dpool,
                                   hipStream_t st) {
    if (dpool ? !c.bits : !c.dz) return hipErrorInvalidValue;
    FlatArgs a = make_args(c, plan, frag);
    const size_t rows = (size_t)c.B * c.H * c.W;
    a.in = (const uint16_t*)c.dz; a.in_lstride = rows * c.c_out; a.c_k = c.c_out;
    a.bits = c.bits; a.bits_pitch = conv_bits_pitch(c.c_out); a.bits_lstride = rows * a.bits_pitch;
    a.dpool = (const uint16_t*)dpool; a.dpool_lstride = (size_t)c.B * c.c_out; a.inv = 1.0f / (float)(c.H * c.W);
    a.images = c.B; a.places = tile_images(plan.PWAVES * a.PB * 32 + 2 * (c.W + 1) + 2, c.H, c.W);
    a.act = (const uint16_t*)c.in;
    a.out = (uint16_t*)c.dz_in; a.out_lstride = rows * c.c_in; a.c_n = c.c_in;
    a.sign = -1;
    return dpool ? run<BWD_POOL>(a, plan, st) : run<BWD>(a, plan, st);
}

}  // namespace kavg
