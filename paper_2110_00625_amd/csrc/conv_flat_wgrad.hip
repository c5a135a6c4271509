// Weight gradient of a 3x3 convolution (stride 1, zero padding 1) on channels-last bf16 images of any size, all nine
// taps from one pass over the images:
//
//     dW[o][tap][c] = sum over positions p of dZ[p][o] * A[p + (dy, dx)][c],   tap = 3 (dy+1) + (dx+1)
//
// (the learner update of Algorithm 1 for a convolutional layer: the contraction runs over the positions of the
// minibatch).  Positions are numbered with margins, as in conv_flat.hip, so that the pixel a tap points at lies a constant
// distance away: a workgroup walks over a range of positions 64 at a time with those 64 rows of dZ in LDS (two
// buffers) and the pixels around them in a ring of LDS rows, of which every slice replaces 64.  Each pixel and each row of
// dZ is then brought in once per workgroup, and every tap reads the ring at its own distance.
//
// Workgroup = (learner, range of positions, up to 64 input channels); 3 * OB wavefronts for OB blocks of 32 output
// channels: a wavefront owns the taps with dx = tl - 1 (dy = -1, 0, 1) for one output block and all input blocks, or --
// with two input blocks and an even number of output blocks -- two output blocks and one input block (five operand reads
// per slab of 16 positions instead of seven for the same six matrix instructions).  MFMA 32x32x16 bf16, M = output
// channel, N = input channel, K = position; both operands come out of LDS by transpose reads.  FIRST: 8 input channels,
// gathered images; the three dy of a tap column share one block of 32 columns.
// The bias gradient is the product of dZ with ones: one more matrix instruction per slab and output block, taken by the
// wavefronts of the three dx in turn.  (Adding up rows of dZ by hand read a quarter more LDS words than the products.)
// The fp32 sums of a workgroup go to partial[learner * splits + range][o][9 c_in] and partial_bias, which
// conv_step_kernel adds up and applies to the master.
#include "kavg_internal.h"
#include "conv_flat.h"
#include "conv_pool.h"
#include "fastdiv.h"
#include <algorithm>

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int SLP = 64;                      // positions per slice
constexpr int LDS_MAX = 160 * 1024;

template <int IB, int OB, bool FIRST>
struct WgradShape {
    static constexpr int NT = 64 * 3 * OB;
    static constexpr int ZP = OB * 32 + 32, AP = FIRST ? 16 : IB * 32 + 32;    // LDS rows: channels plus 64 bytes (transpose reads stay off each other's banks)
    static constexpr int AC = FIRST ? 1 : IB * 4;                              // 16-byte pieces of a pixel
    static constexpr int ZN = (SLP * OB * 4 + NT - 1) / NT, AN = (SLP * AC + NT - 1) / NT;
    static constexpr int smem(int ring) { return 2 * SLP * ZP * 2 + ring * AP * 2; }
};

struct WgradArgs {
    const uint16_t* dz; size_t dz_lstride; int c_out;    // [learner][pixel][c_out]
    const uint16_t* in; size_t in_lstride; int c_in;     // [learner][pixel][c_in]
    const int32_t* gather; long gather_lstride;          // FIRST: images are rows of `in`
    const int32_t* table; int table_len;                 // pixel of position i - pitch - 1
    int pitch, HW, end, slices, splits, groups;          // slices per range; ranges per learner; groups of input channels
    int ring, lead;                                      // rows of the ring (a power of two); slices of pixels that the first slice needs
    uint32_t div_hw_m; int div_hw_s;
    float* partial; float* partial_bias;
    const uint16_t* dpool; size_t dpool_lstride; float inv;          // POOL: dZ from the bits and these
    const uint8_t* bits; size_t bits_lstride; int bits_pitch;        // bytes
};

// Fragment of a [position][channel] LDS tile for one 16-position slab: lane l receives channel x0 + l%32 at positions
// row0 + 8 (l/32) .. +7.  In its 16-lane group, lane t = 4a + b fetches channels 4b .. 4b+3 of row a and receives the
// four rows of channel t.  Rows wrap at mask + 1.
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* tile, int pitch, int mask, int row, int col) {
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(tile + (row & mask) * pitch + col));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(tile + ((row + 4) & mask) * pitch + col));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

template <int IB, int OB, bool FIRST, bool POOL>
__global__ void __launch_bounds__(64 * 3 * OB) conv_flat_wgrad_kernel(WgradArgs a) {
    typedef WgradShape<IB, OB, FIRST> SH;
    constexpr int NT = SH::NT, ZP = SH::ZP, AP = SH::AP, AC = SH::AC;
    constexpr bool PAIR = IB == 2 && OB % 2 == 0;
    constexpr int OI = PAIR ? 2 : 1, NI = PAIR ? 1 : IB, TY = FIRST ? 1 : 3;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* const Z = (uint16_t*)smem;                 // [2][SLP][ZP]
    uint16_t* const A = Z + 2 * SLP * ZP;                // [ring][AP]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tl = wave / OB;
    const int ob0 = PAIR ? ((wave % OB) >> 1) * 2 : wave % OB, nb0 = PAIR ? (wave % OB) & 1 : 0;
    int at = blockIdx.x;
    const int grp = at % a.groups; at /= a.groups;       // (ranges of a learner next to each other)
    const int learner = at / a.splits, range = at - learner * a.splits;
    const int q0 = range * a.slices * SLP, q_end = min(q0 + a.slices * SLP, a.end);
    const int n = (q_end - q0 + SLP - 1) / SLP;          // slices of this range (0: an empty last range)
    const uint16_t* dz = a.dz + (size_t)learner * a.dz_lstride;
    const uint16_t* in = a.in + (size_t)learner * a.in_lstride;
    const int ch0 = grp * 64;

    // piece i of this thread: row of the slice and 16-byte chunk, for dZ and for the pixels
    const int mask = a.ring - 1;
    u32x4 zr[POOL ? 1 : SH::ZN], ar[SH::AN], gr[POOL ? SH::ZN : 1];
    uint8_t br[POOL ? SH::ZN : 1];
    int zi[SH::ZN], ai[SH::AN];                          // pixels of the slice that is requested next
    unsigned z_ok = 0, a_ok = 0;
    auto look_up = [&](int s) __attribute__((always_inline)) {       // dZ slice s, pixel slice s + lead
#pragma unroll
        for (int i = 0; i < SH::ZN; ++i) {
            const int q = q0 + s * SLP + min(tid + NT * i, SLP * OB * 4 - 1) / (OB * 4);
            zi[i] = a.table[min(q + a.pitch + 1, a.table_len - 1)];
        }
#pragma unroll
        for (int i = 0; i < SH::AN; ++i) {
            const int t = q0 + (s + a.lead) * SLP + min(tid + NT * i, SLP * AC - 1) / AC;
            ai[i] = a.table[min(t, a.table_len - 1)];
        }
    };
    const u32x4 zero = {0u, 0u, 0u, 0u};
    // 16-byte chunk of the pixel px of the table (anything where there is none)
    auto pixel_piece = [&](int px, int chunk) __attribute__((always_inline)) {
        const int ch = ch0 + chunk * 8;
        const bool ok = px >= 0 && ch < a.c_in;
        int64_t p = ok ? px : 0;
        if constexpr (FIRST) {
            const int img = (int)fastdiv((uint32_t)p, a.div_hw_m, a.div_hw_s);
            p += ((int64_t)a.gather[(long)learner * a.gather_lstride + img] - img) * a.HW;
        }
        return (const u32x4*)(in + p * a.c_in + (ok ? ch : 0));
    };
    auto fetch_pixels = [&]() __attribute__((always_inline)) {
        a_ok = 0;
#pragma unroll
        for (int i = 0; i < SH::AN; ++i) {
            const int chunk = min(tid + NT * i, SLP * AC - 1) % AC;
            if (ai[i] >= 0 && ch0 + chunk * 8 < a.c_in) a_ok |= 1u << i;
            ar[i] = *pixel_piece(ai[i], chunk);
        }
    };
    auto fetch_dz = [&](int s) __attribute__((always_inline)) {
        z_ok = 0;
#pragma unroll
        for (int i = 0; i < SH::ZN; ++i) {
            const int e = min(tid + NT * i, SLP * OB * 4 - 1), q = q0 + s * SLP + e / (OB * 4), ch = (e % (OB * 4)) * 8;
            const bool ok = zi[i] >= 0 && ch < a.c_out && q < q_end;
            if (ok) z_ok |= 1u << i;
            const int px = ok ? zi[i] : 0, c = ok ? ch : 0;
            if constexpr (!POOL) zr[i] = *(const u32x4*)(dz + (int64_t)px * a.c_out + c);
            if constexpr (POOL) br[i] = a.bits[(size_t)learner * a.bits_lstride + (size_t)px * a.bits_pitch + (c >> 3)];
            if constexpr (POOL)
                gr[i] = *(const u32x4*)(a.dpool + (size_t)learner * a.dpool_lstride +
                                        (size_t)fastdiv((uint32_t)px, a.div_hw_m, a.div_hw_s) * a.c_out + c);
        }
    };
    auto stash_pixels = [&](int slice) __attribute__((always_inline)) {     // slice: of 64 rows of the ring
#pragma unroll
        for (int i = 0; i < SH::AN; ++i) {
            const int e = tid + NT * i;
            if (e < SLP * AC) *(u32x4*)(A + ((slice * SLP + e / AC) & mask) * AP + (e % AC) * 8) = (a_ok >> i) & 1u ? ar[i] : zero;
        }
    };
    auto stash_dz = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < SH::ZN; ++i) {
            const int e = tid + NT * i;
            u32x4 v;
            if constexpr (POOL) v = pool_grad_bits((z_ok >> i) & 1u ? br[i] : 0u, gr[i], a.inv);
            else v = (z_ok >> i) & 1u ? zr[i] : zero;
            if (e < SLP * OB * 4) *(u32x4*)(Z + (buf * SLP + e / (OB * 4)) * ZP + (e % (OB * 4)) * 8) = v;
        }
    };

    f32x16 acc[TY][OI][NI], bacc;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        bacc[e] = 0.f;
#pragma unroll
        for (int ty = 0; ty < TY; ++ty)
#pragma unroll
            for (int oi = 0; oi < OI; ++oi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) acc[ty][oi][ni][e] = 0.f;
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    const int b_oi = PAIR ? nb0 : 0;                     // the output block whose bias this wavefront sums (of its OI)

    if (n > 0) {
        // the pixels around the first slice: rows 0 .. 64 lead - 1 of the ring
        for (int e0 = tid; e0 < a.lead * SLP * AC; e0 += NT * 4) {
            int pi[4];
            u32x4 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) pi[i] = a.table[min(q0 + min(e0 + NT * i, a.lead * SLP * AC - 1) / AC, a.table_len - 1)];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = *pixel_piece(pi[i], (e0 + NT * i) % AC);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = e0 + NT * i;
                if (e < a.lead * SLP * AC) *(u32x4*)(A + (e / AC) * AP + (e % AC) * 8) = pi[i] >= 0 && ch0 + (e % AC) * 8 < a.c_in ? v[i] : zero;
            }
        }
        look_up(0);
        fetch_dz(0);
        fetch_pixels();
        look_up(1);
        stash_dz(0);
        stash_pixels(a.lead);
        __syncthreads();
        // lane's row and column inside an operand block (see frag_tr)
        const int t16 = lane & 15, lrow = (lane >> 5) * 8 + (t16 >> 2), lcol = ((lane >> 4) & 1) * 16 + (t16 & 3) * 4;
        const int arow = lrow + (FIRST ? min(lcol >> 3, 2) * a.pitch : 0) + tl, acol = FIRST ? lcol & 7 : nb0 * 32 + lcol;
        for (int s = 0; s < n; ++s) {
            fetch_dz(s + 1);                             // in flight during the MFMAs (beyond the range: zeros, not used)
            fetch_pixels();
            look_up(s + 2);
            const uint16_t* Zs = Z + (s & 1) * SLP * ZP;
#pragma unroll
            for (int kq = 0; kq < SLP / 16; ++kq) {
                bf16x8 zf[OI];
#pragma unroll
                for (int oi = 0; oi < OI; ++oi) zf[oi] = frag_tr(Zs, ZP, SLP - 1, kq * 16 + lrow, (ob0 + oi) * 32 + lcol);
#pragma unroll
                for (int ty = 0; ty < TY; ++ty) {
                    // tap (dy, dx) = (ty - 1, tl - 1): position + pitch + 1 + dy * pitch + dx of the ring
                    const int row = s * SLP + kq * 16 + ty * a.pitch + arow;
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni) {
                        const bf16x8 af = frag_tr(A, AP, mask, row, acol + ni * 32);
#pragma unroll
                        for (int oi = 0; oi < OI; ++oi)
                            acc[ty][oi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zf[oi], af, acc[ty][oi][ni], 0, 0, 0);
                    }
                }
                if ((s + kq) % 3 == tl) bacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b_oi ? zf[OI - 1] : zf[0], ones, bacc, 0, 0, 0);
            }
            stash_dz((s + 1) & 1);                       // the other buffer: last read before the previous barrier
            stash_pixels(s + 1 + a.lead);                // (rows that no tap of this slice or the next reads)
            __syncthreads();
        }
    }

    // accumulator e of a block: output channel 8 (e/4) + 4 (lane/32) + e%4, input channel lane%32
    const size_t part = (size_t)learner * a.splits + range;
    float* out = a.partial + part * a.c_out * 9 * a.c_in;
    // Distances of 32 bits from the range's sums, a test for eight channels at a time: with 64 bits and a test per value ten instructions of each of
    // up to 96 stores.  (28x28, 32 -> 64 channels, 8 learners of 32 images 27.2 -> 26.6 us, the first layer 12.8 -> 12.4; rounds of two steps, channels
    // 8-64-64-64 on 14x14, 4 of 60 257 -> 249.)
    const int tap_row = 9 * a.c_in, o0 = ob0 * 32 + 4 * (lane >> 5);
#pragma unroll
    for (int ty = 0; ty < TY; ++ty)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
            const int c = FIRST ? lane & 7 : ch0 + (nb0 + ni) * 32 + (lane & 31), dy = FIRST ? (lane & 31) >> 3 : ty;
            if (c < a.c_in && dy < 3) {
                const int at0 = o0 * tap_row + (dy * 3 + tl) * a.c_in + c;
#pragma unroll
                for (int oi = 0; oi < OI; ++oi)
#pragma unroll
                    for (int g = 0; g < 4; ++g)          // (eight output channels are there or not for the whole wavefront)
                        if ((ob0 + oi) * 32 + 8 * g < a.c_out) {
#pragma unroll
                            for (int e = 0; e < 4; ++e) out[at0 + (oi * 32 + 8 * g + e) * tap_row] = acc[ty][oi][ni][4 * g + e];
                        }
            }
        }
    float* red = (float*)smem;                           // [tl][output channel] (the tiles are dead: the loop ended with a barrier)
    if ((lane & 31) == 0) {                              // every column of bacc holds the same sums
#pragma unroll
        for (int e = 0; e < 16; ++e) red[tl * OB * 32 + (ob0 + b_oi) * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)] = bacc[e];
    }
    __syncthreads();
    if (grp == 0 && tid < a.c_out) a.partial_bias[part * a.c_out + tid] = red[tid] + red[OB * 32 + tid] + red[2 * OB * 32 + tid];
}

int ring_rows(int W, int* lead) {
    const int l = (SLP + 2 * (W + 1) + 2 + SLP - 1) / SLP - 1;       // slices beyond the one at the same place
    int ring = 256;
    while (ring < (l + 2) * SLP) ring *= 2;
    if (lead) *lead = l;
    return ring;
}

int smem_of(int IB, int OB, bool first, int ring) { return 2 * SLP * (OB * 32 + 32) * 2 + ring * (first ? 16 : IB * 32 + 32) * 2; }

template <int IB, int OB, bool FIRST, bool POOL>
hipError_t launch(const WgradArgs& a, int wgs, hipStream_t st) {
    const int smem = WgradShape<IB, OB, FIRST>::smem(a.ring);
    if (smem > 64 * 1024) {
        static hipError_t raised = hipFuncSetAttribute((const void*)conv_flat_wgrad_kernel<IB, OB, FIRST, POOL>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MAX);
        if (raised != hipSuccess) return raised;
    }
    hipLaunchKernelGGL((conv_flat_wgrad_kernel<IB, OB, FIRST, POOL>), dim3(wgs), dim3(64 * 3 * OB), smem, st, a);
    return hipGetLastError();
}
template <int IB, bool FIRST, bool POOL>
hipError_t launch_ob(const WgradArgs& a, int OB, int wgs, hipStream_t st) {
    if (OB == 1) return launch<IB, 1, FIRST, POOL>(a, wgs, st);
    if (OB == 2) return launch<IB, 2, FIRST, POOL>(a, wgs, st);
    if (OB == 3) return launch<IB, 3, FIRST, POOL>(a, wgs, st);
    return launch<IB, 4, FIRST, POOL>(a, wgs, st);
}

}  // namespace

int conv_flat_wgrad_splits(int P, int B, int H, int W, int c_in, int c_out, bool first) {
    if ((first && c_in != 8) || c_out > 128 || (size_t)B * (H + 1) * (W + 1) >= ((size_t)1 << 30) || W > 4096) return 0;
    const int IB = c_in <= 32 ? 1 : 2, OB = (c_out + 31) / 32, groups = (c_in + 63) / 64;
    const int smem = smem_of(IB, OB, first, ring_rows(W, nullptr));
    if (smem > LDS_MAX) return 0;
    // Ranges: one round of workgroups over the 256 compute units, f of them on each, and at least four slices each, since every
    // range brings in its margins.  More workgroups per compute unit hide more of each other's waits (up to as many as fit
    // into its LDS, 16 wavefronts at most), but each writes partial sums that conv_step_kernel reads again.  The better f: a slice
    // takes 1 us of a compute unit, f workgroups are 1 .. 1.7 times as fast as one, the sums move at 3.5 TB/s.  (us per step of
    // nets, f as many as fit / 1: 28x28 32 -> 64, 8 learners of 32 images 130 / 123; 32x32 64 -> 64, 15 of 6 177 / 149; but
    // 60x32 8 -> 32, 8 of 62 98 / 119; 32x32 24 -> 24 -> 40, 12 of 35 244 / 251.)
    const int end = ((B - 1) * (H + 1) + H - 1) * (W + 1) + W, all = (end + SLP - 1) / SLP;
    const int fit = std::max(1, std::min({LDS_MAX / smem, 16 / (3 * OB), 5}));
    const double faster[6] = {0, 1, 1.35, 1.5, 1.6, 1.7}, slices = (double)all * P * groups / 256, sums = (double)P * c_out * 9 * c_in * 8 / 3.5e6;
    int best = 1;
    double least = 0;
    for (int f = 1; f <= fit; ++f) {
        const int S = std::max(1, std::min(std::max(1, 256 * f / (P * groups)), all / 4));
        const double us = slices / faster[f] + S * sums;
        if (f == 1 || us < least) { best = S; least = us; }
    }
    return best;
}

hipError_t conv_flat_wgrad(const ConvCall& c, const int32_t* table, const void* X, const int32_t* gather, long gstride,
                           const void* dpool, hipStream_t st) {
    if (c.splits < 1 || !c.partial || !c.partial_bias || (dpool ? !c.bits : !c.dz) || (gather && c.c_in != 8))
        return hipErrorInvalidValue;
    WgradArgs a = {};
    const size_t rows = (size_t)c.B * c.H * c.W;
    a.dz = (const uint16_t*)c.dz; a.dz_lstride = rows * c.c_out; a.c_out = c.c_out;
    a.in = (const uint16_t*)(gather ? X : c.in); a.in_lstride = gather ? 0 : rows * c.c_in; a.c_in = c.c_in;
    a.gather = gather; a.gather_lstride = gstride;
    a.table = table; a.table_len = conv_flat_table_len(c.B, c.H, c.W);
    a.pitch = c.W + 1; a.HW = c.H * c.W;
    a.end = ((c.B - 1) * (c.H + 1) + c.H - 1) * (c.W + 1) + c.W;
    a.splits = c.splits; a.groups = (c.c_in + 63) / 64;
    a.slices = ((a.end + SLP - 1) / SLP + a.splits - 1) / a.splits;
    a.ring = ring_rows(c.W, &a.lead);
    fastdiv_make((uint32_t)a.HW, &a.div_hw_m, &a.div_hw_s);
    a.partial = c.partial; a.partial_bias = c.partial_bias;
    a.dpool = (const uint16_t*)dpool; a.dpool_lstride = (size_t)c.B * c.c_out; a.inv = 1.0f / (float)a.HW;
    a.bits = (const uint8_t*)c.bits; a.bits_pitch = conv_bits_pitch(c.c_out) * 4; a.bits_lstride = rows * a.bits_pitch;
    const int OB = (c.c_out + 31) / 32, wgs = c.P * a.splits * a.groups;
    if (gather) return dpool ? launch_ob<1, true, true>(a, OB, wgs, st) : launch_ob<1, true, false>(a, OB, wgs, st);
    if (c.c_in <= 32) return dpool ? launch_ob<1, false, true>(a, OB, wgs, st) : launch_ob<1, false, false>(a, OB, wgs, st);
    return dpool ? launch_ob<2, false, true>(a, OB, wgs, st) : launch_ob<2, false, false>(a, OB, wgs, st);
}

}  // namespace kavg
