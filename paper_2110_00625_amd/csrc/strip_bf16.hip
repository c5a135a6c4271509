// One pass over a layer's weights per local step (KAVG_BF16), layers above the first: the data gradient, which needs the
// weights of before the update, and the SGD update of the learner:
//
//     dZ_{l-1} = bf16((dZ_l W_l) * [A_{l-1} > 0]);    W_l <- W_l - lr * dZ_l^T A_{l-1};    b_l <- b_l - lr * colsum(dZ_l)
//
// (the last two lines of a local step of Algorithm 1; W_l is the fp32 master in two 16-bit planes, split.h).
//
// A workgroup owns a strip of 128 input units and walks down the output units RC at a time.  The strip's activations
// (up to 256 samples) stay in LDS; a chunk brings in RC columns of dZ, which both products use, and RC x 128 weights, which
// are multiplied, updated and written back while they are at hand.  Chunks are requested ahead in registers.
//
//   update:        four wavefronts; rows = input units (32 each), columns = output units, k = samples, MFMA 32x32x16.  The
//                  activations stay in registers; the chunk's gradient passes through LDS so that a thread then holds
//                  eight consecutive columns of both planes (256 bytes per row and plane).
//   data gradient: four wavefronts; rows = input units (transpose reads of the weights in LDS), columns = samples, k = units
//                  of the chunk; the sums of the whole strip stay in accumulators (BT/32 blocks per wavefront).
//
// Every sum is one chain over ascending samples or units, as in the separate kernels (gemm_bf16.hip; their data gradient
// splits its contraction where a launch is small): with the samples split over two wavefronts instead, both kinds of
// product on each, the results moved by half a per cent of the block momentum within a round, and with 256 samples it was
// slower (2048 -> 2048, 16 learners: 87 against 75 us).
//
// Why: with the weights streaming from memory the separate kernels read the hi plane twice (2 of 12 bytes per weight and
// step), and with 256 samples what they pull out of L2 for each tile of weights -- both operands of every tile, 128 KB per
// 128 KB of master traffic -- held the update to 4.5 - 5 TB/s.  Here a chunk costs its dZ columns only.
// Measured, both products of a layer, us (separate kernels -> this one): 4096 -> 4096, 32 learners of 64 samples 745 + 207 ->
// 787; 8 of 256, mean with 4096 -> 1000: 149 + 70 -> 165.  Rounds of four steps, 256-1024-1024-1024-40: 24 learners of 128 936 ->
// 881, of 200 1198 -> 1085.
// What bounds it: up to 128 samples the traffic of the weights itself (5.0 - 5.9 TB/s; without the products the same time);
// with 256 samples the two barriers per chunk on top.
#include "kavg_internal.h"
#include "column_sum.h"
#include "split.h"

namespace kavg {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int NT = 512;
constexpr int SC = 128;                      // input units of a strip
constexpr int XP = SC + 32;                  // LDS rows of activations and weights: 64 bytes of padding (transpose reads)
constexpr int PP = SC + 4;                   // LDS rows of the gradient (fp32)

constexpr int RC = 32;                       // output units per chunk
constexpr int ZP = RC + 16;                  // LDS rows of dZ: read along the units and across them

template <int BT>
struct StripShape {
    static constexpr int ZN = (BT * RC / 8 + NT - 1) / NT, AN = BT * SC / 8 / NT;
    static constexpr int SMEM = BT * XP * 2 + BT * ZP * 2 + RC * XP * 2 + RC * (PP + 1) * 4;
};
static_assert(RC * SC / 8 == NT, "one 16-byte piece of each plane per thread and chunk");

struct StripArgs {
    const uint16_t* dz; size_t dz_lstride; int ld_dz;                // [learner][B][ld_dz]
    const uint16_t* in; size_t in_lstride; int ld_in;                // [learner][B][ld_in]
    uint16_t* hi; uint16_t* lo; uint16_t* bhi; uint16_t* blo; size_t lstride;
    uint16_t* dz_prev; size_t dz_prev_lstride;                       // [learner][B][ld_in]
    int B, d_in, d_out;
    int strips, total, padded;                                       // strips per learner; workgroups
    float lr;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));      // round to nearest even
}

// fragment of a [k][x] tile by transpose reads: lane l receives x0 + l%32 at k = k0 + 8 (l/32) .. +7
__device__ __forceinline__ bf16x8 frag_tr(const uint16_t* tile, int pitch, int k0, int x0, int lane) {
    const int t = lane & 15, grp = lane >> 4;
    const uint16_t* p = tile + (k0 + (grp >> 1) * 8 + (t >> 2)) * pitch + x0 + (grp & 1) * 16 + (t & 3) * 4;
    typedef bf16x4 __attribute__((address_space(3))) * lds_ptr;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_ptr)(p + 4 * pitch));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// STREAM: how the planes are accessed (stream_policy).  CHAINS: the data gradient's sums, one chain over the units, or two (even and odd chunks) that are added up at the end.
template <int BT, int STREAM, int CHAINS>
__global__ void __launch_bounds__(NT) strip_kernel(StripArgs a) {
    typedef StripShape<BT> SH;
    constexpr int ZN = SH::ZN, KS = BT / 16;                 // slabs of 16 samples
    // Chunks in registers, the one at hand and those requested ahead.  More than 64 samples: a third is slower (70 against 66 us
    // with 1024 -> 1024, 32 learners of 128) or has no registers left beside the accumulators.  64: two where a second
    // workgroup per compute unit counts for more (planes that stream: 0.3 % of a round), else three (58 against 59 us); with
    // two chains there are hardly more strips than compute units, and four are 1 - 2 % of a round faster than two.
    constexpr int SETS = BT > 64 ? 2 : CHAINS == 2 ? 4 : STREAM == STREAM_LO ? 3 : 2;
    static_assert(CHAINS == 1 || SETS % 2 == 0, "a chunk's set has its parity");
    // blocks of a wavefront's data gradient: input units x samples
    constexpr int CBW = BT == 64 ? 1 : 2, SBW = BT / 32 / CBW;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    uint16_t* const X = (uint16_t*)smem;                     // [BT][XP] activations
    uint16_t* const Z = X + BT * XP;                         // [BT][ZP] dZ of the chunk
    uint16_t* const W = Z + BT * ZP;                         // [RC][XP] hi plane of the chunk
    float* const G = (float*)(W + RC * XP);                  // [RC][PP] gradient of the chunk
    float* const GB = G + RC * PP;                           // [RC] column sums of dZ
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // workgroup g runs on XCD g mod 8: each XCD gets one contiguous range of (learner, strip)
    const int at = (blockIdx.x & 7) * (a.padded >> 3) + (blockIdx.x >> 3);
    if (at >= a.total) return;
    const int learner = at / a.strips, strip = at - learner * a.strips;
    const int c0 = strip * SC;
    const int wrow = tid >> 4, wcol = (tid & 15) * 8;        // this thread's piece of a chunk's weights
    const uint16_t* dz = a.dz + (size_t)learner * a.dz_lstride;
    const uint16_t* in = a.in + (size_t)learner * a.in_lstride;
    uint16_t* hi = a.hi + (size_t)learner * a.lstride;
    uint16_t* lo = a.lo + (size_t)learner * a.lstride;
    uint16_t* bhi = a.bhi + (size_t)learner * a.lstride;
    uint16_t* blo = a.blo + (size_t)learner * a.lstride;
    const u32x4 zero = {0u, 0u, 0u, 0u};

    u32x4 zr[SETS][ZN], hr[SETS], lr_[SETS];
    uint16_t br[SETS][2];                                    // bias of unit tid % RC of the chunk (both planes)
    // No load is predicated: places outside are read from clamped ones and dropped later.
    auto load = [&](int set, int r0) __attribute__((always_inline)) {
        const size_t p = (size_t)min(r0 + wrow, a.d_out - 1) * a.d_in + min(c0 + wcol, a.d_in - 8);
        hr[set] = plane_get<STREAM == STREAM_BOTH>((const u32x4*)(hi + p));
        lr_[set] = plane_get<STREAM != STREAM_NONE>((const u32x4*)(lo + p));
#pragma unroll
        for (int i = 0; i < ZN; ++i) {
            const int e = tid + NT * i, s = e / (RC / 8), r = r0 + (e % (RC / 8)) * 8;
            zr[set][i] = *(const u32x4*)(dz + (size_t)min(s, a.B - 1) * a.ld_dz + min(r, a.ld_dz - 8));
        }
        const int b = min(r0 + tid % RC, a.d_out - 1);
        br[set][0] = bhi[b];
        br[set][1] = blo[b];
    };
#pragma unroll
    for (int s = 0; s + 1 < SETS; ++s) load(s, s * RC);

    // the strip's activations
    {
        u32x4 v[SH::AN];
#pragma unroll
        for (int i = 0; i < SH::AN; ++i) {
            const int e = tid + NT * i, s = min(e / 16, a.B - 1), c = c0 + (e & 15) * 8;
            v[i] = *(const u32x4*)(in + (size_t)s * a.ld_in + min(c, a.d_in - 8));
        }
#pragma unroll
        for (int i = 0; i < SH::AN; ++i) {
            const int e = tid + NT * i;
            *(u32x4*)(X + (e / 16) * XP + (e & 15) * 8) = e / 16 < a.B && c0 + (e & 15) * 8 < a.d_in ? v[i] : zero;
        }
    }

    __syncthreads();

    // A chunk: its pieces from registers to LDS, the next one requested, the products (each kind of wavefront its own), and
    // the master's step from the gradient in LDS.
    auto stage = [&](int set, int r0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ZN; ++i) {
            const int e = tid + NT * i, s = e / (RC / 8), r = r0 + (e % (RC / 8)) * 8;
            if (BT * RC / 8 % NT == 0 || e < BT * RC / 8)
                *(u32x4*)(Z + s * ZP + (e % (RC / 8)) * 8) = s < a.B && r < a.ld_dz ? zr[set][i] : zero;
        }
        *(u32x4*)(W + wrow * XP + wcol) = r0 + wrow < a.d_out ? hr[set] : zero;      // (an infinite weight times no gradient is not zero)
        __syncthreads();
        load((set + SETS - 1) % SETS, r0 + (SETS - 1) * RC);
        __builtin_amdgcn_sched_barrier(0);                   // (left alone, the compiler moves the requests to their use)
    };
    // The bias of a chunk's units belongs to one of the learner's strips, in turn.
    auto owns_bias = [&](int r0) __attribute__((always_inline)) { return r0 / RC % a.strips == strip; };
    auto step = [&](int set, int r0) __attribute__((always_inline)) {
        __syncthreads();
        const float* gp = G + wrow * PP + wcol;
        const f32x4 g0 = *(const f32x4*)gp, g1 = *(const f32x4*)(gp + 4);
        const float gs[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
        u32x4 oh, ol;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t b0, b1, h2, l2;
            split_join2(hr[set][q], lr_[set][q], b0, b1);
            const float w0 = __builtin_bit_cast(float, b0) - a.lr * gs[2 * q], w1 = __builtin_bit_cast(float, b1) - a.lr * gs[2 * q + 1];
            split_pack2(__builtin_bit_cast(uint32_t, w0), __builtin_bit_cast(uint32_t, w1), h2, l2);
            oh[q] = h2; ol[q] = l2;
        }
        if (r0 + wrow < a.d_out && c0 + wcol < a.d_in) {
            const size_t p = (size_t)(r0 + wrow) * a.d_in + c0 + wcol;
            plane_put<STREAM == STREAM_BOTH>((u32x4*)(hi + p), oh);
            plane_put<STREAM != STREAM_NONE>((u32x4*)(lo + p), ol);
        }
        if (tid < RC && r0 + tid < a.d_out && owns_bias(r0)) {
            const float b = __builtin_bit_cast(float, split_join(br[set][0], br[set][1])) - a.lr * GB[tid];
            bhi[r0 + tid] = (uint16_t)split_hi(__builtin_bit_cast(uint32_t, b));
            blo[r0 + tid] = (uint16_t)split_lo(__builtin_bit_cast(uint32_t, b));
        }
    };
    // (chunks beyond the last unit multiply zeros and store nothing; leaving the loop at each of them costs the compiler
    // a copy of the accumulators per exit)

    if (wave < 4) {
        // update: input units 32 wave .. +31 of the strip, all samples in one chain; its activations stay in registers
        const int cb = wave;
        bf16x8 xf[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) xf[k] = frag_tr(X, XP, k * 16, cb * 32, lane);
        auto chunk = [&](int set, int r0) __attribute__((always_inline)) {
            stage(set, r0);
            f32x16 g;
#pragma unroll
            for (int e = 0; e < 16; ++e) g[e] = 0.f;
#pragma unroll
            for (int k = 0; k < KS; ++k) g = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[k], frag_tr(Z, ZP, k * 16, 0, lane), g, 0, 0, 0);
            // accumulator e: input unit 8 (e/4) + 4 (lane/32) + e%4 of the block, output unit lane%32
            float* p = G + (lane & 31) * PP + cb * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q) *(f32x4*)(p + 8 * q) = (f32x4){g[4 * q], g[4 * q + 1], g[4 * q + 2], g[4 * q + 3]};
            if (cb == 0 && owns_bias(r0)) {
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < KS; ++k) sum = column_sum16(frag_tr(Z, ZP, k * 16, 0, lane), sum);
                if (lane < RC) GB[lane] = sum;
            }
            step(set, r0);
        };
        for (int r0 = 0; r0 < a.d_out; r0 += SETS * RC) {
#pragma unroll
            for (int s = 0; s < SETS; ++s) chunk(s, r0 + s * RC);
        }
        return;
    }

    // data gradient: input units 32 bc .. and samples 32 bs .. , CBW x SBW blocks
    const int bc = (wave - 4) % (4 / CBW) * CBW, bs = (wave - 4) / (4 / CBW) * SBW;
    f32x16 back[CHAINS][CBW][SBW];
#pragma unroll
    for (int h = 0; h < CHAINS; ++h)
#pragma unroll
        for (int c = 0; c < CBW; ++c)
#pragma unroll
            for (int s = 0; s < SBW; ++s)
#pragma unroll
                for (int e = 0; e < 16; ++e) back[h][c][s][e] = 0.f;
    auto chunk = [&](int set, int r0) __attribute__((always_inline)) {
        stage(set, r0);
        const int h = CHAINS == 2 ? set & 1 : 0;
#pragma unroll
        for (int k = 0; k < RC / 16; ++k) {
            bf16x8 wf[CBW], zf[SBW];
#pragma unroll
            for (int c = 0; c < CBW; ++c) wf[c] = frag_tr(W, XP, k * 16, (bc + c) * 32, lane);
#pragma unroll
            for (int s = 0; s < SBW; ++s) zf[s] = *(const bf16x8*)(Z + ((bs + s) * 32 + (lane & 31)) * ZP + k * 16 + (lane >> 5) * 8);
#pragma unroll
            for (int c = 0; c < CBW; ++c)
#pragma unroll
                for (int s = 0; s < SBW; ++s)
                    back[h][c][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[c], zf[s], back[h][c][s], 0, 0, 0);
        }
        step(set, r0);
    };
    for (int r0 = 0; r0 < a.d_out; r0 += SETS * RC) {
#pragma unroll
        for (int s = 0; s < SETS; ++s) chunk(s, r0 + s * RC);
    }

    uint16_t* out = a.dz_prev + (size_t)learner * a.dz_prev_lstride;
#pragma unroll
    for (int cc = 0; cc < CBW; ++cc)
#pragma unroll
        for (int s = 0; s < SBW; ++s) {
            const int row = (bs + s) * 32 + (lane & 31);
            const f32x16 d = CHAINS == 2 ? back[0][cc][s] + back[CHAINS - 1][cc][s] : back[0][cc][s];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int cl = (bc + cc) * 32 + 8 * q + 4 * (lane >> 5);
                const u32x2 m = *(const u32x2*)(X + row * XP + cl);
                // stored activations are ReLU outputs (never negative): positive <=> non-zero magnitude
                const float v0 = (m.x & 0x7FFFu) ? d[4 * q + 0] : 0.f, v1 = (m.x & 0x7FFF0000u) ? d[4 * q + 1] : 0.f;
                const float v2 = (m.y & 0x7FFFu) ? d[4 * q + 2] : 0.f, v3 = (m.y & 0x7FFF0000u) ? d[4 * q + 3] : 0.f;
                if (row < a.B && c0 + cl < a.d_in)
                    *(u32x2*)(out + (size_t)row * a.ld_in + c0 + cl) = (u32x2){pack_bf16x2(v0, v1), pack_bf16x2(v2, v3)};
            }
        }
}

template <int BT, int STREAM, int CHAINS>
hipError_t launch(const StripArgs& a, hipStream_t st) {
    constexpr int SMEM = StripShape<BT>::SMEM;
    static_assert(SMEM <= 160 * 1024, "more LDS than a compute unit has");
    if (SMEM > 64 * 1024) {
        static hipError_t raised = hipFuncSetAttribute((const void*)strip_kernel<BT, STREAM, CHAINS>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, SMEM);
        if (raised != hipSuccess) return raised;
    }
    hipLaunchKernelGGL((strip_kernel<BT, STREAM, CHAINS>), dim3(a.padded), dim3(NT), SMEM, st, a);
    return hipGetLastError();
}
template <int BT, int CHAINS>
hipError_t launch_stream(const StripArgs& a, int stream, hipStream_t st) {
    if (stream == STREAM_NONE) return launch<BT, STREAM_NONE, CHAINS>(a, st);
    return stream == STREAM_LO ? launch<BT, STREAM_LO, CHAINS>(a, st) : launch<BT, STREAM_BOTH, CHAINS>(a, st);
}

}  // namespace

bool bf16_strip_ok(const LayerCall& c) {
    if (c.gather || !c.dz_prev || c.B > 256 || c.u || c.rows || c.partial || c.skip_bias || c.shared_w || c.d_in < 8 || c.ld_dz < 8) return false;
    // One workgroup per strip, so the strips have to fill the 256 compute units: at three quarters of the last round and more
    // this is at least as fast (rounds of 256-1024-1024-1024-40, separate kernels against this one, us: 192 strips, 128 samples
    // 936 / 881, 64 samples 769 / 760; 384 strips 1709 / 1708, 1470 / 1481; 448 of 64 1685 / 1582), below it is not (a layer: 128
    // strips 42 / 50; 320: 93 / 95; 264 strips of 4104 -> 2056: 160 / 173).
    const long strips = (long)((c.d_in + SC - 1) / SC) * c.P, rounds = (strips + 255) / 256;
    return 4 * strips >= 3 * 256 * rounds;
}

hipError_t bf16_strip(const LayerCall& c, hipStream_t st) {
    if (!bf16_strip_ok(c)) return hipErrorInvalidValue;
    StripArgs a = {};
    a.dz = (const uint16_t*)c.dz; a.dz_lstride = c.dz_stride; a.ld_dz = c.ld_dz;
    a.in = (const uint16_t*)c.in; a.in_lstride = c.in_stride; a.ld_in = c.ld_in;
    a.hi = c.ws; a.lo = c.wlo; a.bhi = c.bhi; a.blo = c.blo; a.lstride = c.ws_stride;
    a.dz_prev = (uint16_t*)c.dz_prev; a.dz_prev_lstride = c.dz_prev_stride;
    a.B = c.B; a.d_in = c.d_in; a.d_out = c.d_out; a.lr = c.lr;
    a.strips = (c.d_in + SC - 1) / SC;
    a.total = a.strips * c.P;
    a.padded = (a.total + 7) / 8 * 8;
    // where the separate data gradient would split its contraction (small launches, up to 128 samples), so does this one
    const bool two = bf16_backward_splits(c.P, c.B, c.d_in, c.d_out);
    const int stream = stream_policy(c, false);
    if (c.B <= 64) return two ? launch_stream<64, 2>(a, stream, st) : launch_stream<64, 1>(a, stream, st);
    if (c.B <= 128) return two ? launch_stream<128, 2>(a, stream, st) : launch_stream<128, 1>(a, stream, st);
    if (two) return hipErrorInvalidValue;                    // (never: 192 strips of more than 128 samples are 384 tiles)
    return launch_stream<256, 1>(a, stream, st);
}

}  // namespace kavg
