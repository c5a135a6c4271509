// fp32 path of the learner step (KAVG_FP32): forward, backward-data and the
// fused weight-gradient + SGD update, batched over learners.
//
// All three are products O[r][c] = sum_k R(r,k) * Cm(c,k) on the matrix cores in full fp32
// (v_mfma_f32_32x32x2_f32: exact fp32 products, fp32 accumulation; no reduced precision):
//
//   forward        r = sample, c = output unit, k = input unit
//                  O = act(A_{l-1} W_l^T + b_l)
//   backward-data  r = sample, c = input unit,  k = output unit
//                  dZ_{l-1} = (dZ_l W_l) * [A_{l-1} > 0]
//   update         r = output unit, c = input unit, k = sample
//                  W_l <- W_l - lr * dZ_l^T A_{l-1};  b_l <- b_l - lr * colsum(dZ_l)
//                  (the learner update of Algorithm 1; 1/B already sits in dZ_L)
//
// Operands move in 16-byte pieces, global -> registers (two slices ahead) -> LDS (two buffers, one barrier per slice).
// A piece needs 4-byte alignment only, so rows of any length take the same path; only the last slice of a contraction
// and tiles at the edge of an operand are read word by word, and nothing outside an operand is read at all.  An
// operand with k contiguous in memory ("K": activations, dZ, W of the forward pass) lies in LDS as [x][k] and a lane
// reads four k at once; one with x contiguous ("X": W of backward-data, both operands of the update) as [k][x].
// Every output is one chain of matrix instructions over ascending pairs of k (per split, see below), whatever the tile, so
// results depend on neither tiles nor timing.  (In fp32 a pre-activation whose sum is taken in another order can fall on
// the other side of zero, once in some ten million, and moves a row of a gradient by a sample's share.)
//
// What bounds these kernels: 3072-512 with 64 rows and 8 learners is 1.6 GFLOP per product, 10 us of the matrix
// cores' fp32 rate; the update also moves 100 MB of weights, 15 us out of the memory-side cache.  Measured on
// 3072-512-256-10 (8 learners, 64 rows): split forward product 24 -> 14 us per launch (mean of the two layers),
// backward-data 24 -> 11 us, the updates of a step 75 -> 30 us; a round of four steps 657 -> 325 us.  (Before: 64x64
// tiles everywhere, operands moved word by word, one slice ahead, the weights read after the contraction.)
//
// The forward pass may split the contraction over several workgroups where a layer has few output tiles: each writes
// its partial tile to a scratch buffer and a second small kernel (below a head: the head's, f32_head_finishes) adds the
// partials in ascending split order, then applies bias and ReLU.  The updates of all layers of a step are one launch: they
// depend on nothing but the backward pass, and on small models each launch is a few microseconds of latency.
#include "kavg_internal.h"
#include "head_update.h"
#include "loss_mean.h"

namespace kavg {

namespace {

constexpr int BK = 32;         // contraction slice
constexpr int UR = 64, UC = 128;   // tile of the update: units x inputs
constexpr int KPITCH = BK + 4; // [x][k] rows: 16-byte reads of 16 lanes fall on 16 different groups of four banks
__host__ __device__ constexpr int xpitch(int X) { return X + 8; }   // [k][x] rows

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

enum { EPI_FWD = 0, EPI_BWD = 1, EPI_PARTIAL = 2 };

// Workgroup -> piece of work: workgroup g runs on XCD g mod 8, so each XCD gets one contiguous range and the operands
// of a learner stay in one L2.
__device__ __forceinline__ int xcd_range(int g, int n_padded) { return (g & 7) * (n_padded >> 3) + (g >> 3); }

// The loaders issue no load behind a branch: a wait for one slice is then a counted wait and not a wait for everything
// in flight.  A piece that would leave its operand is read from the last place where it fits and shifted on its way to
// LDS; what lies outside the contraction becomes zero there.  WORDS: an extent is below 4, no piece fits, words are
// read one by one (from clamped places).

// elements sh .. of a piece, for sh in 0..3 (what is shifted in is not used)
__device__ __forceinline__ f32x4 shifted(const f32x4& v, int sh) {
    f32x4 o;
    o[0] = sh == 0 ? v[0] : sh == 1 ? v[1] : sh == 2 ? v[2] : v[3];
    o[1] = sh == 0 ? v[1] : sh == 1 ? v[2] : v[3];
    o[2] = sh == 0 ? v[2] : v[3];
    o[3] = v[3];
    return o;
}

// k-contiguous operand, X rows: thread t moves pieces (row t/8 + 32 i, k 4*(t%8))
template <int X, bool WORDS>
struct KLoader {
    static constexpr int N = X / 32;
    const float* p[N];
    int k4, at, nK, k_end;
    __device__ __forceinline__ void init(const float* base, long ld, const int32_t* gather, int x0, int nX, int nK_, int k_end_, int tid) {
        k4 = (tid & 7) * 4;
        // in LDS the even k of a group of eight come first, then the odd ones: a half wavefront reads every second k
        at = (tid >> 3) * KPITCH + (k4 & ~7) + (k4 & 7) / 2;
        nK = nK_; k_end = k_end_;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int x = min(x0 + (tid >> 3) + 32 * i, nX - 1);      // rows beyond the operand only reach outputs that are not stored
            p[i] = base + (gather ? (long)gather[x] : (long)x) * ld;
        }
    }
    __device__ __forceinline__ void load(f32x4 (&v)[N], int k0) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (WORDS) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = p[i][min(k0 + k4 + e, nK - 1)];
            } else {
                v[i] = *(const f32x4u*)(p[i] + min(k0 + k4, nK - 4));
            }
        }
    }
    __device__ __forceinline__ void store(f32x4 (&v)[N], float* lds, int k0) const {
        if (k0 + BK > k_end) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if constexpr (!WORDS) v[i] = shifted(v[i], max(k0 + k4 - (nK - 4), 0));
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = k0 + k4 + e < k_end ? v[i][e] : 0.f;
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            *(float2*)(lds + at + 32 * i * KPITCH) = make_float2(v[i][0], v[i][2]);
            *(float2*)(lds + at + 32 * i * KPITCH + 4) = make_float2(v[i][1], v[i][3]);
        }
    }
};

// x-contiguous operand, X columns: thread t moves pieces (row t/(X/4) + (1024/X) i, columns 4*(t%(X/4)))
template <int X, bool WORDS, bool EDGE>
struct XLoader {
    static constexpr int PPR = X / 4, ROWS = 256 / PPR, N = BK / ROWS;
    const float* p;          // base, at the piece's (clamped) columns
    long ld;
    int kr, at, nK, sh;      // sh: how far the piece was moved to fit
    int xw[4];               // WORDS: the (clamped) columns
    bool edge;
    // nX: readable columns of a row
    __device__ __forceinline__ void init(const float* base, long ld_, int x0, int nX, int nK_, int tid) {
        const int x = x0 + (tid % PPR) * 4;
        kr = tid / PPR;
        at = kr * xpitch(X) + (tid % PPR) * 4;
        nK = nK_;
        ld = ld_;
        edge = x0 + X > nX;
        sh = max(x - (nX - 4), 0);
        p = WORDS ? base : base + min(x, nX - 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) xw[e] = min(x + e, nX - 1);
    }
    // row[i]: memory row of the piece in the slice, inside the operand
    __device__ __forceinline__ void load(f32x4 (&v)[N], const int (&row)[N]) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float* r = p + row[i] * ld;
            if constexpr (WORDS) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[i][e] = r[xw[e]];
            } else {
                v[i] = *(const f32x4u*)r;
            }
        }
    }
    __device__ __forceinline__ void rows(int (&row)[N], int k0) const {
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = min(k0 + kr + ROWS * i, nK - 1);
    }
    // take: -1 where the rows are looked up in the table, 0 where the table is ignored
    __device__ __forceinline__ void rows(int (&row)[N], int k0, const int32_t* table, int take) const {
        rows(row, k0);
#pragma unroll
        for (int i = 0; i < N; ++i) row[i] = (table[row[i]] & take) | (row[i] & ~take);
    }
    __device__ __forceinline__ void store(f32x4 (&v)[N], float* lds, int k0) const {
        if (!WORDS && EDGE && edge) {
#pragma unroll
            for (int i = 0; i < N; ++i) v[i] = shifted(v[i], sh);
        }
        if (k0 + BK > nK) {
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (k0 + kr + ROWS * i >= nK) v[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < N; ++i) *(f32x4*)(lds + at + ROWS * i * xpitch(X)) = v[i];
    }
};

// The slices of a contraction, two ahead in registers: step(set, slice, request the slice after next).  Straight-line code around every request, see the loaders.
template <class Load, class Step>
__device__ __forceinline__ void pipeline(int n, Load load, Step step) {
    load(0, 0);
    if (n == 1) {
        step(0, 0, false);
        return;
    }
    load(1, 1);
    int s = 0;
    for (; s + 3 < n; s += 2) { step(0, s, true); step(1, s + 1, true); }
    if (s + 2 < n) { step(0, s, true); step(1, s + 1, false); step(0, s + 2, false); }
    else { step(0, s, false); step(1, s + 1, false); }
}

struct RowArgs {
    const float* R; size_t r_lstride; int ldR; const int32_t* gather; long gather_lstride;   // [r][k], k contiguous
    const float* C; size_t c_lstride; long ldC;                     // forward: [c][k]; backward: [k][c]
    int nR, nC, nK;
    int k_chunk, splits;                                            // contraction range of one split (nK: not split)
    int tiles_r, tiles_c, total, padded;
    float* out; size_t out_lstride; int ld_out; size_t split_stride;
    const float* bias; size_t bias_lstride; int relu;               // forward
    const float* mask; size_t mask_lstride; int ld_mask;            // backward: previous activations
};

// 64 x 64 tile in quarters, or 32 x 128 with the four wavefronts side by side (for batches whose last 64-row tile would be
// at most half full).
template <int EPI, int TR, bool WORDS>
__global__ void __launch_bounds__(256, WORDS || TR == 32 ? 3 : 4) rows_kernel(RowArgs a) {
    constexpr bool CK = EPI != EPI_BWD;
    constexpr int TC = TR == 64 ? 64 : 128;
    constexpr int CSZ = CK ? TC * KPITCH : BK * xpitch(TC);
    __shared__ __align__(16) float lds[2][TR * KPITCH + CSZ];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 31, half = lane >> 5;
    int at = xcd_range(blockIdx.x, a.padded);
    if (at >= a.total) return;
    const int ct = at % a.tiles_c; at /= a.tiles_c;
    const int rt = at % a.tiles_r; at /= a.tiles_r;
    const int split = at % a.splits, learner = at / a.splits;
    const int r0 = rt * TR, c0 = ct * TC;
    const int rq = TR == 64 ? (wave >> 1) * 32 : 0, cq = TR == 64 ? (wave & 1) * 32 : wave * 32;
    const int k_begin = split * a.k_chunk, k_end = min(k_begin + a.k_chunk, a.nK);

    typedef KLoader<TR, WORDS> RLoader;
    typedef KLoader<TC, WORDS> CKLoader;
    typedef XLoader<TC, WORDS, true> CXLoader;
    RLoader lr;
    CKLoader lck;
    CXLoader lcx;
    lr.init(a.R + (size_t)learner * a.r_lstride, a.ldR, a.gather ? a.gather + learner * a.gather_lstride : nullptr, r0, a.nR, a.nK, k_end, tid);
    if constexpr (CK) lck.init(a.C + (size_t)learner * a.c_lstride, a.ldC, nullptr, c0, a.nC, a.nK, k_end, tid);
    else lcx.init(a.C + (size_t)learner * a.c_lstride, a.ldC, c0, a.nC, a.nK, tid);

    f32x16 acc = {};
    f32x4 rv[2][RLoader::N], cv[2][TC / 32];
    auto load = [&](int set, int s) __attribute__((always_inline)) {
        const int k0 = k_begin + s * BK;
        lr.load(rv[set], k0);
        if constexpr (CK) lck.load(cv[set], k0);
        else {
            int row[CXLoader::N];
            lcx.rows(row, k0);
            lcx.load(cv[set], row);
        }
    };
    auto step = [&](int set, int s, bool more) __attribute__((always_inline)) {
        const int k0 = k_begin + s * BK;
        float* R = lds[set];
        float* C = lds[set] + TR * KPITCH;
        lr.store(rv[set], R, k0);
        if constexpr (CK) lck.store(cv[set], C, k0); else lcx.store(cv[set], C, k0);
        if (more) load(set, s + 2);
        __syncthreads();
#pragma unroll
        for (int g = 0; g < BK / 8; ++g) {                            // half a wavefront: k = 8 g + half, + 2, + 4, + 6
            const f32x4 r4 = *(const f32x4*)(R + (rq + m) * KPITCH + 8 * g + 4 * half);
            f32x4 c4;
            if constexpr (CK) c4 = *(const f32x4*)(C + (cq + m) * KPITCH + 8 * g + 4 * half);
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i) c4[i] = C[(8 * g + 2 * i + half) * xpitch(TC) + cq + m];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(r4[i], c4[i], acc, 0, 0, 0);
        }
    };
    pipeline((k_end - k_begin + BK - 1) / BK, load, step);

    // accumulator v of lane l is the output (row 8*(v/4) + 4*(l/32) + v%4, column l%32) of the wavefront's block
    const int c = c0 + cq + m;
    if (c >= a.nC) return;
    float* out = a.out + (size_t)learner * a.out_lstride + c;
    if (EPI == EPI_PARTIAL) out += (size_t)split * a.split_stride;
    const float b = EPI == EPI_FWD ? a.bias[(size_t)learner * a.bias_lstride + c] : 0.f;
    const float* mask = EPI == EPI_BWD ? a.mask + (size_t)learner * a.mask_lstride + c : nullptr;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = r0 + rq + 8 * (v >> 2) + 4 * half + (v & 3);
        if (r >= a.nR) continue;
        float z = acc[v];
        if (EPI == EPI_FWD) { z += b; if (a.relu) z = fmaxf(z, 0.f); }
        if (EPI == EPI_BWD) z = mask[(size_t)r * a.ld_mask] > 0.f ? z : 0.f;
        out[(size_t)r * a.ld_out] = z;
    }
}

struct UpdLayer {
    const float* dz; size_t dz_lstride; int ld_dz;                  // [k][r]
    const float* in; size_t in_lstride; int ld_in; const int32_t* gather; long gather_lstride;   // [k][c]
    float* w; float* b; float* u; float* ub;                        // u, ub: velocities, null: plain SGD
    int d_out, d_in, tiles_r, tiles_c, total, padded;
    int head;                                                       // the last layer, of few classes: head_tile
};
constexpr int GROUP = 8;       // layers per launch
struct UpdArgs {
    UpdLayer layer[GROUP];
    int n_layers, B;
    size_t lstride;            // between learners, in weights and velocities
    float lr, beta;
    LossMeans losses;          // n > 0: computed by the workgroups behind those of the layers, four each
};

// 64 x 128 tile of a layer's weights (53 KB of LDS, 168 registers: three workgroups per compute unit).  A wavefront owns
// 32 x 64: two column blocks interleaved (column 2m + i), so that a lane holds pairs of neighbouring columns and moves
// them in 8-byte pieces, 256 bytes per row and half wavefront.  The weights are requested right after the first operand
// slice and arrive under the contraction.  One slice ahead in registers: two ahead cost the third workgroup (31 -> 37 us).
// INSIDE: the whole tile lies inside the layer.
template <bool WORDS, bool INSIDE>
__device__ __forceinline__ void update_tile(const UpdArgs& a, const UpdLayer& q, int learner, int rt, int ct, float* lds) {
    constexpr int RSZ = BK * xpitch(UR), CSZ = BK * xpitch(UC);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m = lane & 31, half = lane >> 5;
    const int r0 = rt * UR, c0 = ct * UC, nK = a.B;
    const int rq = (wave >> 1) * 32, cq = (wave & 1) * 64;

    typedef XLoader<UR, WORDS, !INSIDE> RLoader;
    typedef XLoader<UC, WORDS, !INSIDE> CLoader;
    RLoader lr;
    CLoader lc;
    // (without a gather the look-ups read, and ignore, words of dZ: no branch around a load)
    const int32_t* table = q.gather ? q.gather + learner * q.gather_lstride : (const int32_t*)q.dz;
    lr.init(q.dz + (size_t)learner * q.dz_lstride, q.ld_dz, r0, q.ld_dz, nK, tid);
    lc.init(q.in + (size_t)learner * q.in_lstride, q.ld_in, c0, q.d_in, nK, tid);

    f32x4 rv[RLoader::N], cv[CLoader::N];
    int row[2][CLoader::N];      // memory rows of a slice, looked up before the slice that precedes it is requested
    const int take = q.gather ? -1 : 0;
    lc.rows(row[0], 0, table, take);
    auto load = [&](int s) __attribute__((always_inline)) {
        int rr[RLoader::N];
        lc.rows(row[1], (s + 1) * BK, table, take);
        lr.rows(rr, s * BK);
        lr.load(rv, rr);
        lc.load(cv, row[0]);
#pragma unroll
        for (int i = 0; i < CLoader::N; ++i) row[0][i] = row[1][i];
    };

    // the tile's weights: rows rb + 8*(v/4) + v%4, columns c and c+1; places outside are read clamped, never stored
    const int c = c0 + cq + 2 * m, rb = r0 + rq + 4 * half;
    const size_t wat = (size_t)learner * a.lstride, tat = wat + (size_t)r0 * q.d_in + c0;
    const unsigned lane_at = (unsigned)(rq + 4 * half) * (unsigned)q.d_in + cq + 2 * m;      // inside the tile
    float w0[16], w1[16];
    const int cl = WORDS ? min(c, q.d_in - 1) : min(c, q.d_in - 2), ch = min(c + 1, q.d_in - 1);
    auto fetch = [&](const float* src, float (&x0)[16], float (&x1)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if constexpr (INSIDE) {
                const f32x2u t = *(const f32x2u*)(src + tat + (size_t)(8 * (v >> 2) + (v & 3)) * q.d_in + lane_at);
                x0[v] = t.x; x1[v] = t.y;
            } else {
                const float* s = src + wat + (size_t)min(rb + 8 * (v >> 2) + (v & 3), q.d_out - 1) * q.d_in;
                if constexpr (WORDS) { x0[v] = s[cl]; x1[v] = s[ch]; }
                else { const f32x2u t = *(const f32x2u*)(s + cl); x0[v] = t.x; x1[v] = t.y; }
            }
        }
    };
    const bool last_odd = !INSIDE && !WORDS && c == q.d_in - 1;     // this pair was read one column to the left
    auto put = [&](float* dst, const float (&x0)[16], const float (&x1)[16]) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if constexpr (INSIDE) {
                const f32x2u t = {x0[v], x1[v]};
                *(f32x2u*)(dst + tat + (size_t)(8 * (v >> 2) + (v & 3)) * q.d_in + lane_at) = t;
            } else {
                const int r = rb + 8 * (v >> 2) + (v & 3);
                float* d = dst + wat + (size_t)r * q.d_in + c;
                if (r < q.d_out && c < q.d_in) d[0] = x0[v];
                if (r < q.d_out && c + 1 < q.d_in) d[1] = x1[v];
            }
        }
    };

    f32x16 acc0 = {}, acc1 = {};
    float bsum = 0.f;                                               // column sum of dZ: unit r0 + tid, samples ascending
    const bool bias = ct == 0 && tid < UR;
    auto step = [&](int s, bool more) __attribute__((always_inline)) {
        float* R = lds + (s & 1) * (RSZ + CSZ);
        float* C = R + RSZ;
        lr.store(rv, R, s * BK);
        lc.store(cv, C, s * BK);
        if (more) load(s + 1);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < BK / 2; ++t) {
            const int k = 2 * t + half;
            const float r1 = R[k * xpitch(UR) + rq + m];
            const float2 c2 = *(const float2*)(C + k * xpitch(UC) + cq + 2 * m);
            acc0 = __builtin_amdgcn_mfma_f32_32x32x2f32(r1, c2.x, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(r1, c2.y, acc1, 0, 0, 0);
        }
        if (bias) {
#pragma unroll 8
            for (int k = 0; k < BK; ++k) bsum += R[k * xpitch(UR) + tid];
        }
    };
    load(0);
    fetch(q.w, w0, w1);
    const int n = (nK + BK - 1) / BK;
    step(0, true);               // outside the loop: its waits leave the weights in flight (and no branch: the request is
                                 // for the last row over and over where there is one slice only)
    for (int s = 1; s + 1 < n; ++s) step(s, true);
    if (n > 1) step(n - 1, false);

    float g0[16], g1[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) { g0[v] = acc0[v]; g1[v] = acc1[v]; }
    if (q.u) {                                                      // heavy ball inside the learner
        float u0[16], u1[16];
        fetch(q.u, u0, u1);
#pragma unroll
        for (int v = 0; v < 16; ++v) { g0[v] = a.beta * (last_odd ? u1[v] : u0[v]) + g0[v]; g1[v] = a.beta * u1[v] + g1[v]; }
        put(q.u, g0, g1);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) { w0[v] = (last_odd ? w1[v] : w0[v]) - a.lr * g0[v]; w1[v] -= a.lr * g1[v]; }
    put(q.w, w0, w1);
    if (bias && r0 + tid < q.d_out) {
        const size_t bat = wat + r0 + tid;
        if (q.ub) { bsum = a.beta * q.ub[bat] + bsum; q.ub[bat] = bsum; }
        q.b[bat] = q.b[bat] - a.lr * bsum;
    }
}

// The step of a last layer of at most CT classes on sixteen of its input units.  Lane = 4*g + pl: sample group g (samples
// s = g mod 16) and input unit 16 block + 4 wave + pl.  Every lane sums dZ_L[s][c] * A[s][unit] over its samples in ascending
// order; a butterfly over the group bits of the lane index adds the sixteen groups, after which lane group g applies the update
// of class c = g.  What waits here is a chain of latencies; as a launch of its own it was 5 us and a gap of every step
// (rounds, us, with that launch and without: 3072-512-256-10, 8 learners of 64 346 / 331; 300-500-10, 2 of 16 236 / 208;
// 500-700-16, 30 of 20 203 / 188).
template <int CT>
__device__ __forceinline__ void head_tile(const UpdArgs& a, const UpdLayer& q, int learner, int block) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int grp = lane >> 2, pl = lane & 3;
    const int unit = block * 16 + wave * 4 + pl;
    const bool live = unit < q.d_in;
    const int uu = live ? unit : q.d_in - 1;                        // out-of-range lanes shadow the last unit, never store
    const int32_t* g = q.gather + (long)learner * q.gather_lstride;
    const float* in = q.in + (size_t)learner * q.in_lstride;
    const float* dz = q.dz + (size_t)learner * q.dz_lstride;
    const size_t lat = (size_t)learner * a.lstride;

    float acc[CT], bsum[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = bsum[c] = 0.f;
#pragma unroll 4
    for (int s = grp; s < a.B; s += 16) {
        const float x = in[(size_t)(q.gather ? g[s] : s) * q.ld_in + uu];
        float gz[CT];                                               // one row of dZ_L; entries beyond ld_dz are zero
#pragma unroll
        for (int i = 0; i < CT / 4; ++i) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (4 * i < q.ld_dz) v = *(const f32x4*)(dz + (size_t)s * q.ld_dz + 4 * i);      // (ld_dz is a multiple of 8)
            gz[4 * i] = v.x; gz[4 * i + 1] = v.y; gz[4 * i + 2] = v.z; gz[4 * i + 3] = v.w;
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            bsum[c] += gz[c];                                       // bias gradient: column sum of dZ_L
            acc[c] = fmaf(gz[c], x, acc[c]);
        }
    }
    float mine = 0.f;
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const float v = groups_sum(acc[c]);
        if (c == grp) mine = v;
    }
    if (live && grp < q.d_out) {
        const size_t at = lat + (size_t)grp * q.d_in + unit;
        if (q.u) { mine = a.beta * q.u[at] + mine; q.u[at] = mine; }       // heavy ball inside the learner
        q.w[at] = q.w[at] - a.lr * mine;
    }
    if (block == 0 && wave == 0) {
        float sum = 0.f;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const float v = groups_sum(bsum[c]);
            if (c == grp) sum = v;
        }
        if (pl == 0 && grp < q.d_out) {
            const size_t at = lat + grp;
            if (q.ub) { sum = a.beta * q.ub[at] + sum; q.ub[at] = sum; }
            q.b[at] = q.b[at] - a.lr * sum;
        }
    }
}

template <bool WORDS>
__global__ void __launch_bounds__(256, WORDS ? 2 : 3) update_kernel(UpdArgs a) {
    __shared__ __align__(16) float lds[2 * BK * (xpitch(UR) + xpitch(UC))];
    int g = blockIdx.x, li = 0;
    while (li + 1 < a.n_layers && g >= a.layer[li].padded) g -= a.layer[li++].padded;
    const UpdLayer& q = a.layer[li];
    if (g >= q.padded) {
        const int r = (g - q.padded) * 4 + (threadIdx.x >> 6);
        if (r < a.losses.n) loss_mean_wave(a.losses, r, threadIdx.x & 63);
        return;
    }
    int at = xcd_range(g, q.padded);
    if (at >= q.total) return;
    const int rt = at % q.tiles_r; at /= q.tiles_r;
    const int ct = at % q.tiles_c, learner = at / q.tiles_c;
    if (q.head) {
        if (q.d_out <= 8) head_tile<8>(a, q, learner, ct); else head_tile<16>(a, q, learner, ct);
        return;
    }
    if (!WORDS && (rt + 1) * UR <= q.d_out && (ct + 1) * UC <= q.d_in) update_tile<WORDS, !WORDS>(a, q, learner, rt, ct, lds);
    else update_tile<WORDS, false>(a, q, learner, rt, ct, lds);
}

// out[j][r][c] = act(sum_s partial[s][j][r][c] + bias[j][c]), splits added in ascending order
__global__ void __launch_bounds__(256)
finish_forward_kernel(const float* __restrict__ partial, size_t split_stride, int splits, const float* __restrict__ bias,
                      size_t bias_stride, float* __restrict__ out, int P, int B, int ld_out, int nC, int relu) {
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    const size_t per_learner = (size_t)B * ld_out;
    if (e >= (size_t)P * per_learner) return;
    const int c = (int)(e % ld_out);
    if (c >= nC) return;
    const int learner = (int)(e / per_learner);
    // eight partials are requested together, then added in ascending order (same sum, one round trip
    // to memory per eight splits instead of one per split)
    float z = 0.f;
    int s = 0;
    for (; s + 8 <= splits; s += 8) {
        float t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = partial[(size_t)(s + u) * split_stride + e];
#pragma unroll
        for (int u = 0; u < 8; ++u) z += t[u];
    }
    for (; s < splits; ++s) z += partial[(size_t)s * split_stride + e];
    z += bias[(size_t)learner * bias_stride + c];
    if (relu) z = fmaxf(z, 0.f);
    out[e] = z;
}

int div_up(int a, int b) { return (a + b - 1) / b; }

template <int EPI>
hipError_t run_rows(RowArgs& a, int P, hipStream_t st) {
    const int TR = div_up(a.nR, 32) & 1 ? 32 : 64;      // 32: a last tile of 64 rows would be at most half full
    a.tiles_r = div_up(a.nR, TR);
    a.tiles_c = div_up(a.nC, TR == 64 ? 64 : 128);
    a.total = a.tiles_r * a.tiles_c * a.splits * P;
    a.padded = div_up(a.total, 8) * 8;
    const bool words = a.nK < 4 || (EPI == EPI_BWD && a.nC < 4);
    if (words && TR == 64) hipLaunchKernelGGL((rows_kernel<EPI, 64, true>), dim3(a.padded), dim3(256), 0, st, a);
    else if (words) hipLaunchKernelGGL((rows_kernel<EPI, 32, true>), dim3(a.padded), dim3(256), 0, st, a);
    else if (TR == 64) hipLaunchKernelGGL((rows_kernel<EPI, 64, false>), dim3(a.padded), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((rows_kernel<EPI, 32, false>), dim3(a.padded), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace

// How the forward pass of a layer splits its contraction: returns the number of splits and the
// contraction range of each (a multiple of the slice length).  Depends on the shapes only.
int f32_forward_plan(int P, int B, int d_in, int d_out, int* chunk_out) {
    const long tiles = (long)div_up(B, 64) * div_up(d_out, 64) * P;
    long s = 1;
    if (tiles < 256 && d_in > 4 * BK) {
        s = (512 + tiles - 1) / tiles;               // aim at ~512 workgroups
        const long max_s = d_in / (2 * BK);          // at least two slices per split
        if (s > max_s) s = max_s;
        if (s > 64) s = 64;
        if (s < 1) s = 1;
    }
    int chunk = (int)((d_in + s - 1) / s);
    chunk = (chunk + BK - 1) / BK * BK;
    if (chunk_out) *chunk_out = chunk;
    return (d_in + chunk - 1) / chunk;               // splits that actually receive work
}

// Up to sixteen partial products of a unit arrive in one round trip, beside the head's weights; more would be a round trip each
// eight of every 64 units, in one wavefront per sample, where finish_forward_kernel has a lane for every unit.  Rounds, us, with
// that launch and with the sums in the head: 3072-512-256-10, 8 learners of 64 (8 splits) 331 / 324; 300-500-10, 2 of 16 (4)
// 210 / 196; 784-300-10, 4 of 16 (9) 103 / 97; 900-100-16, 2 of 32 (10) 95.5 / 85.5; 1024-1000-8, 2 of 32 (16) 132 / 131.
bool f32_head_finishes(int P, int B, int d_in, int d_out) {
    const int splits = f32_forward_plan(P, B, d_in, d_out, nullptr);
    return splits > 1 && splits <= HEAD_SPLITS;
}

hipError_t f32_forward(const LayerCall& c, hipStream_t st) {
    RowArgs a = {};
    a.R = (const float*)c.in; a.r_lstride = c.gather ? 0 : c.in_stride; a.ldR = c.ld_in;    // gathered: one data set for all
    a.gather = c.gather; a.gather_lstride = c.gather_stride;
    a.C = c.w; a.c_lstride = c.w_stride; a.ldC = c.d_in;
    a.nR = c.B; a.nC = c.d_out; a.nK = c.d_in;
    a.out = (float*)c.out; a.out_lstride = c.out_stride; a.ld_out = c.ld_out;
    a.bias = c.b; a.bias_lstride = c.w_stride;
    a.relu = c.relu;
    a.splits = f32_forward_plan(c.P, c.B, c.d_in, c.d_out, &a.k_chunk);
    if (a.splits == 1 || !c.scratch) {
        a.k_chunk = a.nK; a.splits = 1;
        return run_rows<EPI_FWD>(a, c.P, st);
    }
    a.out = (float*)c.scratch;
    a.split_stride = (size_t)c.P * c.out_stride;
    hipError_t e = run_rows<EPI_PARTIAL>(a, c.P, st);
    if (e != hipSuccess || c.unfinished) return e;
    const size_t total = (size_t)c.P * c.out_stride;
    hipLaunchKernelGGL(finish_forward_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                       (const float*)c.scratch, a.split_stride, a.splits, c.b, c.w_stride, (float*)c.out, c.P, c.B,
                       c.ld_out, c.d_out, c.relu);
    return hipGetLastError();
}

hipError_t f32_backward_data(const LayerCall& c, hipStream_t st) {
    RowArgs a = {};
    a.R = (const float*)c.dz; a.r_lstride = c.dz_stride; a.ldR = c.ld_dz;
    a.C = c.w; a.c_lstride = c.w_stride; a.ldC = c.d_in;             // Cm(c = input unit, k = output unit) = W[k][c]
    a.nR = c.B; a.nC = c.d_in; a.nK = c.d_out; a.k_chunk = a.nK; a.splits = 1;
    a.out = (float*)c.dz_prev; a.out_lstride = c.dz_prev_stride; a.ld_out = c.ld_in;
    a.mask = (const float*)c.in; a.mask_lstride = c.in_stride; a.ld_mask = c.ld_in;
    return run_rows<EPI_BWD>(a, c.P, st);
}

hipError_t f32_update(const LayerCall* calls, int n, const LossMeans* losses, hipStream_t st) {
    for (int at = 0; at < n; at += GROUP) {
        UpdArgs a = {};
        a.n_layers = n - at < GROUP ? n - at : GROUP;
        a.B = calls[at].B; a.lstride = calls[at].w_stride; a.lr = calls[at].lr; a.beta = calls[at].beta;
        int wgs = 0;
        bool words = false;
        for (int i = 0; i < a.n_layers; ++i) {
            const LayerCall& c = calls[at + i];
            UpdLayer& q = a.layer[i];
            q.dz = (const float*)c.dz; q.dz_lstride = c.dz_stride; q.ld_dz = c.ld_dz;
            q.in = (const float*)c.in; q.in_lstride = c.gather ? 0 : c.in_stride; q.ld_in = c.ld_in;
            q.gather = c.gather; q.gather_lstride = c.gather_stride;
            q.w = c.w; q.b = c.b; q.u = c.u; q.ub = c.ub;
            q.d_out = c.d_out; q.d_in = c.d_in;
            q.head = c.head;
            q.tiles_r = c.head ? 1 : div_up(c.d_out, UR); q.tiles_c = div_up(c.d_in, c.head ? 16 : UC);
            q.total = q.tiles_r * q.tiles_c * c.P;
            q.padded = div_up(q.total, 8) * 8;
            wgs += q.padded;
            words = words || (!c.head && (c.d_in < 4 || c.ld_dz < 4 || c.d_in >= 1 << 24));      // (2^24: reach of lane_at)
        }
        if (losses && at + a.n_layers == n) {
            a.losses = *losses;
            wgs += (losses->n + 3) / 4;
        }
        if (words) hipLaunchKernelGGL(update_kernel<true>, dim3(wgs), dim3(256), 0, st, a);
        else hipLaunchKernelGGL(update_kernel<false>, dim3(wgs), dim3(256), 0, st, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace kavg
