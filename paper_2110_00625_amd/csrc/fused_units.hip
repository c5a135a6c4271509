// All K local steps of Algorithm 1 in ONE launch, for fp32 models with one hidden layer that is wide and inputs that are
// short: d_0 <= 512 inputs, any number of hidden units, at most 16 classes, minibatches of at most 64 rows.
//
// fused_small.hip cuts W_1 into column chunks, so its workgroups exchange B x (hidden units) partial pre-activations per
// step and its hidden layer is bounded by what one workgroup can hold.  Here W_1 is cut into groups of UN hidden units (16,
// 32 or 64): workgroup (j, g) keeps the UN rows of learner j's W_1 and the UN columns of its W_2 in LDS for the whole call
// and forms its units' activations completely; what it lacks is the rest of the logits.  The exchange of a step is one
// B x C tile of partial logits per workgroup (a few KB) instead of a B x 64 tile per column chunk:
//   1. A_1[:, own units] = relu(X[idx] W_1^T + b_1) by fp32 matrix instructions, the contraction spread over the wavefronts;
//   2. partial logits A_1 W_2^T of the own units, written to device memory as tagged words;
//   3. the G partials of every logit are collected and added in ascending group order (+ b_2), then softmax
//      cross-entropy and dZ_2 -- identically in each of the learner's workgroups;
//   4. dZ_1[:, own units] = (dZ_2 W_2) masked by the ReLU; SGD steps on the own rows of W_1, columns of W_2, b_1 and
//      (identically everywhere) b_2.
// With G = 1 nothing is exchanged.  Tags, buffers and the bounded polls are those of fused_small.hip: a word (value, tag)
// validates itself, two buffers alternate (one is overwritten at step k+2, which its writer reaches only after every reader
// has finished step k), all P*G workgroups are resident because there are no more of them than compute units (launches of
// several contexts that do not fit together take turns, kavg_api.hip), and a wait that runs out of polls raises an error word
// and carries on, so every wavefront reaches the end.
//
// What bounds it: the chain of phases inside a step, each of them a few dependent LDS round trips and matrix instructions on
// eight wavefronts, not a throughput.  Measured per step on 256-256-10 with 6 learners, B = 32 (16 groups of 16 units), us:
// pre-activations 0.95, their sum and ReLU 0.3, partial logits 1.0, exchange and softmax 1.5, dZ_1 1.0, step of W_1 1.3; loading
// and storing the parameters 10 per launch.  A round (K = 4) with the meta step and the read-back of the losses: 79 us, as
// launches per layer (six dependent kernels of 4-17 us per step) 180 us; 48 learners, B = 4, K = 8: 153 against 419 us.
// What it took: all workgroups of a learner on one XCD (88 -> 79), no division by a run-time number in a phase (64 -> 42 us for
// the launch), parameters requested all at once (48 learners: 9 -> 4 us per launch), sums over the rows that exist and not
// over whole blocks (minibatches of 4), the next step's rows written to a second LDS buffer while the partial logits travel, biases as a column of the
// products instead of serial sums at the end of a step.
#include "kavg_internal.h"
#include "fused_common.h"

#include <type_traits>

namespace kavg {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 512, NW = NT / 64;
constexpr int CLS = 16;          // classes (upper bound)
constexpr int ROWS = 64;         // minibatch rows (upper bound)
constexpr int KBMAX = 1024;      // K*B, at most
constexpr int D0MAX = 512;       // inputs (upper bound): two 16-byte pieces per lane and row
constexpr int GMAX = 16;         // workgroups per learner, at most
constexpr int PD = CLS + 4;      // row pitch of dZ_2

// Row pitches (in words) are 4 modulo 8: the sixteen rows of an operand block then start in sixteen different groups of four
// banks, so 16-byte operand reads are conflict-free.
struct UnitsLayout {
    int UN, G, D, PW, PU, R;     // units per workgroup, workgroups per learner, inputs + 1 rounded up to 16, pitches of tiles D / UN wide, rows rounded up to 16
    int NX;                      // buffers of X: two where they fit
    int W1, X, Z, A1, D1, W2, D2, b2, rowloss, y, idx, gave_up, words;     // offsets in 4-byte words, total
};
constexpr int LDS_WORDS = 160 * 1024 / 4;

__host__ __device__ inline UnitsLayout units_layout(int B, int K, int d0, int d1, int UN) {
    UnitsLayout q{};
    q.UN = UN; q.G = (d1 + UN - 1) / UN;
    q.D = (d0 + 16) / 16 * 16; q.PW = q.D + 4; q.PU = UN + 4; q.R = (B + 15) / 16 * 16;
    int p = 0;
    auto take = [&](int words) { const int at = p; p += (words + 3) / 4 * 4; return at; };
    q.W1 = take(UN * q.PW);
    const int blocks = (q.R / 16) * (UN / 16);
    q.Z = take((blocks > NW ? blocks : NW) * 256);
    q.A1 = take(q.R * q.PU);
    q.D1 = take(q.R * q.PU);
    q.W2 = take(2 * CLS * q.PU);
    q.D2 = take(q.R * PD);
    q.b2 = take(CLS); q.rowloss = take(ROWS); q.y = take(2 * ROWS);
    q.idx = take(K * B);
    q.gave_up = take(1);
    q.NX = p + 2 * q.R * q.PW <= LDS_WORDS ? 2 : 1;
    q.X = take(q.NX * q.R * q.PW);
    q.words = p;
    return q;
}

// VEC: rows of W_1 and X are read and written 16 bytes at a time (d_0 a multiple of 4), else word by word.
// UN is a template parameter so that no index below needs a division by it (a step is a chain of short phases: each
// division by a run-time number in a phase shows).
template <bool VEC, int UN>
__global__ void __launch_bounds__(NT) fused_units_kernel(FusedSmallCall a, int spread) {
    extern __shared__ __align__(16) float sm[];
    const UnitsLayout q = units_layout(a.B, a.K, a.d0, a.d1, UN);
    constexpr int PU = UN + 4, ublocks = UN / 16;
    const int G = q.G, PW = q.PW;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Workgroups are dealt round-robin to the 8 XCDs: with spread = 0 all workgroups of a learner run on one of them, so
    // that what they exchange meets in one L2.  (Nothing but the time depends on it.)
    const int j = spread ? blockIdx.x / G : (int)(blockIdx.x >> 3) / G * 8 + (int)(blockIdx.x & 7);
    const int g = spread ? blockIdx.x % G : (int)(blockIdx.x >> 3) % G;
    if (j >= a.P) return;
    const int ub = g * UN, un = min(UN, a.d1 - ub);             // units ub .. ub+un-1 are this workgroup's
    const int l16 = lane & 15, lq = lane >> 4;
    float* rep = a.reps + (size_t)j * a.rep_stride;
    float *W1 = sm + q.W1, *Z = sm + q.Z, *A1 = sm + q.A1, *D1 = sm + q.D1, *D2 = sm + q.D2;
    float *b2 = sm + q.b2, *rowloss = sm + q.rowloss;
    int *idx = (int*)(sm + q.idx), *gave_up_word = (int*)(sm + q.gave_up);

    // ---- parameters: requested together, ahead of everything else; places outside the model are read from inside and dropped
    constexpr int RW = UN / NW, W2N = (CLS * UN + NT - 1) / NT;
    f32x4 wv[2][RW];
    float bv[RW], w2v[W2N];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const float* src = rep + a.w1_off + (size_t)(ub + min(wave + NW * i, un - 1)) * a.d0;
            const int c = h * 256 + lane * 4;
            if (VEC) wv[h][i] = *(const f32x4*)(src + min(c, a.d0 - 4));
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) wv[h][i][e] = src[min(c + e, a.d0 - 1)];
            }
        }
#pragma unroll
    for (int i = 0; i < RW; ++i) bv[i] = rep[a.b1_off + ub + min(wave + NW * i, un - 1)];
#pragma unroll
    for (int i = 0; i < W2N; ++i) {
        const int e = tid + NT * i;
        w2v[i] = rep[a.w2_off + (size_t)min(e / UN, a.C - 1) * a.d1 + ub + min(e % UN, un - 1)];
    }
    const float b2v = rep[a.b2_off + min(tid, a.C - 1)];

    // ---- the learner's minibatch indices: draw (j, t0 + k, m) of the counter-based stream, or the caller's ----
    for (int e = tid; e < a.K * a.B; e += NT) {
        int32_t v;
        if (a.generate_idx) {
            v = index_draw(a.seed, (uint32_t)j, a.t0 + (uint32_t)(e / a.B), (uint32_t)(e % a.B), a.N);
            if (g == 0) a.idx[(size_t)j * a.K * a.B + e] = v;
        } else {
            v = a.idx[(size_t)j * a.K * a.B + e];
        }
        idx[e] = v;
    }

    // ---- parameters into LDS; positions outside the model (and rows of the minibatch beyond B) are zero throughout.
    // Column d_0 of W_1 is b_1 and column d_0 of every row of X is 1: the bias is added and stepped by the products. ----
    static_assert(D0MAX + 16 <= 2 * 256 + 16, "two pieces per lane and row, and the last sixteen columns");
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const int r = wave + NW * i;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int c = h * 256 + lane * 4;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = r < un ? (c + e < a.d0 ? wv[h][i][e] : c + e == a.d0 ? bv[i] : 0.f) : 0.f;
            if (c < q.D) *(f32x4*)(W1 + r * PW + c) = v;
        }
        const int c = 512 + lane;                               // (columns 512 .. 527 of inputs of 512)
        if (c < q.D) W1[r * PW + c] = r < un && c == a.d0 ? bv[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < W2N; ++i) {
        const int e = tid + NT * i, c = e / UN, u = e % UN;
        if (e < CLS * UN) sm[q.W2 + c * PU + u] = (c < a.C && u < un) ? w2v[i] : 0.f;
    }
    if (tid == 0) *gave_up_word = 0;
    if (tid < CLS) b2[tid] = tid < a.C ? b2v : 0.f;
    for (int e = tid; e < q.R * PD; e += NT) D2[e] = 0.f;
    for (int r = wave; r < q.NX * q.R; r += NW)
        for (int c = lane; c < q.D; c += 64) sm[q.X + r * PW + c] = c == a.d0 ? 1.f : 0.f;
    __syncthreads();                                            // idx is complete

    // The rows of a step: wavefront w fetches rows w, w + 8, ..., its lanes 16 consecutive bytes each; requested one step
    // ahead, so that a cold row costs nothing.
    constexpr int RPW = ROWS / NW;
    f32x4 xnext[RPW][2];
    int ynext = 0;
    const int halves = a.d0 > 256 ? 2 : 1;
    auto fetch_rows = [&](int k) {
        const int* ik = idx + k * a.B;
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int m = wave + NW * i, c = h * 256 + lane * 4;
                if (m < a.B && h < halves) {                    // (wave-uniform)
                    const float* src = a.X + (size_t)ik[m] * a.d0;
                    if (VEC) xnext[i][h] = *(const f32x4*)(src + min(c, a.d0 - 4));
                    else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) xnext[i][h][e] = src[min(c + e, a.d0 - 1)];
                    }
                }
            }
        ynext = a.y[ik[min(tid, a.B - 1)]];
    };
    auto store_rows = [&](int k) {                              // the fetched rows of step k into their LDS buffer
        float* X = sm + q.X + (q.NX == 2 ? (k & 1) * q.R * PW : 0);
#pragma unroll
        for (int i = 0; i < RPW; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int m = wave + NW * i, c = h * 256 + lane * 4;
                if (m < a.B && h < halves && c < a.d0) {
                    f32x4 v = xnext[i][h];
                    if (!VEC) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = c + e < a.d0 ? v[e] : c + e == a.d0 ? 1.f : 0.f;
                    }
                    *(f32x4*)(X + m * PW + c) = v;
                }
            }
        if (tid < a.B) ((int*)(sm + q.y))[(k & 1) * ROWS + tid] = ynext;
    };
    fetch_rows(0);
    store_rows(0);

    bool gave_up = false;                                       // a wait ran out of polls: the results are void, finish quickly
    const int rblocks = q.R / 16, blocks = rblocks * ublocks;   // blocks in {1, 2, 3, 4, 6, 8, 12, 16}
    const int kslog = blocks >= 5 ? 0 : blocks >= 3 ? 1 : blocks == 2 ? 2 : 3, KS = 1 << kslog;   // wavefronts that share a block's contraction
    const int kspan = ((q.D / 16 + KS - 1) >> kslog) * 16;
    const float invB = 1.f / (float)a.B;
    const int tile = a.B * CLS;                                 // words of a workgroup's partial logits

    for (int k = 0; k < a.K; ++k) {
        const float* X = sm + q.X + (q.NX == 2 ? (k & 1) * q.R * PW : 0);
        const float* W2 = sm + q.W2 + (k & 1) * CLS * PU;
        float* W2next = sm + q.W2 + ((k & 1) ^ 1) * CLS * PU;
        __syncthreads();
        if (k + 1 < a.K) fetch_rows(k + 1);

        // 1. pre-activations in 16x16 blocks (matrix instruction 16x16x4; lane l supplies row l%16 of either operand, and
        //    sixteen consecutive k serve four instructions: instruction i contracts k = 4*(l/16) + i)
        for (int w = wave; w < blocks * KS; w += NW) {
            const int blk = w >> kslog, ks = w & (KS - 1);
            const int m0 = (blk / ublocks) * 16, u0 = (blk % ublocks) * 16;
            const int cb = ks * kspan, ce = min(cb + kspan, q.D);
            f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
            const float* xp = X + (m0 + l16) * PW + lq * 4;
            const float* wp = W1 + (u0 + l16) * PW + lq * 4;
#pragma unroll 4
            for (int c = cb; c < ce; c += 16) {
                const f32x4 x = *(const f32x4*)(xp + c), v = *(const f32x4*)(wp + c);
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[0], v[0], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[1], v[1], acc1, 0, 0, 0);
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[2], v[2], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[3], v[3], acc1, 0, 0, 0);
            }
            acc0 += acc1;
#pragma unroll
            for (int v = 0; v < 4; ++v) Z[(blk * KS + ks) * 256 + (4 * lq + v) * 16 + l16] = acc0[v];     // [row][unit] of the block
        }
        __syncthreads();
        for (int e = tid; e < blocks * 256; e += NT) {
            const int blk = e >> 8, at = e & 255;
            const int m = (blk / ublocks) * 16 + (at >> 4), u = (blk % ublocks) * 16 + (at & 15);
            float z = Z[blk * KS * 256 + at];
            for (int s = 1; s < KS; ++s) z += Z[(blk * KS + s) * 256 + at];
            A1[m * PU + u] = m < a.B ? fmaxf(z, 0.f) : 0.f;
        }
        __syncthreads();

        // 2. this group's share of the logits, one 16-row block per wavefront
        const uint32_t tag = a.tag0 + (uint32_t)k + 1u;
        uint64_t* parts = a.partial + ((size_t)(k & 1) * a.P + j) * G * tile;
        if (wave < rblocks) {
            const int m0 = wave * 16;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float* ap = A1 + (m0 + l16) * PU + lq * 4;
            const float* wp = W2 + l16 * PU + lq * 4;
            for (int u = 0; u < UN; u += 16) {
                const f32x4 x = *(const f32x4*)(ap + u), v = *(const f32x4*)(wp + u);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], v[i], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + 4 * lq + v;
                if (G > 1) { if (m < a.B && l16 < a.C) st_tagged(parts + (size_t)g * tile + m * CLS + l16, acc[v], tag); }
                else Z[m * CLS + l16] = acc[v];
            }
        }
        if (q.NX == 2 && k + 1 < a.K) store_rows(k + 1);        // (while the partials travel)
        if (G == 1) __syncthreads();                            // (Z's pre-activations were read before the last barrier)

        // 3. logits: thread = (row, class), the classes of a row in the 16 lanes of a wavefront row; the partials of up to
        //    eight groups are requested together and asked for again until all carry this step's tag
        for (int e = tid; e < q.R * CLS; e += NT) {
            const int m = e >> 4, c = e & 15;
            const bool live = c < a.C && m < a.B;
            float z = 0.f;
            if (G == 1) {
                z = Z[e];
            } else {
                const uint64_t* src = parts + min(m, a.B - 1) * CLS + min(c, a.C - 1);
                for (int g0 = 0; g0 < G; g0 += 8) {
                    uint64_t t[8];
                    unsigned spins = 0;
                    for (;;) {
                        bool ok = true;
#pragma unroll
                        for (int u = 0; u < 8; ++u) t[u] = ld_tagged(src + (size_t)min(g0 + u, G - 1) * tile);
#pragma unroll
                        for (int u = 0; u < 8; ++u) ok = ok && (uint32_t)(t[u] >> 32) == tag;
                        if (ok || gave_up) break;
                        if (++spins >= a.spin_limit) { atomicOr(a.err, 1); gave_up = true; *gave_up_word = 1; break; }   // and never wait again
                        __builtin_amdgcn_s_sleep(1);
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");       // discard cached copies of the lines (see fused_small.hip)
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) z += g0 + u < G ? __builtin_bit_cast(float, (uint32_t)t[u]) : 0.f;
                }
            }
            z += b2[c];
            const float mx = row16_max(live ? z : -INFINITY);
            const float ex = live ? expf(z - mx) : 0.f;
            const float den = row16_sum(ex);
            if (m < a.B) {
                const int yy = ((const int*)(sm + q.y))[(k & 1) * ROWS + m];
                D2[m * PD + c] = live ? (ex / den - (c == yy ? 1.f : 0.f)) * invB : 0.f;          // dZ_2 = (p - onehot) / B
                if (c == yy) rowloss[m] = logf(den) + mx - z;
            }
        }
        __syncthreads();
        gave_up = gave_up || *gave_up_word != 0;

        // 4. dZ_1 = (dZ_2 W_2) masked by the ReLU; meanwhile, from the last wavefront backwards, the SGD steps of W_2 (into
        //    its other buffer), b_2, and the mean loss
        for (int w = wave; w < blocks; w += NW) {
            const int m0 = (w / ublocks) * 16, u0 = (w % ublocks) * 16;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float* dp = D2 + (m0 + l16) * PD + lq;
            const float* wp = W2 + lq * PU + u0 + l16;
#pragma unroll
            for (int c = 0; c < CLS; c += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[c], wp[c * PU], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = (m0 + 4 * lq + v) * PU + u0 + l16;
                D1[at] = A1[at] > 0.f ? acc[v] : 0.f;            // rows beyond B: A_1 is zero there
            }
        }
        if (NW - 1 - wave <= ublocks) {     // W_2[c][u] -= lr sum_m dZ_2[m][c] A_1[m][u]; wavefront NW-1-ublocks: b_2, a column of ones for A_1
            const int ublk = NW - 1 - wave, u0 = min(ublk, ublocks - 1) * 16;
            const bool bias = ublk == ublocks;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
            for (int m = 0; m < a.B; m += 4)                    // (beyond B: zeros)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(D2[(m + lq) * PD + l16], bias ? 1.f : A1[(m + lq) * PU + u0 + l16], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = 4 * lq + v;
                if (bias) { if (l16 == 0) b2[c] -= a.lr * acc[v]; }
                else W2next[c * PU + u0 + l16] = W2[c * PU + u0 + l16] - a.lr * acc[v];
            }
        } else if (wave == 0 && g == 0) {
            float l = lane < a.B ? rowloss[lane] : 0.f;
            l = row16_sum(l);
            l += __shfl_xor(l, 16, 64);
            l += __shfl_xor(l, 32, 64);
            if (lane == 0) a.losses[(size_t)k * a.P + j] = l * invB;
        }
        __syncthreads();

        // 5. W_1[u][c] -= lr sum_m dZ_1[m][u] X[m][c]: a wavefront owns one 16-unit block and every (NW/ublocks)-th
        //    16-column block, up to four of them at a time on one dZ_1 operand
        {
            const int u0 = (wave % ublocks) * 16, cstep = 16 * (NW / ublocks);
            const float* dp = D1 + lq * PU + u0 + l16;
            int cb = (wave / ublocks) * 16;
            auto columns = [&](auto nb_tag) {
                constexpr int NB = decltype(nb_tag)::value;
                f32x4 acc[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
                const float* xp = X + lq * PW + cb + l16;
#pragma unroll 4
                for (int m = 0; m < a.B; m += 4) {              // (beyond B dZ_1 is zero)
                    const float d = dp[m * PU];
#pragma unroll
                    for (int i = 0; i < NB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, xp[m * PW + i * cstep], acc[i], 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v) W1[(u0 + 4 * lq + v) * PW + cb + i * cstep + l16] -= a.lr * acc[i][v];
                cb += NB * cstep;
            };
            while (cb + 3 * cstep < q.D) columns(std::integral_constant<int, 4>{});
            if (cb + 2 * cstep < q.D) columns(std::integral_constant<int, 3>{});
            else if (cb + cstep < q.D) columns(std::integral_constant<int, 2>{});
            else if (cb < q.D) columns(std::integral_constant<int, 1>{});
        }
        if (q.NX == 1 && k + 1 < a.K) {
            __syncthreads();                                    // X is no longer read
            store_rows(k + 1);
        }
    }
    __syncthreads();

    // ---- parameters back to the replica ----
    for (int r = wave; r < un; r += NW)
        for (int c = lane * 4; c < q.D; c += 256) {
            float* dst = rep + a.w1_off + (size_t)(ub + r) * a.d0 + c;
            const f32x4 v = *(const f32x4*)(W1 + r * PW + c);
            if (VEC && c < a.d0) *(f32x4*)dst = v;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (!VEC && c + i < a.d0) dst[i] = v[i];
                if (c + i == a.d0) rep[a.b1_off + ub + r] = v[i];
            }
        }
    for (int e = tid; e < CLS * UN; e += NT) {
        const int c = e / UN, u = e % UN;
        if (c < a.C && u < un) rep[a.w2_off + (size_t)c * a.d1 + ub + u] = sm[q.W2 + (a.K & 1) * CLS * PU + c * PU + u];
    }
    if (g == 0 && tid < a.C) rep[a.b2_off + tid] = b2[tid];
}

}  // namespace

// Units per workgroup: the fewest (16, 32 or 64) that give every workgroup of the launch a compute unit of its own, at most
// GMAX workgroups per learner, and fit the LDS; 0: shape not covered.
int fused_units_plan(int P, int K, int B, int d0, int d1, int C, int compute_units) {
    if (d1 < 1 || C < 1 || C > CLS || B < 1 || B > ROWS || d0 < 4 || d0 > D0MAX || (long)K * B > KBMAX) return 0;
    for (int UN = 16; UN <= 64; UN *= 2) {
        const int G = (d1 + UN - 1) / UN;
        if (G > GMAX || (long)P * G > compute_units) continue;
        if (units_layout(B, K, d0, d1, UN).words <= LDS_WORDS) return UN;
    }
    return 0;
}

// Where fused_small.hip covers the shape as well.  That kernel exchanges 64 pre-activations per row and workgroup instead of
// C logits, but its workgroups hold 64 to 192 inputs of all units where these hold all inputs of few units, and many of
// these on the chip slow each other's exchange.  Measured at K = 4 on 2 - 250 learners, 8 - 512 inputs, 8 - 64 units and
// batches of 2 - 64 (1578 shapes; us for the K steps, this kernel / that one): 64-8-10, 2 learners of 32 rows 22 / 42;
// 256-64-10, 8 of 32 34 / 40; but 512-64-10, 2 of 32 47 / 42; 320-64-10, 24 of 48 67 / 58; 64-64-10, 48 of 24 53 / 39;
// 128-48-10, 128 of 16 50 / 41.  Inside the lines below it was the faster one at every shape (1.5 times in the mean), outside
// them not always.
bool fused_units_faster(int P, int K, int B, int d0, int d1, int C, int compute_units) {
    const int UN = fused_units_plan(P, K, B, d0, d1, C, compute_units), G = UN ? (d1 + UN - 1) / UN : 0;
    if (G == 0) return false;
    if (B <= 16) return G == 1 || 4 * P * G <= 3 * compute_units;
    return 4 * P * G <= compute_units && (B + 15) / 16 * 16 * d0 <= 12288;
}

// two buffers of P x G tiles of B x CLS (value, tag) words; UN from fused_units_plan
size_t fused_units_scratch_bytes(int P, int B, int d1, int UN) { return (size_t)2 * P * ((d1 + UN - 1) / UN) * B * CLS * 8; }

namespace {
// Workgroups of a launch.  One XCD per learner where its compute units hold all workgroups that then fall to it and there
// are enough partners for it to matter (rounds of 256-256-10, us: 6 learners x 16 groups 79 on one XCD, 88 spread;
// 6 x 8 groups 81 / 83; 48 x 4 groups 159 / 153).
int units_grid(int P, int G, int compute_units, int* spread) {
    const int per_xcd = (P + 7) / 8 * G;
    *spread = per_xcd > compute_units / 8 || G < 8 ? 1 : 0;
    return *spread ? P * G : 8 * per_xcd;
}

template <bool VEC, int UN>
hipError_t launch_units(const FusedSmallCall& c, hipStream_t st) {
    const UnitsLayout q = units_layout(c.B, c.K, c.d0, c.d1, UN);
    static hipError_t raised = hipFuncSetAttribute((const void*)fused_units_kernel<VEC, UN>,
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, LDS_WORDS * 4);
    if (raised != hipSuccess) return raised;
    int spread;
    const int grid = units_grid(c.P, q.G, c.compute_units, &spread);
    hipLaunchKernelGGL((fused_units_kernel<VEC, UN>), dim3(grid), dim3(NT), q.words * 4, st, c, spread);
    return hipGetLastError();
}
}  // namespace

int fused_units_workgroups(int P, int d1, int UN, int compute_units) {
    int spread;
    return units_grid(P, (d1 + UN - 1) / UN, compute_units, &spread);
}

hipError_t launch_fused_units(const FusedSmallCall& c, hipStream_t st) {
    const bool vec = c.d0 % 4 == 0;
    switch (fused_units_plan(c.P, c.K, c.B, c.d0, c.d1, c.C, c.compute_units)) {
        case 16: return vec ? launch_units<true, 16>(c, st) : launch_units<false, 16>(c, st);
        case 32: return vec ? launch_units<true, 32>(c, st) : launch_units<false, 32>(c, st);
        case 64: return vec ? launch_units<true, 64>(c, st) : launch_units<false, 64>(c, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace kavg
