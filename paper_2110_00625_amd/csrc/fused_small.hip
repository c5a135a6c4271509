// All K local steps of Algorithm 1 in ONE launch, for fp32 models small enough to live on chip:
// one hidden layer of at most 64 units, at most 16 classes, minibatches of at most 64 rows.
//
// Such a model (d_0 x 64 + 64 x C weights per learner) takes a few microseconds of arithmetic per
// step; run as a chain of generic kernels it is bound by ~6 dependent launches per step.  Here the
// learner's first-layer weights are cut into S column chunks of CW input features (CW a multiple of
// 64, at most 192, or 384 where four workgroups share a chunk); workgroup (j, s) keeps chunk s of learner j's W_1 in LDS for the whole call,
// together with private copies of b_1, W_2 and b_2.  (Where the device has the compute units for it and the
// layer has more than 32 units, two or four workgroups share a chunk, each with half or a quarter of the hidden units: "its chunk"
// is then those units' rows of the chunk; everything else is unchanged.)  Per step
//   1. the workgroup multiplies its CW columns of the gathered rows X[idx] with its chunk of W_1
//      (fp32 matrix instructions) and writes the B x 64 partial pre-activations to device memory;
//   2. it collects the partials of all S workgroups of its learner and adds them in ascending chunk
//      order (bias, ReLU): every workgroup now holds the same A_1;
//   3. it runs the head -- logits, softmax cross-entropy, dZ_2, dZ_1, the SGD step on its copies of
//      W_2, b_2, b_1 -- redundantly: same inputs, same instruction sequence in every workgroup, so
//      the copies stay bit-identical without further communication;
//   4. and takes the SGD step on its own chunk of W_1 in LDS (dZ_1^T times its columns of X[idx]).
// Only after the K steps do the parameters go back to the replica in device memory.
//
// One exchange per step, without flags that anything depends on: a partial is written as a 64-bit word
// (value, tag) by one device-scope atomic store, the tag being the number of the step counted over all launches of the
// context.  A reader requests the S words of an element with device-scope atomic loads and asks again
// (a bounded number of times, after a device-scope acquire that discards cached copies of the lines)
// until every tag shows the current step; each word validates itself, so nothing depends on the order
// in which different addresses become visible.  (Each wavefront also raises a hint word after its stores, and
// wavefront 0 waits for the learner's hints before anyone gathers -- the other wavefronts finish the previous
// step's W_2, b_1, b_2 and loss meanwhile; the hints only time the first request, the tags decide.)  Partials
// alternate between two buffers: a workgroup overwrites the buffer of step k only when it computes step k+2,
// which it starts after it has read every partial of step k+1, each of which was written after its
// writer had read the partials of step k.  All workgroups must be resident at once: the host
// launches this kernel only when their number does not exceed the number of compute units, and launches of several
// contexts that do not fit on the chip together take turns (kavg_api.hip).  A reader that
// runs out of polls raises an error word and carries on, so every wavefront reaches the end of the
// kernel whatever happens.
//
// The minibatch indices of the learner's K steps are produced here as well (same counter-based
// stream as index_stream_kernel; workgroup 0 of a learner also stores them for kavg_indices), unless
// the caller supplied its own.
#include "kavg_internal.h"
#include "fused_common.h"

#include <type_traits>

namespace kavg {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NT = 512;         // threads per workgroup (8 wavefronts)
constexpr int CWMAX = 192;      // input features per workgroup, at most (WIDE: twice as many)
constexpr int HID = 64;         // hidden units (upper bound)
constexpr int CLS = 16;         // classes (upper bound)
constexpr int MAXROWS = 64;     // minibatch rows (upper bound)
// Row pitches of the LDS tiles, in words.  A matrix instruction reads a tile either as (16 rows) x (4 consecutive
// words) or as (4 rows) x (16 consecutive words); pitches of 12 or 4 modulo the 64 banks spread the first pattern
// over all banks (the hot one: the operands of the two big products) and the second over most.
__host__ __device__ constexpr int pw_of(bool wide) { return (wide ? 2 * CWMAX : CWMAX) + 12; }      // tiles CW wide
constexpr int PH = HID + 4;     // tiles 64 wide
constexpr int PD = CLS + 4;     // dZ_2
constexpr int TILE = MAXROWS * HID;
constexpr int KBMAX = 1024;     // K*B, at most

// WIDE: a quarter of the units, minibatches of at most half as many rows
template <bool WIDE>
struct Smem {
    static constexpr int PW = pw_of(WIDE), ROWS = MAXROWS / (WIDE ? 2 : 1), UNITS = WIDE ? HID / 4 : HID;
    float W1[UNITS * PW];       // chunk of W_1: [unit][feature]
    float X[ROWS * PW];         // gathered rows, this chunk's columns: [row][feature]
    float A1[ROWS * PH];        // hidden activations [row][unit]
    float D1[ROWS * PH];        // dZ_1 [row][unit]
    float W2[CLS * PH];         // [class][unit]
    float D2[ROWS * PD];        // dZ_2 [row][class]
    float b1[HID], b2[CLS], rowloss[ROWS];
    int y[ROWS];
    int idx[KBMAX];             // the learner's minibatch indices [K][B]
    int gave_up;                // a wait ran out of polls
    float sums[WIDE ? 4 * ROWS * UNITS : 1];     // pre-activations of the four quarters of the chunk's columns
};

// acc + acc1 += sum over `columns` (a multiple of 32) of x[row][c] w[unit][c], in two chains so that the matrix pipeline does not wait for its
// own result.  (The compiler does not unroll a loop of unknown length around matrix instructions: the operands of the next 32 columns
// are requested by hand before those at hand are used.)
__device__ __forceinline__ void contract(const float* xp, const float* wp, int columns, f32x4& acc, f32x4& acc1) {
    float x[2][8], w[2][8];
    auto request = [&](int set, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { x[set][i] = xp[c + 4 * i]; w[set][i] = wp[c + 4 * i]; }
    };
    auto use = [&](int set) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[set][i], w[set][i], acc, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(x[set][i + 1], w[set][i + 1], acc1, 0, 0, 0);
        }
    };
    request(0, 0);
    for (int c = 0; c < columns; c += 64) {
        request(1, min(c + 32, columns - 32));
        __builtin_amdgcn_sched_barrier(0);
        use(0);
        if (c + 32 < columns) {
            request(0, min(c + 64, columns - 32));
            __builtin_amdgcn_sched_barrier(0);
            use(1);
        }
    }
}

// WIDE: chunks of up to 384 columns, each shared by four workgroups of 16 units, for minibatches of at most 32 rows.  A
// workgroup then gathers the partials of half as many chunks (131 instead of 262 KB per step for 32 rows of 3072, all requested at once): the
// exchange, not the arithmetic, is the longest part of a step.  us per round of four steps: 3072-64-10, 4 learners of 32 rows 72.2 -> 65.0,
// 1024-64-10, 8 learners 62.0 -> 55.1, 784-64-10, 4 of 24 rows 56.2 -> 50.7.
// BATCH (WIDE, and chunks of more than 64 columns): the operands of 16 rows of the update of W_1 are requested before those at hand are
// used.  With 64 columns a wavefront has one or two blocks of them to a row, and four rows at a time are faster.  (us per round of four steps,
// eight and more where stated, four rows / 16: 128 columns, 1836-54-4, 10 learners of 32 rows, eight 129.8 / 123.5, 1500-32-10, 16 of 20,
// eight 125.7 / 120.5, 192, 3072-64-10, 4 of 64 101.2 / 96.5; 64, 256-64-10, 60 of 32 53.7 / 55.1, 64-52-16, 51 of 39, fourteen 154.8 / 158.5,
// 784-64-10, 16 of 64 89.6 / 88.9.)  The products' loop by hand in chunks of up to 192 columns: 784-64-10, 16 of 32 64.0 / 64.7,
// 512-32-10, 30 of 24 55.7 / 57.5.
template <bool WIDE, bool BATCH>
__global__ void __launch_bounds__(NT)
fused_small_kernel(FusedSmallCall a, int S, int CW, int UH) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    typedef Smem<WIDE> Lds;
    Lds& sm = *(Lds*)smem_raw;
    constexpr int PW = Lds::PW, ROWS = Lds::ROWS;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // workgroup (j, s, h): learner j, column chunk s, and -- with UH = 2 or 4 -- half or quarter h of the hidden units (the chunk's
    // two products are then shared by several compute units; everything else is as if UH were 1)
    const int j = blockIdx.x / (S * UH), s = (blockIdx.x / UH) % S, h = blockIdx.x % UH;
    const int UN = HID / UH, ub = h * UN;                       // hidden units ub .. ub+UN-1 are this workgroup's
    const bool first = s == 0 && h == 0;                        // the learner's workgroup that writes what all of them hold
    const int c0 = s * CW;
    const int cw = min(CW, a.d0 - c0);                          // valid columns of this chunk (a multiple of 4)
    const int CW4 = CW / 4;
    float* rep = a.reps + (size_t)j * a.rep_stride;

    // ---- the learner's minibatch indices: draw (j, t0 + k, m) of the counter-based stream, or the caller's ----
    for (int e = tid; e < a.K * a.B; e += NT) {
        int32_t v;
        if (a.generate_idx) {
            v = index_draw(a.seed, (uint32_t)j, a.t0 + (uint32_t)(e / a.B), (uint32_t)(e % a.B), a.N);
            if (first) a.idx[(size_t)j * a.K * a.B + e] = v;
        } else {
            v = a.idx[(size_t)j * a.K * a.B + e];
        }
        sm.idx[e] = v;
    }

    // ---- parameters into LDS ----
    for (int e = tid; e < UN * CW4; e += NT) {                  // sm.W1 row r holds unit ub + r
        const int r = e / CW4, c = (e % CW4) * 4;
        f32x4 v = {0.f, 0.f, 0.f, 0.f};
        if (ub + r < a.d1 && c < cw) v = *(const f32x4*)(rep + a.w1_off + (size_t)(ub + r) * a.d0 + c0 + c);
        *(f32x4*)(sm.W1 + r * PW + c) = v;
    }
    for (int e = tid; e < CLS * HID; e += NT) {
        const int c = e / HID, u = e % HID;
        sm.W2[c * PH + u] = (c < a.C && u < a.d1) ? rep[a.w2_off + (size_t)c * a.d1 + u] : 0.f;
    }
    if (tid == 0) sm.gave_up = 0;
    if (tid < HID) sm.b1[tid] = tid < a.d1 ? rep[a.b1_off + tid] : 0.f;
    if (tid < CLS) sm.b2[tid] = tid < a.C ? rep[a.b2_off + tid] : 0.f;
    for (int e = tid; e < ROWS * PH; e += NT) { sm.D1[e] = 0.f; sm.A1[e] = 0.f; }   // rows beyond B stay zero throughout
    for (int e = tid; e < ROWS * PD; e += NT) sm.D2[e] = 0.f;
    for (int e = tid; e < ROWS * PW; e += NT) sm.X[e] = 0.f;

    // The thread's 16-byte pieces of a step's X tile: piece i covers row (tid / CW4 + i * (NT / CW4)) ... laid
    // out so that consecutive threads read consecutive 16 bytes of a row.
    const int rows_per_pass = NT / CW4;                         // CW4 in {16, 32, 48}: 32, 16, 10 rows per pass; WIDE, up to 96: at least 5
    const int xr = tid / CW4, xc = (tid % CW4) * 4;
    constexpr int XMAX = 7;                                     // passes: ceil(64 / 10), ceil(32 / 5)
    const int xpasses = (a.B + rows_per_pass - 1) / rows_per_pass;
    // the next step's pieces (and label) are requested one step ahead
    int ynext = 0;
    f32x4 xnext[XMAX];
    auto fetch_x = [&](int k) {
        const int* idx = sm.idx + k * a.B;
#pragma unroll
        for (int i = 0; i < XMAX; ++i) {
            const int m = xr + i * rows_per_pass;
            if (i < xpasses && xr < rows_per_pass) {
                const f32x4 x = *(const f32x4*)(a.X + (size_t)idx[min(m, a.B - 1)] * a.d0 + c0 + min(xc, cw - 4));
                xnext[i] = (m < a.B && xc < cw) ? x : (f32x4){0.f, 0.f, 0.f, 0.f};
            }
        }
        ynext = a.y[idx[min(tid, a.B - 1)]];
    };
    __syncthreads();                                            // sm.idx is complete
    fetch_x(0);

    bool gave_up = false;                                       // a wait ran out of polls: the results are void, finish quickly
    const int Bk = (a.B + 7) & ~7;                              // rows as a contraction length (rows beyond B are zero)
    const int rblocks = (a.B + 15) / 16;                        // 16-row blocks of the minibatch
    const float invB = 1.f / (float)a.B;

    // The small parameters of step kk, from what its head left in LDS: W_2 <- W_2 - lr dZ_2^T A_1 as four 16x16 blocks
    // (wavefronts 1..4), b_1 (5), b_2 (6), the loss (7).  Runs while wavefront 0 waits for the next step's partials.
    auto small_updates = [&](int kk) {
        if (wave >= 1 && wave <= HID / 16) {
            const int u0 = (wave - 1) * 16;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float* dp = sm.D2 + (lane >> 4) * PD + (lane & 15);           // dZ_2[m][c]: row c of the product
            const float* ap = sm.A1 + (lane >> 4) * PH + u0 + (lane & 15);
            for (int m = 0; m < Bk; m += 8) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[m * PD], ap[m * PH], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[(m + 4) * PD], ap[(m + 4) * PH], acc, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) sm.W2[(4 * (lane >> 4) + v) * PH + u0 + (lane & 15)] -= a.lr * acc[v];
        } else if (wave == 5) {                                 // b_1 <- b_1 - lr colsum(dZ_1)
            float g = 0.f;
#pragma unroll 8
            for (int m = 0; m < Bk; ++m) g += sm.D1[m * PH + lane];
            sm.b1[lane] -= a.lr * g;
        } else if (wave == 6) {                                 // b_2 <- b_2 - lr colsum(dZ_2)
            if (lane < CLS) {
                float g = 0.f;
#pragma unroll 8
                for (int m = 0; m < Bk; ++m) g += sm.D2[m * PD + lane];
                sm.b2[lane] -= a.lr * g;
            }
        } else if (wave == 7 && first && lane == 0) {           // mean loss of this learner's step
            float l = 0.f;
            for (int m = 0; m < a.B; ++m) l += sm.rowloss[m];
            a.losses[(size_t)kk * a.P + j] = l * invB;
        }
    };

    for (int k = 0; k < a.K; ++k) {
        __syncthreads();                                        // previous step is done with sm.X
#pragma unroll
        for (int i = 0; i < XMAX; ++i) {
            const int m = xr + i * rows_per_pass;
            if (i < xpasses && xr < rows_per_pass && m < ROWS) {
                *(f32x4*)(sm.X + m * PW + xc) = xnext[i];
            }
        }
        if (tid < ROWS) sm.y[tid] = tid < a.B ? ynext : 0;
        __syncthreads();
        if (k + 1 < a.K) fetch_x(k + 1);                        // the next step's rows: requested now, used a step later

        // 1. partial pre-activations of this chunk, Zp[m][u] = sum_c X[m][c] W1[u][c], in 16x16 blocks
        //    (matrix instruction 16x16x4: lane l supplies X[m0 + l%16][c + l/16] and W1[u0 + l%16][c + l/16],
        //     and receives Zp[m0 + 4*(l/16) + v][u0 + l%16] in accumulator v)
        const uint32_t tag = a.tag0 + (uint32_t)k + 1u;
        uint64_t* part = a.partial + (((size_t)(k & 1) * a.P + j) * S + s) * TILE;
        if constexpr (WIDE) {                                   // one block of units, at most two of rows: eight wavefronts take a quarter of the columns of a block each
            const int m0 = (wave & 1) * 16, c0w = (wave >> 1) * (CW / 4);
            if (m0 < a.B) {
                f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
                const float* xp = sm.X + (m0 + (lane & 15)) * PW + c0w + (lane >> 4);
                const float* wp = sm.W1 + (lane & 15) * PW + c0w + (lane >> 4);
                contract(xp, wp, CW / 4, acc, acc1);
                acc += acc1;
#pragma unroll
                for (int v = 0; v < 4; ++v) sm.sums[((wave >> 1) * ROWS + m0 + 4 * (lane >> 4) + v) * Lds::UNITS + (lane & 15)] = acc[v];
            }
            __syncthreads();
            const int m = tid / Lds::UNITS, u = tid % Lds::UNITS;
            static_assert(NT == ROWS * Lds::UNITS, "a thread per partial");
            const float* q = sm.sums + m * Lds::UNITS + u;
            constexpr int Q = ROWS * Lds::UNITS;
            if (m < a.B) st_tagged(part + m * HID + ub + u, (q[0] + q[Q]) + (q[2 * Q] + q[3 * Q]), tag);
        } else
        for (int blk = wave; blk < rblocks * (UN / 16); blk += NT / 64) {
            const int m0 = (blk / (UN / 16)) * 16, u0 = (blk % (UN / 16)) * 16;        // u0: row of sm.W1, unit ub + u0
            f32x4 acc = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};   // two chains: the matrix pipeline never waits for its own result
            const float* xp = sm.X + (m0 + (lane & 15)) * PW + (lane >> 4);
            const float* wp = sm.W1 + (u0 + (lane & 15)) * PW + (lane >> 4);
#pragma unroll 4
            for (int c = 0; c < CW; c += 8) {
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xp[c], wp[c], acc, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(xp[c + 4], wp[c + 4], acc1, 0, 0, 0);
            }
            acc += acc1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + 4 * (lane >> 4) + v;
                if (m < a.B) st_tagged(part + m * HID + ub + u0 + (lane & 15), acc[v], tag);
            }
        }

        // This wavefront's partials are on their way: say so in its hint word (a separate address: only a hint --
        // the words of the partials validate themselves).  Then, while wavefront 0 waits for the hints of all
        // wavefronts of the learner's S workgroups, the others finish the previous step's small parameters.
        uint32_t* hints = a.hints + ((size_t)(k & 1) * a.P + j) * S * UH * (NT / 64);
        if (lane == 0) __hip_atomic_store(hints + (s * UH + h) * (NT / 64) + wave, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wave == 0) {
            unsigned spins = 0;
            for (;;) {
                bool ok = true;
                for (int i = lane; i < S * UH * (NT / 64); i += 64)
                    ok = ok && __hip_atomic_load(hints + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
                if (__builtin_amdgcn_ballot_w64(!ok) == 0 || gave_up) break;
                if (++spins >= a.spin_limit) { atomicOr(a.err, 1); sm.gave_up = 1; break; }
                __builtin_amdgcn_s_sleep(1);
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");       // discard cached copies (see below)
            }
        } else if (k > 0) {
            small_updates(k - 1);
        }
        __syncthreads();
        gave_up = gave_up || sm.gave_up != 0;

        // 2. A_1 = relu(sum of the learner's S partials + b_1).  Element e = tid + i*NT of the B x 64 tile; eight
        //    partials of each of four elements are requested together and asked for again until all carry this
        //    step's tag; they are added in ascending chunk order.
        {
            const uint64_t* base = a.partial + ((size_t)(k & 1) * a.P + j) * S * TILE;
            const int n_el = a.B * HID;
            for (int g0 = 0; g0 * NT < n_el; g0 += 4) {
                float z[4] = {0.f, 0.f, 0.f, 0.f};
                for (int q0 = 0; q0 < S; q0 += 8) {
                    const int nq = min(8, S - q0);
                    uint64_t t[4][8];
                    unsigned spins = 0;
                    for (;;) {
                        bool ok = true;
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int u = 0; u < 8; ++u)
                                t[i][u] = ld_tagged(base + (size_t)(q0 + min(u, nq - 1)) * TILE + min(tid + (g0 + i) * NT, n_el - 1));
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int u = 0; u < 8; ++u) ok = ok && (uint32_t)(t[i][u] >> 32) == tag;
                        if (ok || gave_up) break;
                        if (++spins >= a.spin_limit) { atomicOr(a.err, 1); gave_up = true; break; }   // and never wait again
                        __builtin_amdgcn_s_sleep(1);
                        // Without this a reader can be served the same cached copy of a line again and again (seen on
                        // the device: waits that never ended although the words had long been written); the acquire
                        // discards the cached copies, so the next request goes to memory.
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int u = 0; u < 8; ++u) z[i] += u < nq ? __builtin_bit_cast(float, (uint32_t)t[i][u]) : 0.f;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = tid + (g0 + i) * NT;
                    if (e < n_el) sm.A1[(e / HID) * PH + e % HID] = fmaxf(z[i] + sm.b1[e % HID], 0.f);
                }
            }
        }
        __syncthreads();

        // 3. the head, identically in every workgroup of the learner.  Logits in 16-row blocks, one per wavefront:
        //    lane l receives rows m0 + 4*(l/16) + v (v = 0..3) of class l%16, so the 16 classes of a row sit in the
        //    16 lanes of one row of the wavefront and its softmax is a reduction over that row.
        if (wave < rblocks) {
            const int m0 = wave * 16, c = lane & 15;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float* ap = sm.A1 + (m0 + c) * PH + (lane >> 4);
            const float* wp = sm.W2 + c * PH + (lane >> 4);
#pragma unroll
            for (int u = 0; u < HID; u += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ap[u], wp[u], acc, 0, 0, 0);
            const bool live = c < a.C;
            const float bias = sm.b2[c];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + 4 * (lane >> 4) + v;
                const float z = acc[v] + bias;
                const float mx = row16_max(live ? z : -INFINITY);
                const float ex = live ? expf(z - mx) : 0.f;
                const float den = row16_sum(ex);
                const int yy = sm.y[m];
                if (m < a.B) {
                    sm.D2[m * PD + c] = live ? (ex / den - (c == yy ? 1.f : 0.f)) * invB : 0.f;   // dZ_2 = (p - onehot) / B
                    if (c == yy) sm.rowloss[m] = logf(den) + mx - z;
                }
            }
        }
        __syncthreads();
        for (int blk = wave; blk < rblocks * (HID / 16); blk += NT / 64) {      // dZ_1 = (dZ_2 W_2) masked by the ReLU
            const int m0 = (blk / (HID / 16)) * 16, u0 = (blk % (HID / 16)) * 16;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            const float* dp = sm.D2 + (m0 + (lane & 15)) * PD + (lane >> 4);
            const float* wp = sm.W2 + (lane >> 4) * PH + u0 + (lane & 15);
#pragma unroll
            for (int c = 0; c < CLS; c += 4) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dp[c], wp[c * PH], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int at = (m0 + 4 * (lane >> 4) + v) * PH + u0 + (lane & 15);
                sm.D1[at] = sm.A1[at] > 0.f ? acc[v] : 0.f;      // rows beyond B: A_1 is zero there
            }
        }
        __syncthreads();

        // 4. W_1[u][c] <- W_1[u][c] - lr sum_m dZ_1[m][u] X[m][c] on this workgroup's units and columns.  A wavefront
        //    owns one 16-unit block and every G-th 16-column block (G = wavefronts per unit block): one dZ_1 operand
        //    feeds all its blocks.
        {
            const int nub = UN / 16, G = (NT / 64) / nub;       // 4 unit blocks x 2 column groups, or 2 x 4, or 1 x 8
            const int u0 = (wave % nub) * 16, cb0 = (wave / nub) * 16;
            const float* dp = sm.D1 + (lane >> 4) * PH + ub + u0 + (lane & 15);
            const float* xp = sm.X + (lane >> 4) * PW + cb0 + (lane & 15);
            const int cstep = 16 * G;
            auto update_w1 = [&](auto nb_tag) {
                constexpr int NB = decltype(nb_tag)::value;
                f32x4 acc[NB];
#pragma unroll
                for (int i = 0; i < NB; ++i) acc[i] = (f32x4){0.f, 0.f, 0.f, 0.f};
                if constexpr (!BATCH) {
#pragma unroll 2
                    for (int m = 0; m < Bk; m += 4) {
                        const float d = dp[m * PH];
#pragma unroll
                        for (int i = 0; i < NB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, xp[m * PW + cstep * i], acc[i], 0, 0, 0);
                    }
                } else {
                    auto rows = [&](auto count, int m) __attribute__((always_inline)) {
                        constexpr int N = decltype(count)::value / 4;
                        float d[N], x[N][NB];
#pragma unroll
                        for (int t = 0; t < N; ++t) {
                            d[t] = dp[(m + 4 * t) * PH];
#pragma unroll
                            for (int i = 0; i < NB; ++i) x[t][i] = xp[(m + 4 * t) * PW + cstep * i];
                        }
#pragma unroll
                        for (int t = 0; t < N; ++t)
#pragma unroll
                            for (int i = 0; i < NB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[t], x[t][i], acc[i], 0, 0, 0);
                    };
                    int m = 0;
                    for (; m + 16 <= Bk; m += 16) rows(std::integral_constant<int, 16>(), m);
                    if (m < Bk) rows(std::integral_constant<int, 8>(), m);
                }
#pragma unroll
                for (int i = 0; i < NB; ++i)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        sm.W1[(u0 + 4 * (lane >> 4) + v) * PW + cb0 + cstep * i + (lane & 15)] -= a.lr * acc[i][v];
            };
            switch ((CW / 16) / G) {                            // column blocks per wavefront
                case 1: update_w1(std::integral_constant<int, 1>{}); break;
                case 2: update_w1(std::integral_constant<int, 2>{}); break;
                case 3: update_w1(std::integral_constant<int, 3>{}); break;
                case 4: update_w1(std::integral_constant<int, 4>{}); break;
                default: update_w1(std::integral_constant<int, 6>{}); break;
            }
        }
    }
    __syncthreads();
    small_updates(a.K - 1);
    __syncthreads();

    // ---- parameters back to the replica ----
    for (int e = tid; e < UN * CW4; e += NT) {
        const int r = e / CW4, c = (e % CW4) * 4;
        if (ub + r < a.d1 && c < cw) {
            *(f32x4*)(rep + a.w1_off + (size_t)(ub + r) * a.d0 + c0 + c) = *(const f32x4*)(sm.W1 + r * PW + c);
        }
    }
    if (first) {
        for (int e = tid; e < a.C * a.d1; e += NT) rep[a.w2_off + e] = sm.W2[(e / a.d1) * PH + e % a.d1];
        if (tid < a.d1) rep[a.b1_off + tid] = sm.b1[tid];
        if (tid < a.C) rep[a.b2_off + tid] = sm.b2[tid];
    }
}

}  // namespace

// Columns per workgroup: the fewest multiples of 64 (at most 192) that leave at most 16 chunks, else 192.
int fused_small_chunk_width(int d0) {
    for (int cw = 64; cw < CWMAX; cw += 64)
        if ((d0 + cw - 1) / cw <= 16) return cw;
    return CWMAX;
}
int fused_small_chunks(int d0) { const int cw = fused_small_chunk_width(d0); return (d0 + cw - 1) / cw; }

bool fused_small_shape_ok(int P, int K, int B, int d0, int d1, int C, int compute_units) {
    if (d1 < 1 || d1 > HID || C < 1 || C > CLS || B < 1 || B > MAXROWS || d0 < 4 || d0 % 4 != 0) return false;
    if ((long)K * B > KBMAX) return false;
    return (long)P * fused_small_chunks(d0) <= compute_units;
}

namespace {

// How a learner's workgroups share W_1: S chunks of CW columns, each in the hands of UH workgroups with 64 / UH units.
struct Split { int S, CW, UH; bool wide; };

// Two workgroups per chunk when the layer is wider than 32 units and the device has the compute units for it; with more than eight
// chunks and at most 32 rows, half as many chunks with four workgroups each.
Split split_of(int P, int B, int d0, int d1, int compute_units) {
    const int CW = fused_small_chunk_width(d0), S = fused_small_chunks(d0), half = (S + 1) / 2;
    if (d1 > HID / 2 && S > 8 && B <= MAXROWS / 2 && (long)4 * P * half <= compute_units) {
        for (int cw = 128; cw <= 2 * CWMAX; cw += 128)         // (16 columns for each of eight wavefronts)
            if ((d0 + cw - 1) / cw <= half) return {(d0 + cw - 1) / cw, cw, 4, true};
    }
    return {S, CW, d1 > HID / 2 && (long)2 * P * S <= compute_units ? 2 : 1, false};
}

template <bool WIDE, bool BATCH>
hipError_t launch_split(const FusedSmallCall& c, const Split& p, hipStream_t st) {
    static hipError_t raised = hipFuncSetAttribute((const void*)fused_small_kernel<WIDE, BATCH>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                   (int)sizeof(Smem<WIDE>));
    if (raised != hipSuccess) return raised;
    hipLaunchKernelGGL((fused_small_kernel<WIDE, BATCH>), dim3(c.P * p.S * p.UH), dim3(NT), sizeof(Smem<WIDE>), st, c, p.S, p.CW, p.UH);
    return hipGetLastError();
}

}  // namespace

// two buffers of P x chunks tiles of (value, tag) words, then two of P x chunks x wavefronts hint words
size_t fused_small_partial_words(int P, int d0) { return (size_t)2 * P * fused_small_chunks(d0) * TILE; }
size_t fused_small_scratch_bytes(int P, int d0) {          // (hint words for a unit split of two, or of four and half as many chunks)
    return fused_small_partial_words(P, d0) * 8 + (size_t)2 * P * ((fused_small_chunks(d0) + 1) / 2 * 2) * 2 * (NT / 64) * 4;
}

int fused_small_workgroups(int P, int B, int d0, int d1, int compute_units) {
    const Split p = split_of(P, B, d0, d1, compute_units);
    return P * p.S * p.UH;
}

hipError_t launch_fused_small(const FusedSmallCall& c, hipStream_t st) {
    const Split p = split_of(c.P, c.B, c.d0, c.d1, c.compute_units);
    if (p.wide) return launch_split<true, true>(c, p, st);
    return p.CW > 64 ? launch_split<false, true>(c, p, st) : launch_split<false, false>(c, p, st);
}

}  // namespace kavg
