// The meta level of Algorithm 1 as one bandwidth-bound pass:
//     a = (1/P) sum_j w^j;  d = a - w~;  v <- mu v + d;  w~ <- w~ + v;  w^j <- w~ for all j.
// a and d never reach memory.  The displacement is formed as
//     d = (1/P) sum_j (w^j - w~),
// which equals a - w~ in exact arithmetic, keeps the small quantity d at full
// fp32 precision, and is exactly zero when all replicas equal w~ (so lr = 0
// leaves every parameter bit-identical for any P).
//
// Traffic per parameter and pass: read P replicas + w~ + v, write w~ + v + P
// replicas = (2P+4)*4 bytes (+2P bytes when bf16 shadows are refreshed).
// Each lane owns four consecutive parameters (16-byte accesses), on long vectors
// eight such pieces 4 KB apart, on short ones a single parameter (two in planes),
// so that there are some hundred workgroups; the replica loads are issued sixteen
// at a time so that many are in flight per lane.  TOGETHER: so are the last of
// them, those beyond the last replica for that one over and over (one by one they
// cost a round trip to memory each; on long vectors other workgroups hide it).
// us per pass: 48 replicas of 68 362 floats 11.2 -> 5.0, in planes 16.4 -> 7.0.
// Replica loads and stores are streaming (non-temporal): nothing is reused.
#include "kavg_internal.h"
#include "split.h"
#include <type_traits>

namespace kavg {

__device__ __forceinline__ uint16_t to_bf16_bits(float x) {     // weights: nearest, ties away from zero
    return (uint16_t)split_hi(__builtin_bit_cast(uint32_t, x));
}

// One parameter.  A vector whose length is no multiple of the parameters per lane ends in up to seven of them, and the step ends
// with the lane that takes the last one: its loads go out sixteen at a time as well (one by one they were a round trip each: 48
// replicas of 220 001 floats, four per lane, 17.0 -> 14.7 us; 64 of 240 001 in planes, eight per lane, 35.7 -> 22.7).
__device__ __forceinline__ void meta_scalar_element(float* w_tilde, float* v, float* reps, size_t stride,
                                                    uint16_t* shadow, size_t sstride, int P, size_t e,
                                                    float mu, float invP) {
    const float wt = w_tilde[e];
    float acc = 0.f;
#pragma unroll 16
    for (int j = 0; j < P; ++j) acc += reps[(size_t)j * stride + e] - wt;
    const float vn = mu * v[e] + acc * invP;
    const float wn = wt + vn;
    v[e] = vn;
    w_tilde[e] = wn;
    for (int j = 0; j < P; ++j) reps[(size_t)j * stride + e] = wn;
    if (shadow) {
        const uint16_t h = to_bf16_bits(wn);
        for (int j = 0; j < P; ++j) shadow[(size_t)j * sstride + e] = h;
    }
}

// V: pieces of W parameters per lane, 256 lanes apart, so that a workgroup covers V*W KB of consecutive
// addresses in every replica (longer runs inside one DRAM row per stream).
template <bool SHADOW, int UNROLL, bool SHADOW_CACHED, int V, int W, bool TOGETHER>
__global__ void __launch_bounds__(256)
meta_update_vec_kernel(float* __restrict__ w_tilde, float* __restrict__ v, float* __restrict__ reps,
                       size_t stride, uint16_t* __restrict__ shadow, size_t sstride, int P,
                       size_t n4, size_t n, float mu, float invP) {      // n4: whole pieces
    typedef float fvec __attribute__((ext_vector_type(W)));
    typedef uint16_t hvec __attribute__((ext_vector_type(W)));
    const size_t i0 = (size_t)blockIdx.x * (256 * V) + threadIdx.x;
    const size_t s4 = stride / W;
    if (i0 + (size_t)(V - 1) * 256 < n4) {                  // all V pieces are whole vectors
        fvec wt[V], acc[V];
#pragma unroll
        for (int q = 0; q < V; ++q) { wt[q] = ((const fvec*)w_tilde)[i0 + q * 256]; acc[q] = 0.f; }
        const fvec* r = (const fvec*)reps + i0;
        int j = 0;
        for (; j + UNROLL <= P; j += UNROLL) {
            fvec t[UNROLL][V];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int q = 0; q < V; ++q) t[u][q] = __builtin_nontemporal_load(r + (size_t)(j + u) * s4 + q * 256);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int q = 0; q < V; ++q) acc[q] += t[u][q] - wt[q];
        }
        if constexpr (!TOGETHER) {
            for (; j < P; ++j)
#pragma unroll
                for (int q = 0; q < V; ++q) acc[q] += __builtin_nontemporal_load(r + (size_t)j * s4 + q * 256) - wt[q];
        } else if (j < P) {
            fvec t[UNROLL][V];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
#pragma unroll
                for (int q = 0; q < V; ++q) t[u][q] = __builtin_nontemporal_load(r + (size_t)min(j + u, P - 1) * s4 + q * 256);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u)
                if (j + u < P)
#pragma unroll
                    for (int q = 0; q < V; ++q) acc[q] += t[u][q] - wt[q];
        }
        fvec wn[V];
#pragma unroll
        for (int q = 0; q < V; ++q) {
            const fvec vn = mu * ((const fvec*)v)[i0 + q * 256] + acc[q] * invP;
            wn[q] = wt[q] + vn;
            ((fvec*)v)[i0 + q * 256] = vn;
            ((fvec*)w_tilde)[i0 + q * 256] = wn[q];
        }
        fvec* o = (fvec*)reps + i0;
        for (int jj = 0; jj < P; ++jj)
#pragma unroll
            for (int q = 0; q < V; ++q) __builtin_nontemporal_store(wn[q], o + (size_t)jj * s4 + q * 256);
        if (SHADOW) {
            const size_t ss4 = sstride / W;
#pragma unroll
            for (int q = 0; q < V; ++q) {
                hvec h;
#pragma unroll
                for (int e = 0; e < W; ++e) h[e] = to_bf16_bits(wn[q][e]);
                hvec* so = (hvec*)shadow + i0 + q * 256;
                // The shadows are what the next forward pass reads: when they all fit in the memory-side
                // cache they are written with ordinary stores and stay there (the replicas above, read
                // again only by the updates, always bypass it).
                if (SHADOW_CACHED) { for (int jj = 0; jj < P; ++jj) so[(size_t)jj * ss4] = h; }
                else { for (int jj = 0; jj < P; ++jj) __builtin_nontemporal_store(h, so + (size_t)jj * ss4); }
            }
        }
        return;
    }
    if constexpr (V * W == 1) return;                       // (nothing is smaller than a parameter)
    // the last workgroups: piece by piece, whole vectors first, then the ragged tail of at most 3 parameters
    for (int q = 0; q < V; ++q) {
        const size_t i = i0 + (size_t)q * 256;
        if (i < n4) {
            for (int e = 0; e < W; ++e)
                meta_scalar_element(w_tilde, v, reps, stride, SHADOW ? shadow : nullptr, sstride, P, W * i + e, mu, invP);
        } else {
            const size_t e = W * n4 + (i - n4);
            if (e < n) meta_scalar_element(w_tilde, v, reps, stride, SHADOW ? shadow : nullptr, sstride, P, e, mu, invP);
        }
    }
}

__global__ void __launch_bounds__(256)
meta_update_scalar_kernel(float* w_tilde, float* v, float* reps, size_t stride, uint16_t* shadow,
                          size_t sstride, int P, size_t n, float mu, float invP) {
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e < n) meta_scalar_element(w_tilde, v, reps, stride, shadow, sstride, P, e, mu, invP);
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

hipError_t launch_meta_update(float* w_tilde, float* v, float* reps, size_t stride,
                              uint16_t* shadow, size_t sstride, int P, size_t n, float mu,
                              int shadow_cached, hipStream_t st) {
    const float invP = 1.0f / (float)P;
    bool vec = aligned16(w_tilde) && aligned16(v) && aligned16(reps) && (stride % 4 == 0);
    if (shadow) vec = vec && (((uintptr_t)shadow & 7) == 0) && (sstride % 4 == 0);
    if (vec) {
        // Long vectors: eight pieces per lane, so that a workgroup reads and writes 32 KB of consecutive
        // addresses per replica (meta-only workload, 64 replicas: 0.665 -> 0.70 of the HBM peak); others one piece per
        // lane.  A parameter per lane up to four workgroups per compute unit: beyond, four times as many requests cost more than
        // the workgroups hide; up to three of very few replicas, whose latency is soon hidden, and of many in whole pieces, where
        // the requests count sooner.  us, four per lane / one: 31 replicas of 250 001 18.1 / 8.4, 16 of 196 607 5.3 / 4.2, 48 of 68 362
        // 11.2 / 5.0; 64 of 230 000 16.7 / 21.7, 48 of 210 000 11.8 / 13.9, 2 of 230 000 2.7 / 3.2; 64 of 410 000 (and two per lane)
        // 35.6 / 43.9 (40.7); rounds of one step on 504-504-10, 259 570 parameters, 48 learners 78.9 / 76.2.
        // The last replicas together: one by one / together, a parameter per lane: 31 of 68 362 5.2 / 4.2, 33 4.3 / 4.6 (rounds of
        // four steps on 3072-64-10, 4 learners, 72.4 / 72.1); four per lane: 12 of 410 000 6.6 / 6.0, 31 of 350 001 26.8 / 17.2, but 17
        // of 410 000 9.9 / 11.0, 24 of 700 000 23.0 / 26.3.
        const bool wide = n / 4 >= (size_t)256 * 8 * 1024;
        const int W = n < (size_t)(P >= 4 && (P < 32 || n % 4) ? 4 : 3) * 256 * 256 ? 1 : 4, rest = P % 16;
        const bool together = W == 1 ? rest >= 4 : rest >= 8 && n < (size_t)2 * 256 * 1024;
        const size_t nw = n / W, threads = nw + (n - W * nw);
        const unsigned grid = (unsigned)((threads + (wide ? 2048 : 256) - 1) / (wide ? 2048 : 256));
#define KAVG_META_AS(SH, SC, U, V, W, T)                                                                      \
        hipLaunchKernelGGL((meta_update_vec_kernel<SH, U, SC, V, W, T>), dim3(grid), dim3(256), 0, st, w_tilde, v, reps, stride, \
                           shadow, sstride, P, nw, n, mu, invP)
#define KAVG_META_LAUNCH(SH, SC)                                                                              \
        do {                                                                                                  \
            if (wide) KAVG_META_AS(SH, SC, 2, 8, 4, false);                                                   \
            else if (W == 4 && together) KAVG_META_AS(SH, SC, 16, 1, 4, true);                                \
            else if (W == 4) KAVG_META_AS(SH, SC, 16, 1, 4, false);                                           \
            else if (together) KAVG_META_AS(SH, SC, 16, 1, 1, true);                                          \
            else KAVG_META_AS(SH, SC, 16, 1, 1, false);                                                       \
        } while (0)
        if (shadow && shadow_cached) KAVG_META_LAUNCH(true, true);
        else if (shadow) KAVG_META_LAUNCH(true, false);
        else KAVG_META_LAUNCH(false, false);
#undef KAVG_META_AS
#undef KAVG_META_LAUNCH
    } else {
        const unsigned grid = (unsigned)((n + 255) / 256);
        hipLaunchKernelGGL(meta_update_scalar_kernel, dim3(grid), dim3(256), 0, st, w_tilde, v, reps,
                           stride, shadow, sstride, P, n, mu, invP);
    }
    return hipGetLastError();
}

// ---- the same step on replicas stored as hi / lo planes -------------------------------------
// Each lane owns eight consecutive parameters: 16 bytes of either plane per learner.  Traffic per
// parameter and pass: P*(2+2) bytes read, P*(2+2) written, plus w~ and v: (2P+4)*4 bytes -- the
// refreshed bf16 values are part of the replicas, not an extra copy.  The hi planes are what the
// next forward pass reads (ordinary stores when they fit the memory-side cache); the lo planes
// are only read again by the updates and are streamed.
__device__ __forceinline__ void meta_split_scalar_element(float* w_tilde, float* v, uint16_t* hi, uint16_t* lo,
                                                          size_t stride, int P, size_t e, float mu, float invP) {
    const float wt = w_tilde[e];
    float acc = 0.f;
#pragma unroll 16
    for (int j = 0; j < P; ++j) {
        const size_t at = (size_t)j * stride + e;
        acc += __builtin_bit_cast(float, split_join(hi[at], lo[at])) - wt;
    }
    const float vn = mu * v[e] + acc * invP;
    const float wn = wt + vn;
    v[e] = vn;
    w_tilde[e] = wn;
    const uint32_t b = __builtin_bit_cast(uint32_t, wn);
    for (int j = 0; j < P; ++j) {
        const size_t at = (size_t)j * stride + e;
        hi[at] = (uint16_t)split_hi(b);
        lo[at] = (uint16_t)split_lo(b);
    }
}

// W: parameters per lane
template <int UNROLL, bool HI_CACHED, int W, bool TOGETHER>
__global__ void __launch_bounds__(256)
meta_update_split_kernel(float* __restrict__ w_tilde, float* __restrict__ v, uint16_t* __restrict__ hi,
                         uint16_t* __restrict__ lo, size_t stride, int P, size_t nw, size_t n, float mu,
                         float invP) {
    typedef uint32_t words __attribute__((ext_vector_type(W / 2)));          // pairs of 16 bits
    constexpr int F = W < 4 ? W : 4;
    typedef float fvec __attribute__((ext_vector_type(F)));
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < nw) {
        float wt[W], acc[W];
#pragma unroll
        for (int f = 0; f < W / F; ++f) {
            const fvec x = ((const fvec*)w_tilde)[i * (W / F) + f];
#pragma unroll
            for (int e = 0; e < F; ++e) wt[f * F + e] = x[e];
        }
#pragma unroll
        for (int e = 0; e < W; ++e) acc[e] = 0.f;
        const words* ph = (const words*)hi + i;
        const words* pl = (const words*)lo + i;
        const size_t s8 = stride / W;
        auto add = [&](const words& h, const words& l) {
#pragma unroll
            for (int q = 0; q < W / 2; ++q) {
                uint32_t b0, b1;
                split_join2(h[q], l[q], b0, b1);
                acc[2 * q] += __builtin_bit_cast(float, b0) - wt[2 * q];
                acc[2 * q + 1] += __builtin_bit_cast(float, b1) - wt[2 * q + 1];
            }
        };
        int j = 0;
        auto batch = [&](auto whole) __attribute__((always_inline)) {           // not whole: the last learner over and over, added once
            words th[UNROLL], tl[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const size_t at = (size_t)(whole ? j + u : min(j + u, P - 1)) * s8;
                th[u] = HI_CACHED ? ph[at] : __builtin_nontemporal_load(ph + at);
                tl[u] = __builtin_nontemporal_load(pl + at);
            }
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) if (whole || j + u < P) add(th[u], tl[u]);
        };
        for (; j + UNROLL <= P; j += UNROLL) batch(std::true_type{});
        if constexpr (!TOGETHER) {
            for (; j < P; ++j)
                add(HI_CACHED ? ph[(size_t)j * s8] : __builtin_nontemporal_load(ph + (size_t)j * s8),
                    __builtin_nontemporal_load(pl + (size_t)j * s8));
        } else {
            if (j < P) batch(std::false_type{});
        }
        float wn[W];
        fvec vo[W / F];                                         // (all before the first store: a wait for a load is one for older stores, too)
#pragma unroll
        for (int f = 0; f < W / F; ++f) vo[f] = ((const fvec*)v)[i * (W / F) + f];
#pragma unroll
        for (int f = 0; f < W / F; ++f) {
            fvec vn, w;
#pragma unroll
            for (int e = 0; e < F; ++e) {
                vn[e] = mu * vo[f][e] + acc[f * F + e] * invP;
                w[e] = wn[f * F + e] = wt[f * F + e] + vn[e];
            }
            ((fvec*)v)[i * (W / F) + f] = vn;
            ((fvec*)w_tilde)[i * (W / F) + f] = w;
        }
        words oh, ol;
#pragma unroll
        for (int q = 0; q < W / 2; ++q) {
            uint32_t h2, l2;
            split_pack2(__builtin_bit_cast(uint32_t, wn[2 * q]), __builtin_bit_cast(uint32_t, wn[2 * q + 1]), h2, l2);
            oh[q] = h2; ol[q] = l2;
        }
        words* qh = (words*)hi + i;
        words* ql = (words*)lo + i;
        if (HI_CACHED) { for (int jj = 0; jj < P; ++jj) qh[(size_t)jj * s8] = oh; }
        else { for (int jj = 0; jj < P; ++jj) __builtin_nontemporal_store(oh, qh + (size_t)jj * s8); }
        for (int jj = 0; jj < P; ++jj) __builtin_nontemporal_store(ol, ql + (size_t)jj * s8);
    } else {
        const size_t e = W * nw + (i - nw);               // ragged tail: fewer than W parameters
        if (e < n) meta_split_scalar_element(w_tilde, v, hi, lo, stride, P, e, mu, invP);
    }
}

hipError_t launch_meta_update_split(float* w_tilde, float* v, uint16_t* hi, uint16_t* lo, size_t stride,
                                    int P, size_t n, float mu, int hi_cached, hipStream_t st) {
    // planes and vectors come out of the 256-byte aligned workspace; stride is a multiple of 64
    const float invP = 1.0f / (float)P;
    // Two parameters per lane up to two workgroups per compute unit, beyond that the requests cost more than the workgroups hide
    // (us, eight per lane / two: 16 replicas of 240 001 7.5 / 5.5, 48 of 68 362 16.4 / 7.0; 64 of 470 000 36.4 / 45.0, 33 of 410 000
    // 17.2 / 20.9; four per lane: 8 of 1 000 000 10.5 / 13.3).  The last replicas together: one by one / together, eight per lane:
    // 12 of 300 000 7.7 / 7.4, 31 of 410 000 18.6 / 16.5; but 37 of 817 000 40.0 / 46.7.
    const int W = hi_cached && n < (size_t)2 * 256 * 512 ? 2 : 8;
    const bool together = W == 2 ? P % 16 > 4 : P % 8 >= 4 && hi_cached && n < (size_t)2 * 256 * 1024;
    const size_t nw = n / W, threads = nw + (n - W * nw);
    const dim3 grid((unsigned)((threads + 255) / 256));
#define KAVG_META_SPLIT(U, HC, W, T) \
    hipLaunchKernelGGL((meta_update_split_kernel<U, HC, W, T>), grid, dim3(256), 0, st, w_tilde, v, hi, lo, stride, P, nw, n, mu, invP)
    if (!hi_cached) KAVG_META_SPLIT(8, false, 8, false);
    else if (W == 8 && together) KAVG_META_SPLIT(8, true, 8, true);
    else if (W == 8) KAVG_META_SPLIT(8, true, 8, false);
    else if (together) KAVG_META_SPLIT(16, true, 2, true);
    else KAVG_META_SPLIT(16, true, 2, false);
#undef KAVG_META_SPLIT
    return hipGetLastError();
}

__global__ void __launch_bounds__(256)
broadcast_split_kernel(const float* __restrict__ w_tilde, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo,
                       size_t stride, int P, size_t n) {
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const uint32_t b = __builtin_bit_cast(uint32_t, w_tilde[e]);
    for (int j = 0; j < P; ++j) {
        hi[(size_t)j * stride + e] = (uint16_t)split_hi(b);
        lo[(size_t)j * stride + e] = (uint16_t)split_lo(b);
    }
}

hipError_t launch_broadcast_split(const float* w_tilde, uint16_t* hi, uint16_t* lo, size_t stride, int P,
                                  size_t n, hipStream_t st) {
    const unsigned grid = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(broadcast_split_kernel, dim3(grid), dim3(256), 0, st, w_tilde, hi, lo, stride, P, n);
    return hipGetLastError();
}

// "set w^j = w~_n" for every learner (first round, or after a state restore).
__global__ void __launch_bounds__(256)
broadcast_kernel(const float* __restrict__ w_tilde, float* __restrict__ reps, size_t stride,
                 uint16_t* __restrict__ shadow, size_t sstride, int P, size_t n) {
    const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const float w = w_tilde[e];
    for (int j = 0; j < P; ++j) reps[(size_t)j * stride + e] = w;
    if (shadow) {
        const uint16_t h = to_bf16_bits(w);
        for (int j = 0; j < P; ++j) shadow[(size_t)j * sstride + e] = h;
    }
}

hipError_t launch_broadcast(const float* w_tilde, float* reps, size_t stride, uint16_t* shadow,
                            size_t sstride, int P, size_t n, hipStream_t st) {
    const unsigned grid = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(broadcast_kernel, dim3(grid), dim3(256), 0, st, w_tilde, reps, stride, shadow,
                       sstride, P, n);
    return hipGetLastError();
}

}  // namespace kavg
