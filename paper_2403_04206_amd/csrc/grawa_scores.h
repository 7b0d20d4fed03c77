// From tile sums to scores and weights on the device (gfx950, wave64): the weight formula, and the pieces that
// let one launch do what needs a second one otherwise.
//
// Values pass between blocks of one launch (which may run on different XCDs, each with an L2 of its own) only
// through device-scope atomic read-modify-writes, which always act on the latest value.  A thread that hands
// a value over waits for the exchange to return before its block counts itself in, and the block that arrives last
// reads after its count has returned.  No block ever waits for another: one that is not last leaves, so nothing
// depends on which blocks are resident and nothing can hang.  Which block comes last varies from run to run;
// what it adds and in which order does not, so results are bit-reproducible.  Release and acquire fences at
// device scope would do instead of the read-modify-writes, but write back and invalidate a whole L2 per block
// (one acquire per layer alone: 16 us instead of 8 for the norm pass of a 270 k-parameter model).
#pragma once
#include "grawa_device.h"

// The values below pass through registers that the compiler cannot see through: an exchange whose result is unused
// may be lowered to a plain store, and the addition of a known zero is lowered to a plain load.
__device__ __forceinline__ void hand_over(double *p, double v)
{
    const unsigned long long before =
        __hip_atomic_exchange(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(v),
                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("" ::"v"(before) : "memory"); // also: the exchange has been performed from here on
}
__device__ __forceinline__ double take_over(double *p)
{
    unsigned long long zero = 0ull;
    asm volatile("" : "+v"(zero)::"memory");
    return __longlong_as_double((long long)__hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(p), zero,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Counts the block in; true in every thread of the block that is the n-th.  What the block publishes was
// handed over, by any of its threads, before the call.  The launch before this one has set the counter to zero (k_sumsq),
// so that nothing a launch leaves behind, complete or not, reaches the next call.
// `sh` is one word of LDS.
__device__ __forceinline__ bool last_to_arrive(unsigned *counter, unsigned n, unsigned *sh)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *sh = before == n - 1 ? 1u : 0u;
    }
    __syncthreads();
    return *sh != 0u;
}

// Weights of one group of K scores held in LDS (sA[k], k < K): beta_k proportional to
// 1/A_k, summing to one, evaluated as (A_min/A_k) / sum_j (A_min/A_j) so that nothing
// overflows.  Scores of exactly zero share the weight equally and take all of it (the
// limit A -> 0+).  Called by ONE full wave (all 64 lanes); lanes stride over the workers.
// A score that is +inf or NaN sets `bit` in the plan's flag word (flags may be null).
__device__ __forceinline__ void group_weights(const double *sA, int K, float *beta, int64_t stride,
                                              float *beta_user, unsigned *flags, unsigned bit)
{
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    double mn = INFINITY, nz = 0.0, bad = 0.0;
    for (int k = lane; k < K; k += GRAWA_WAVE) {
        const double a = sA[k];
        mn = fmin(mn, a);
        nz += (a == 0.0) ? 1.0 : 0.0;
        bad += isfinite(a) ? 0.0 : 1.0;
    }
    const double a_min = wave_min(mn);
    const double n_zero = wave_sum(nz);
    if (flags && wave_sum(bad) > 0.0 && lane == 0) atomicOr(flags, bit);
    double z = 0.0;
    if (n_zero == 0.0)
        for (int k = lane; k < K; k += GRAWA_WAVE) z += a_min / sA[k];
    const double zsum = wave_sum(z);
    for (int k = lane; k < K; k += GRAWA_WAVE) {
        const double a = sA[k];
        double b;
        if (n_zero > 0.0)
            b = (a == 0.0) ? 1.0 / n_zero : 0.0;
        else
            b = (a_min / a) / zsum;
        beta[(int64_t)k * stride] = (float)b;
        if (beta_user) beta_user[(int64_t)k * stride] = (float)b;
    }
}

// The score of a worker and layer from its sum of squares: its norm.  load() comes before the sums are read, publish() where the weights
// are written out.
struct NormScore {
    struct State {};
    __device__ __forceinline__ State load(int, int) const { return State{}; }
    __device__ __forceinline__ double score(const State &, double sum) const { return sqrt(sum); }
    __device__ __forceinline__ void publish(int, int, double) const {}
};

// The same weights for one layer l straight from its tile sums, by one full wave (K <= 64): `group` = the largest
// power of two not above 64 / K lanes share a worker's tiles t0 .. t1 - 1.  out[k] (LDS) receives beta_k;
// beta_user[k * L] too if not null, and a score that is not finite is flagged then.
template <typename Score>
__device__ __forceinline__ void wave_layer_weights(const Score &scores, int l, const double *__restrict__ partials, int64_t pitch,
                                                   int t0, int t1, int K, int group, float *out, bool owner,
                                                   float *beta_user, int L, unsigned *flags)
{
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int k = lane / group, i = lane % group;
    const bool active = k < K, head = active && i == 0;
    const double *p = partials + (int64_t)(active ? k : 0) * pitch;
    const typename Score::State state = scores.load(active ? k : 0, l);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int t = t0 + i;
    for (; t + 3 * group < t1; t += 4 * group) {
        s0 += p[t];
        s1 += p[t + group];
        s2 += p[t + 2 * group];
        s3 += p[t + 3 * group];
    }
    for (; t < t1; t += group) s0 += p[t];
    double s = (s0 + s1) + (s2 + s3);
    for (int m = 1; m < group; m <<= 1) s += __shfl_xor(s, m, GRAWA_WAVE);
    const double a = scores.score(state, s);
    const double a_min = wave_min(active ? a : (double)INFINITY);
    const double n_zero = __popcll(__ballot(head && a == 0.0));
    const double z = wave_sum(head && n_zero == 0.0 ? a_min / a : 0.0);
    if (head) {
        const double b = n_zero > 0.0 ? (a == 0.0 ? 1.0 / n_zero : 0.0) : (a_min / a) / z;
        out[k] = (float)b;
        if (owner && beta_user) beta_user[(int64_t)k * L] = (float)b;
        if (owner && flags && !isfinite(a)) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
        if (owner) scores.publish(k, l, a);
    }
}

// The same by a segment of G lanes, the smallest power of two not below K, one worker each; a wave takes 64 / G layers at a time, and all
// its lanes take part (`here`: the segment has a layer).  For layers of few tiles; the whole row of weights.
template <int K> struct Segment {
    static constexpr int G = K <= 1 ? 1 : K <= 2 ? 2 : K <= 4 ? 4 : K <= 8 ? 8 : 16;
};
template <int G, typename Op> __device__ __forceinline__ double segment_reduce(double v, const Op &op)
{
    static_assert(G <= 16, "within a row of lanes");
    if constexpr (G > 1) v = op(v, dpp_move_f64<0xB1>(v));  // lane ^ 1
    if constexpr (G > 2) v = op(v, dpp_move_f64<0x4E>(v));  // lane ^ 2
    if constexpr (G > 4) v = op(v, dpp_move_f64<0x141>(v)); // other quad of the half row
    if constexpr (G > 8) v = op(v, dpp_move_f64<0x140>(v)); // other half of the row
    return v;
}
template <int K, typename Score>
__device__ __forceinline__ void segment_layer_weights(const Score &scores, int l, bool here, const double *__restrict__ partials,
                                                      int64_t pitch, int t0, int t1, float *out, float *beta_user, int L,
                                                      unsigned *flags)
{
    constexpr int G = Segment<K>::G;
    const int lane = threadIdx.x & (GRAWA_WAVE - 1), k = lane % G;
    const bool active = here && k < K;
    double a = INFINITY;
    if (active) {
        const typename Score::State state = scores.load(k, l);
        double s = 0.0;
        for (int t = t0; t < t1; ++t) s += partials[(int64_t)k * pitch + t];
        a = scores.score(state, s);
    }
    const double a_min = segment_reduce<G>(a, [](double p, double q) { return fmin(p, q); });
    const unsigned long long zero = __ballot(active && a == 0.0) >> (lane - k) & (~0ull >> (GRAWA_WAVE - G));
    const double n_zero = __popcll(zero);
    const double z = segment_reduce<G>(active && n_zero == 0.0 ? a_min / a : 0.0, [](double p, double q) { return p + q; });
    if (active) {
        const float b = (float)(n_zero > 0.0 ? (a == 0.0 ? 1.0 / n_zero : 0.0) : (a_min / a) / z);
        out[k] = b;
        if (beta_user) beta_user[(int64_t)k * L] = b;
        if (flags && !isfinite(a)) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
        scores.publish(k, l, a);
    }
}

// The same by one lane, which walks the workers.
template <int K, typename Score>
__device__ __forceinline__ void lane_layer_weights(const Score &scores, int l, const double *__restrict__ partials, int64_t pitch,
                                                   int t0, int t1, float *out, float *beta_user, int L, unsigned *flags)
{
    double a[K];
#pragma unroll
    for (int k = 0; k < K; ++k) a[k] = 0.0;
    for (int t = t0; t < t1; ++t)
#pragma unroll
        for (int k = 0; k < K; ++k) a[k] += partials[(int64_t)k * pitch + t];
    double a_min = INFINITY, n_zero = 0.0, z = 0.0;
    bool bad = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        a[k] = scores.score(scores.load(k, l), a[k]);
        scores.publish(k, l, a[k]);
        a_min = fmin(a_min, a[k]);
        n_zero += a[k] == 0.0 ? 1.0 : 0.0;
        bad = bad || !isfinite(a[k]);
    }
    if (n_zero == 0.0) {
#pragma unroll
        for (int k = 0; k < K; ++k) z += a_min / a[k];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float b = (float)(n_zero > 0.0 ? (a[k] == 0.0 ? 1.0 / n_zero : 0.0) : (a_min / a[k]) / z);
        out[k] = b;
        if (beta_user) beta_user[(int64_t)k * L] = b;
    }
    if (flags && bad) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
}
