// Running norm estimate of Appendix G where a scored step leaves its tile sums to the launch that needs them next (gfx950,
// wave64): the next scored step folds them into g_mvg in a few blocks of its own, the communication in the launch that forms
// the weights.  A step is then one launch, whatever the layers are, and no block waits for another.
//
// The step counts live on the device, so that replayed calls count.  What a launch folds in lies in another buffer than the sums
// that it writes (grawa_step_buffer).
// A communication writes nothing but counts (d_consumed, d_seen), which say that everything up to that step is used up; what is left
// of mvg is then taken as zero.  Every sum runs in the same order wherever it is formed, so that a replay gives the bits of the calls.
#pragma once
#include "grawa_route.h"
#include "grawa_scores.h"

struct GrawaFold {
    GrawaEstimate *est;
    double *value; // [K][L] the estimates once more, packed: written by k_fold, for the model level
    const uint64_t *consumed; // [2 L]
    const int32_t *layer_tile0; // [L+1]
    unsigned *flags;
    int64_t pitch; // sums in one of the buffers
    int K, L;
    int by_wave;     // no layer has more than GRAWA_FOLD_WAVE_TILES tiles
    int lanes;       // of a wave that add the tiles of a worker: as many as in the pull, where that folds in (wave_layer_weights)
    unsigned buffer; // that the sums of this launch go to
    unsigned blocks, rows; // of a step's grid that fold (grawa_fold_blocks)
    double gamma;    // of the step that this launch takes
};

enum { GRAWA_SCORE_NONE = 0, GRAWA_SCORE_SUMS = 1, GRAWA_SCORE_LATER = 2 }; // k_row_step: no scores; sums for the launch after it; sums for the next call

#define GRAWA_FOLD_LANES 512 // that share a long layer's tiles

// Sum of p[t0 + first], p[t0 + first + step], ... below t1 over the lanes of one wave, four
// independent loads in flight per lane; every lane gets the total.
__device__ __forceinline__ double wave_strided_sum(const double *__restrict__ p, int t0, int t1, int first,
                                                   int step)
{
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int t = t0 + first;
    for (; t + 3 * step < t1; t += 4 * step) {
        s0 += p[t];
        s1 += p[t + step];
        s2 += p[t + 2 * step];
        s3 += p[t + 3 * step];
    }
    for (; t < t1; t += step) s0 += p[t];
    return wave_sum((s0 + s1) + (s2 + s3));
}

// The same sum as that of a wave from t0 on, where it has up to N = 4 or 16 terms, by one thread: the order of wave_sum.
template <int N> __device__ __forceinline__ double few_tiles_sum(const double *__restrict__ p, int t0, int t1)
{
    double s[N];
#pragma unroll
    for (int i = 0; i < N; ++i) s[i] = t0 + i < t1 ? p[t0 + i] : 0.0;
#pragma unroll
    for (int m = 1; m < N; m <<= 1)
#pragma unroll
        for (int i = 0; i < N; i += 2 * m) s[i] += s[i + m];
    return s[0];
}

// Sum of p[t0] .. p[t1 - 1] by GRAWA_FOLD_LANES threads of a block, or by one of 256, each of which does what two of those do.
// Called by the whole block; every thread gets the total.  `part`: one double per wave of GRAWA_FOLD_LANES threads.
template <int THREADS>
__device__ __forceinline__ double block_tile_sum(const double *__restrict__ p, int t0, int t1, double *part)
{
    __syncthreads(); // the parts of the sum before have been read
#pragma unroll 1 // few registers: a step that folds on the way keeps its waves
    for (int first = (int)threadIdx.x; first < GRAWA_FOLD_LANES; first += THREADS) {
        double s[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) s[u] = 0.0;
        int t = t0 + first;
        for (; t + 7 * GRAWA_FOLD_LANES < t1; t += 8 * GRAWA_FOLD_LANES)
#pragma unroll
            for (int u = 0; u < 8; ++u) s[u] += p[t + u * GRAWA_FOLD_LANES];
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (t + u * GRAWA_FOLD_LANES < t1) s[u] += p[t + u * GRAWA_FOLD_LANES];
        const double w = wave_sum(((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])));
        if ((threadIdx.x & (GRAWA_WAVE - 1)) == 0) part[first / GRAWA_WAVE] = w;
    }
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < GRAWA_FOLD_LANES / GRAWA_WAVE; ++w) tot += part[w];
    return tot;
}

// Brings the estimates of all workers and layers up to the last step: block `first` of `blocks`, of THREADS threads.  A wave takes a worker
// and layer, or, where some layer is longer than a wave adds, the block.
//   FOLD_STEP   and this launch takes the next step, whose sums stay pending
//   FOLD_ONLY   nothing more
//   FOLD_SUMS   and the sums of the next step, in f.buffer, are folded in as well
enum { GRAWA_FOLD_STEP, GRAWA_FOLD_ONLY, GRAWA_FOLD_SUMS };
template <int THREADS, int MODE>
__device__ __forceinline__ void fold_all(const GrawaFold &f, const double *__restrict__ sums, int64_t n_tiles, unsigned first, unsigned blocks)
{
    __shared__ double part[GRAWA_FOLD_LANES / GRAWA_WAVE];
    constexpr unsigned WAVES = THREADS / GRAWA_WAVE;
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const unsigned wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / GRAWA_WAVE));
    const unsigned units = (unsigned)f.K * (unsigned)f.L; // at most GRAWA_FOLD_MAX_UNITS
    const unsigned step = f.by_wave ? blocks * WAVES : blocks;
    for (unsigned u = f.by_wave ? first * WAVES + wave : first; u < units; u += step) {
        const unsigned k = u / (unsigned)f.L, l = u - k * (unsigned)f.L;
        GrawaEstimate e = f.est[u];
        const uint64_t used = grawa_last_used(f.consumed[l], f.consumed[f.L + l]);
        const int t0 = f.layer_tile0[l], t1 = f.layer_tile0[l + 1];
        const double *p = sums + (int64_t)k * n_tiles;
        if (!f.by_wave) __syncthreads(); // every wave has read what thread 0 writes below
        double next = 0.0, tot = 0.0;
        const auto sum = [&](unsigned buffer) {
            return t1 - t0 > GRAWA_FOLD_WAVE_TILES ? block_tile_sum<THREADS>(p + buffer * f.pitch, t0, t1, part)
                                                   : wave_strided_sum(p + buffer * f.pitch, lane < f.lanes ? t0 : t1, t1, lane, f.lanes);
        };
        if (MODE == GRAWA_FOLD_SUMS) next = sum(f.buffer);
        if (grawa_estimate_pending(e, used)) tot = sum(e.buffer); // the same for all units
        if (f.by_wave ? lane == 0 : threadIdx.x == 0) {
            e.mvg = grawa_estimate_value(e, used, sqrt(tot));
            e.left = 0;
            if (MODE != GRAWA_FOLD_ONLY) {
                e.gamma = f.gamma;
                e.buffer = f.buffer;
                e.n += 1;
                e.left = 1;
            }
            if (MODE == GRAWA_FOLD_SUMS) {
                e.mvg = grawa_estimate_value(e, used, sqrt(next));
                e.left = 0;
            }
            f.est[u] = e;
            if (MODE != GRAWA_FOLD_STEP) f.value[u] = e.mvg;
        }
    }
}

static inline GrawaFold grawa_fold_of(const grawa_plan *p, double gamma, unsigned buffer, unsigned blocks, unsigned rows)
{
    return GrawaFold{p->d_est, p->d_mvg, p->d_consumed, p->d_layer_rtile0, p->d_flags, (int64_t)p->K * p->n_rtiles, p->K, p->L,
                     p->max_rtiles <= GRAWA_FOLD_WAVE_TILES, p->d_seen ? grawa_group_lanes(p->K) : 64, buffer, blocks, rows, gamma};
}
