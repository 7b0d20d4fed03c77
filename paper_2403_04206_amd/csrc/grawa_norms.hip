// Gradient norms and weights of the GRAWA update (gfx950, wave64).
//
//   k_sumsq            per (tile, worker) sum of squares of the gradient   [eq. (3), (5)]
//   k_finalize_layers  tile sums -> ||G||_F, per-layer or model-level weights [eq. (2)-(7)]
//   k_finalize_model   ||G||_F -> model-level weights, many layers         [eq. (2)-(4)]
//   k_estimate         tile sums of a scored step -> running norm estimate [App. G]
//   k_local_weights    weights from the running norm estimate              [App. G]
//   k_leader_weights   LSGD (leader) weights                               [App. F]
//
// The norm pass is a read-only stream: it runs fastest with several non-temporal loads per
// lane in flight and a capped occupancy; what a fused pull reads again is read through the caches (grawa_cached_grad_cols).  Squares and sums are fp64 throughout, added in a
// fixed order (no sum is formed by atomics; how norms pass between the blocks of a launch: grawa_scores.h),
// so results are bit-reproducible.
#include "grawa_fold.h"
#include "grawa_offsets.h"
#include "grawa_route.h"

// ---------------------------------------------------------------------------------
// gradient norms: per-tile sums of squares
// ---------------------------------------------------------------------------------

// grid (n_tiles, K), block 256.  partials[k][tile] = sum over the tile of g[k][i]^2.  Also clears the arrival counter
// of the launch that follows (null where none arrives).  Tiles that start before cached_cols are read with cached loads.
// Each lane issues 8 independent 8-byte streaming loads per trip and keeps one accumulator
// per load; with the occupancy capped at 4 waves per SIMD this shape measured fastest for a
// read-only stream on this part (7.3-7.4 TB/s; 16-byte loads at full occupancy 6.9-7.0).
// Every value is widened to fp64 before it is squared and every sum is fp64: the squares are
// exact, so gradients of any magnitude the input type holds (1e-38 .. 3e38) give the same
// norms as a float64 evaluation up to the order of the additions.  The pass needs under a
// fifth of the fp64 rate at full HBM speed, so this costs no time.
#define GRAWA_SUMSQ_U 8

// The last, partial trip of up to N loads per lane: a lane past the end loads a clamped (valid) address and
// discards the value.
template <typename GT, bool NT, int N>
__device__ __forceinline__ void sumsq_rest(const GT *body, int j0, int nvec, double (&acc)[GRAWA_SUMSQ_U])
{
    if (j0 >= nvec) return;
    typename Grad<GT>::Vec8 q[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const int j = j0 + u * GRAWA_BLOCK;
        q[u] = Grad<GT>::template load8<NT>(body + (int64_t)(j < nvec ? j : j0) * Grad<GT>::VEC8);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const double r = Grad<GT>::sumsq8(q[u], 0.0);
        acc[u] += (j0 + u * GRAWA_BLOCK < nvec) ? r : 0.0;
    }
}

// The 8-byte vectors 0 .. nvec - 1 of a tile.
template <typename GT, bool NT>
__device__ __forceinline__ void sumsq_body(const GT *body, int nvec, double (&acc)[GRAWA_SUMSQ_U])
{
    constexpr int V = Grad<GT>::VEC8;
    const int tid = threadIdx.x;
    // All loads of a trip are issued before any is used.  Full trips need no bounds checks.
    typename Grad<GT>::Vec8 q[GRAWA_SUMSQ_U];
    int j0 = tid;
    for (; j0 + (GRAWA_SUMSQ_U - 1) * GRAWA_BLOCK < nvec; j0 += GRAWA_SUMSQ_U * GRAWA_BLOCK) {
#pragma unroll
        for (int u = 0; u < GRAWA_SUMSQ_U; ++u)
            q[u] = Grad<GT>::template load8<NT>(body + (int64_t)(j0 + u * GRAWA_BLOCK) * V);
        __builtin_amdgcn_sched_barrier(0); // keep the arithmetic from being hoisted between the loads
#pragma unroll
        for (int u = 0; u < GRAWA_SUMSQ_U; ++u) acc[u] = Grad<GT>::sumsq8(q[u], acc[u]);
    }
    // What is left is less than a trip: a trip of as few loads as hold it, so that a short tile does not load, convert and
    // discard values.  (All lanes of a block take the same one, except that with more than 7 loads left the lanes that
    // have all 8 took them as a full trip above and have nothing left.)
    const int left = nvec - (j0 - tid);
    if (left > 4 * GRAWA_BLOCK) sumsq_rest<GT, NT, 8>(body, j0, nvec, acc);
    else if (left > 2 * GRAWA_BLOCK) sumsq_rest<GT, NT, 4>(body, j0, nvec, acc);
    else if (left > GRAWA_BLOCK) sumsq_rest<GT, NT, 2>(body, j0, nvec, acc);
    else sumsq_rest<GT, NT, 1>(body, j0, nvec, acc);
}

// MIX: cached_cols may be above 0.
template <typename GT, bool MIX>
__device__ __forceinline__ void sumsq_tile(const GrawaTile t, const GT *__restrict__ g, int64_t ldg, int64_t n_tiles,
                                           double *__restrict__ partials, unsigned *__restrict__ cnt_all, int64_t cached_cols)
{
    constexpr int V = Grad<GT>::VEC8;
    const int k = blockIdx.y;
    const GT *row = g + (int64_t)k * ldg;
    const int tid = threadIdx.x;

    const int64_t a = t.start, b = t.start + t.len;
    int64_t a_al = (a + V - 1) / V * V;
    if (a_al > b) a_al = b;
    int64_t b_al = b / V * V;
    if (b_al < a_al) b_al = a_al;

    double acc[GRAWA_SUMSQ_U];
#pragma unroll
    for (int u = 0; u < GRAWA_SUMSQ_U; ++u) acc[u] = 0.0;

    // unaligned head (< V elements) on the first lanes, tail on the lanes of the second wave
    if (tid < (int)(a_al - a)) {
        acc[0] = sq_add(Grad<GT>::one(row + a + tid), 0.0);
    }
    if (tid >= GRAWA_WAVE && tid - GRAWA_WAVE < (int)(b - b_al)) {
        acc[1] = sq_add(Grad<GT>::one(row + b_al + (tid - GRAWA_WAVE)), 0.0);
    }

    const int nvec = (int)((b_al - a_al) / V);
    if (MIX && a < cached_cols) sumsq_body<GT, false>(row + a_al, nvec, acc);
    else sumsq_body<GT, true>(row + a_al, nvec, acc);

    __shared__ double sm[GRAWA_BLOCK / GRAWA_WAVE];
    double lane = 0.0;
#pragma unroll
    for (int u = 0; u < GRAWA_SUMSQ_U; ++u) lane += acc[u];
    const double total = block_sum<GRAWA_BLOCK>(lane, sm);
    if (tid == 0) partials[(int64_t)k * n_tiles + blockIdx.x] = total;
    if (cnt_all && tid == 0 && k == 0 && blockIdx.x == 0) *cnt_all = 0u;
}

template <typename GT, bool MIX>
__global__ __launch_bounds__(GRAWA_BLOCK) __attribute__((amdgpu_waves_per_eu(1, 4))) void k_sumsq(
    const GT *__restrict__ g, int64_t ldg, const GrawaTile *__restrict__ tiles, int64_t n_tiles,
    double *__restrict__ partials, unsigned *__restrict__ cnt_all, int64_t cached_cols)
{
    sumsq_tile<GT, MIX>(tiles[blockIdx.x], g, ldg, n_tiles, partials, cnt_all, cached_cols);
}

// The same without a map: every block finds its tile in the layer offsets.
template <typename GT>
__global__ __launch_bounds__(GRAWA_BLOCK) __attribute__((amdgpu_waves_per_eu(1, 4))) void k_sumsq_slots(
    const GT *__restrict__ g, int64_t ldg, const int64_t *__restrict__ off, int L, int64_t P, int shift, int64_t n_tiles,
    double *__restrict__ partials)
{
    const int64_t i = blockIdx.x;
    const int layer = wave_last_layer(off, L, [&](int l, int64_t o) { return first_slot(o, l, P, shift) <= i; });
    sumsq_tile<GT, false>(slot_tile(i, layer, off[layer], off[layer + 1], P, shift), g, ldg, n_tiles, partials, nullptr, 0);
}

// ---------------------------------------------------------------------------------
// scores and weights
// ---------------------------------------------------------------------------------

#define GRAWA_FIN_BLOCK 1024
#define GRAWA_FIN_WAVES (GRAWA_FIN_BLOCK / GRAWA_WAVE)

// Score of every worker (the sum of its layer norms, or the norm of the flattened gradient) from S[k][l], then the K
// weights, by one block of 1024.
template <typename Read>
__device__ __forceinline__ void model_weights(double *S, int K, int L, int goal, Read read, double *sA, float *beta,
                                              float *beta_user, unsigned *flags)
{
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = threadIdx.x / GRAWA_WAVE;
    for (int k = wave; k < K; k += GRAWA_FIN_WAVES) {
        double *p = S + (int64_t)k * L;
        double s = 0.0;
        for (int l = lane; l < L; l += GRAWA_WAVE) {
            const double v = read(p + l);
            s += goal == GRAWA_GOAL_MODEL_SUM ? sqrt(v) : v;
        }
        s = wave_sum(s);
        if (goal == GRAWA_GOAL_MODEL_FLAT) s = sqrt(s);
        if (lane == 0) sA[k] = s;
    }
    __syncthreads();
    if (wave == 0) group_weights(sA, K, beta, 1, beta_user, flags, GRAWA_NONFINITE_MODEL_SCORE);
}

// grid L, block 1024 (16 waves).  Block l adds the tile partials of layer l for every worker
// and turns the K layer norms into the K per-layer weights.  With K >= 16 every wave takes
// workers w, w+16, ...; with fewer workers 16/K waves share one worker's tiles and their
// results are added in wave order.  All sums are fp64 in a fixed order.
// Model level (goal): the blocks hand their squared norms S[k][l] over, and the last one forms the model-level weights;
// cnt_all null: S is only stored, for k_finalize_model (grawa_model_weights_by_last_block).
__global__ __launch_bounds__(GRAWA_FIN_BLOCK) void k_finalize_layers(
    const double *__restrict__ partials, int64_t n_tiles, const int32_t *__restrict__ tile_begin,
    const int32_t *__restrict__ tile_end, int K, int L, int goal, double *__restrict__ S, float *__restrict__ A_user,
    float *__restrict__ beta, float *__restrict__ beta_user, unsigned *__restrict__ cnt_all,
    unsigned *__restrict__ flags)
{
    __shared__ double sA[GRAWA_MAX_WORKERS];
    __shared__ double sw[GRAWA_FIN_WAVES];
    __shared__ unsigned sh_last;
    const int l = blockIdx.x;
    const int t0 = tile_begin[l], t1 = tile_end[l];
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = threadIdx.x / GRAWA_WAVE;
    if (K >= GRAWA_FIN_WAVES) {
        for (int k = wave; k < K; k += GRAWA_FIN_WAVES) {
            const double s = wave_strided_sum(partials + (int64_t)k * n_tiles, t0, t1, lane, GRAWA_WAVE);
            if (lane == 0) sA[k] = s;
        }
        __syncthreads();
    } else {
        const int share = GRAWA_FIN_WAVES / K; // waves per worker
        const int k = wave % K, part = wave / K;
        double s = 0.0;
        if (part < share)
            s = wave_strided_sum(partials + (int64_t)k * n_tiles, t0, t1, part * GRAWA_WAVE + lane,
                                 share * GRAWA_WAVE);
        if (lane == 0) sw[wave] = s;
        __syncthreads();
        if ((int)threadIdx.x < K) {
            double tot = 0.0;
            for (int j = 0; j < share; ++j) tot += sw[threadIdx.x + j * K];
            sA[threadIdx.x] = tot;
        }
        __syncthreads();
    }
    // sA[k] holds the squared norm; publish it, replace it by the norm, then the weights
    const bool model = goal >= GRAWA_GOAL_MODEL_SUM;
    for (int k = threadIdx.x; k < K; k += GRAWA_FIN_BLOCK) {
        const double s = sA[k];
        const double a = sqrt(s);
        if (model && cnt_all) hand_over(S + (int64_t)k * L + l, s);
        else if (model) S[(int64_t)k * L + l] = s;
        if (A_user) A_user[(int64_t)k * L + l] = (float)a;
        if (goal != GRAWA_GOAL_LAYER_WEIGHTS && flags && !isfinite(a)) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
        sA[k] = a;
    }
    if (goal == GRAWA_GOAL_SCORES) return;
    if (!model) {
        __syncthreads();
        if (wave == 0) group_weights(sA, K, beta + l, L, beta_user ? beta_user + l : nullptr, flags, GRAWA_NONFINITE_LAYER_SCORE);
        return;
    }
    if (!cnt_all || !last_to_arrive(cnt_all, (unsigned)L, &sh_last)) return;
    model_weights(S, K, L, goal, [](double *p) { return take_over(p); }, sA, beta, beta_user, flags);
}

// grid 1, block 1024: the model-level weights from the squared layer norms.
__global__ __launch_bounds__(GRAWA_FIN_BLOCK) void k_finalize_model(double *__restrict__ S, int K, int L, int goal,
                                                                    float *__restrict__ beta,
                                                                    float *__restrict__ beta_user,
                                                                    unsigned *__restrict__ flags)
{
    __shared__ double sA[GRAWA_MAX_WORKERS];
    model_weights(S, K, L, goal, [](double *p) { return *p; }, sA, beta, beta_user, flags);
}

// grid (L, y) and block from grawa_estimate_shape: the tile sums of a scored local step -> running estimate of
// Appendix G, g_mvg <- gamma g_mvg + (1 - gamma) g_cur, t <- t + 1.  The tiles of this step are short (1024 columns).
// A layer of up to wave_tiles of them is a wave's work for one worker; of a longer one the whole block adds
// the tiles of one worker at a time (the 50 000 tiles of the largest layer of the 350 M transformer for each of 8 workers
// took one block 72 us).
// The counts t (one per layer, see k_local_weights) live on the device so that a recorded and replayed call still counts.
__global__ __launch_bounds__(GRAWA_EST_MAX_THREADS) void k_estimate(const double *__restrict__ partials, int64_t n_tiles,
                                                                    const int32_t *__restrict__ layer_tile0, int K, int L,
                                                                    int wave_tiles, double *__restrict__ mvg, double gamma,
                                                                    int64_t *__restrict__ local_t,
                                                                    unsigned *__restrict__ flags)
{
    __shared__ double sm[GRAWA_MAX_WORKERS];
    const int l = blockIdx.x, y = blockIdx.y, rows = gridDim.y, threads = blockDim.x;
    const int t0 = layer_tile0[l], t1 = layer_tile0[l + 1];
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = threadIdx.x / GRAWA_WAVE, waves = threads / GRAWA_WAVE;
    const auto step = [&](int k, double tot) {
        const double norm = sqrt(tot);
        mvg[(int64_t)k * L + l] = gamma * mvg[(int64_t)k * L + l] + (1.0 - gamma) * norm;
        if (flags && !isfinite(norm)) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
    };
    if (t1 - t0 <= wave_tiles || K > 4 * rows) {
        // The sums first, then every worker's update by a thread of its own, side by side.
        int n = wave;
        for (int k = y * waves + wave; k < K; k += rows * waves, n += waves) {
            const double tot = wave_strided_sum(partials + (int64_t)k * n_tiles, t0, t1, lane, GRAWA_WAVE);
            if (lane == 0) sm[n] = tot;
        }
        __syncthreads();
        for (int j = threadIdx.x; j < K; j += threads) {
            const int k = (j / waves * rows + y) * waves + j % waves;
            if (k < K) step(k, sm[j]);
        }
    } else {
        for (int k = y; k < K; k += rows) {
            const double *p = partials + (int64_t)k * n_tiles;
            double s[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) s[u] = 0.0;
            int t = t0 + (int)threadIdx.x;
            for (; t + 7 * threads < t1; t += 8 * threads)
#pragma unroll
                for (int u = 0; u < 8; ++u) s[u] += p[t + u * threads];
            for (; t < t1; t += threads) s[0] += p[t];
            const double part = wave_sum(((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7])));
            __syncthreads(); // the last worker's sums have been read
            if (lane == 0) sm[wave] = part;
            __syncthreads();
            if (threadIdx.x == 0) {
                double tot = 0.0;
                for (int i = 0; i < waves; ++i) tot += sm[i];
                step(k, tot);
            }
        }
    }
    if (y == 0 && threadIdx.x == 0) local_t[l] += 1;
}

// Weights from the running norm estimate g_est = gamma g_mvg / (1 - gamma^t) (Appendix G), t =
// the device-side count of local steps since the last communication, and then g_mvg <- 0, t <- 0.
// per_layer: grid L, block l normalises column l over the workers (eq. (7)); otherwise grid 1: score of worker k
// is the sum of its layer estimates (eq. (3) applied to the estimates), then eq. (4).  est_user (float
// [K][L], may be null) receives g_est.  With t = 0 (no step was counted) the estimates are taken
// as zero, which the zero-norm rule turns into the plain average.
// Every layer has a count t of its own (all equal), so that the block that reads one also resets it and no block
// needs to know of the others: one count for all needs the blocks to arrive at a counter, which from some thousand layers
// on takes longer than the reset as a launch of its own.
// Block: 256 per layer (starting the blocks is what takes the time), 1024 for the one of the model level, where a wave
// takes a worker at a time (256 threads there: 4 waves, 16 workers and 3000 layers of 300 k columns 108 us the step and
// the communication, with 1024 threads 64; the launch apart that reset the estimate before: 75).
#define GRAWA_LW_BLOCK_LAYER 256
#define GRAWA_LW_BLOCK_MODEL 1024
__global__ __launch_bounds__(GRAWA_LW_BLOCK_MODEL) void k_local_weights(double *__restrict__ mvg, double gamma,
                                                                  int64_t *__restrict__ local_t, int K, int L,
                                                                  int per_layer, float *__restrict__ beta,
                                                                  float *__restrict__ beta_user,
                                                                  float *__restrict__ est_user,
                                                                  unsigned *__restrict__ flags)
{
    __shared__ double sA[GRAWA_MAX_WORKERS];
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = threadIdx.x / GRAWA_WAVE, waves = (int)blockDim.x / GRAWA_WAVE;
    const int l0 = per_layer ? (int)blockIdx.x : 0;
    const int64_t t = local_t[l0];
    const double scale = t > 0 ? gamma / grawa_one_minus_power(gamma, t) : 0.0;
    if (per_layer) {
        for (int k = threadIdx.x; k < K; k += blockDim.x) {
            const int64_t at = (int64_t)k * L + l0;
            const double e = scale * mvg[at];
            sA[k] = e;
            if (est_user) est_user[at] = (float)e;
            mvg[at] = 0.0;
        }
        __syncthreads(); // also: every thread has read t
        if (threadIdx.x == 0) local_t[l0] = 0;
        if (wave == 0)
            group_weights(sA, K, beta + l0, L, beta_user ? beta_user + l0 : nullptr, flags, GRAWA_NONFINITE_LAYER_SCORE);
    } else {
        for (int k = wave; k < K; k += waves) {
            double *row = mvg + (int64_t)k * L;
            float *est = est_user ? est_user + (int64_t)k * L : nullptr;
            double s = 0.0;
            const auto take = [&](int l, double v) {
                const double e = scale * v;
                s += e;
                if (est) est[l] = (float)e;
                row[l] = 0.0;
            };
            int l = lane;
            for (; l + 3 * GRAWA_WAVE < L; l += 4 * GRAWA_WAVE) { // four loads in flight: none may pass the stores
                const double v0 = row[l], v1 = row[l + GRAWA_WAVE], v2 = row[l + 2 * GRAWA_WAVE], v3 = row[l + 3 * GRAWA_WAVE];
                take(l, v0);
                take(l + GRAWA_WAVE, v1);
                take(l + 2 * GRAWA_WAVE, v2);
                take(l + 3 * GRAWA_WAVE, v3);
            }
            for (; l < L; l += GRAWA_WAVE) take(l, row[l]);
            s = wave_sum(s);
            if (lane == 0) sA[k] = s;
        }
        __syncthreads(); // also: every thread has read t
        for (int l = threadIdx.x; l < L; l += blockDim.x) local_t[l] = 0;
        if (wave == 0) group_weights(sA, K, beta, 1, beta_user, flags, GRAWA_NONFINITE_MODEL_SCORE);
    }
}

// The same where the last step's sums may not be folded in yet (grawa_fold.h).  per_layer: grid L, and what is pending is folded in on the way: by a
// thread per worker, a wave per worker in turn, or, for a layer of more than GRAWA_FOLD_WAVE_TILES tiles, all waves for the workers' parts, N
// parts of a worker side by side (each what a wave of block_tile_sum adds, so that the sum is the same; two side by side take 5.9 us for 8
// workers and 586 tiles, four 5.0), as long as grawa_fold_in_weights; beyond, k_fold goes before.  Model level: grid 1, from the packed table that
// k_fold, or here (fold_here) the block itself, writes: 32 bytes an estimate, read by one block one after the other, made a round of one step of
// 8 workers and 2000 layers 54 us, now 39.  A thread's first estimate brings the counts too, instead of a load before it (4 workers, 2000 layers 26.6 ->
// 25.7, 16 workers, 1000 32.0 -> 31.7).
__global__ __launch_bounds__(GRAWA_FIN_BLOCK) void k_fold_weights(const GrawaFold f, const double *__restrict__ sums, int64_t n_tiles,
                                                                   int per_layer, int fold_here, uint64_t *__restrict__ consumed,
                                                                   float *__restrict__ beta, float *__restrict__ beta_user,
                                                                   float *__restrict__ est_user)
{
    constexpr int PARTS = GRAWA_FOLD_LANES / GRAWA_WAVE, N = 4;
    __shared__ double sA[GRAWA_MAX_WORKERS];
    __shared__ double part[GRAWA_FOLD_LONG_WORKERS * PARTS];
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / GRAWA_WAVE)), waves = (int)blockDim.x / GRAWA_WAVE;
    const int l0 = per_layer ? (int)blockIdx.x : 0;
    const int K = f.K, L = f.L;
    const GrawaEstimate mine = f.est[(int64_t)((int)threadIdx.x < K ? threadIdx.x : 0) * L + l0];
    const auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    GrawaEstimate e0 = {}; // counts and buffer: the same for all workers and layers
    e0.n = (uint64_t)uniform((uint32_t)(mine.n >> 32)) << 32 | uniform((uint32_t)mine.n);
    e0.buffer = uniform(mine.buffer);
    e0.left = uniform(mine.left);
    const uint64_t n = e0.n, used = grawa_last_used(consumed[l0], consumed[L + l0]);
    if (per_layer) {
        const bool pending = grawa_estimate_pending(e0, used);
        const int t0 = f.layer_tile0[l0], t1 = f.layer_tile0[l0 + 1], tiles = t1 - t0;
        const double *p = sums + e0.buffer * f.pitch;
        if (pending && tiles > GRAWA_FOLD_WAVE_TILES) { // grawa_fold_in_weights
            for (int j = N * wave; j < K * PARTS; j += N * waves) {
                const double *row = p + (int64_t)(j / PARTS) * n_tiles;
                const int first = t0 + (j % PARTS) * GRAWA_WAVE + lane;
                double w[N], half[2][N];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    double s[N][4];
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int h = 0; h < N; ++h) {
                            const int at = first + h * GRAWA_WAVE + (4 * u + v) * GRAWA_FOLD_LANES;
                            s[h][v] = at < t1 ? row[at] : 0.0;
                        }
#pragma unroll
                    for (int h = 0; h < N; ++h) half[u][h] = (s[h][0] + s[h][1]) + (s[h][2] + s[h][3]);
                }
#pragma unroll
                for (int h = 0; h < N; ++h) w[h] = half[0][h] + half[1][h];
                wave_sums<N>(w);
#pragma unroll
                for (int h = 0; h < N; ++h)
                    if (lane == 0) part[j + h] = w[h];
            }
            __syncthreads();
            if ((int)threadIdx.x < K) { // in the order of block_tile_sum
                double tot = 0.0;
                for (int w = 0; w < PARTS; ++w) tot += part[threadIdx.x * PARTS + w];
                sA[threadIdx.x] = tot;
            }
        } else if (pending && tiles > 16) {
            for (int k = wave; k < K; k += waves) {
                const double s = wave_strided_sum(p + (int64_t)k * n_tiles, t0, t1, lane, GRAWA_WAVE);
                if (lane == 0) sA[k] = s;
            }
        }
        const double scale = n != used ? f.gamma / grawa_one_minus_power(f.gamma, (int64_t)(n - used)) : 0.0;
        __syncthreads(); // also: every thread has read `used`
        if (threadIdx.x == 0) consumed[l0] = n;
        for (int k = (int)threadIdx.x; k < K; k += (int)blockDim.x) {
            double s = 0.0;
            if (pending) s = tiles <= 4    ? few_tiles_sum<4>(p + (int64_t)k * n_tiles, t0, t1)
                             : tiles <= 16 ? few_tiles_sum<16>(p + (int64_t)k * n_tiles, t0, t1)
                                           : sA[k];
            e0.mvg = k == (int)threadIdx.x ? mine.mvg : f.est[(int64_t)k * L + l0].mvg;
            e0.gamma = mine.gamma;
            const double v = scale * grawa_estimate_value(e0, used, sqrt(s));
            sA[k] = v;
            if (est_user) est_user[(int64_t)k * L + l0] = (float)v;
        }
        __syncthreads();
        if (wave == 0)
            group_weights(sA, K, beta + l0, L, beta_user ? beta_user + l0 : nullptr, f.flags, GRAWA_NONFINITE_LAYER_SCORE);
    } else {
        if (fold_here) { // a thread for each worker and layer; the longer ones of a wave by all of it, one after the other
            const unsigned units = (unsigned)K * (unsigned)L;
            const int few = (int)grawa_thread_tiles(f.lanes);
            for (unsigned base = 0; base < units; base += blockDim.x) {
                const unsigned u = base + lane * waves + wave, k = u / (unsigned)L, l = u - k * (unsigned)L;
                GrawaEstimate e = {};
                int t0 = 0, t1 = 0;
                if (u < units) {
                    e = f.est[u];
                    t0 = f.layer_tile0[l];
                    t1 = f.layer_tile0[l + 1];
                }
                const double *p = sums + e0.buffer * f.pitch;
                const bool pending = u < units && grawa_estimate_pending(e, used);
                double s = 0.0;
                if (pending && t1 - t0 <= few) s = few_tiles_sum<16>(p + (int64_t)k * n_tiles, t0, t1);
                for (unsigned long long todo = __ballot(pending && t1 - t0 > few); todo; todo &= todo - 1) {
                    const int j = __builtin_ctzll(todo), a = __builtin_amdgcn_readlane(t0, j), b = __builtin_amdgcn_readlane(t1, j);
                    const double tot = wave_strided_sum(p + (int64_t)__builtin_amdgcn_readlane((int)k, j) * n_tiles, lane < f.lanes ? a : b, b, lane, f.lanes);
                    if (lane == j) s = tot;
                }
                if (u < units) f.value[u] = grawa_estimate_value(e, used, sqrt(s));
            }
            __syncthreads();
        }
        const double scale = n != used ? f.gamma / grawa_one_minus_power(f.gamma, (int64_t)(n - used)) : 0.0;
        for (int k = wave; k < K; k += waves) {
            const double *row = f.value + (int64_t)k * L;
            float *est = est_user ? est_user + (int64_t)k * L : nullptr;
            double s = 0.0;
            const auto take = [&](int l, double value) {
                const double v = scale * value;
                s += v;
                if (est) est[l] = (float)v;
            };
            int l = lane;
            for (; l + 3 * GRAWA_WAVE < L; l += 4 * GRAWA_WAVE) { // four loads in flight: none may pass the stores
                const double v0 = row[l], v1 = row[l + GRAWA_WAVE], v2 = row[l + 2 * GRAWA_WAVE], v3 = row[l + 3 * GRAWA_WAVE];
                take(l, v0);
                take(l + GRAWA_WAVE, v1);
                take(l + 2 * GRAWA_WAVE, v2);
                take(l + 3 * GRAWA_WAVE, v3);
            }
            for (; l < L; l += GRAWA_WAVE) take(l, row[l]);
            s = wave_sum(s);
            if (lane == 0) sA[k] = s;
        }
        __syncthreads(); // also: every thread has read `used`
        for (int l = threadIdx.x; l < L; l += blockDim.x) consumed[l] = n;
        if (wave == 0) group_weights(sA, K, beta, 1, beta_user, f.flags, GRAWA_NONFINITE_MODEL_SCORE);
    }
}

// The estimates up to the last step, in a launch of its own; FOLD_SUMS: of a recorded step.
template <int THREADS, int MODE>
__global__ __launch_bounds__(THREADS) void k_fold(const GrawaFold f, const double *__restrict__ sums, int64_t n_tiles)
{
    fold_all<THREADS, MODE>(f, sums, n_tiles, blockIdx.x, gridDim.x);
}

// An explicit reset: everything so far is used up.
__global__ __launch_bounds__(GRAWA_BLOCK) void k_fold_reset(const GrawaEstimate *__restrict__ est, int L, uint64_t *__restrict__ consumed)
{
    const int l = blockIdx.x * GRAWA_BLOCK + threadIdx.x;
    if (l < L) consumed[l] = est[l].n;
}

// g_mvg <- 0 and t <- 0 (an explicit reset).
__global__ __launch_bounds__(GRAWA_BLOCK) void k_zero_estimate(double *__restrict__ p, int64_t n,
                                                               int64_t *__restrict__ local_t, int L)
{
    const int64_t i = (int64_t)blockIdx.x * GRAWA_BLOCK + threadIdx.x;
    if (i < n) p[i] = 0.0;
    if (i < L) local_t[i] = 0;
}

// flag word <- 0
__global__ void k_clear_flags(unsigned *__restrict__ flags)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *flags = 0u;
}

// Weights of the LSGD center (Appendix F), written where the pull kernel reads its model-level
// weights: 1 for the worker with the smallest loss (the first one on ties), 0 for the rest; its index goes to
// leader_out when given.  A NaN loss never leads, except that worker 0 leads when its own loss is NaN (the rule
// of a scan that starts at worker 0 and moves on strictly smaller losses).  One wave.  Up to 8 workers every lane scans
// them all, with all loads in flight; beyond, a lane scans the workers lane, lane + 64, ..., then as many lanes as hold
// workers are combined.  On the device, with the pull of 20 k columns, us, one thread / lanes combined / this: 1 worker
// 3.5 / 3.9 / 3.5, 4 3.7 / 4.0 / 3.7, 8 4.2 / 4.3 / 3.6, 16 5.1 / 4.6 / 4.5.
#define GRAWA_LEADER_SCAN 8
__global__ __launch_bounds__(GRAWA_WAVE) void k_leader_weights(const float *__restrict__ loss, int K,
                                                              float *__restrict__ beta, int *__restrict__ leader_out)
{
    const int lane = threadIdx.x;
    int best;
    if (K <= GRAWA_LEADER_SCAN) {
        float v[GRAWA_LEADER_SCAN];
#pragma unroll
        for (int k = 0; k < GRAWA_LEADER_SCAN; ++k) v[k] = loss[k < K ? k : 0];
        float low = v[0];
        best = 0;
#pragma unroll
        for (int k = 1; k < GRAWA_LEADER_SCAN; ++k)
            if (k < K && v[k] < low) {
                low = v[k];
                best = k;
            }
    } else {
        const float first = loss[0];
        float low = INFINITY;
        best = K;
        for (int k = lane; k < K; k += GRAWA_WAVE) {
            const float v = loss[k];
            if (v < low || (v == low && best == K)) { // the second: a loss of +inf may still lead
                low = v;
                best = k;
            }
        }
        for (int m = 1; m < GRAWA_WAVE && m < K; m <<= 1) { // lanes from K on hold nothing
            const float v = __shfl_xor(low, m, GRAWA_WAVE);
            const int k = __shfl_xor(best, m, GRAWA_WAVE);
            if (k < K && (best == K || v < low || (v == low && k < best))) {
                low = v;
                best = k;
            }
        }
        if (best == K || !(first == first)) best = 0;
    }
    if (lane == 0 && leader_out) *leader_out = best;
    for (int k = lane; k < K; k += GRAWA_WAVE) beta[k] = k == best ? 1.f : 0.f;
}

// ---------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------

// Kernels that are timed carry their own start/stop events (taken from the dispatch itself,
// so nothing extra is queued on the stream); both may be null.
hipError_t grawa_launch_sumsq(const grawa_plan *p, const void *g, int64_t ldg, grawa_dtype_t dt, int64_t cached_cols,
                              hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    const dim3 grid((unsigned)p->n_tiles, (unsigned)p->K), block(GRAWA_BLOCK);
    if (p->tile_shift) {
        if (dt == GRAWA_BF16)
            k_sumsq_slots<uint16_t><<<grid, block, 0, s>>>((const uint16_t *)g, ldg, p->d_off, p->L, p->P, p->tile_shift, p->n_tiles,
                                                           p->d_partials);
        else
            k_sumsq_slots<float><<<grid, block, 0, s>>>((const float *)g, ldg, p->d_off, p->L, p->P, p->tile_shift, p->n_tiles,
                                                        p->d_partials);
        return hipGetLastError();
    }
#define GRAWA_SUMSQ_GO(GT, MIX)                                                                              \
    hipExtLaunchKernelGGL((k_sumsq<GT, MIX>), grid, block, 0, s, e0, e1, 0, (const GT *)g, ldg,              \
                          (const GrawaTile *)p->d_tiles, p->n_tiles, p->d_partials, p->d_cnt_all, cached_cols)
    if (dt == GRAWA_BF16) {
        if (cached_cols) GRAWA_SUMSQ_GO(uint16_t, true);
        else GRAWA_SUMSQ_GO(uint16_t, false);
    } else {
        if (cached_cols) GRAWA_SUMSQ_GO(float, true);
        else GRAWA_SUMSQ_GO(float, false);
    }
#undef GRAWA_SUMSQ_GO
    return hipGetLastError();
}

hipError_t grawa_launch_finalize_layers(const grawa_plan *p, int goal, float *norms_user, float *beta_user,
                                        hipStream_t s)
{
    const bool model = goal >= GRAWA_GOAL_MODEL_SUM;
    const bool apart = model && !grawa_model_weights_by_last_block(p->L);
    float *beta = model ? p->d_beta_model : p->d_beta_layer;
    k_finalize_layers<<<dim3((unsigned)p->L), dim3(GRAWA_FIN_BLOCK), 0, s>>>(
        p->d_partials, p->n_tiles, p->d_layer_tile0, p->d_layer_tile1, p->K, p->L, goal, p->d_S, norms_user, beta,
        beta_user, apart ? nullptr : p->d_cnt_all, p->d_flags);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !apart) return e;
    k_finalize_model<<<dim3(1), dim3(GRAWA_FIN_BLOCK), 0, s>>>(p->d_S, p->K, p->L, goal, beta, beta_user, p->d_flags);
    return hipGetLastError();
}

hipError_t grawa_launch_estimate(const grawa_plan *p, double gamma, hipStream_t s)
{
    int rows, threads, wave_tiles;
    grawa_estimate_shape(p->K, p->L, p->max_rtiles, &rows, &threads, &wave_tiles);
    k_estimate<<<dim3((unsigned)p->L, (unsigned)rows), dim3((unsigned)threads), 0, s>>>(
        p->d_partials, p->n_rtiles, p->d_layer_rtile0, p->K, p->L, wave_tiles, p->d_mvg, gamma, p->d_local_t, p->d_flags);
    return hipGetLastError();
}

// step: a recorded step, whose sums are to be folded in; null: only what is pending.
hipError_t grawa_launch_fold(const grawa_plan *p, const GrawaFold *step, hipStream_t s)
{
    const GrawaFold f = step ? *step : grawa_fold_of(p, 0.0, 0, 0, 0);
    const unsigned units = (unsigned)p->K * (unsigned)p->L;
    const dim3 grid(f.by_wave ? (units + 3) / 4 : units), block(f.by_wave ? 256 : GRAWA_FOLD_LANES);
#define GRAWA_FOLD_GO(THREADS, MODE) k_fold<THREADS, MODE><<<grid, block, 0, s>>>(f, p->d_sums, p->n_rtiles)
    if (f.by_wave && step) GRAWA_FOLD_GO(256, GRAWA_FOLD_SUMS);
    else if (f.by_wave) GRAWA_FOLD_GO(256, GRAWA_FOLD_ONLY);
    else if (step) GRAWA_FOLD_GO(GRAWA_FOLD_LANES, GRAWA_FOLD_SUMS);
    else GRAWA_FOLD_GO(GRAWA_FOLD_LANES, GRAWA_FOLD_ONLY);
#undef GRAWA_FOLD_GO
    return hipGetLastError();
}

// Whether what is sent to the stream is recorded into a graph, and a number of the recording that is not 0.
bool grawa_is_recorded(hipStream_t s, unsigned long long *id)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    const hipError_t e = hipStreamGetCaptureInfo(s, &st, id);
    *id += 1;
    if (e == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError(); // the launch then fails as well
    return false;
}

hipError_t grawa_launch_local_weights(const grawa_plan *p, double gamma, int per_layer, float *beta_user,
                                      float *est_user, hipStream_t s)
{
    if (p->fold_later) {
        unsigned long long id = 0;
        const bool recorded = grawa_is_recorded(s, &id);
        const GrawaFold f = grawa_fold_of(p, gamma, 0, 0, 0);
        const bool folded = grawa_all_folded(p->steps, recorded, id);
        const bool here = !per_layer && !folded && grawa_fold_in_model_weights(p->K, p->L, p->max_rtiles, p->n_longer);
        const bool before = per_layer ? !grawa_fold_in_weights(p->K, p->max_rtiles) : !here;
        if (before && !folded) {
            const hipError_t e = grawa_launch_fold(p, nullptr, s);
            if (e != hipSuccess) return e;
        }
        const int want = !per_layer ? GRAWA_FIN_WAVES : p->max_rtiles <= 16 || before || folded ? 4 : f.by_wave ? p->K : 4 * p->K;
        const int waves = want < 4 ? 4 : want < GRAWA_FIN_WAVES ? want : GRAWA_FIN_WAVES;
        k_fold_weights<<<dim3(per_layer ? (unsigned)p->L : 1u), dim3(waves * GRAWA_WAVE), 0, s>>>(
            f, p->d_sums, p->n_rtiles, per_layer, here, p->d_consumed, per_layer ? p->d_beta_layer : p->d_beta_model, beta_user, est_user);
        return hipGetLastError();
    }
    k_local_weights<<<dim3(per_layer ? (unsigned)p->L : 1u), dim3(per_layer ? GRAWA_LW_BLOCK_LAYER : GRAWA_LW_BLOCK_MODEL), 0, s>>>(
        p->d_mvg, gamma, p->d_local_t, p->K, p->L, per_layer, per_layer ? p->d_beta_layer : p->d_beta_model,
        beta_user, est_user, p->d_flags);
    return hipGetLastError();
}

hipError_t grawa_launch_zero_estimate(const grawa_plan *p, hipStream_t s)
{
    if (p->fold_later) {
        k_fold_reset<<<dim3((unsigned)((p->L + GRAWA_BLOCK - 1) / GRAWA_BLOCK)), dim3(GRAWA_BLOCK), 0, s>>>(p->d_est, p->L, p->d_consumed);
        return hipGetLastError();
    }
    const int64_t n = (int64_t)p->K * p->L;
    k_zero_estimate<<<dim3((unsigned)((n + GRAWA_BLOCK - 1) / GRAWA_BLOCK)), dim3(GRAWA_BLOCK), 0, s>>>(p->d_mvg, n,
                                                                                                    p->d_local_t, p->L);
    return hipGetLastError();
}

hipError_t grawa_launch_clear_flags(const grawa_plan *p, hipStream_t s)
{
    k_clear_flags<<<dim3(1), dim3(GRAWA_WAVE), 0, s>>>(p->d_flags);
    return hipGetLastError();
}

hipError_t grawa_launch_leader_weights(const grawa_plan *p, const float *loss, int *leader_out, hipStream_t s)
{
    k_leader_weights<<<dim3(1), dim3(GRAWA_WAVE), 0, s>>>(loss, p->K, p->d_beta_model, leader_out);
    return hipGetLastError();
}
