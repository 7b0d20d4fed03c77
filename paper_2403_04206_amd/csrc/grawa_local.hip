// Local-phase kernels of the GRAWA training loop (gfx950, wave64):
//   k_row_step     x_k <- x_k - lr g_k                                            [Alg. 1, 2]
//                  (+ proximity step toward the stored center)                    [Alg. 1, 2, "Prox."]
//                  (+ per-tile sums of squares of the gradient, for the running
//                     norm estimate of Local-GRAWA)                               [App. G]
//   k_layer_step   the scored step of a small model, estimate included           [App. G]
//   k_nesterov     SGD with Nesterov momentum and weight decay                   [App. B.2.2]
//   k_stream_copy  plain copy (measurement aid)
// All are read-modify-write streams with no reuse: global loads and stores kept in flight, one
// row (worker) per block, which is the access shape that streams fastest on this part.
#include "grawa_fold.h"
#include "grawa_route.h"

// ---------------------------------------------------------------------------------
// local step, row by row
// ---------------------------------------------------------------------------------

#define GRAWA_ROW_BLOCK 1024 // columns per block
#define GRAWA_ROW_GROUP 4096 // column blocks of one row launched back to back (4 Mi columns)

// One block = one aligned block of 1024 columns of one worker; V * U * 256 = 1024, a lane handles U
// vectors of V adjacent columns.  All loads are issued at once, then
//     x <- x - lr g ;   PROX: x <- x + w (c - x), c the stored center, w = mu/tau ;
//     SCORE: partials[k][tile] = sum over the tile of g^2 in fp64, from the values in registers.
// grid (group, K, n_groups): the column blocks are cut into groups of gridDim.x; blocks are started
// with x fastest, so within a group the blocks of worker 0 come first, then worker 1, ..., and no
// index arithmetic is needed to find a block's place.  Blocks that run together therefore stream one
// row (the fastest shape: 6.4-6.6 TB/s against 5.2-6.0 for a block that owns all K rows of a
// tile), and the piece of the center a group needs (16 MB) is re-read by the other K-1 workers
// from cache instead of HBM.  With one group per row pass (k slowest) the center is re-read from
// HBM once it outgrows the last-level cache (measured 4.5 TB/s at P = 354 M); with k fastest the
// blocks in flight spread over all K rows (5.8-6.0).
// SCORE: only after its loads are issued does a block consult the 1024-column tile map (tiles
// block_tile0[m] .. block_tile0[m+1]-1 lie in aligned block m, each inside one layer).  Nearly
// every block holds one tile; in a block that contains layer boundaries every wave adds the tiles of its own columns (the block
// reducing once per tile, with two barriers each: 4 workers, ResNet-20's 59 tensors 6.1 us, now 5.4; one tile a block would take 4.3).
// The tile sums go to k_estimate, to k_fold or, GRAWA_SCORE_LATER, to the launch that needs them next (grawa_fold.h): a few blocks ahead of
// the others (grawa_fold_blocks) fold in those of the step before, a launch of 5 us that this one hides.  (Updating the estimate inside this launch, by the block that brings the last tile of a (worker, layer), was
// tried: its device-scope traffic costs more than the launch from about 1000 blocks or 30 tiles per layer on, 4 steps and
// the communication on 8 workers 117 us instead of 45.)  The maps are parameters of their own, each __restrict__: as
// members of a struct they may alias the stores, and a block with many tiles then reads them by vector loads that wait for
// its stores (64 workers, 300 k columns, 5000 layers: this kernel 141 us for 114).
// The last P % V columns of a row are handled element by element.
template <typename GT, int V, int U, bool LNT, int ST, bool PROX, int SCORE>
__global__ __launch_bounds__(GRAWA_CELL) __attribute__((amdgpu_waves_per_eu(1, PROX && !SCORE ? 7 : 8))) void k_row_step(float *__restrict__ x, int64_t ldx,
                                                         const GT *__restrict__ g, int64_t ldg, float lr,
                                                         const float *__restrict__ center, float w, int64_t P,
                                                         unsigned n_blocks,
                                                         const GrawaTile *__restrict__ tiles,
                                                         const int32_t *__restrict__ block_tile0, int64_t n_tiles,
                                                         double *__restrict__ partials, const GrawaFold fold)
{
    static_assert(V * U * GRAWA_CELL == GRAWA_ROW_BLOCK, "one trip covers one aligned block of columns");
    typedef typename FloatVec<V>::T XV;
    unsigned k = blockIdx.y;
    unsigned m = blockIdx.z * gridDim.x + blockIdx.x;
    if constexpr (SCORE == GRAWA_SCORE_LATER) {
        if (blockIdx.x < fold.blocks || k < fold.rows) { // these fold in the sums of the step before
            const unsigned width = fold.rows ? gridDim.x : fold.blocks, height = fold.rows ? fold.rows : gridDim.y;
            fold_all<GRAWA_CELL, GRAWA_FOLD_STEP>(fold, partials, n_tiles, (blockIdx.z * height + k) * width + blockIdx.x,
                                                  gridDim.z * height * width);
            return;
        }
        m = blockIdx.z * (gridDim.x - fold.blocks) + blockIdx.x - fold.blocks;
        k -= fold.rows;
    }
    if (m >= n_blocks) return; // the last group may be short (whole block leaves, before any barrier)
    const int64_t c0 = (int64_t)m * GRAWA_ROW_BLOCK + (int64_t)threadIdx.x * V;
    float *xr = x + (int64_t)k * ldx;
    const GT *gr = g + (int64_t)k * ldg;
    XV xv[U], cv[U];
    float gf[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + (int64_t)u * (GRAWA_CELL * V);
        if (c + V <= P) {
            const XV *xp = reinterpret_cast<const XV *>(xr + c);
            xv[u] = LNT ? __builtin_nontemporal_load(xp) : *xp;
            GradVec<GT, V, LNT>::load(gr + c, gf[u]);
            if (PROX) cv[u] = *reinterpret_cast<const XV *>(center + c); // cached: shared by the K rows
        } else {
#pragma unroll
            for (int e = 0; e < V; ++e) gf[u][e] = 0.f;
        }
    }
    int r0 = 0, r1 = 1;
    if (SCORE) {
        r0 = block_tile0[m];
        r1 = block_tile0[m + 1];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = c0 + (int64_t)u * (GRAWA_CELL * V);
        if (c + V <= P) {
            XV o = xv[u];
#pragma unroll
            for (int e = 0; e < V; ++e) {
                float v = fmaf(-lr, gf[u][e], vec_get<V>(xv[u], e));
                if (PROX) v = fmaf(w, vec_get<V>(cv[u], e) - v, v);
                vec_set<V>(o, e, v);
            }
            if (ST)
                st_lane<ST, XV>(uniform_base(xr + (int64_t)m * GRAWA_ROW_BLOCK), (threadIdx.x + u * GRAWA_CELL) * (V * 4u), o);
            else
                *reinterpret_cast<XV *>(xr + c) = o;
        } else if (V > 1 && c < P) { // the vector that holds the row's last columns
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (c + e < P) {
                    gf[u][e] = Grad<GT>::one(gr + c + e);
                    float v = fmaf(-lr, gf[u][e], xr[c + e]);
                    if (PROX) v = fmaf(w, center[c + e] - v, v);
                    xr[c + e] = v;
                }
        }
    }
    if constexpr (SCORE) {
        static_assert(V == 4 && U == 1, "a wave holds 256 adjacent columns");
        __shared__ double sm[GRAWA_BLOCK / GRAWA_WAVE];
        double *out = partials + (int64_t)k * n_tiles;
        out += fold.buffer * fold.pitch;
        const auto put = [&](int t, double tot) {
            out[t] = tot;
            if (fold.flags && !isfinite(tot)) atomicOr(fold.flags, GRAWA_NONFINITE_LAYER_SCORE); // null: k_estimate looks
        };
        if (r1 - r0 == 1) { // the usual case: the whole block lies in one tile
            double acc = 0.0; // squares and sums in fp64: exact squares at any gradient magnitude
#pragma unroll
            for (int e = 0; e < V; ++e) acc = sq_add(gf[0][e], acc);
            const double tot = block_sum<GRAWA_BLOCK>(acc, sm);
            if (threadIdx.x == 0) put(r0, tot);
        } else {
            // Every wave adds the tiles of its own 256 columns; the sums of a tile that goes on in other waves are added
            // in wave order.
            __shared__ double tail[GRAWA_BLOCK / GRAWA_WAVE];
            __shared__ int head_tile[GRAWA_BLOCK / GRAWA_WAVE], tail_tile[GRAWA_BLOCK / GRAWA_WAVE];
            const int lane = threadIdx.x & (GRAWA_WAVE - 1);
            const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / GRAWA_WAVE));
            const int begin = wave * (GRAWA_WAVE * V), end = begin + GRAWA_WAVE * V, at = threadIdx.x * V; // in the block
            int head_at = -1, tail_at = -1;
            for (int t = r0; t < r1; t += GRAWA_WAVE) {
                int lo = GRAWA_ROW_BLOCK, hi = lo;
                if (t + lane < r1) {
                    const GrawaTile tile = tiles[t + lane];
                    lo = (int)(tile.start - (int64_t)m * GRAWA_ROW_BLOCK);
                    hi = lo + tile.len;
                }
                constexpr int N = 2; // tiles whose sums go on together: a round of four steps 28.9 -> 28.0 us (ResNet-20, 4 workers); 4: 27.9, but with few layers 26.6 -> 27.4
                for (unsigned long long in = __ballot(lo < end && hi > begin); in;) {
                    double acc[N];
                    int id[N], from[N], to[N];
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        acc[j] = 0.0;
                        id[j] = in ? __builtin_ctzll(in) : -1;
                        in &= in - 1; // 0 stays 0
                        from[j] = id[j] < 0 ? 0 : __builtin_amdgcn_readlane(lo, id[j]);
                        to[j] = id[j] < 0 ? 0 : __builtin_amdgcn_readlane(hi, id[j]);
                    }
#pragma unroll
                    for (int e = 0; e < V; ++e)
#pragma unroll
                        for (int j = 0; j < N; ++j)
                            acc[j] = (at + e >= from[j] && at + e < to[j]) ? sq_add(gf[0][e], acc[j]) : acc[j];
                    if (id[N - 1] < 0) acc[0] = wave_sum(acc[0]);
                    else wave_sums<N>(acc);
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        if (id[j] < 0) continue;
                        if (from[j] < begin) {
                            head_at = t + id[j];
                            if (lane == 0) sm[wave] = acc[j];
                        } else if (to[j] > end) {
                            tail_at = t + id[j];
                            if (lane == 0) tail[wave] = acc[j];
                        } else if (lane == 0) {
                            put(t + id[j], acc[j]);
                        }
                    }
                }
            }
            if (lane == 0) {
                head_tile[wave] = head_at;
                tail_tile[wave] = tail_at;
            }
            __syncthreads();
            if (threadIdx.x < GRAWA_BLOCK / GRAWA_WAVE && tail_tile[threadIdx.x] >= 0) { // a tile that goes on begins in this wave
                const int t = tail_tile[threadIdx.x];
                double tot = tail[threadIdx.x];
#pragma unroll
                for (int w = 1; w < GRAWA_BLOCK / GRAWA_WAVE; ++w) // no tile begins before the block
                    if (w > (int)threadIdx.x && head_tile[w] == t) tot += sm[w];
                put(t, tot);
            }
        }
    }
}

// Scored step of a small model in one launch: a block owns a whole layer of one worker, so that the norm of its gradient, and
// with it the running estimate, need no second launch and no exchange between blocks.  grid (L, K), block 256; a lane handles
// vectors of 4 adjacent columns (rows are aligned to 16 bytes), U of them in flight at a time; a vector that the layer shares
// with a neighbour is handled element by element.  What bounds it is the longest layer, at the rate of one CU: so it serves where all
// layers are short (grawa_fold_later).  More vectors in flight cost registers and gain nothing: round of four steps and the
// communication, 4 workers, 270 k columns, U = 2 42.9 us, 3 43.5, 5 43.7, 10 56.
#define GRAWA_LAYER_U 2
#define GRAWA_LAYER_THREADS 256
template <typename GT, bool PROX>
__global__ __launch_bounds__(GRAWA_LAYER_THREADS) void k_layer_step(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr, const float *__restrict__ center, float w,
    const int64_t *__restrict__ off, int L, double *__restrict__ mvg, double gamma, int64_t *__restrict__ local_t,
    unsigned *__restrict__ flags)
{
    constexpr int V = 4, U = GRAWA_LAYER_U, T = GRAWA_LAYER_THREADS;
    typedef typename FloatVec<V>::T XV;
    const int l = blockIdx.x, k = blockIdx.y;
    const int64_t a = off[l], b = off[l + 1];
    const int64_t va = (a + V - 1) / V, vb = b / V; // whole vectors [va, vb), none where vb <= va
    float *xr = x + (int64_t)k * ldx;
    const GT *gr = g + (int64_t)k * ldg;
    const double before = threadIdx.x == 0 ? mvg[(int64_t)k * L + l] : 0.0;
    double acc = 0.0;
    const auto one = [&](int64_t c) {
        const float gv = Grad<GT>::one(gr + c);
        float v = fmaf(-lr, gv, xr[c]);
        if (PROX) v = fmaf(w, center[c] - v, v);
        xr[c] = v;
        acc = sq_add(gv, acc);
    };
    // The columns outside whole vectors: up to 3 at either end (a layer inside one vector: up to 3 in all).
    const int64_t head = vb > va ? va * V : b < va * V ? b : va * V, tail = vb > va ? vb * V : head;
    if (threadIdx.x < GRAWA_WAVE) {
        if (a + (int64_t)threadIdx.x < head) one(a + threadIdx.x);
        else if (threadIdx.x >= GRAWA_WAVE / 2 && tail + (int64_t)threadIdx.x - GRAWA_WAVE / 2 < b) one(tail + threadIdx.x - GRAWA_WAVE / 2);
    }
    for (int64_t v0 = va + threadIdx.x; v0 - (int64_t)threadIdx.x < vb; v0 += U * T) {
        XV xv[U], cv[U];
        float gf[U][V];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t v = v0 + u * T;
            if (v < vb) {
                xv[u] = *reinterpret_cast<const XV *>(xr + v * V);
                GradVec<GT, V, false>::load(gr + v * V, gf[u]);
                if (PROX) cv[u] = *reinterpret_cast<const XV *>(center + v * V);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t v = v0 + u * T;
            if (v < vb) {
                XV o = xv[u];
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    float t = fmaf(-lr, gf[u][e], vec_get<V>(xv[u], e));
                    if (PROX) t = fmaf(w, vec_get<V>(cv[u], e) - t, t);
                    vec_set<V>(o, e, t);
                    acc = sq_add(gf[u][e], acc);
                }
                *reinterpret_cast<XV *>(xr + v * V) = o;
            }
        }
    }
    __shared__ double sm[T / GRAWA_WAVE];
    const double tot = block_sum<T>(acc, sm);
    if (threadIdx.x == 0) {
        const double norm = sqrt(tot);
        mvg[(int64_t)k * L + l] = gamma * before + (1.0 - gamma) * norm;
        if (flags && !isfinite(norm)) atomicOr(flags, GRAWA_NONFINITE_LAYER_SCORE);
        if (k == 0) local_t[l] += 1;
    }
}

// ---------------------------------------------------------------------------------
// Nesterov-momentum SGD step
// ---------------------------------------------------------------------------------

// Vector shape of the Nesterov step: fp32 gradients V = 1, U = 4; bf16 V = 2, U = 2 (bf16 at V = 4, U = 4
// 5.6 TB/s: more bytes in flight per lane cost bandwidth at full occupancy, and 2-byte loads (V = 1) waste
// requests).  Waves per SIMD: bf16 6 (36.5 M columns x 8 workers 795 us; 5: 810, 7: 810, 8: 825), fp32 8 (889; 6: 914).
// Large rows off the cache-line grid: V = 4, streaming loads and stores that the L2 merges (GRAWA_ST_MERGE); with bf16 gradients
// up to 192 MB cached loads and stores written through, which find part of the arrays in the cache.  Three sets in turn, us:
// fp32 against cached accesses with V = 1, 140 MB 126 -> 119, 400 MB 361 -> 348, 1.5 GB 1367 -> 1335; bf16, the form up to 192 MB
// against the one beyond, 3 and 16 workers: 140 MB 100 / 106 and 93 / 103, 180 MB 136 / 137 and 130 / 134, 260 MB 208 / 200 and
// 201 / 194, 1.5 GB 1216 / 1163.  One set again and again, 3 and 16 workers: bf16 260 MB 191 / 200 and 189 / 197, fp32, against cached accesses,
// 500 MB 462 / 468 and 462 / 482 (three sets 468 / 468 and 464 / 463).
#define GRAWA_NAG_CACHED_LOADS_BYTES ((int64_t)192 << 20)
#define GRAWA_SGD_V_F32 1
#define GRAWA_SGD_U_F32 4
#define GRAWA_SGD_V_BF16 2
#define GRAWA_SGD_U_BF16 2

// grid (ceil(P / (256*U*V)), K), block 256; a lane handles U vectors of V adjacent columns, vectors of a
// block 256*V columns apart; the last P % V columns of a row take a scalar path.  One step of SGD with Nesterov momentum and weight decay
// (the local optimizer of Appendix B.2.2), buf = momentum buffer [K][ldb], zero before the first step:
//     d = g + wd x ;  buf <- momentum buf + d ;  x <- x - lr (d + momentum buf).
template <typename GT, int V, int U, bool LNT, int ST>
__global__ __launch_bounds__(GRAWA_CELL) __attribute__((amdgpu_waves_per_eu(1, sizeof(GT) == 2 ? 6 : 8))) void k_nesterov(float *__restrict__ x, int64_t ldx,
                                                         const GT *__restrict__ g, int64_t ldg,
                                                         float *__restrict__ buf, int64_t ldb, int64_t P,
                                                         float lr, float momentum, float wd)
{
    typedef typename FloatVec<V>::T XV;
    const int64_t nvec = P / V;
    const int64_t j0 = (int64_t)blockIdx.x * (GRAWA_CELL * U) + threadIdx.x;
    float *xr = x + (int64_t)blockIdx.y * ldx;
    float *br = buf + (int64_t)blockIdx.y * ldb;
    const GT *gr = g + (int64_t)blockIdx.y * ldg;
    XV xv[U], bv[U];
    float gf[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + u * GRAWA_CELL;
        if (j < nvec) {
            const XV *xp = reinterpret_cast<const XV *>(xr + j * V);
            const XV *bp = reinterpret_cast<const XV *>(br + j * V);
            xv[u] = LNT ? __builtin_nontemporal_load(xp) : *xp;
            bv[u] = LNT ? __builtin_nontemporal_load(bp) : *bp;
            GradVec<GT, V, LNT>::load(gr + j * V, gf[u]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t j = j0 + u * GRAWA_CELL;
        if (j < nvec) {
            XV xo = xv[u], bo = bv[u];
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const float xc = vec_get<V>(xv[u], c);
                const float d = fmaf(wd, xc, gf[u][c]);
                const float b = fmaf(momentum, vec_get<V>(bv[u], c), d);
                vec_set<V>(bo, c, b);
                vec_set<V>(xo, c, fmaf(-lr, fmaf(momentum, b, d), xc));
            }
            if (ST) {
                const int64_t c0 = (int64_t)blockIdx.x * (GRAWA_CELL * U * V);
                const unsigned o = (threadIdx.x + u * GRAWA_CELL) * (V * 4u);
                st_lane<ST, XV>(uniform_base(xr + c0), o, xo);
                st_lane<ST, XV>(uniform_base(br + c0), o, bo);
            } else {
                *reinterpret_cast<XV *>(xr + j * V) = xo;
                *reinterpret_cast<XV *>(br + j * V) = bo;
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x < (unsigned)(P - nvec * V)) {
        const int64_t i = nvec * V + threadIdx.x;
        const float xc = xr[i];
        const float d = fmaf(wd, xc, Grad<GT>::one(gr + i));
        const float b = fmaf(momentum, br[i], d);
        br[i] = b;
        xr[i] = fmaf(-lr, fmaf(momentum, b, d), xc);
    }
}

// ---------------------------------------------------------------------------------
// plain copy (measurement aid)
// ---------------------------------------------------------------------------------

// grid ceil(n/64), block 64 (one wave): one streaming 16-byte load and store per lane, the
// shape that measured fastest for a two-stream copy on this part.
#define GRAWA_COPY_BLOCK 64
__global__ __launch_bounds__(GRAWA_COPY_BLOCK) void k_stream_copy(v4u *__restrict__ dst,
                                                                  const v4u *__restrict__ src, int64_t n)
{
    const int64_t j = (int64_t)blockIdx.x * GRAWA_COPY_BLOCK + threadIdx.x;
    if (j < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + j), dst + j);
}

// ---------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------

// center == nullptr: no proximity step.  p == nullptr: no scores; otherwise the plan's 1024-column tile map and
// workspace take them.  Vector shapes: fp32 gradients V = 1, U = 4 for the plain step,
// V = 4, U = 1 with the proximity step or the scores; bf16 V = 2, U = 2 for the plain step, else
// V = 4, U = 1 (each the fastest measured for its case on arrays of random values; the spread
// between shapes is 3-10 %).
// Large rows off the cache-line grid (wide): 16-byte lanes, streaming loads, and stores that the L2 merges (GRAWA_ST_MERGE), up to some
// sizes cached loads and stores written through (grawa_row_step_merges_from).  Three sets of arrays in turn, us, these / those, rows 4 or
// 12 bytes off a line: with the center fp32 100 MB 58.7 -> 51.8, 200 MB 120 -> 103, 1.5 GB 879 -> 815; bf16, 3 and 16 workers, 200 MB
// 97.4 -> 89.8 and 99.4 -> 87.1, 1.5 GB 729 -> 705; scored step with the center and the communication fp32 70 MB 79.9 -> 72.8,
// 400 MB 378 -> 357, bf16 100 MB 97.7 -> 94.2 and 100.0 -> 93.1.
// The plain step only from 512 MB on: below, the pull that follows would lose the part of x a cached step leaves in the
// cache (step and LSGD phase, bf16, 3 and 16 workers: 300 MB 210 / 222 and 216 / 229, 520 MB 364 / 376 and 388 / 402, 800 MB
// 609 / 596 and 638 / 626).
static hipError_t launch_row_step(grawa_plan *p, float *x, int64_t ldx, const void *g, int64_t ldg,
                                  grawa_dtype_t dt, float lr, const float *center, float w, int K, int64_t P,
                                  double gamma, hipStream_t s)
{
    const int64_t nb = (P + GRAWA_ROW_BLOCK - 1) / GRAWA_ROW_BLOCK;
    const bool prox = center != nullptr;
    const bool later = p && p->fold_later;
    if (p && !later && grawa_step_by_layers(K, p->L, P, p->max_rtiles)) {
#define GRAWA_LS_GO(GT, PROX)                                                                                              \
    k_layer_step<GT, PROX><<<dim3((unsigned)p->L, (unsigned)K), dim3(GRAWA_LAYER_THREADS), 0, s>>>(                        \
        x, ldx, (const GT *)g, ldg, lr, center, w, p->d_off, p->L, p->d_mvg, gamma, p->d_local_t, p->d_flags)
        if (dt == GRAWA_BF16) {
            if (prox) GRAWA_LS_GO(uint16_t, true);
            else GRAWA_LS_GO(uint16_t, false);
        } else {
            if (prox) GRAWA_LS_GO(float, true);
            else GRAWA_LS_GO(float, false);
        }
#undef GRAWA_LS_GO
        return hipGetLastError();
    }
    // Nothing is shared between the rows without a center: one group, i.e. row after row (3 % faster).
    const int64_t group = (prox && nb > GRAWA_ROW_GROUP) ? GRAWA_ROW_GROUP : nb;
    const int64_t n_groups = (nb + group - 1) / group;
    if (K > 65535 || n_groups > 65535 || group >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
    unsigned long long id = 0;
    const bool recorded = later && grawa_is_recorded(s, &id);
    bool at_once = false;
    const unsigned buffer = later ? grawa_step_buffer(p->steps, recorded, id, &at_once) : 0;
    unsigned fold_blocks = 0, fold_rows = 0;
    if (later && !at_once) grawa_fold_blocks(K, p->L, p->max_rtiles, prox, group, n_groups, &fold_blocks, &fold_rows);
    GrawaFold fold = {}; // no flags either: k_estimate looks at the norms
    if (later) fold = grawa_fold_of(p, gamma, buffer, fold_blocks, fold_rows);
    const dim3 grid((unsigned)group + fold_blocks, (unsigned)K + fold_rows, (unsigned)n_groups), block(GRAWA_CELL);
    const bool aligned = rows_line_aligned(x, ldx, 4) && rows_line_aligned(g, ldg, dt == GRAWA_BF16 ? 2 : 4);
    const int64_t bytes = (int64_t)K * P * 4;
    const bool plain = !prox && !p;
    const bool nt = aligned && bytes > (plain ? GRAWA_STREAMING_MIN_SGD_BYTES : GRAWA_STREAMING_MIN_ROW_BYTES);
    const bool wide = !aligned && bytes > (plain ? 2 * GRAWA_STREAMING_MIN_SGD_BYTES : GRAWA_STREAMING_MIN_ROW_BYTES);
    const GrawaTile *tiles = p ? p->d_rtiles : nullptr;
    const int32_t *block_tile0 = p ? p->d_block_rtile0 : nullptr;
    double *partials = later ? p->d_sums : p ? p->d_partials : nullptr;
    const int64_t n_tiles = p ? p->n_rtiles : 0;
#define GRAWA_RS_GO(GT, V, U, LNT, ST, PROX, SCORE)                                                                    \
    k_row_step<GT, V, U, LNT, ST, PROX, SCORE><<<grid, block, 0, s>>>(x, ldx, (const GT *)g, ldg, lr, center, w, P, \
                                                                       (unsigned)nb, tiles, block_tile0, n_tiles,  \
                                                                       partials, fold)
#define GRAWA_RS_NT(GT, V, U, PROX, SCORE)                                                                            \
    do {                                                                                                              \
        constexpr int64_t FROM = grawa_row_step_merges_from(sizeof(GT) == 2, PROX, SCORE);                            \
        constexpr bool NEVER = FROM == GRAWA_ROW_STEP_NEVER, ALWAYS = FROM == 0;                                      \
        if (nt) GRAWA_RS_GO(GT, V, U, true, GRAWA_ST_STREAM, PROX, SCORE);                                            \
        else if (!wide) GRAWA_RS_GO(GT, V, U, false, GRAWA_ST_CACHED, PROX, SCORE);                                   \
        else if (bytes > FROM) GRAWA_RS_GO(GT, 4, 1, !NEVER, (NEVER ? GRAWA_ST_STREAM : GRAWA_ST_MERGE), PROX, SCORE); \
        else GRAWA_RS_GO(GT, 4, 1, ALWAYS, (ALWAYS ? GRAWA_ST_MERGE : GRAWA_ST_STREAM), PROX, SCORE);                 \
    } while (0)
    if (dt == GRAWA_BF16) {
        if (prox && later && !at_once) GRAWA_RS_NT(uint16_t, 4, 1, true, GRAWA_SCORE_LATER);
        else if (later && !at_once) GRAWA_RS_NT(uint16_t, 4, 1, false, GRAWA_SCORE_LATER);
        else if (prox && p) GRAWA_RS_NT(uint16_t, 4, 1, true, GRAWA_SCORE_SUMS);
        else if (prox) GRAWA_RS_NT(uint16_t, 4, 1, true, GRAWA_SCORE_NONE);
        else if (p) GRAWA_RS_NT(uint16_t, 4, 1, false, GRAWA_SCORE_SUMS);
        else GRAWA_RS_NT(uint16_t, 2, 2, false, GRAWA_SCORE_NONE);
    } else {
        if (prox && later && !at_once) GRAWA_RS_NT(float, 4, 1, true, GRAWA_SCORE_LATER);
        else if (later && !at_once) GRAWA_RS_NT(float, 4, 1, false, GRAWA_SCORE_LATER);
        else if (prox && p) GRAWA_RS_NT(float, 4, 1, true, GRAWA_SCORE_SUMS);
        else if (prox) GRAWA_RS_NT(float, 4, 1, true, GRAWA_SCORE_NONE);
        else if (p) GRAWA_RS_NT(float, 4, 1, false, GRAWA_SCORE_SUMS);
        else GRAWA_RS_NT(float, 1, 4, false, GRAWA_SCORE_NONE);
    }
#undef GRAWA_RS_NT
#undef GRAWA_RS_GO
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !p) return e;
    if (later) {
        grawa_step_sent(p->steps, recorded, id);
        return at_once ? grawa_launch_fold(p, &fold, s) : e;
    }
    return grawa_launch_estimate(p, gamma, s);
}

hipError_t grawa_launch_row_step(float *x, int64_t ldx, const void *g, int64_t ldg, grawa_dtype_t dt, float lr,
                                 const float *center, float w, int K, int64_t P, hipStream_t s)
{
    return launch_row_step(nullptr, x, ldx, g, ldg, dt, lr, center, w, K, P, 0.0, s);
}

hipError_t grawa_launch_row_step_scored(grawa_plan *p, float *x, int64_t ldx, const void *g, int64_t ldg,
                                        grawa_dtype_t dt, float lr, const float *center, float w, double gamma,
                                        hipStream_t s)
{
    return launch_row_step(p, x, ldx, g, ldg, dt, lr, center, w, p->K, p->P, gamma, s);
}

hipError_t grawa_launch_nesterov(float *x, int64_t ldx, const void *g, int64_t ldg, grawa_dtype_t dt, float *buf,
                                 int64_t ldb, int K, int64_t P, float lr, float momentum, float wd, hipStream_t s)
{
    const int64_t bytes = (int64_t)K * P * 4;
    const bool large = bytes > GRAWA_STREAMING_MIN_BYTES;
    const bool nt = large && rows_line_aligned(x, ldx, 4) && rows_line_aligned(buf, ldb, 4) &&
                    rows_line_aligned(g, ldg, dt == GRAWA_BF16 ? 2 : 4);
#define GRAWA_NAG_GO(GT, V, U, LNT, ST)                                                                          \
    k_nesterov<GT, V, U, LNT, ST><<<dim3((unsigned)((P + GRAWA_CELL * (U) * (V) - 1) / (GRAWA_CELL * (U) * (V))), \
                                         (unsigned)K), dim3(GRAWA_CELL), 0, s>>>(                               \
        x, ldx, (const GT *)g, ldg, buf, ldb, P, lr, momentum, wd)
    if (dt == GRAWA_BF16) {
        if (nt) GRAWA_NAG_GO(uint16_t, GRAWA_SGD_V_BF16, GRAWA_SGD_U_BF16, true, GRAWA_ST_STREAM);
        else if (large && bytes <= GRAWA_NAG_CACHED_LOADS_BYTES) GRAWA_NAG_GO(uint16_t, 4, 1, false, GRAWA_ST_STREAM);
        else if (large) GRAWA_NAG_GO(uint16_t, 4, 1, true, GRAWA_ST_MERGE);
        else GRAWA_NAG_GO(uint16_t, GRAWA_SGD_V_BF16, GRAWA_SGD_U_BF16, false, GRAWA_ST_CACHED);
    } else {
        if (nt) GRAWA_NAG_GO(float, GRAWA_SGD_V_F32, GRAWA_SGD_U_F32, true, GRAWA_ST_STREAM);
        else if (large) GRAWA_NAG_GO(float, 4, 1, true, GRAWA_ST_MERGE);
        else GRAWA_NAG_GO(float, GRAWA_SGD_V_F32, GRAWA_SGD_U_F32, false, GRAWA_ST_CACHED);
    }
#undef GRAWA_NAG_GO
    return hipGetLastError();
}

hipError_t grawa_launch_stream_copy(void *dst, const void *src, int64_t nbytes, hipStream_t s)
{
    const int64_t n = nbytes / 16;
    const int64_t gx = (n + GRAWA_COPY_BLOCK - 1) / GRAWA_COPY_BLOCK;
    if (gx > 0)
        k_stream_copy<<<dim3((unsigned)gx), dim3(GRAWA_COPY_BLOCK), 0, s>>>((v4u *)dst, (const v4u *)src, n);
    return hipGetLastError();
}
