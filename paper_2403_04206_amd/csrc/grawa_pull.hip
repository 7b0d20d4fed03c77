// Center and pull of the GRAWA update (gfx950, wave64):
//   x_C = sum_k beta_k x_k ;  x_k <- x_k + lambda (x_C - x_k)      [display after eq. (2); eq. (7)]
// with the local SGD step x_k - lr g_k optionally applied on the way in (Algorithms 1 and 2) and,
// for EASGD (Appendix F), the center averaged in time.
//
// A read-modify-write pass over K far-apart rows: it runs fastest when a wave touches one aligned
// 256-byte piece of every row (one 32-bit element per lane per row), blocks are small and many,
// and accesses are non-temporal -- provided every row starts on a 128-byte boundary, so that no
// cache line is written in two parts.  There is no dense contraction, hence no matrix-core code.
#include "grawa_fold.h"
#include "grawa_offsets.h"
#include "grawa_route.h"

// ---------------------------------------------------------------------------------
// center + pull (+ SGD on the way in)
// ---------------------------------------------------------------------------------

// Layer of column i, given a layer at or before it (cells that contain a layer boundary).
__device__ __forceinline__ int layer_of(const int64_t *__restrict__ off, int layer, int L, int64_t i)
{
    while (layer + 1 < L && off[layer + 1] <= i) ++layer;
    return layer;
}

// The layers of V adjacent columns from `col` on; the start of the next layer is loaded only where a column reaches it.
// Columns past the row get the layer of its last column (their weights are loaded and not used).
template <int V>
__device__ __forceinline__ void layers_of(const int64_t *__restrict__ off, int layer, int L, int64_t col, int64_t P,
                                          int (&layers)[V])
{
    int64_t next = layer + 1 < L ? off[layer + 1] : P;
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const int64_t i = col + e < P ? col + e : P - 1;
        while (layer + 1 < L && next <= i) {
            ++layer;
            next = layer + 1 < L ? off[layer + 1] : P;
        }
        layers[e] = layer;
    }
}

// Center of the V columns from `col` of a cell that holds layer boundaries, over R rows of v (rows for which has(k) is
// false excepted), weights beta[k * stride + layer].  c must be 0.  A cell of few layers goes through them one by one, the
// weights by scalar loads, and every column keeps the sum of its own layer; with more layers every column fetches its own
// weights, all of them loaded before one is used.  (Every column fetching its own, one after the other: pull of 4 rows of
// 10 M columns off the line grid, 3000 layers 52.6 -> 73.4 us against the one-column form, 100 000 layers 60.3 -> 129;
// now 58 and 69, which is what streaming a 160 MB array that was in the cache costs: 30 M columns 168 -> 166 and 198 -> 197.)  Lanes past the row take part and are not used.
#define GRAWA_FEW_LAYERS 8
template <int R, int V, bool FEW, typename Has>
__device__ __forceinline__ void center_by_layer(const float *beta, int64_t stride, const int64_t *__restrict__ off, int L,
                                                int64_t P, int64_t cell0, int first, int64_t col, const Has &has,
                                                const typename FloatVec<V>::T (&v)[R], typename FloatVec<V>::T &c)
{
    const int64_t end = cell0 + GRAWA_CELL < P ? cell0 + GRAWA_CELL : P;
    const int l0 = __builtin_amdgcn_readfirstlane(first);
    const __attribute__((address_space(4))) int64_t *starts = (const __attribute__((address_space(4))) int64_t *)uniform_base(off);
    if (FEW && (l0 + GRAWA_FEW_LAYERS >= L || starts[l0 + GRAWA_FEW_LAYERS] >= end)) {
        int64_t start = cell0;
        for (int l = l0;; ++l) {
            const uint64_t bb = uniform_base(beta + l);
            typename FloatVec<V>::T t = typename FloatVec<V>::T{};
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (has(k)) {
                    const float w = ld_uniform_f32(bb, (int64_t)k * stride);
#pragma unroll
                    for (int e = 0; e < V; ++e) vec_set<V>(t, e, fmaf(w, vec_get<V>(v[k], e), vec_get<V>(t, e)));
                }
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (col + e >= start) vec_set<V>(c, e, vec_get<V>(t, e));
            if (l + 1 >= L) break;
            start = starts[l + 1];
            if (start >= end) break;
        }
        return;
    }
    int layers[V];
    layers_of<V>(off, l0, L, col, P, layers);
    float w[R][V];
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int e = 0; e < V; ++e) w[k][e] = has(k) ? beta[(int64_t)k * stride + layers[e]] : 0.f;
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (has(k)) {
#pragma unroll
            for (int e = 0; e < V; ++e) vec_set<V>(c, e, fmaf(w[k][e], vec_get<V>(v[k], e), vec_get<V>(c, e)));
        }
}

// Per-layer weights straight from the tile sums of the norm pass, computed by every block for the layers of its own
// cell (TILES).  A small update is a chain of short launches, and this one drops a link: for 270 k parameters and
// 4 workers the weights as a launch of their own took 4.0 us plus the boundary.  The loads of x are in flight
// meanwhile.  The cell that a layer starts in writes its row of weights_out.
struct TileWeights {
    const double *partials;
    int64_t pitch;
    const int32_t *tile_begin, *tile_end; // [L]
    float *weights_out;                   // [K][L] or null
    unsigned *flags;
    int group;                            // lanes per worker: the largest power of two not above 64 / K
    int shift;                            // without the maps: tiles of 2^shift columns, found in the offsets
};

// The same from the running estimate (the communication of a local round): what a scored step left pending is folded in on
// the way.  Every block keeps the step that it has used everything up to (`seen`), since no block may write what another one of
// the launch reads; the cell that a layer starts in tells the other launches.
struct EstimateWeights : TileWeights { // partials: the buffers of sums
    const GrawaEstimate *est;
    const uint64_t *consumed;    // [2 L]
    uint64_t *consumed_by_pulls; // [L], the second half
    uint64_t *seen;              // [cells]
    float *est_out;              // [K][L] or null
    int64_t buffer;              // sums in one
    double gamma;
};
struct EstimateScore {
    typedef GrawaEstimate State;
    const EstimateWeights &w;
    int L;
    uint64_t n, used;
    double scale;
    __device__ __forceinline__ State load(int k, int l) const { return w.est[(int64_t)k * L + l]; }
    __device__ __forceinline__ double score(const State &e, double sum) const { return scale * grawa_estimate_value(e, used, sqrt(sum)); }
    __device__ __forceinline__ void publish(int k, int l, double a) const
    {
        if (k == 0) w.consumed_by_pulls[l] = n;
        if (w.est_out) w.est_out[(int64_t)k * L + l] = (float)a;
    }
};

template <int K> struct CellWeights {
    float beta[GRAWA_CELL * K]; // [layer of the cell][K]
    int start[GRAWA_CELL];      // first column of the layer, relative to the cell
};

// Fills `sh` for the cell at column cell0 whose first layer is l0; returns the number of layers.  Called by the whole
// block (4 waves); ends with a barrier.  The first and the last layer of the cell may have tiles in other cells, any
// number of them: a wave for each.  The layers between have all their columns in the cell, so one tile each (tiles are
// cut at multiples of at least 1024): a segment of lanes for each, a lane per worker, as long as that takes two rounds, else a
// lane for each, with the loads of its K workers in flight together.  (A lane's K roots and quotients, one after the other, are the longest
// chain of the launch.  Update, us, a lane for each / segments: ResNet-20, 59 layers, 8 workers 10.3 / 9.5, without maps and with the center
// 11.5 / 10.7; 15 workers, 170 k columns, 60 layers 13.5 / 11.6; 4 workers, 200 k, 150 layers 8.1 / 7.9.)  So a cell takes two rounds at most, for 3 layers as for 256 (a wave per layer in turn took 16 rounds, and lanes that walked
// all tiles of their layer more: 4 workers, 600 k columns, of which the first 60 or 100 are layers of their own, update on the
// device 24.6 and 174 us; with the weights as a launch 17.3 and 21.8; now 11.4 and 11.7).
template <int K, bool SLOTS, typename Score>
__device__ __forceinline__ int cell_weights(const TileWeights &w, const Score &scores, const double *partials,
                                            const int64_t *__restrict__ off, int L, int64_t P, int64_t cell0, int l0, bool boundary,
                                            CellWeights<K> &sh)
{
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / GRAWA_WAVE));
    int nl = 1;
    if (boundary) {
        const int64_t end = cell0 + GRAWA_CELL < P ? cell0 + GRAWA_CELL : P;
        for (int l = l0 + 1;; l += GRAWA_WAVE) {
            const unsigned long long in = __ballot(l + lane < L && off[l + lane] < end);
            nl += __popcll(in);
            if (in != ~0ull) break;
        }
        if (nl > GRAWA_CELL) nl = GRAWA_CELL; // only with offsets that break the rules
        if ((int)threadIdx.x < nl) sh.start[threadIdx.x] = threadIdx.x ? (int)(off[l0 + (int)threadIdx.x] - cell0) : 0;
    }
    if (wave == 0 || (wave == 1 && nl > 1)) {
        const int i = wave == 0 ? 0 : nl - 1, l = l0 + i;
        int t0, t1;
        if constexpr (SLOTS) layer_slots(off, l, P, w.shift, t0, t1);
        else t0 = w.tile_begin[l], t1 = w.tile_end[l];
        wave_layer_weights(scores, l, partials, w.pitch, t0, t1, K, w.group, sh.beta + i * K,
                           off[l] >= cell0, w.weights_out ? w.weights_out + l : nullptr, L, w.flags);
    } else if (wave >= 2) {
        const auto at = [&](int i, bool segment, bool here) {
            const int l = l0 + i;
            int t0, t1;
            if constexpr (SLOTS) layer_slots(off, l, P, w.shift, t0, t1);
            else t0 = w.tile_begin[l], t1 = w.tile_end[l];
            float *out = sh.beta + i * K, *user = w.weights_out ? w.weights_out + l : nullptr;
            if (segment) segment_layer_weights<K>(scores, l, here, partials, w.pitch, t0, t1, out, user, L, w.flags);
            else lane_layer_weights<K>(scores, l, partials, w.pitch, t0, t1, out, user, L, w.flags);
        };
        constexpr int G = Segment<K>::G, ROUND = 2 * (GRAWA_WAVE / G); // layers that two waves take at a time
        const int lane2 = (int)threadIdx.x - 2 * GRAWA_WAVE;
        if (nl - 2 <= 2 * ROUND) {
            for (int base = 1; base < nl - 1; base += ROUND) {
                const int i = base + lane2 / G;
                at(i < nl - 1 ? i : 1, true, i < nl - 1);
            }
        } else {
            for (int i = 1 + lane2; i < nl - 1; i += GRAWA_CELL - 2 * GRAWA_WAVE) at(i, false, true);
        }
    }
    __syncthreads();
    return nl;
}

// Which of the nl layers of the cell column `col` (relative to the cell) lies in.
template <int K> __device__ __forceinline__ int cell_layer_of(const CellWeights<K> &sh, int nl, int col)
{
    int i = 0;
    for (int step = nl > 1 ? 1 << (31 - __builtin_clz(nl - 1)) : 0; step; step >>= 1)
        if (i + step < nl && sh.start[i + step] <= col) i += step;
    return i;
}

// Plain form, K <= 23 (16 without the SGD step excepted), on few cells to 32 (grawa_plain_form).  grid ceil(P/256), block 256: a lane owns one
// column.  It loads x[k][i] for its K workers (all loads in flight together; with SGD also g[k][i] and
// applies x - lr g), forms c = sum_k beta_k x_k and writes x_k + lambda (c - x_k) back, so every
// parameter is read once and written once.  A wave touches one 256-byte piece per row.
// NT = streaming loads/stores, chosen by the host only when every row
// starts on a 128-byte boundary.  Row bases are wave-uniform, the lane adds only its index.
// cell_layer[j] describes the 256-column cell j: >= 0: the whole cell lies in that layer (weights
// come through scalar loads); < 0: the cell contains a layer boundary, ~cell_layer[j] is the layer of
// its first column and each lane finds its own layer.  Model-level weights pass cell_layer = nullptr.
// The pull is x + lambda (c - x), one fma, which leaves a single worker exactly unchanged.
// moving != 0 (EASGD, Appendix F): center_out holds the previous center c0 on entry and the
// center used and stored is c0 + rho (c - c0).
// WPE caps the waves per SIMD (grawa_waves_for; cached accesses: launch_plain): more only queues requests to K far-apart rows and costs DRAM
// efficiency (measured: K = 16 at 3 waves 6.1 TB/s, at 8 waves 5.7; K = 8 at 4 waves 6.5, at 8 waves 6.2).
// TILES: weights from the tile sums, by the maps of a plan or found in the offsets (GRAWA_TILES_SLOTS), or from the running estimate.
enum { GRAWA_TILES_NONE = 0, GRAWA_TILES_MAPS = 1, GRAWA_TILES_SLOTS = 2, GRAWA_TILES_ESTIMATE = 3 };
template <int TILES> struct WeightsOf { typedef TileWeights T; };
template <> struct WeightsOf<GRAWA_TILES_ESTIMATE> { typedef EstimateWeights T; };
template <int K, bool SGD, typename GT, bool NT, int WPE, int TILES>
__global__ __launch_bounds__(GRAWA_CELL) __attribute__((amdgpu_waves_per_eu(1, WPE))) void k_center_pull(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving, const typename WeightsOf<TILES>::T tw)
{
    const int64_t cell0 = (int64_t)blockIdx.x * GRAWA_CELL; // wave-uniform
    const unsigned col = threadIdx.x;
    const bool ok = cell0 + col < P;
    float *xb = x + cell0;
    const GT *gb = g + cell0;
    const unsigned xoff = col * 4u, goff = col * (unsigned)sizeof(GT);

    float v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = 0.f;
    if (ok) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = ld_lane<NT, float>(uniform_base(xb + (int64_t)k * ldx), xoff);
        if (SGD) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[k] = fmaf(-lr, Grad<GT>::template lane<NT>(uniform_base(gb + (int64_t)k * ldg), goff), v[k]);
        }
    }
    float cprev = 0.f;
    if (moving && ok) cprev = ld_lane<NT, float>(uniform_base(center_out + cell0), xoff);

    int info = 0;
    if constexpr (TILES == GRAWA_TILES_SLOTS) {
        const int l = wave_last_layer(off, L, [&](int, int64_t o) { return o <= cell0; });
        info = off[l + 1] >= (cell0 + GRAWA_CELL < P ? cell0 + GRAWA_CELL : P) ? l : ~l;
    } else {
        info = cell_layer ? cell_layer[blockIdx.x] : 0;
    }
    float c = 0.f;
    if constexpr (TILES) {
        __shared__ CellWeights<K> cw;
        const int l0 = info >= 0 ? info : ~info;
        int nl;
        if constexpr (TILES == GRAWA_TILES_ESTIMATE) {
            const GrawaEstimate e = tw.est[l0]; // counts and buffer: the same for all workers and layers
            const uint64_t used = grawa_last_used(tw.consumed[l0], tw.seen[blockIdx.x]);
            const double scale = e.n != used ? tw.gamma / grawa_one_minus_power(tw.gamma, (int64_t)(e.n - used)) : 0.0;
            nl = cell_weights<K, false>(tw, EstimateScore{tw, L, e.n, used, scale}, tw.partials + e.buffer * tw.buffer, off, L, P, cell0, l0,
                                        info < 0, cw);
            if (threadIdx.x == 0) tw.seen[blockIdx.x] = e.n; // after the barrier at whose end every thread has read it
        } else {
            nl = cell_weights<K, TILES == GRAWA_TILES_SLOTS>(tw, NormScore{}, tw.partials, off, L, P, cell0, l0, info < 0, cw);
        }
        const float *b = cw.beta + cell_layer_of<K>(cw, nl, (int)col) * K;
#pragma unroll
        for (int k = 0; k < K; ++k) c = fmaf(b[k], v[k], c);
    } else if (info >= 0) { // one layer for the whole cell: weights through scalar loads
        const uint64_t bb = uniform_base(beta + info);
#pragma unroll
        for (int k = 0; k < K; ++k) c = fmaf(ld_uniform_f32(bb, (int64_t)k * beta_stride), v[k], c);
    } else if (ok) { // the cell holds a layer boundary: each lane looks up its own layer
        const float *b = beta + layer_of(off, ~info, L, cell0 + col);
#pragma unroll
        for (int k = 0; k < K; ++k) c = fmaf(b[(int64_t)k * beta_stride], v[k], c);
    }
    if (moving) c = fmaf(rho, c - cprev, cprev);

    if (ok) {
#pragma unroll
        for (int k = 0; k < K; ++k)
            st_lane<NT ? GRAWA_ST_STREAM : GRAWA_ST_CACHED, float>(uniform_base(xb + (int64_t)k * ldx), xoff, fmaf(lambda, c - v[k], v[k]));
        if (center_out) st_lane<NT ? GRAWA_ST_STREAM : GRAWA_ST_CACHED, float>(uniform_base(center_out + cell0), xoff, c);
    }
}

// Wide form, up to 5 workers and with the fp32 SGD step 12 to 23, for arrays beyond the last-level cache whose rows do not start on line boundaries (a plain
// [K, P] tensor).  grid ceil(P/1024), block 256: a lane owns four adjacent columns (16-byte accesses are always aligned:
// the ABI asks for it), a wave 1 KiB per row and the block 4 KiB, so that one line in 32 instead of one in 8 is shared
// with another block.  Otherwise as the plain form; a wave's 256 columns are one cell.  With streaming loads and stores written
// through (LNT, GRAWA_ST_STREAM) it also serves line-aligned rows of one or two workers, where a 4-byte load per row and lane
// leaves too little in flight: K = 1 3.64 -> 6.69 TB/s, K = 2 5.71 -> 6.64, with the SGD step on bf16 gradients 5.77 -> 6.46.
// Off the line grid: measured on 1.2 to 2 GB of random values, pitch 16 bytes off a line, TB/s, plain form / this one (WPE in
// grawa_waves_wide), cached loads: K = 2 5.46/6.27, 3 5.73/6.26, 4 5.71/5.96; with the SGD step 2 5.60/6.28, 4 5.69/5.97,
// 12 5.29/5.58, 16 5.35/5.67.
// These are passes in a row over several arrays.  The plain form's cached stores leave up to 256 MB in the last-level
// cache, which a later pass has to write back; after a read of other memory a single pass of it looks faster than it is.
// One LGRAWA update, and a read of 1 GB after it, 4 workers, 75 M columns, plain / wide: 597 / 613 and 313 / 277 us.
template <int K, bool SGD, typename GT, bool LNT, int ST, int WPE>
__global__ __launch_bounds__(GRAWA_BLOCK) __attribute__((amdgpu_waves_per_eu(1, WPE))) void k_center_pull_wide(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving)
{
    constexpr int V = 4;
    typedef typename FloatVec<V>::T XV;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / GRAWA_WAVE));
    const int64_t cell = (int64_t)blockIdx.x * V + wave; // wave-uniform
    const int64_t cell0 = cell * GRAWA_CELL;
    if (cell0 >= P) return;
    const unsigned lane = threadIdx.x & (GRAWA_WAVE - 1);
    const int64_t col = cell0 + lane * V;
    const int n = col + V <= P ? V : (col < P ? (int)(P - col) : 0); // columns of this lane inside the row
    float *xb = x + cell0;
    const GT *gb = g + cell0;
    const unsigned xoff = lane * (V * 4u), goff = lane * (V * (unsigned)sizeof(GT));

    XV v[K];
    XV cprev = XV{};
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = XV{};
    if (n == V) {
#pragma unroll
        for (int k = 0; k < K; ++k) v[k] = ld_lane<LNT, XV>(uniform_base(xb + (int64_t)k * ldx), xoff);
        if constexpr (SGD) {
            float f[K][V];
#pragma unroll
            for (int k = 0; k < K; ++k) GradVec<GT, V, LNT>::lane(uniform_base(gb + (int64_t)k * ldg), goff, f[k]);
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int e = 0; e < V; ++e) vec_set<V>(v[k], e, fmaf(-lr, f[k][e], vec_get<V>(v[k], e)));
        }
        if (moving) cprev = ld_lane<LNT, XV>(uniform_base(center_out + cell0), xoff);
    } else if (n > 0) { // the lane that holds the row's last columns
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < n) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float t = xb[(int64_t)k * ldx + lane * V + e];
                    if (SGD) t = fmaf(-lr, Grad<GT>::one(gb + (int64_t)k * ldg + lane * V + e), t);
                    vec_set<V>(v[k], e, t);
                }
                if (moving) vec_set<V>(cprev, e, center_out[col + e]);
            }
    }

    const int info = cell_layer ? cell_layer[cell] : 0;
    XV c = XV{};
    if (info >= 0) { // one layer for the whole cell: weights through scalar loads
        const uint64_t bb = uniform_base(beta + info);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float w = ld_uniform_f32(bb, (int64_t)k * beta_stride);
#pragma unroll
            for (int e = 0; e < V; ++e) vec_set<V>(c, e, fmaf(w, vec_get<V>(v[k], e), vec_get<V>(c, e)));
        }
    } else { // the cell holds a layer boundary
        center_by_layer<K, V, true>(beta, beta_stride, off, L, P, cell0, ~info, col, [](int) { return true; }, v, c);
    }
    if (moving) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            vec_set<V>(c, e, fmaf(rho, vec_get<V>(c, e) - vec_get<V>(cprev, e), vec_get<V>(cprev, e)));
    }
    if (n == V) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            XV o = v[k];
#pragma unroll
            for (int e = 0; e < V; ++e)
                vec_set<V>(o, e, fmaf(lambda, vec_get<V>(c, e) - vec_get<V>(v[k], e), vec_get<V>(v[k], e)));
            st_lane<ST, XV>(uniform_base(xb + (int64_t)k * ldx), xoff, o);
        }
        if (center_out) st_lane<ST, XV>(uniform_base(center_out + cell0), xoff, c);
    } else if (n > 0) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < n) {
#pragma unroll
                for (int k = 0; k < K; ++k)
                    xb[(int64_t)k * ldx + lane * V + e] =
                        fmaf(lambda, vec_get<V>(c, e) - vec_get<V>(v[k], e), vec_get<V>(v[k], e));
                if (center_out) center_out[col + e] = vec_get<V>(c, e);
            }
    }
}

// Row-split form: the rows of W adjacent 256-column cells are divided over S groups of waves.  grid: one block per W cells
// from first_cell on (grawa_split_blocks), block S * W * 256 / V = 1024 threads.  A lane owns V adjacent columns of its group's
// rows: Q of them, and one more for the first K - S Q groups when REM (K is then S Q + 1 .. S Q + S - 1).  Each group forms its
// part of the center, the parts are added in group order through LDS, every group pulls and stores its own rows.  A wave
// touches one piece of 256 V bytes per row, the block starts its loads, and after the barrier its stores, together.
// Two uses:
// * One cell a block (W = 1), K >= 24 with S = 8, V = 2, and K = 16 without the SGD step with S = 4, V = 1.
//   Measured on 4.5 GB of random values, TB/s, this form against the plain one at its best cap: K = 24 5.94/5.85,
//   28 5.97/5.84, 32 5.89/5.88, 33 5.93/5.78, 44 5.91/5.94, 56 5.59/5.62, 64 5.50/5.52; with the SGD step (fp32)
//   24 6.00/5.75, 32 5.91/5.44, 33 6.03/5.49, 44 5.56/5.72, 63 5.45/5.53; below 24 the plain form is faster.  One
//   kernel serves eight worker counts, with one guarded row instead of a guard on each: a form that
//   guards every row (its loads then wait for one another) ran at 4.1 TB/s, 2.0 with the SGD step.  Whole MGRAWA update,
//   11.7 M columns, K = 48, bf16 gradients: 1266 us with that form, 986 with this one.
// * Bursts (V = 4, S W = 16, WPE = 4), for large rows off the line grid: one block of 16 waves per CU, so that each CU reads
//   and then writes W KiB of a row at once and lines are shared at the ends of those pieces only.  What bounds it is the
//   memory's handling of the parts of lines and of the many rows.  MGRAWA update, arrays of 1.2 GB, us, the forms before / this one:
//   7 workers 513 / 499, 8 538 / 520, 10 535 / 522, 11 525 / 513, 12 533 / 512, 16 542 / 544, 23 534 / 520, 24 582 / 561, 27 630 / 564,
//   32 607 / 554, 48 617 / 558, 64 644 / 550; with the fp32 SGD step 9 861 / 837, 10 887 / 833, 32 963 / 877, 48 1013 / 891, 64 1015 / 892;
//   fused, fp32, 200 MB 8 151 / 135, 9 152 / 133, 32 170 / 148 (without the step: GRAWA_BURST_MIN_BYTES).  Two blocks per CU are slower than the forms before.  Up to 15
//   workers streaming loads and stores that the L2 merges; beyond, cached loads and stores written through (12 workers 5.81 / 5.99
//   TB/s against these, 20 workers 5.85 / 5.33).  S: 2 up to 9 workers, 4 up to 23, 8 beyond (10 workers with 2: 540 us, 9 with
//   4 and the SGD step: 918 for 894).  With the fp32 SGD step the wide form stays for 12 to 23 workers (12, 1.2 GB: 861 / 882, 855 /
//   848 on rows 32 and 16 bytes off a line; 15 853 / 862, 20 855 / 860).  On line-aligned rows of 40 to 64 workers bursts are no faster.
template <int Q, bool REM, int S, int V, int W, int WPE, bool SGD, typename GT, bool NT, int ST>
__global__ __launch_bounds__(S *W *GRAWA_CELL / V) __attribute__((amdgpu_waves_per_eu(4, WPE))) void k_center_pull_split(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int K, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving, unsigned first_cell)
{
    typedef typename FloatVec<V>::T XV;
    constexpr int CELL_LANES = GRAWA_CELL / V;
    constexpr int LANES = W * CELL_LANES; // lanes of a group
    constexpr int R = REM ? Q + 1 : Q;    // register slots per lane
    static_assert(CELL_LANES % GRAWA_WAVE == 0, "a cell is made of whole waves");
    static_assert(S * LANES == GRAWA_SPLIT_THREADS, "the grid is chosen for this many threads");
    const int group = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / LANES)); // wave-uniform
    const unsigned at = threadIdx.x % LANES; // the lane's place in its group, and in its cell:
    const unsigned lane = at % CELL_LANES;
    unsigned cell = first_cell + blockIdx.x; // wave-uniform; below 2^24 + W
    if constexpr (W > 1) cell = first_cell + blockIdx.x * W + __builtin_amdgcn_readfirstlane((int)(at / CELL_LANES));
    const int64_t cell0 = (int64_t)cell * GRAWA_CELL; // W > 1: may lie past the row, whose lanes then take part in the barrier only
    const int rem = REM ? K - S * Q : 0;
    const bool more = REM && group < rem; // this group owns one row more
    const int k0 = group * Q + (REM ? (group < rem ? group : rem) : 0);
    const int64_t col = cell0 + lane * V;
    const int n = col + V <= P ? V : (col < P ? (int)(P - col) : 0); // columns of this lane inside the row
    float *xb = x + cell0 + (int64_t)k0 * ldx;
    const GT *gb = g + cell0 + (int64_t)k0 * ldg;
    const unsigned xoff = lane * (V * 4u), goff = lane * (V * (unsigned)sizeof(GT));

    XV v[R];
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = XV{};
    if (n == V) {
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (k < Q || more) v[k] = ld_lane<NT, XV>(uniform_base(xb + (int64_t)k * ldx), xoff);
        if constexpr (SGD) {
            float f[R][V];
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < Q || more) GradVec<GT, V, NT>::lane(uniform_base(gb + (int64_t)k * ldg), goff, f[k]);
#pragma unroll
            for (int k = 0; k < R; ++k)
                if (k < Q || more) {
#pragma unroll
                    for (int e = 0; e < V; ++e) vec_set<V>(v[k], e, fmaf(-lr, f[k][e], vec_get<V>(v[k], e)));
                }
        }
    } else if (n > 0) { // the lane that holds the row's last columns
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (k < Q || more) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    if (e < n) {
                        float t = xb[(int64_t)k * ldx + lane * V + e];
                        if (SGD) t = fmaf(-lr, Grad<GT>::one(gb + (int64_t)k * ldg + lane * V + e), t);
                        vec_set<V>(v[k], e, t);
                    }
            }
    }

    XV cprev = XV{}; // read before the barrier: group 0 overwrites it after the barrier
    if (moving) {
        if (n == V) cprev = ld_lane<NT, XV>(uniform_base(center_out + cell0), xoff);
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (n < V && e < n) vec_set<V>(cprev, e, center_out[col + e]);
    }

    const int info = cell_layer && (W == 1 || cell0 < P) ? cell_layer[cell] : 0;
    XV c = XV{};
    if (info >= 0) { // one layer for the whole cell: weights through scalar loads
        const uint64_t bb = uniform_base(beta + info + (int64_t)k0 * beta_stride);
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (k < Q || more) {
                const float w = ld_uniform_f32(bb, (int64_t)k * beta_stride);
#pragma unroll
                for (int e = 0; e < V; ++e) vec_set<V>(c, e, fmaf(w, vec_get<V>(v[k], e), vec_get<V>(c, e)));
            }
    } else { // the cell holds a layer boundary
        center_by_layer<R, V, (W > 1)>(beta + (int64_t)k0 * beta_stride, beta_stride, off, L, P, cell0, ~info, col,
                              [&](int k) { return k < Q || more; }, v, c);
    }
    __shared__ XV part[S][LANES];
    part[group][at] = c;
    __syncthreads();
    c = part[0][at];
#pragma unroll
    for (int s = 1; s < S; ++s) c += part[s][at];
    if (moving) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            vec_set<V>(c, e, fmaf(rho, vec_get<V>(c, e) - vec_get<V>(cprev, e), vec_get<V>(cprev, e)));
    }
    if (n == V) {
#pragma unroll
        for (int k = 0; k < R; ++k)
            if (k < Q || more) {
                XV o = v[k];
#pragma unroll
                for (int e = 0; e < V; ++e)
                    vec_set<V>(o, e, fmaf(lambda, vec_get<V>(c, e) - vec_get<V>(v[k], e), vec_get<V>(v[k], e)));
                st_lane<ST, XV>(uniform_base(xb + (int64_t)k * ldx), xoff, o);
            }
        if (center_out && group == 0) st_lane<ST, XV>(uniform_base(center_out + cell0), xoff, c);
    } else if (n > 0) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < n) {
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if (k < Q || more)
                        xb[(int64_t)k * ldx + lane * V + e] =
                            fmaf(lambda, vec_get<V>(c, e) - vec_get<V>(v[k], e), vec_get<V>(v[k], e));
                if (center_out && group == 0) center_out[col + e] = vec_get<V>(c, e);
            }
    }
}

// Any number of workers: two sweeps over k per column (the second sweep re-reads what the
// first just fetched, normally from cache).  Used only when K exceeds the register-resident
// variants above.
template <bool SGD, typename GT>
__global__ __launch_bounds__(GRAWA_CELL) void k_center_pull_any(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int K, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving)
{
    const int64_t i = (int64_t)blockIdx.x * GRAWA_CELL + threadIdx.x;
    if (i >= P) return;
    int layer = 0;
    if (cell_layer) {
        const int info = cell_layer[blockIdx.x];
        layer = info >= 0 ? info : layer_of(off, ~info, L, i);
    }
    const float *b = beta + layer;
    float c = 0.f;
    for (int k = 0; k < K; ++k) {
        float v = x[(int64_t)k * ldx + i];
        if (SGD) v = fmaf(-lr, Grad<GT>::one(g + (int64_t)k * ldg + i), v);
        c = fmaf(b[(int64_t)k * beta_stride], v, c);
    }
    if (moving) c = fmaf(rho, c - center_out[i], center_out[i]);
    for (int k = 0; k < K; ++k) {
        float v = x[(int64_t)k * ldx + i];
        if (SGD) v = fmaf(-lr, Grad<GT>::one(g + (int64_t)k * ldg + i), v);
        x[(int64_t)k * ldx + i] = fmaf(lambda, c - v, v);
    }
    if (center_out) center_out[i] = c;
}

// ---------------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------------

// Waves per SIMD the plain form is capped at on large arrays, from sweeps of this kernel over K and the cap on the part, on arrays
// of 1 to 2 GB holding random values and three row lengths (best throughput at roughly 24 to 36 four-byte row
// loads in flight per SIMD; a two-byte load counts half).  The best caps, TB/s at the best and one wave more:
// K = 4 6.71 (8), 6 6.66/6.57, 8 6.57/6.46, 12 6.41/6.28, 22 6.16/5.95; with the fp32 SGD step
// 4 6.60/6.57, 8 6.43/6.30, 12 6.13/6.07, 16 6.04/5.73; with bf16 gradients 4 6.73/6.68, 8 6.51/6.43 (one wave
// fewer: 6.09), 12 6.28/6.25 (one fewer: 5.61), 16 5.96/5.92.
// The values matter: arrays of zeros stream about 4 % faster on this part and shift some of the optima, so
// sweeps over cleared memory mislead.
constexpr int grawa_waves_for(int k, bool sgd, bool bf16)
{
    if (sgd && bf16) return k <= 3 ? 8 : k == 4 ? 7 : k == 5 ? 6 : k == 6 ? 5 : k <= 11 ? 4 : k <= 16 ? 3 : 2;
    if (sgd) return k <= 2 ? 8 : k == 3 ? 7 : k <= 5 ? 5 : k <= 7 ? 4 : k <= 11 ? 3 : 2;
    return k <= 4 ? 8 : k == 5 ? 6 : k == 6 ? 5 : k <= 8 ? 4 : k <= 16 ? 3 : 2;
}

#define GRAWA_CP_ARGS                                                                                                 \
    const grawa_plan *p, float *x, int64_t ldx, const void *g, int64_t ldg, float lr, const float *beta, int per_layer, \
        float lambda, float *center_out, float rho, int moving, [[maybe_unused]] const TileWeights &tw,                     \
        [[maybe_unused]] bool capped, hipStream_t s,                                                                   \
        hipEvent_t e0, hipEvent_t e1
#define GRAWA_CP_PASS p, x, ldx, g, ldg, lr, beta, per_layer, lambda, center_out, rho, moving, tw, capped, s, e0, e1
#define GRAWA_CP_STRIDE per_layer ? (int64_t)p->L : (int64_t)1
#define GRAWA_CP_CELLS per_layer ? (const int32_t *)p->d_cell_layer : (const int32_t *)nullptr

template <int K, bool SGD, typename GT, bool NT, int TILES> static void launch_plain(GRAWA_CP_ARGS)
{
    constexpr int CAP = grawa_waves_for(K, SGD, sizeof(GT) == 2), WPE = NT ? CAP : 8;
    // Cached accesses: the cap, where it is wanted, is set by the LDS a block asks for, of the CU's 160 KB.  Up to 128 MB the
    // caches answer, and what counts is that all blocks of a small array run at once (1054 blocks of 8 workers are one more
    // round than 4 per CU hold).  LGRAWA with the fp32 SGD step, us, capped / not: 8 workers, 270 k columns 13.9 / 12.0,
    // 317 k 14.9 / 13.1, 10 workers 256 k 15.6 / 13.7, 15 workers 174 k 17.3 / 15.4; MGRAWA 8 workers, 1.6 M 35.0 / 31.4, 3.1 M
    // 58.8 / 54.7, 20 workers 312 k 23.3 / 21.9; LGRAWA with the weights in the pull 12 workers, 218 k, 20 layers 10.8 / 9.4, 200 layers 14.4 /
    // 13.2, 13 workers, 201 k 10.9 / 9.6 and 15.4 / 14.2 (fewer columns, and 14 and 15 workers, 0 to 0.2 us slower).  Rows off the grid from 64 MB on: 15 workers, 90 MB 55.5 / 57.4, 6 workers with
    // the fp32 step 72.6 / 74.6.
    const size_t lds = WPE > CAP && capped ? ((size_t)160 << 10) / (CAP + 1) + 1024 : 0;
    hipExtLaunchKernelGGL((k_center_pull<K, SGD, GT, NT, WPE, TILES>), dim3((unsigned)p->n_cells), dim3(GRAWA_CELL), lds, s, e0,
                          e1, 0, x, ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE, GRAWA_CP_CELLS,
                          (const int64_t *)p->d_off, p->L, p->P, lambda, center_out, rho, moving, tw);
}

// The wide form's cap (best of 2, 3, 4 and 8 waves; one too many costs 3 to 5 %, and more than it gains over the plain form).
constexpr int grawa_waves_wide(int k, bool sgd /* fp32 gradients */)
{
    if (k == 1) return 8;
    if (k == 2) return sgd ? 3 : 4;
    if (k == 3) return sgd ? 2 : 3;
    return k <= 5 ? 2 : 1;
}

template <int K, bool SGD, typename GT, bool LNT, int ST> static void launch_wide(GRAWA_CP_ARGS)
{
    hipExtLaunchKernelGGL((k_center_pull_wide<K, SGD, GT, LNT, ST, grawa_waves_wide(K, SGD && sizeof(GT) == 4)>), dim3((unsigned)((p->n_cells + 3) / 4)),
                          dim3(GRAWA_BLOCK), 0, s, e0, e1, 0, x, ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE,
                          GRAWA_CP_CELLS, (const int64_t *)p->d_off, p->L, p->P, lambda, center_out, rho, moving);
}

// W cells a block; WPE caps the waves per SIMD.
template <int Q, bool REM, int S, int V, int W, int WPE, bool SGD, typename GT, bool NT, int ST> static void launch_split(GRAWA_CP_ARGS)
{
    static_assert(GRAWA_SPLIT_LAUNCH_CELLS % W == 0, "a launch begins with the first cell of a block");
    for (int64_t at = 0; at < p->n_cells;) { // one launch but for the longest rows
        const int64_t n = grawa_split_blocks(p->n_cells, at);
        hipExtLaunchKernelGGL((k_center_pull_split<Q, REM, S, V, W, WPE, SGD, GT, NT, ST>), dim3((unsigned)((n + W - 1) / W)),
                              dim3(GRAWA_SPLIT_THREADS), 0, s, at == 0 ? e0 : nullptr, at + n == p->n_cells ? e1 : nullptr, 0,
                              x, ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE, GRAWA_CP_CELLS,
                              (const int64_t *)p->d_off, p->L, p->K, p->P, lambda, center_out, rho, moving, (unsigned)at);
        at += n;
    }
}

// Row-split, 8-byte lanes, one cell a block.
template <int Q, bool REM, bool SGD, typename GT, bool NT> static void launch_cell(GRAWA_CP_ARGS)
{
    launch_split<Q, REM, 8, 2, 1, 8, SGD, GT, NT, NT ? GRAWA_ST_STREAM : GRAWA_ST_CACHED>(GRAWA_CP_PASS);
}

// Row-split, 16-byte lanes, W cells a block and one block per CU: S W = 16 waves, 4 per SIMD.
template <int Q, bool REM, int S, bool SGD, typename GT, bool NT, int ST> static void launch_burst(GRAWA_CP_ARGS)
{
    launch_split<Q, REM, S, 4, 16 / S, 4, SGD, GT, NT, ST>(GRAWA_CP_PASS);
}

// One plain kernel per worker count up to 23, on few cells up to 32 (fully unrolled); the rest up to 71 workers share the
// row-split kernels by K / 8; beyond that the two-sweep kernel.
template <bool SGD, typename GT, bool NT> static hipError_t dispatch_cp(GRAWA_CP_ARGS)
{
    // Line-aligned streaming rows of one worker, and of two unless fused with fp32 gradients: the wide form.
    constexpr int WIDE_TO = !NT ? 0 : SGD && sizeof(GT) == 4 ? 1 : 2;
#define GRAWA_CP_PLAIN(N)                                                                       \
    case N:                                                                                     \
        if constexpr (N <= WIDE_TO) launch_wide<N, SGD, GT, true, GRAWA_ST_STREAM>(GRAWA_CP_PASS);               \
        else launch_plain<N, SGD, GT, NT, GRAWA_TILES_NONE>(GRAWA_CP_PASS);                                \
        return hipGetLastError();
#define GRAWA_CP_SPLIT(N)                                                     \
    case N:                                                                   \
        if (p->K % 8 == 0) launch_cell<N, false, SGD, GT, NT>(GRAWA_CP_PASS); \
        else launch_cell<N, true, SGD, GT, NT>(GRAWA_CP_PASS);               \
        return hipGetLastError();
    switch (p->K) {
        GRAWA_CP_PLAIN(1) GRAWA_CP_PLAIN(2) GRAWA_CP_PLAIN(3) GRAWA_CP_PLAIN(4) GRAWA_CP_PLAIN(5) GRAWA_CP_PLAIN(6)
        GRAWA_CP_PLAIN(7) GRAWA_CP_PLAIN(8) GRAWA_CP_PLAIN(9) GRAWA_CP_PLAIN(10) GRAWA_CP_PLAIN(11) GRAWA_CP_PLAIN(12)
        GRAWA_CP_PLAIN(13) GRAWA_CP_PLAIN(14) GRAWA_CP_PLAIN(15) GRAWA_CP_PLAIN(17) GRAWA_CP_PLAIN(18)
        GRAWA_CP_PLAIN(19) GRAWA_CP_PLAIN(20) GRAWA_CP_PLAIN(21) GRAWA_CP_PLAIN(22) GRAWA_CP_PLAIN(23)
    case 16:
        if constexpr (SGD) launch_plain<16, SGD, GT, NT, GRAWA_TILES_NONE>(GRAWA_CP_PASS);
        else launch_split<4, false, 4, 1, 1, 8, SGD, GT, NT, NT ? GRAWA_ST_STREAM : GRAWA_ST_CACHED>(GRAWA_CP_PASS);
        return hipGetLastError();
    }
    if constexpr (!NT) // never as large as the streaming passes
        if (grawa_plain_form(p->K, p->n_cells)) switch (p->K) {
                GRAWA_CP_PLAIN(24) GRAWA_CP_PLAIN(25) GRAWA_CP_PLAIN(26) GRAWA_CP_PLAIN(27) GRAWA_CP_PLAIN(28)
                GRAWA_CP_PLAIN(29) GRAWA_CP_PLAIN(30) GRAWA_CP_PLAIN(31) GRAWA_CP_PLAIN(32)
            }
    switch (p->K / 8) {
        GRAWA_CP_SPLIT(3) GRAWA_CP_SPLIT(4) GRAWA_CP_SPLIT(5) GRAWA_CP_SPLIT(6) GRAWA_CP_SPLIT(7) GRAWA_CP_SPLIT(8)
    }
    hipExtLaunchKernelGGL((k_center_pull_any<SGD, GT>), dim3((unsigned)p->n_cells), dim3(GRAWA_CELL), 0, s, e0, e1, 0, x,
                          ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE, GRAWA_CP_CELLS,
                          (const int64_t *)p->d_off, p->L, p->K, p->P, lambda, center_out, rho, moving);
    return hipGetLastError();
#undef GRAWA_CP_PLAIN
#undef GRAWA_CP_SPLIT
}

// Large rows off the line grid, 16-byte lanes: the forms of grawa_off_grid, whose plain ones do not come here.  A worker count
// without a kernel is an error, never a call that does nothing.
template <bool SGD, typename GT> static hipError_t dispatch_cp_off_grid(GRAWA_CP_ARGS)
{
    constexpr bool F32_SGD = SGD && sizeof(GT) == 4;
#define GRAWA_CP_EACH(N)                                                                                                     \
    case N: {                                                                                                                \
        constexpr GrawaOffGrid F = grawa_off_grid(N, F32_SGD);                                                               \
        constexpr int ST = F.merge ? GRAWA_ST_MERGE : GRAWA_ST_STREAM;                                                       \
        if constexpr (F.form == GRAWA_OFF_GRID_WIDE) launch_wide<N, SGD, GT, F.merge, ST>(GRAWA_CP_PASS);                    \
        else if constexpr (F.form == GRAWA_OFF_GRID_BURST)                                                                   \
            launch_burst<N / F.groups, (N % F.groups != 0), F.groups, SGD, GT, F.merge, ST>(GRAWA_CP_PASS);                  \
        else return hipErrorInvalidValue;                                                                                    \
        return hipGetLastError();                                                                                            \
    }
#define GRAWA_CP_EIGHTH(N)                                                                                 \
    case N:                                                                                                \
        if (p->K % 8 == 0) launch_burst<N, false, 8, SGD, GT, false, GRAWA_ST_STREAM>(GRAWA_CP_PASS);      \
        else launch_burst<N, true, 8, SGD, GT, false, GRAWA_ST_STREAM>(GRAWA_CP_PASS);                     \
        return hipGetLastError();
    switch (p->K) {
        GRAWA_OFF_GRID_EACH(GRAWA_CP_EACH)
    }
    switch (p->K / 8) {
        GRAWA_OFF_GRID_EIGHTHS(GRAWA_CP_EIGHTH)
    }
    return hipErrorInvalidValue;
#undef GRAWA_CP_EACH
#undef GRAWA_CP_EIGHTH
}

// Weights straight from the tile sums (GRAWA_TILES_COUNTS), cached accesses.
template <bool SGD, typename GT> static hipError_t dispatch_cp_tiles(GRAWA_CP_ARGS)
{
#define GRAWA_CP_TILES(N)                                                                                      \
    case N:                                                                                                    \
        if constexpr (!SGD) /* the call without maps has no fused step */                                      \
            if (p->tile_shift) {                                                                               \
                launch_plain<N, SGD, GT, false, GRAWA_TILES_SLOTS>(GRAWA_CP_PASS);                             \
                return hipGetLastError();                                                                      \
            }                                                                                                  \
        launch_plain<N, SGD, GT, false, GRAWA_TILES_MAPS>(GRAWA_CP_PASS);                                      \
        return hipGetLastError();
    switch (p->K) {
        GRAWA_TILES_COUNTS(GRAWA_CP_TILES)
    }
    return hipErrorInvalidValue;
#undef GRAWA_CP_TILES
}

// Weights from the running estimate (EstimateWeights): arrays of at most 10 MB, so cached accesses without a cap.
hipError_t grawa_launch_local_pull(const grawa_plan *p, float *x, int64_t ldx, double gamma, float lambda, float *center_out,
                                   float *weights_out, float *est_out, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    EstimateWeights w = {};
    static_cast<TileWeights &>(w) = TileWeights{p->d_sums, p->n_rtiles, p->d_layer_rtile0, p->d_layer_rtile0 + 1, weights_out, p->d_flags,
                                                grawa_group_lanes(p->K), 0};
    w.est = p->d_est;
    w.consumed = p->d_consumed;
    w.consumed_by_pulls = p->d_consumed + p->L;
    w.seen = p->d_seen;
    w.est_out = est_out;
    w.buffer = (int64_t)p->K * p->n_rtiles;
    w.gamma = gamma;
#define GRAWA_LOCAL_PULL(N)                                                                                                  \
    case N:                                                                                                                  \
        hipExtLaunchKernelGGL((k_center_pull<N, false, float, false, 8, GRAWA_TILES_ESTIMATE>), dim3((unsigned)p->n_cells),  \
                              dim3(GRAWA_CELL), 0, s, e0, e1, 0, x, ldx, (const float *)nullptr, (int64_t)0, 0.f,            \
                              (const float *)nullptr, (int64_t)p->L, (const int32_t *)p->d_cell_layer,                       \
                              (const int64_t *)p->d_off, p->L, p->P, lambda, center_out, 0.f, 0, w);                         \
        return hipGetLastError();
    switch (p->K) {
        GRAWA_TILES_COUNTS(GRAWA_LOCAL_PULL)
    }
    return hipErrorInvalidValue;
#undef GRAWA_LOCAL_PULL
}

bool grawa_pull_from_tiles(const grawa_plan *p) { return grawa_weights_in_pull(p->K, p->n_cells); }

hipError_t grawa_launch_center_pull(const grawa_plan *p, float *x, int64_t ldx, const float *beta,
                                    int per_layer, float lambda, const void *g_sgd, int64_t ldg_sgd,
                                    grawa_dtype_t dt, float lr, int fuse_sgd, float *center_out, float rho,
                                    int moving, float *weights_out, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    TileWeights tw = {};
    if (!beta)
        tw = TileWeights{p->d_partials, p->n_tiles, p->d_layer_tile0, p->d_layer_tile1, weights_out, p->d_flags, grawa_group_lanes(p->K), p->tile_shift};
    // Streaming accesses pay off only when the arrays do not fit the last-level cache anyway: x, and g where the step is fused.
    // (By x alone, fused LGRAWA updates, three sets in turn, us, line-aligned rows / rows off the grid: 70 MB fp32 2 workers 57.3 ->
    // 53.8 / 58.4 -> 52.4, 6 55.2 -> 51.8 / 57.3 -> 56.7, 48 64.4 -> 60.9 / 67.1 -> 60.8; 95 MB bf16 2 68.4 -> 56.6 / 70.2 -> 57.4, 12
    // 64.7 -> 58.6 / 67.4 -> 64.6, 32 68.7 -> 62.6 / 71.4 -> 68.6; 125 MB fp32 6 91.8 -> 84.4 / 94.7 -> 92.0.  What it costs where nothing
    // else is touched between the calls and the last-level cache still holds part of x and g, one set again and again, line-aligned rows, fp32: 2
    // and 4 workers 1 % at most, 8 84 MB 60.8 -> 62.0, 12 70 MB 53.6 -> 56.3, 16 66 MB 51.5 -> 55.6, 32 84 MB 61.6 -> 64.6, 124 MB 85.0 -> 87.1,
    // three sets in turn 69.8 -> 61.8, 61.1 -> 56.9, 58.2 -> 55.3, 76.1 -> 65.5 and 106.6 -> 88.8; rows off the grid 16 66 MB 55.2 -> 61.6 and
    // 60.5 -> 60.4, and, as bursts, 24 130 MB 94.8 -> 102.9 and 112.5 -> 106.0, bf16 24 and 48 130 MB 79.6 -> 87.9 and 79.5 -> 94.8 against
    // 94.8 -> 88.7 and 99.8 -> 93.3, 200 MB 113.1 -> 117.3 and 115.3 -> 118.9 against 132.5 -> 121.5 and 141.5 -> 124.7.)
    const int64_t bytes = (int64_t)p->K * p->P * (4 + (fuse_sgd ? (dt == GRAWA_BF16 ? 2 : 4) : 0));
    const bool large = beta && bytes > GRAWA_STREAMING_MIN_BYTES;
    bool nt = rows_line_aligned(x, ldx, 4) && (!center_out || rows_line_aligned(center_out, 0, 4));
    if (fuse_sgd) nt = nt && rows_line_aligned(g_sgd, ldg_sgd, dt == GRAWA_BF16 ? 2 : 4);
    // Cached accesses of small arrays want no cap, unless rows off the grid make many requests of them (launch_plain).
    const bool capped = large || (!nt && bytes > GRAWA_STREAMING_MIN_BYTES / 2);
    nt = nt && large;
    const bool off_grid = large && !nt && grawa_off_grid_large(p->K, fuse_sgd, bytes, GRAWA_STREAMING_MIN_BYTES) &&
                          grawa_off_grid(p->K, fuse_sgd && dt != GRAWA_BF16).form != GRAWA_OFF_GRID_PLAIN;
    const void *g = g_sgd;
    const int64_t ldg = ldg_sgd;
#define GRAWA_CP_GO(SGD, GT)                                                      \
    (!beta  ? dispatch_cp_tiles<SGD, GT>(GRAWA_CP_PASS)                           \
     : nt   ? dispatch_cp<SGD, GT, true>(GRAWA_CP_PASS)                           \
     : off_grid ? dispatch_cp_off_grid<SGD, GT>(GRAWA_CP_PASS)                    \
            : dispatch_cp<SGD, GT, false>(GRAWA_CP_PASS))
    if (!fuse_sgd) return GRAWA_CP_GO(false, float);
    return dt == GRAWA_BF16 ? GRAWA_CP_GO(true, uint16_t) : GRAWA_CP_GO(true, float);
#undef GRAWA_CP_GO
}
