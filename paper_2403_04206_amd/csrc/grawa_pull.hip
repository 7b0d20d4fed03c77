// Center and pull of the GRAWA update (gfx950, wave64):
//   x_C = sum_k beta_k x_k ;  x_k <- x_k + lambda (x_C - x_k)      [display after eq. (2); eq. (7)]
// with the local SGD step x_k - lr g_k optionally applied on the way in (Algorithms 1 and 2) and,
// for EASGD (Appendix F), the center averaged in time.
//
// A read-modify-write pass over K far-apart rows: it runs fastest when a wave touches one aligned
// 256-byte piece of every row (one 32-bit element per lane per row), blocks are small and many,
// and accesses are non-temporal -- provided every row starts on a 128-byte boundary, so that no
// cache line is written in two parts.  There is no dense contraction, hence no matrix-core code.
#include "grawa_device.h"

// ---------------------------------------------------------------------------------
// center + pull (+ SGD on the way in)
// ---------------------------------------------------------------------------------

// Layer of column i, given a layer at or before it (cells that contain a layer boundary).
__device__ __forceinline__ int layer_of(const int64_t *__restrict__ off, int layer, int L, int64_t i)
{
    while (layer + 1 < L && off[layer + 1] <= i) ++layer;
    return layer;
}

// Plain form, K <= 23 (16 without the SGD step excepted).  grid ceil(P/256), block 256: a lane owns one
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
// WPE caps the waves per SIMD: the form is fastest with roughly 32-48 row loads in flight per
// SIMD (K x WPE); more only queues requests to K far-apart rows and costs DRAM efficiency
// (measured: K = 16 at 3 waves 6.1 TB/s, at 8 waves 5.7; K = 8 at 4 waves 6.5, at 8 waves 6.2).
template <int K, bool SGD, typename GT, bool NT, int WPE>
__global__ __launch_bounds__(GRAWA_CELL) __attribute__((amdgpu_waves_per_eu(1, WPE))) void k_center_pull(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving)
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

    const int info = cell_layer ? cell_layer[blockIdx.x] : 0;
    float c = 0.f;
    if (info >= 0) { // one layer for the whole cell: weights through scalar loads
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
            st_lane<NT, float>(uniform_base(xb + (int64_t)k * ldx), xoff, fmaf(lambda, c - v[k], v[k]));
        if (center_out) st_lane<NT, float>(uniform_base(center_out + cell0), xoff, c);
    }
}

// Row-split form: the rows of a 256-column cell are divided over S groups of waves.  grid ceil(P/256),
// block S * 256 / V.  A lane owns V adjacent columns of its group's rows: Q of them, and one more for the
// first K - S Q groups when REM (K is then S Q + 1 .. S Q + S - 1).  Each group forms its part of the
// center, the parts are added in group order through LDS, every group pulls and stores its own rows.  A
// wave touches one piece of 256 V bytes per row, the block starts its loads, and after the barrier its
// stores, together.
// Used for K >= 24 with S = 8, V = 2 (1024 threads), and for K = 16 without the SGD step with S = 4, V = 1.
// Measured on 4.5 GB of random values, TB/s, this form against the plain one at its best cap: K = 24 5.94/5.85,
// 28 5.97/5.84, 32 5.89/5.88, 33 5.93/5.78, 44 5.91/5.94, 56 5.59/5.62, 64 5.50/5.52; with the SGD step (fp32)
// 24 6.00/5.75, 32 5.91/5.44, 33 6.03/5.49, 44 5.56/5.72, 63 5.45/5.53; below 24 the plain form is faster.  One
// kernel serves eight worker counts, with one guarded row instead of a guard on each: a form that
// guards every row (its loads then wait for one another) ran at 4.1 TB/s, 2.0 with the SGD step.  Whole MGRAWA update,
// 11.7 M columns, K = 48, bf16 gradients: 1266 us with that form, 986 with this one.
template <int Q, bool REM, int S, int V, bool SGD, typename GT, bool NT>
__global__ __launch_bounds__(S *GRAWA_CELL / V) void k_center_pull_split(
    float *__restrict__ x, int64_t ldx, const GT *__restrict__ g, int64_t ldg, float lr,
    const float *__restrict__ beta, int64_t beta_stride, const int32_t *__restrict__ cell_layer,
    const int64_t *__restrict__ off, int L, int K, int64_t P, float lambda,
    float *__restrict__ center_out, float rho, int moving)
{
    typedef typename FloatVec<V>::T XV;
    constexpr int LANES = GRAWA_CELL / V; // lanes of a group
    constexpr int R = REM ? Q + 1 : Q;    // register slots per lane
    static_assert(LANES % GRAWA_WAVE == 0, "a group is made of whole waves");
    const int64_t cell0 = (int64_t)blockIdx.x * GRAWA_CELL; // wave-uniform
    const int group = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / LANES)); // wave-uniform
    const unsigned lane = threadIdx.x % LANES;
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

    const int info = cell_layer ? cell_layer[blockIdx.x] : 0;
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
    } else { // the cell holds a layer boundary: each column looks up its own layer
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (e < n) {
                const float *b = beta + layer_of(off, ~info, L, col + e) + (int64_t)k0 * beta_stride;
                float t = 0.f;
#pragma unroll
                for (int k = 0; k < R; ++k)
                    if (k < Q || more) t = fmaf(b[(int64_t)k * beta_stride], vec_get<V>(v[k], e), t);
                vec_set<V>(c, e, t);
            }
    }
    __shared__ XV part[S][LANES];
    part[group][lane] = c;
    __syncthreads();
    c = part[0][lane];
#pragma unroll
    for (int s = 1; s < S; ++s) c += part[s][lane];
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
                st_lane<NT, XV>(uniform_base(xb + (int64_t)k * ldx), xoff, o);
            }
        if (center_out && group == 0) st_lane<NT, XV>(uniform_base(center_out + cell0), xoff, c);
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

// Waves per SIMD the plain form is capped at, from sweeps of this kernel over K and
// the cap on the part, on arrays of 3 to 11 GB holding random values (best throughput at roughly
// 24-48 row loads in flight per SIMD).  The values matter: arrays of zeros stream about 4 % faster
// on this part and shift some of the optima, so sweeps over cleared memory mislead.
constexpr int grawa_waves_for(int k, bool sgd)
{
    if (sgd) return k <= 3 ? 8 : k <= 5 ? 5 : k <= 7 ? 4 : k <= 11 ? 3 : 2;
    return k <= 4 ? 8 : k == 5 ? 5 : k <= 8 ? 4 : k <= 16 ? 3 : 2;
}

#define GRAWA_CP_ARGS                                                                                                 \
    const grawa_plan *p, float *x, int64_t ldx, const void *g, int64_t ldg, float lr, const float *beta, int per_layer, \
        float lambda, float *center_out, float rho, int moving, hipStream_t s, hipEvent_t e0, hipEvent_t e1
#define GRAWA_CP_PASS p, x, ldx, g, ldg, lr, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1
#define GRAWA_CP_STRIDE per_layer ? (int64_t)p->L : (int64_t)1
#define GRAWA_CP_CELLS per_layer ? (const int32_t *)p->d_cell_layer : (const int32_t *)nullptr

template <int K, bool SGD, typename GT, bool NT> static void launch_plain(GRAWA_CP_ARGS)
{
    hipExtLaunchKernelGGL((k_center_pull<K, SGD, GT, NT, grawa_waves_for(K, SGD)>), dim3((unsigned)p->n_cells),
                          dim3(GRAWA_CELL), 0, s, e0, e1, 0, x, ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE,
                          GRAWA_CP_CELLS, (const int64_t *)p->d_off, p->L, p->P, lambda, center_out, rho, moving);
}

template <int Q, bool REM, int S, int V, bool SGD, typename GT, bool NT> static void launch_split(GRAWA_CP_ARGS)
{
    hipExtLaunchKernelGGL((k_center_pull_split<Q, REM, S, V, SGD, GT, NT>), dim3((unsigned)p->n_cells),
                          dim3(S * GRAWA_CELL / V), 0, s, e0, e1, 0, x, ldx, (const GT *)g, ldg, lr, beta,
                          GRAWA_CP_STRIDE, GRAWA_CP_CELLS, (const int64_t *)p->d_off, p->L, p->K, p->P, lambda,
                          center_out, rho, moving);
}

// One plain kernel per worker count up to 23 (fully unrolled); 24..71 workers share the row-split
// kernels by K / 8; beyond that the two-sweep kernel.
template <bool SGD, typename GT, bool NT> static void dispatch_cp(GRAWA_CP_ARGS)
{
#define GRAWA_CP_PLAIN(N) \
    case N: launch_plain<N, SGD, GT, NT>(GRAWA_CP_PASS); return;
#define GRAWA_CP_SPLIT(N)                                                        \
    case N:                                                                      \
        if (p->K % 8 == 0) launch_split<N, false, 8, 2, SGD, GT, NT>(GRAWA_CP_PASS); \
        else launch_split<N, true, 8, 2, SGD, GT, NT>(GRAWA_CP_PASS);            \
        return;
    switch (p->K) {
        GRAWA_CP_PLAIN(1) GRAWA_CP_PLAIN(2) GRAWA_CP_PLAIN(3) GRAWA_CP_PLAIN(4) GRAWA_CP_PLAIN(5) GRAWA_CP_PLAIN(6)
        GRAWA_CP_PLAIN(7) GRAWA_CP_PLAIN(8) GRAWA_CP_PLAIN(9) GRAWA_CP_PLAIN(10) GRAWA_CP_PLAIN(11) GRAWA_CP_PLAIN(12)
        GRAWA_CP_PLAIN(13) GRAWA_CP_PLAIN(14) GRAWA_CP_PLAIN(15) GRAWA_CP_PLAIN(17) GRAWA_CP_PLAIN(18)
        GRAWA_CP_PLAIN(19) GRAWA_CP_PLAIN(20) GRAWA_CP_PLAIN(21) GRAWA_CP_PLAIN(22)
        GRAWA_CP_PLAIN(23)
    case 16:
        if constexpr (SGD) launch_plain<16, SGD, GT, NT>(GRAWA_CP_PASS);
        else launch_split<4, false, 4, 1, SGD, GT, NT>(GRAWA_CP_PASS);
        return;
    }
    switch (p->K / 8) {
        GRAWA_CP_SPLIT(3) GRAWA_CP_SPLIT(4) GRAWA_CP_SPLIT(5) GRAWA_CP_SPLIT(6) GRAWA_CP_SPLIT(7) GRAWA_CP_SPLIT(8)
    }
    hipExtLaunchKernelGGL((k_center_pull_any<SGD, GT>), dim3((unsigned)p->n_cells), dim3(GRAWA_CELL), 0, s, e0, e1, 0, x,
                          ldx, (const GT *)g, ldg, lr, beta, GRAWA_CP_STRIDE, GRAWA_CP_CELLS,
                          (const int64_t *)p->d_off, p->L, p->K, p->P, lambda, center_out, rho, moving);
#undef GRAWA_CP_PLAIN
#undef GRAWA_CP_SPLIT
}

hipError_t grawa_launch_center_pull(const grawa_plan *p, float *x, int64_t ldx, const float *beta,
                                    int per_layer, float lambda, const void *g_sgd, int64_t ldg_sgd,
                                    grawa_dtype_t dt, float lr, int fuse_sgd, float *center_out, float rho,
                                    int moving, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    // Streaming accesses pay off only when the arrays do not fit the last-level cache anyway.
    bool nt = (int64_t)p->K * p->P * 4 > GRAWA_STREAMING_MIN_BYTES && rows_line_aligned(x, ldx, 4) &&
              (!center_out || rows_line_aligned(center_out, 0, 4));
    if (fuse_sgd) nt = nt && rows_line_aligned(g_sgd, ldg_sgd, dt == GRAWA_BF16 ? 2 : 4);
    if (!fuse_sgd) {
        if (nt) dispatch_cp<false, float, true>(p, x, ldx, nullptr, 0, 0.f, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
        else dispatch_cp<false, float, false>(p, x, ldx, nullptr, 0, 0.f, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
    } else if (dt == GRAWA_BF16) {
        if (nt) dispatch_cp<true, uint16_t, true>(p, x, ldx, g_sgd, ldg_sgd, lr, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
        else dispatch_cp<true, uint16_t, false>(p, x, ldx, g_sgd, ldg_sgd, lr, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
    } else {
        if (nt) dispatch_cp<true, float, true>(p, x, ldx, g_sgd, ldg_sgd, lr, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
        else dispatch_cp<true, float, false>(p, x, ldx, g_sgd, ldg_sgd, lr, beta, per_layer, lambda, center_out, rho, moving, s, e0, e1);
    }
    return hipGetLastError();
}
