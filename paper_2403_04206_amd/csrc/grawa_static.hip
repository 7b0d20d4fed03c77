// LGRAWA update for callers that cannot allocate device memory (code under HIP graph capture,
// tight serving loops, harnesses that forbid hipMalloc): the same kernels as grawa_lgrawa_update,
// with the plan's workspace replaced by a fixed array that lives in the library's device image.
// The index maps a plan builds on the host are built here by one small kernel from layer
// offsets that already sit in device memory, or, for small problems, not at all: so the call enqueues kernels and nothing else.
#include <cstring>
#include <mutex>

#include "grawa_offsets.h"

#define GRAWA_STATIC_SCRATCH_BYTES ((size_t)32 << 20)
#define GRAWA_STATIC_NO_MAPS 2560 // workers times layers

// One copy per GPU the library runs on, held until the process ends.  In host code this name
// is only a handle for the symbol lookup below; the device address comes from that lookup.
static __device__ __align__(256) unsigned char scratch[GRAWA_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices]; // device address of `scratch` on every device, looked up once

hipError_t scratch_of_current_device(int *dev_out, void **ptr_out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *dev_out = dev;
    *ptr_out = g_scratch_ptr[dev];
    return hipSuccess;
}

inline size_t round256(size_t n) { return (n + 255) & ~size_t(255); }

} // namespace

// One entry of each of the maps per thread; `off` may be LDS or global memory.
__device__ __forceinline__ void static_maps_entry(const int64_t *off, int64_t i, int64_t n, int L, int64_t P, int shift,
                                                  int64_t bound, GrawaTile *__restrict__ tiles, int64_t n_cells,
                                                  int32_t *__restrict__ cell_layer, int32_t *__restrict__ tile_begin,
                                                  int32_t *__restrict__ tile_end)
{
    if (i < bound) {
        int lo = 0, hi = L - 1; // the last layer whose first slot is not above i
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (first_slot(off[mid], mid, P, shift) <= i) lo = mid;
            else hi = mid - 1;
        }
        tiles[i] = slot_tile(i, lo, off[lo], off[lo + 1], P, shift);
    }
    if (i < n_cells) {
        const int64_t first = i * GRAWA_CELL;
        const int64_t last = (first + GRAWA_CELL < P ? first + GRAWA_CELL : P) - 1;
        int lo = 0, hi = L - 1; // the last layer that starts at or before `first`
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (off[mid] <= first) lo = mid;
            else hi = mid - 1;
        }
        cell_layer[i] = off[lo + 1] > last ? (int32_t)lo : ~(int32_t)lo;
    }
    for (int64_t l = i; l < L; l += n) layer_slots(off, (int)l, P, shift, tile_begin[l], tile_end[l]);
}

// grid ceil(max(bound, n_cells)/256), block 256.  Tile i of the norm pass, the layer of 256-column cell i of
// the center+pull pass (the layer itself if the cell lies in one layer, else the complement of
// the layer of its first column) and the tile range of every layer.  The searches run in LDS when the
// offsets fit (two launches with a prefix sum and searches in global memory took 6.1 us on the device for 59 layers).
#define GRAWA_MAP_LDS_OFFSETS 2048
__global__ __launch_bounds__(GRAWA_BLOCK) void k_static_maps(const int64_t *__restrict__ off, int L, int64_t P, int shift,
                                                             int64_t bound, GrawaTile *__restrict__ tiles,
                                                             int64_t n_cells, int32_t *__restrict__ cell_layer,
                                                             int32_t *__restrict__ tile_begin,
                                                             int32_t *__restrict__ tile_end)
{
    __shared__ int64_t sm[GRAWA_MAP_LDS_OFFSETS];
    const int64_t i = (int64_t)blockIdx.x * GRAWA_BLOCK + threadIdx.x;
    const int64_t n = (int64_t)gridDim.x * GRAWA_BLOCK;
    if (L + 1 <= GRAWA_MAP_LDS_OFFSETS) {
        for (int l = threadIdx.x; l <= L; l += GRAWA_BLOCK) sm[l] = off[l];
        __syncthreads();
        static_maps_entry(sm, i, n, L, P, shift, bound, tiles, n_cells, cell_layer, tile_begin, tile_end);
    } else {
        static_maps_entry(off, i, n, L, P, shift, bound, tiles, n_cells, cell_layer, tile_begin, tile_end);
    }
}

extern "C" grawa_status_t grawa_lgrawa_update_static(int K, int64_t P, int L, const int64_t *layer_offsets_dev,
                                                     float *x, int64_t ldx, const void *g, int64_t ldg,
                                                     grawa_dtype_t dt, float lambda, float *center_out,
                                                     float *weights_out, void *stream)
{
    if (K < 1 || P < 1 || L < 1 || (int64_t)L > P || !layer_offsets_dev) return GRAWA_ERR_INVALID_ARG;
    if ((reinterpret_cast<uintptr_t>(layer_offsets_dev) & 7u) != 0) return GRAWA_ERR_ALIGNMENT;
    if (K > GRAWA_MAX_WORKERS) return GRAWA_ERR_UNSUPPORTED;
    grawa_status_t st;
    if ((st = grawa_check_params(P, x, ldx)) != GRAWA_OK) return st;
    if ((st = grawa_check_grads(P, g, ldg, dt)) != GRAWA_OK) return st;
    if ((st = grawa_check_lambda(lambda)) != GRAWA_OK) return st;
    if ((st = grawa_check_center(center_out)) != GRAWA_OK) return st;

    // The same tile length a plan would choose, so both paths add the same partial sums in the
    // same order.  Tiles: at most one per started multiple of T plus one per layer.
    const int T = grawa_default_tile_elems(K, P);
    const int64_t bound = P / T + L + 1;
    const int64_t nc = (P + GRAWA_CELL - 1) / GRAWA_CELL;
    if (bound > GRAWA_MAX_TILES || nc >= GRAWA_MAX_TILES) return GRAWA_ERR_UNSUPPORTED;
    const size_t b_cells = round256(sizeof(int32_t) * (size_t)nc);
    const size_t b_tiles = round256(sizeof(GrawaTile) * (size_t)bound);
    const size_t b_lt0 = round256(sizeof(int32_t) * ((size_t)L + 1));
    const size_t b_part = round256(sizeof(double) * (size_t)K * (size_t)bound);
    const size_t b_S = round256(sizeof(double) * (size_t)K * (size_t)L);
    const size_t b_A = round256(sizeof(float) * (size_t)K * (size_t)L);
    const size_t b_bm = round256(sizeof(float) * (size_t)K);
    if (b_cells + b_tiles + b_lt0 + b_part + b_S + 2 * b_A + b_bm > GRAWA_STATIC_SCRATCH_BYTES)
        return GRAWA_ERR_UNSUPPORTED; // the problem needs more scratch than the fixed array holds

    int dev = -1;
    void *base = nullptr;
    if (scratch_of_current_device(&dev, &base) != hipSuccess) return GRAWA_ERR_HIP;

    grawa_plan p;
    std::memset(&p, 0, sizeof(p));
    p.K = K;
    p.L = L;
    p.P = P;
    p.tile_elems = T;
    p.n_tiles = bound;
    p.n_cells = nc;
    p.device = dev;
    char *w = static_cast<char *>(base);
    p.d_off = const_cast<int64_t *>(layer_offsets_dev); // read only
    p.d_cell_layer = reinterpret_cast<int32_t *>(w); w += b_cells;
    p.d_tiles = reinterpret_cast<GrawaTile *>(w); w += b_tiles;
    p.d_layer_tile0 = reinterpret_cast<int32_t *>(w); w += b_lt0;
    p.d_partials = reinterpret_cast<double *>(w); w += b_part;
    p.d_layer_tile1 = reinterpret_cast<int32_t *>(w); w += b_S; // 4 L of the 8 K L bytes that the limit counts for S
    p.d_beta_layer = reinterpret_cast<float *>(w);

    // With the weights worked out in the pull, both kernels find their tile or cell in the offsets themselves, which saves the
    // launch that writes the maps (2.5 us and its boundary); what they repeat for it grows with the workers and the layers of a
    // cell.  Whole call, us, with maps / without, 3 layers, 59 and 200: 4 workers, 640 k columns 16.2 / 13.6, 16.5 / 13.9, 17.5 /
    // 16.0; 8 workers, 320 k 15.5 / 12.0, 16.7 / 13.5, 18.5 / 16.5; 12 workers, 213 k 15.6 / 11.9, 16.3 / 14.0, 20.3 / 18.5; 15
    // workers, 170 k 15.5 / 11.8, 16.8 / 15.1, 20.2 / 20.7.
    p.tile_shift = grawa_pull_from_tiles(&p) && (int64_t)K * L <= GRAWA_STATIC_NO_MAPS ? __builtin_ctz((unsigned)T) : 0;

    // Nothing in the scratch has to start at zero: the maps, every partial that is read and the weights
    // are written in full before they are read.
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool from_tiles = grawa_pull_from_tiles(&p);
    if (!p.tile_shift) {
        const int64_t n_map = bound > nc ? bound : nc;
        k_static_maps<<<dim3((unsigned)((n_map + GRAWA_BLOCK - 1) / GRAWA_BLOCK)), dim3(GRAWA_BLOCK), 0, s>>>(
            layer_offsets_dev, L, P, __builtin_ctz((unsigned)T), bound, p.d_tiles, nc, p.d_cell_layer, p.d_layer_tile0,
            p.d_layer_tile1);
        if (hipGetLastError() != hipSuccess) return GRAWA_ERR_HIP;
    }
    if (grawa_launch_sumsq(&p, g, ldg, dt, 0, s, nullptr, nullptr) != hipSuccess) return GRAWA_ERR_HIP;
    if (!from_tiles && grawa_launch_finalize_layers(&p, GRAWA_GOAL_LAYER_WEIGHTS, nullptr, weights_out, s) != hipSuccess)
        return GRAWA_ERR_HIP;
    if (grawa_launch_center_pull(&p, x, ldx, from_tiles ? nullptr : p.d_beta_layer, 1, lambda, nullptr, 0, GRAWA_F32,
                                 0.f, 0, center_out, 0.f, 0, weights_out, s, nullptr, nullptr) != hipSuccess)
        return GRAWA_ERR_HIP;
    return GRAWA_OK;
}
