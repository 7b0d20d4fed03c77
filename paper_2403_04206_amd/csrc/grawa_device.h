// Device-side helpers shared by the kernel files of the GRAWA update (gfx950, wave64): bf16
// widening, wave and block reductions in fp64, global-memory accessors with wave-uniform row
// bases, gradient loads by dtype and vector width, and the launch-side choice between streaming
// and cached accesses.
#pragma once
#include <hip/hip_ext.h>

#include "grawa_internal.h"

#define GRAWA_BLOCK 256
#define GRAWA_WAVE 64
#define GRAWA_CELL 256 // columns per block of the one-column-per-lane passes

// ---------------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------------

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_one(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Move a double between lanes with a DPP control word (both 32-bit halves).
template <int CTRL> __device__ __forceinline__ double dpp_move_f64(double v)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    hi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

// Sum over the 64 lanes of a wave; every lane gets the total.  Within a row of 16 lanes:
// quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror, row_mirror; across the four
// rows: two butterfly exchanges.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_move_f64<0xB1>(v);  // lane ^ 1
    v += dpp_move_f64<0x4E>(v);  // lane ^ 2
    v += dpp_move_f64<0x141>(v); // other quad of the half row
    v += dpp_move_f64<0x140>(v); // other half of the row
    v += __shfl_xor(v, 16, GRAWA_WAVE);
    v += __shfl_xor(v, 32, GRAWA_WAVE);
    return v;
}

// The same of N values side by side: the steps of one wait for nothing of the others.
template <int N> __device__ __forceinline__ void wave_sums(double (&v)[N])
{
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += dpp_move_f64<0xB1>(v[j]);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += dpp_move_f64<0x4E>(v[j]);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += dpp_move_f64<0x141>(v[j]);
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] += dpp_move_f64<0x140>(v[j]);
#pragma unroll
    for (int m = 16; m < GRAWA_WAVE; m <<= 1) {
        double w[N];
#pragma unroll
        for (int j = 0; j < N; ++j) w[j] = __shfl_xor(v[j], m, GRAWA_WAVE);
#pragma unroll
        for (int j = 0; j < N; ++j) v[j] += w[j];
    }
}

__device__ __forceinline__ double wave_min(double v)
{
    v = fmin(v, dpp_move_f64<0xB1>(v));
    v = fmin(v, dpp_move_f64<0x4E>(v));
    v = fmin(v, dpp_move_f64<0x141>(v));
    v = fmin(v, dpp_move_f64<0x140>(v));
    v = fmin(v, __shfl_xor(v, 16, GRAWA_WAVE));
    v = fmin(v, __shfl_xor(v, 32, GRAWA_WAVE));
    return v;
}

// Sum over a block through LDS; every thread gets the result.  `sm` holds one double per wave.
template <int BLOCK> __device__ __forceinline__ double block_sum(double v, double *sm)
{
    v = wave_sum(v);
    const int w = threadIdx.x / GRAWA_WAVE;
    __syncthreads();
    if ((threadIdx.x & (GRAWA_WAVE - 1)) == 0) sm[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < BLOCK / GRAWA_WAVE; ++i) t += sm[i];
    return t;
}

typedef float v2f __attribute__((ext_vector_type(2)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// Global-memory accessors for the one-element-per-lane kernels.  An address is a wave-uniform
// 64-bit base plus a 32-bit lane byte offset; the base is pinned in a scalar register pair so
// that the access is issued in that form instead of with a 64-bit address computed per lane.
// NT = streaming (non-temporal) access.
#define GRAWA_GLOBAL __attribute__((address_space(1)))

__device__ __forceinline__ uint64_t uniform_base(const void *p)
{
    uint64_t a = reinterpret_cast<uint64_t>(p);
    asm volatile("" : "+s"(a));
    return a;
}
// A float read through the scalar unit from memory this kernel never writes.
__device__ __forceinline__ float ld_uniform_f32(uint64_t base, int64_t index)
{
    return ((const __attribute__((address_space(4))) float *)base)[index];
}
template <bool NT, typename T> __device__ __forceinline__ T ld_lane(uint64_t base, unsigned byte_off)
{
    const GRAWA_GLOBAL T *p = (const GRAWA_GLOBAL T *)(base + byte_off);
    return NT ? __builtin_nontemporal_load(p) : *p;
}
// Stores.  STREAM: written through the L2 (device scope, sc1) on top of the non-temporal hint, instead of being left to the
// L2's replacement; for rows whose lines are written whole.  Only the buffer form lets both bits be asked for.  Against the
// hint alone, random values: pull of 12 rows of 102 MB 6.31 -> 6.43 TB/s (plain stores 5.55), LGRAWA of the 350 M
// transformer with 8 workers 4411 -> 4279 us, Nesterov step of 36.5 M columns x 8 workers 922 -> 889 us; 0 to 2 % elsewhere.
// MERGE: the hint alone.  For rows off the line grid: where a wave's piece ends inside a line, the L2 holds that part
// until the neighbour's part has come, while STREAM sends both parts on as writes of their own.  8 rows of 50 M
// columns, 32 bytes off a line, streaming loads, TB/s, STREAM / MERGE: step with center and scores fp32 5.88 / 6.08, bf16 5.76 / 6.00,
// plain step 5.90 / 6.13.
enum { GRAWA_ST_CACHED = 0, GRAWA_ST_MERGE = 2, GRAWA_ST_STREAM = 18 }; // the cache bits of the buffer store
template <int ST, typename T> __device__ __forceinline__ void st_lane(uint64_t base, unsigned byte_off, T v)
{
    if constexpr (ST != GRAWA_ST_CACHED) {
        __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(base), 0, -1, 0x00020000);
        if constexpr (sizeof(T) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, (int)byte_off, 0, ST);
        else if constexpr (sizeof(T) == 8)
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2u, v), r, (int)byte_off, 0, ST);
        else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), r, (int)byte_off, 0, ST);
    } else {
        *(GRAWA_GLOBAL T *)(base + byte_off) = v;
    }
}

// acc + v^2 with the value widened first: one fp64 fused multiply-add.
__device__ __forceinline__ double sq_add(float v, double acc)
{
    const double d = (double)v;
    return fma(d, d, acc);
}

// Gradient element access.  VEC8 = elements per 8-byte load (norm pass).
template <typename GT> struct Grad;

template <> struct Grad<float> {
    static constexpr int VEC8 = 2;
    static __device__ __forceinline__ float one(const float *p) { return *p; }
    template <bool NT> static __device__ __forceinline__ float lane(uint64_t base, unsigned off)
    {
        return ld_lane<NT, float>(base, off);
    }
    // 8 bytes (2 floats) at p, 8-byte aligned; and their squares added to acc.
    // The square of a widened fp32 (or bf16) value is exact in fp64, so no gradient magnitude
    // that the input type can hold underflows or overflows here.
    typedef v2f Vec8;
    template <bool NT> static __device__ __forceinline__ Vec8 load8(const float *p)
    {
        const v2f *q = reinterpret_cast<const v2f *>(p);
        return NT ? __builtin_nontemporal_load(q) : *q;
    }
    static __device__ __forceinline__ double sumsq8(Vec8 q, double acc)
    {
        acc = sq_add(q.x, acc);
        acc = sq_add(q.y, acc);
        return acc;
    }
};

template <> struct Grad<uint16_t> { // bfloat16 bit patterns
    static constexpr int VEC8 = 4;
    static __device__ __forceinline__ float one(const uint16_t *p) { return bf16_one(*p); }
    template <bool NT> static __device__ __forceinline__ float lane(uint64_t base, unsigned off)
    {
        return bf16_one(ld_lane<NT, uint16_t>(base, off));
    }
    // 8 bytes (4 bf16) at p, 8-byte aligned; and their squares added to acc
    typedef v2u Vec8;
    template <bool NT> static __device__ __forceinline__ Vec8 load8(const uint16_t *p)
    {
        const v2u *q = reinterpret_cast<const v2u *>(p);
        return NT ? __builtin_nontemporal_load(q) : *q;
    }
    static __device__ __forceinline__ double sumsq8(Vec8 q, double acc)
    {
        acc = sq_add(bf16_lo(q.x), acc);
        acc = sq_add(bf16_hi(q.x), acc);
        acc = sq_add(bf16_lo(q.y), acc);
        acc = sq_add(bf16_hi(q.y), acc);
        return acc;
    }
};

// V gradient elements (naturally aligned) widened to float; `lane` takes a wave-uniform base and the
// lane's byte offset.
template <typename GT, int V, bool NT> struct GradVec;
template <bool NT> struct GradVec<float, 2, NT> {
    static __device__ __forceinline__ void lane(uint64_t base, unsigned off, float (&f)[2])
    {
        const v2f w = ld_lane<NT, v2f>(base, off);
        f[0] = w.x;
        f[1] = w.y;
    }
};
template <bool NT> struct GradVec<float, 1, NT> {
    static __device__ __forceinline__ void load(const float *p, float (&f)[1]) { f[0] = NT ? __builtin_nontemporal_load(p) : *p; }
};
template <bool NT> struct GradVec<float, 4, NT> {
    static __device__ __forceinline__ void lane(uint64_t base, unsigned off, float (&f)[4])
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f w = ld_lane<NT, v4f>(base, off);
        f[0] = w.x;
        f[1] = w.y;
        f[2] = w.z;
        f[3] = w.w;
    }
    static __device__ __forceinline__ void load(const float *p, float (&f)[4])
    {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const v4f *q = reinterpret_cast<const v4f *>(p);
        const v4f w = NT ? __builtin_nontemporal_load(q) : *q;
        f[0] = w.x;
        f[1] = w.y;
        f[2] = w.z;
        f[3] = w.w;
    }
};
template <bool NT> struct GradVec<uint16_t, 2, NT> {
    static __device__ __forceinline__ void lane(uint64_t base, unsigned off, float (&f)[2])
    {
        const uint32_t w = ld_lane<NT, uint32_t>(base, off);
        f[0] = bf16_lo(w);
        f[1] = bf16_hi(w);
    }
    static __device__ __forceinline__ void load(const uint16_t *p, float (&f)[2])
    {
        const uint32_t *q = reinterpret_cast<const uint32_t *>(p);
        const uint32_t w = NT ? __builtin_nontemporal_load(q) : *q;
        f[0] = bf16_lo(w);
        f[1] = bf16_hi(w);
    }
};
template <bool NT> struct GradVec<uint16_t, 4, NT> {
    static __device__ __forceinline__ void lane(uint64_t base, unsigned off, float (&f)[4])
    {
        const v2u w = ld_lane<NT, v2u>(base, off);
        f[0] = bf16_lo(w.x);
        f[1] = bf16_hi(w.x);
        f[2] = bf16_lo(w.y);
        f[3] = bf16_hi(w.y);
    }
    static __device__ __forceinline__ void load(const uint16_t *p, float (&f)[4])
    {
        const v2u *q = reinterpret_cast<const v2u *>(p);
        const v2u w = NT ? __builtin_nontemporal_load(q) : *q;
        f[0] = bf16_lo(w.x);
        f[1] = bf16_hi(w.x);
        f[2] = bf16_lo(w.y);
        f[3] = bf16_hi(w.y);
    }
};
template <int V> struct FloatVec { typedef float T __attribute__((ext_vector_type(V))); };
template <> struct FloatVec<1> { typedef float T; };
template <int V> __device__ __forceinline__ float vec_get(const typename FloatVec<V>::T &v, int c)
{
    if constexpr (V == 1) return v;
    else return v[c];
}
template <int V> __device__ __forceinline__ void vec_set(typename FloatVec<V>::T &v, int c, float f)
{
    if constexpr (V == 1) v = f;
    else v[c] = f;
}

// From what size of x (K P floats; of x and g in a pull with the SGD step) on a pass streams past the caches.  The lines lie where the pass is faster on
// arrays that the caches do not hold when it starts, as after a backward pass.  Cached against streaming, us, on three
// such sets in turn (in brackets: one set again and again, which the 256 MB last-level cache partly holds):
//   pull            MGRAWA, 4 workers,  80 MB x: 43.0/42.5 (38/39), 120 MB: 75/69, 187 MB: 102.8/93.2 (87.2/90.5)
//   Nesterov step   8 workers, x 80 MB: 1.13 x faster (0.9), 120 MB 1.13 (1.06), 160 MB 1.15 (1.15)
//   step with center or scores: 80 MB 1.04 to 1.21 (0.98 to 1.12), 160 MB 1.22 (1.12); 40 MB 0.96.  Scored, aligned rows, 4
//   and 52 workers: 90 MB 56.3/49.6 and 55.0/49.1 (45.7/49.2 and 44.7/48.7), after a pass over x, g and 256 MB of other memory
//   67.6/52.0 and 67.3/50.8.  With the center, off the line grid (cached loads, stores written through; fp32 streams its loads now): 90 MB 58.2/53.7 and 49.9/44.9 (49.6/49.9 and 41.1/42.8),
//   after such a pass 72.1/71.8 and 62.0/61.1.  What the line costs: a step that finds its arrays in the cache, two scored steps
//   and the communication, 8 workers, 95 MB 131/140; one scored step after a pass that leaves them there, 70 MB 34.9/38.3.
//   plain SGD step: 187 MB 100.5/90.2 alone, but the pull that follows finds x in the cache after a cached one: step
//   and EASGD phase 158.4/164.0; 400 MB 211/189 alone, 344/347 with the phase.
// A pull of an array of 134 to 250 MB that a small iteration leaves in the cache is slower for its line (4 workers, 140 MB
// 59.6/65.7 with nothing else touched between, 61.8/60.3 with 64 MB per worker).
#define GRAWA_STREAMING_MIN_BYTES ((int64_t)128 << 20)
#define GRAWA_STREAMING_MIN_ROW_BYTES ((int64_t)64 << 20)
#define GRAWA_STREAMING_MIN_SGD_BYTES ((int64_t)256 << 20)

// Streaming accesses are used only when no cache line is shared between two rows or written
// in two parts: base pointers and row pitches are multiples of 128 bytes.
static inline bool rows_line_aligned(const void *base, int64_t ld, int elem_bytes)
{
    return (reinterpret_cast<uintptr_t>(base) % 128u) == 0 && ((ld * elem_bytes) % 128) == 0;
}
