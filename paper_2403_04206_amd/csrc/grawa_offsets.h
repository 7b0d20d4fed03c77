// The index maps of a plan worked out on the device from layer offsets that the host never sees (gfx950, wave64): tiles of the
// norm pass, the layer of a cell, the tiles of a layer.
#pragma once
#include "grawa_device.h"

// Offsets are read from device memory, so they cannot be validated before the launch; they are clamped to [0, P] (and made
// monotone) wherever an address is formed from them, which keeps every access in range whatever they hold.
__device__ __forceinline__ int64_t clamp_off(int64_t v, int64_t lo, int64_t hi) { return v < lo ? lo : (v > hi ? hi : v); }

// Tile slots.  Every layer is cut at the multiples of T = 2^shift (the same cut the host-side plan makes).
// The piece of layer l in the aligned stretch j of T columns gets slot j + l: going along the row, every new piece
// starts a new stretch, a new layer or both, so slots never repeat and those of a layer are consecutive, and a
// slot is found without a count of the pieces before it.  Slots skipped where a layer starts on a multiple of T
// become tiles of length 0, whose blocks add nothing.  No slot exceeds P / T + L - 1.
__device__ __forceinline__ int64_t first_slot(int64_t off_l, int l, int64_t P, int shift) { return (clamp_off(off_l, 0, P) >> shift) + l; }

// The tile in slot i, a slot of the layer that holds columns [a, b).
__device__ __forceinline__ GrawaTile slot_tile(int64_t i, int layer, int64_t a, int64_t b, int64_t P, int shift)
{
    a = clamp_off(a, 0, P);
    b = clamp_off(b, a, P);
    const int64_t j = i - layer;
    int64_t start = j << shift, stop = (j + 1) << shift;
    if (start < a) start = a;
    if (stop > b) stop = b;
    if (stop < start) stop = start;
    GrawaTile t;
    t.start = start;
    t.len = (int32_t)(stop - start);
    t.layer = layer;
    return t;
}

// The slots [begin, end) of layer l.
__device__ __forceinline__ void layer_slots(const int64_t *__restrict__ off, int l, int64_t P, int shift, int &begin, int &end)
{
    const int64_t a = clamp_off(off[l], 0, P), b = clamp_off(off[l + 1], a, P);
    begin = (int)((a >> shift) + l);
    end = b > a ? (int)(((b - 1) >> shift) + l + 1) : begin;
}

// The last l below L for which in(l, off[l]) holds, where it holds for 0 and, in order, for no layer after the first that it
// fails for: 64 places at a time by a whole wave (one round of loads up to 64 layers, two up to 4096; a binary search by
// one lane takes six for 59).  In range whatever the offsets hold.
template <typename In> __device__ __forceinline__ int wave_last_layer(const int64_t *__restrict__ off, int L, const In &in)
{
    const int lane = threadIdx.x & (GRAWA_WAVE - 1);
    int lo = 0, n = L;
    while (n > 1) {
        const int step = (n + GRAWA_WAVE - 1) / GRAWA_WAVE, l = lo + lane * step;
        const int c = __popcll(__ballot(lane * step < n && in(l, off[lane * step < n ? l : lo])));
        const int at = c > 0 ? (c - 1) * step : 0;
        lo += at;
        n = n - at < step ? n - at : step;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}
