// The rules that choose between kernels and launch shapes, and what host and device share of the running estimate.  Plain C++ with no GPU
// dependency, so that they can be checked on the CPU for sizes that no test allocates.
#ifndef GRAWA_ROUTE_H
#define GRAWA_ROUTE_H

#include <stdint.h>

// Blocks of one launch of the row-split form, one per 256-column cell, from cell `at` on.  Its blocks have 1024 threads
// and a launch takes fewer than 2^32 threads in x, which one launch for all would exceed from 2^30 columns on (plans go to
// 2^32): so at most 2^18 cells (67 M columns) a launch, far below the limit so that tests reach a second launch.  (All cells
// in one launch, as rows of a two-dimensional grid, cost the blocks a multiplication and a test: 16 workers, 1.5 M columns
// 29.3 -> 29.9 us.)
#define GRAWA_SPLIT_THREADS 1024
#define GRAWA_SPLIT_LAUNCH_CELLS ((int64_t)1 << 18)
static inline int64_t grawa_split_blocks(int64_t n_cells, int64_t at)
{
    return n_cells - at < GRAWA_SPLIT_LAUNCH_CELLS ? n_cells - at : GRAWA_SPLIT_LAUNCH_CELLS;
}

// Form of the pull of large rows off the line grid (16-byte lanes, grawa_pull.hip): the wide form, or row-split bursts with
// `groups` groups of waves; plain: the forms of the other rows.  merge: streaming loads and stores that the L2 merges, else cached loads and
// stores written through.  The dispatch is made from this rule; why the lines lie here stands at the kernels.
enum { GRAWA_OFF_GRID_PLAIN = 0, GRAWA_OFF_GRID_WIDE = 1, GRAWA_OFF_GRID_BURST = 2 };
struct GrawaOffGrid {
    int form, groups;
    bool merge;
};
// Bursts of a pull without the SGD step, of the counts whose other form leaves x in the last-level cache, from 320 MB of x on.  MGRAWA, us,
// that form / bursts, one set again and again and three sets in turn: 8 workers 134 MB 73 / 78 and 81 / 79, 200 MB 103 / 113 and 118 / 113, 260 MB
// 139 / 145 and 144 / 147, 400 MB 223 / 214 and 227 / 213; 32 workers 134 MB 78 / 88 and 89 / 89, 200 MB 109 / 123 and 128 / 124, 260 MB
// 150 / 156 and 164 / 157, 400 MB 245 / 244 and 250 / 240; 64 workers 200 MB 116 / 136 and 141 / 137, 400 MB 259 / 252 and 264 / 251.
#define GRAWA_BURST_MIN_BYTES ((int64_t)320 << 20)
static constexpr bool grawa_off_grid_large(int K, bool sgd, int64_t bytes, int64_t large)
{
    return bytes > (!sgd && ((K >= 6 && K <= 11) || K >= 24) ? GRAWA_BURST_MIN_BYTES : large);
}
static constexpr GrawaOffGrid grawa_off_grid(int K, bool f32_sgd)
{
    // Wide, up to 5 workers, the step with fp32 gradients.  LGRAWA with the step, us, cached loads / streaming: 2 workers 140 MB
    // 98.2 / 94.1, 1.2 GB 783 / 775, 3 200 MB 137.6 / 133.7, 1.2 GB 808 / 800, 4 99.3 / 98.1 and 789 / 787, 5 100.4 / 98.9 and 820 /
    // 798; MGRAWA without it 2 477 / 481, 3 482 / 489, 4 491 / 507, 5 489 / 498; with bf16 gradients 140 MB 4 workers 80.3 / 83.2, 5
    // 80.1 / 82.5.
    if (K <= 5) return {GRAWA_OFF_GRID_WIDE, 1, f32_sgd};
    if (f32_sgd && K >= 12 && K <= 23) return {GRAWA_OFF_GRID_WIDE, 1, false};
    if (K > 71) return {GRAWA_OFF_GRID_PLAIN, 1, false};
    return {GRAWA_OFF_GRID_BURST, K <= 9 ? 2 : K <= 23 ? 4 : 8, K <= 15};
}
// The counts that have a kernel each; the others share one by K / 8.
#define GRAWA_OFF_GRID_EACH(X) \
    X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20) X(21) X(22) X(23)
#define GRAWA_OFF_GRID_EIGHTHS(X) X(3) X(4) X(5) X(6) X(7) X(8)
static constexpr bool grawa_off_grid_has_kernel(int K, bool f32_sgd)
{
    const GrawaOffGrid f = grawa_off_grid(K, f32_sgd);
    if (f.form == GRAWA_OFF_GRID_PLAIN) return true; // any count
#define GRAWA_COUNT_IS(N) || K == N
#define GRAWA_EIGHTH_IS(N) || K / 8 == N
    if (false GRAWA_OFF_GRID_EACH(GRAWA_COUNT_IS)) return f.form == GRAWA_OFF_GRID_WIDE || K >= f.groups;
    return f.form == GRAWA_OFF_GRID_BURST && f.groups == 8 && !f.merge && (false GRAWA_OFF_GRID_EIGHTHS(GRAWA_EIGHTH_IS));
#undef GRAWA_COUNT_IS
#undef GRAWA_EIGHTH_IS
}

// The worker counts that have a kernel of the form with the weights from the tile sums.  The rule below and the dispatch
// (grawa_pull.hip) are made from the same list.
#define GRAWA_TILES_COUNTS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
#define GRAWA_COUNT_TRUE(N) \
    case N: return true;
static inline bool grawa_tiles_has_kernel(int K)
{
    switch (K) {
        GRAWA_TILES_COUNTS(GRAWA_COUNT_TRUE)
    }
    return false;
}

// Per-layer weights: worked out by every block of the pull for the layers of its own cell, or by a launch of their own.
// The work in the pull grows with the blocks, with the tiles of the longest layer (with one layer, each of the blocks
// adds all tiles of it) and with the workers; what it saves is one launch.  With fewer than 4 workers the lanes of a wave
// share few sums, and the line is that of 4 workers.  Whole update on the device, us, a launch / in the pull, one layer
// and 60 layers: 1 worker, 400 k columns 8.6 / 7.3 and 9.5 / 7.5, 655 k 9.1 / 9.4 and 9.8 / 8.9, 2.6 M 12.8 / 19.2 and
// 13.3 / 16.8; 2 workers, 655 k 9.9 / 9.7 and 10.4 / 9.4, 1.3 M 11.8 / 14.1 and 12.6 / 12.8; 4 workers, 400 k
// 10.2 / 8.6 and 10.9 / 8.6, 655 k 11.3 / 11.6 and 12.2 / 11.0; 15 workers, 175 k 11.4 / 10.0 and 13.9 / 13.1.
// Without the launch the host saves 1 to 4 us of a call as well.  Slower from 4 x 1.2 M (20.3 / 20.8) and 16 x 600 k
// (31.6 / 33.8) on.
#define GRAWA_TILES_MAX_CELLS 10240 // cells times workers
static inline bool grawa_weights_in_pull(int K, int64_t n_cells)
{
    return grawa_tiles_has_kernel(K) && n_cells * (K < 4 ? 4 : K) <= GRAWA_TILES_MAX_CELLS;
}

// The one-column-per-lane (plain) form serves up to 23 workers, and up to 32 on few cells: there a block of the row-split form,
// with its barrier and four times the threads, is the longer chain.  Split against plain, time of the pull by per-layer
// weights, 24 / 28 / 32 workers, 1 layer, 40 layers and 500: 5 k columns 1.04 1.16 1.30 / 1.07 1.21 1.29 / 1.00 1.18 1.31,
// 105 k 1.09 1.17 1.30 / 1.10 1.20 1.30 / 1.06 1.15 1.30, 200 k 1.10 1.07 1.14 / 1.11 1.10 1.16 / 1.07 1.01 1.10,
// 300 k 1.07 1.02 1.05 / 1.03 0.96 0.96 / 0.98 0.92 0.92, 1 M 1.01 0.98 0.92 / 1.01 0.99 0.94 / 1.00 0.99 0.96.  In a local
// round of 31 workers on 252 k columns (985 cells) the split form is 0.4 us faster, so the line lies at 800 cells.
#define GRAWA_PLAIN_MAX_WORKERS 23
#define GRAWA_PLAIN_FEW_CELLS 800
#define GRAWA_PLAIN_FEW_CELLS_MAX_WORKERS 32
static inline bool grawa_plain_form(int K, int64_t n_cells)
{
    return K <= (n_cells <= GRAWA_PLAIN_FEW_CELLS ? GRAWA_PLAIN_FEW_CELLS_MAX_WORKERS : GRAWA_PLAIN_MAX_WORKERS);
}

// Model-level weights: by the last block of the launch that forms the layer norms, or by a launch of its own.  The last
// block saves the host a launch (a call of 4 workers that is host-bound: 17 us for 21) and the device nothing; every
// layer's arrival and every norm handed over cost, so that from about 100 layers on the device loses.  Whole update
// on the device, us, own launch / last block:
//   4 workers, 262 k columns:  20 layers 11.5 / 11.5, 60 11.6 / 11.8, 100 12.2 / 12.5, 160 12.2 / 13.8, 1000 22.4 / 32.5
//   16 workers, 200 k:         20 16.5 / 16.2, 60 17.1 / 17.1, 100 18.2 / 19.0, 160 20.4 / 21.5, 1000 41.5 / 52.1
//   64 workers, 200 k:         20 40.1 / 39.8, 60 44.3 / 44.3, 100 48.9 / 49.8, 160 57.2 / 58.4, 1000 152 / 164
#define GRAWA_LAST_BLOCK_MAX_LAYERS 100
static inline bool grawa_model_weights_by_last_block(int L) { return L <= GRAWA_LAST_BLOCK_MAX_LAYERS; }

// Launch of the running estimate (of plans that neither leave their sums to the next launch nor go by layers, below; of the sizes quoted here those
// with few layers do now): y rows of blocks per layer and threads of a block.  max_tiles: the most 1024-column
// tiles that a layer has.  Layers of up to GRAWA_EST_WAVE_TILES tiles take a wave per worker, or, where there are many
// layers (GRAWA_EST_BLOCKS blocks fill the chip), a wave per few workers: starting a wave costs more than such a sum.
// A longer layer takes a block of 512 threads per worker, as long as that keeps the launch within
// GRAWA_EST_LONG_BLOCKS blocks for all layers.  Scored step and estimate on the device, us, one block of 1024 per layer /
// a block per layer and worker from 2^20 columns on, a wave below / this:
//   8 workers, 1.05 M columns:   250 layers 24.4 / 24.7 / 23.3, 5000 layers 57.5 / 78.6 / 37.5
//   15 workers, 1.05 M:          1000 layers 40.2 / 53.5 / 38.3
//   64 workers, 300 k:           1000 layers 55.6 / 70.6 / 55.5;  1.05 M, 5000 layers 223 / 586 / 196
// With few sums (GRAWA_EST_FEW_BLOCKS) nothing but the longest one counts: the block per worker already from 129 tiles
// on, and waves in blocks of 8.  A block or wave as above / the rule for many / this: 7 workers, 2.1 M
// columns, 11 layers 29.8 / 31.0 / 29.9; 8 workers, 1.1 M, 3 layers 20.3 / 21.2 / 20.5; 31 workers, 252 k, 6 layers
// 19.2 / 19.9 / 19.5; from 256 tiles on 30.0, 20.6 and 19.9.
#define GRAWA_EST_MAX_THREADS 1024
#define GRAWA_EST_WAVE_TILES 1024
#define GRAWA_EST_BLOCKS 512
#define GRAWA_EST_LONG_BLOCKS 4096
#define GRAWA_EST_FEW_BLOCKS 512
#define GRAWA_EST_WAVE_TILES_FEW 128
static inline void grawa_estimate_shape(int K, int L, int64_t max_tiles, int *rows, int *threads, int *wave_tiles)
{
    const bool few = (int64_t)K * L <= GRAWA_EST_FEW_BLOCKS;
    *wave_tiles = few ? GRAWA_EST_WAVE_TILES_FEW : GRAWA_EST_WAVE_TILES;
    const bool longest = max_tiles > *wave_tiles;
    const int most = few ? 8 : 16;
    const int waves = longest ? 8 : K < most ? K : most;
    const int all = (K + waves - 1) / waves, fill = (longest ? GRAWA_EST_LONG_BLOCKS : GRAWA_EST_BLOCKS) / L;
    const int want = longest ? K : all;
    *rows = fill < 1 ? 1 : fill < want ? fill : want;
    *threads = waves * 64;
}

// Columns of g that the norm pass of an update fused with the step on the same g reads through the caches, so that the pull
// finds them in the 256 MB last-level cache; what is streamed does not displace them.  Bounded by bytes: beyond the
// cache's size it only costs the norm pass its streaming rate (7.1 against 6.2 TB/s).  Whole update, three sets in turn, us, x and
// gradient type, none / 64 / 128 / 192 / 224 / 256 MB cached: 4 workers 20 MB fp32 21.5 / 20.5 / 20.5 / 20.6 / 20.3 / 20.6, 200 MB
// bf16 100.3 / 97.1 / 95.9 / 95.9 / 95.8 / 95.9, 400 MB fp32 246 / 244 / 243 / 243 / 243 / 250; 12 workers 200 MB fp32 147 / 141 / 136
// / 135 / 135 / 134, 400 MB bf16 206 / 197 / 189 / 185 / 185 / 183; 32 workers 150 MB fp32 126 / 118 / 106 / 104 / 104 / 105, 260 MB
// 179 / 175 / 169 / 163 / 162 / 161, 800 MB 536 / 528 / 522 / 517 / 512 / 509, 3.2 GB 2166 / 2157 / 2155 / 2154 / 2143 / 2146, no more than runs
// differ by.  Norm pass and pull apart, 32 workers, none / 224 MB: 150 MB 26.9 / 27.6 and 84.6 / 71.1, 260 MB 43.8 / 45.7 and 138.7 / 119.5, 3.1 GB
// 464 / 471 and 1714 / 1715.  (The L2's traffic counters do not tell: they count what it asks for, whoever answers.)
#define GRAWA_CACHED_GRAD_BYTES ((int64_t)224 << 20)
static inline int64_t grawa_cached_grad_cols(int K, int64_t P, int elem_bytes)
{
    const int64_t cols = GRAWA_CACHED_GRAD_BYTES / ((int64_t)K * elem_bytes);
    return cols < P ? cols : P;
}

// Local steps (k_row_step) over large rows off the line grid: the bytes of x beyond which loads stream and the L2 merges the stores.  Up to
// there loads are cached and stores written through, which leaves part of the arrays to the next pass.  0: at any size.  Three sets in
// turn, us, up to the line / beyond it, 3 to 5 workers (in brackets one set again and again):
//   scored, a round of four steps and the communication: fp32 100 MB 258 / 259 (250 / 261), 180 MB 435 / 443 (424 / 450), 260 MB 624 / 635
//   (582 / 618), 300 MB 736 / 725 (700 / 721), 350 MB 875 / 845 (868 / 835), 1.5 GB 3695 / 3535; of one step and it: 100 MB 104 / 94
//   (90 / 92), 260 MB 235 / 226 (216 / 225), 350 MB 311 / 303.  bf16 four steps 100 MB 227 / 231 (218 / 229), 260 MB 535 / 547 (526 / 548),
//   400 MB 789 / 819 (776 / 821), 700 MB 1425 / 1421, 1.5 GB 3097 / 3068, 2.5 GB 4945 / 4995; one step 100 MB 94 / 88 (84 / 87), 260 MB
//   210 / 208 (202 / 208)
//   scored with the center, four steps: fp32 260 MB 729 / 665 (718 / 658); bf16 260 MB 599 / 596 (581 / 596), 500 MB 1205 / 1137; one step
//   231 / 222 (216 / 220) and 433 / 421; 40 workers, four steps, 220 MB 564 / 578, 400 MB 1001 / 1017
//   with the center alone: fp32 100 MB 58.7 / 51.8, bf16 70 MB 32.2 / 33.8, 100 MB 44.0 / 45.8, 180 MB 91.7 / 84.9 (82.7 / 84.1)
#define GRAWA_ROW_STEP_NEVER INT64_MAX
static constexpr int64_t grawa_row_step_merges_from(bool bf16, bool center, bool scored)
{
    if (scored && !center) return bf16 ? GRAWA_ROW_STEP_NEVER : (int64_t)320 << 20;
    return bf16 && center && !scored ? (int64_t)128 << 20 : 0;
}

// Scored step: whether a block of 256 threads owns a layer of one worker and updates the estimate itself.  One launch saves the other and its
// boundary; what it costs is that the longest layer takes one block, at the rate of one CU.  max_tiles: the most 1024-column tiles of a
// layer.  (Of the most blocks that are accepted a fifth starts in a second round.)  A round of four steps and the communication, fp32, us:
//   up to 7 tiles, against the estimate as a launch of its own: 2 workers, 200 k columns, 300 layers 47.3 / 39.0; 8 workers, 200 k, 20 layers
//   52.5 / 43.8, 300 layers 55.2 / 40.4; against sums left to the next launch (below), replayed: 4 workers, 200 k, 300 layers 34 / 29.4
//   8 to 10 tiles, sums left to the next launch / by layers, without and with the center: with many columns 4 workers, 100 layers of 9 k 43.5 /
//   41.6 and 55.4 / 47.0, 2 workers, 220 of them 46.1 / 43.9 and 59.4 / 57.0; with fewer 8 workers, 30 of them 32.8 / 34.6 and 33.3 / 37.0, 16
//   workers, 14 of them 35.1 / 34.0 and 35.6 / 36.7; with many blocks 16 workers, 4 of them and 60 of 2 k 39.5 / 43.5 and 39.9 / 47.8
#define GRAWA_LAYER_TILES 7
#define GRAWA_LAYER_MAX_ELEMS ((int64_t)1 << 22)
#define GRAWA_LAYER_MAX_BLOCKS 2560
#define GRAWA_LAYER_MANY_TILES 10
#define GRAWA_LAYER_MANY_ELEMS ((int64_t)3 << 20)
#define GRAWA_LAYER_MANY_MAX_BLOCKS 640
static inline bool grawa_step_by_layers(int K, int L, int64_t P, int64_t max_tiles)
{
    const int64_t blocks = (int64_t)K * L, elems = (int64_t)K * P;
    if (elems > GRAWA_LAYER_MAX_ELEMS) return false;
    if (elems > GRAWA_LAYER_MANY_ELEMS && blocks <= GRAWA_LAYER_MANY_MAX_BLOCKS) return max_tiles <= GRAWA_LAYER_MANY_TILES;
    return max_tiles <= GRAWA_LAYER_TILES && blocks <= GRAWA_LAYER_MAX_BLOCKS;
}

// Scored step: whether its tile sums are left to the launch that needs them next (grawa_fold.h) instead of a launch of their own.
// It saves that launch and its boundary, about 5 us on the device and 3 on the host, for every step but the last of a round, and
// against a block per layer (k_layer_step with 1024 threads, which it replaced) the time one CU takes for the longest layer.  A round of four
// steps with the center and the communication, fp32, us, before / now (in brackets replayed as a graph): ResNet-20, 59 layers, 4 workers 42.7 / 28.1
// (42.7 / 28.0), 8 workers 48.0 / 34.3 (48.1 / 34.5), both with the weights in the pull (below); 16 workers, 200 k columns, 150 layers 68.7 / 49.5 (69.1 / 50.2); 4 workers, 1 M, one layer 67.3 /
// 59.7 (67.9 / 60.6), 60 layers 71.9 / 61.0; 64 workers, 300 k, 100 layers 198 / 188; 16 workers, 3 M 510 / 493; 2 workers, 20 M, one layer 428 / 409.
// What it costs: a recording's first step has a launch of its own as well (grawa_step_buffer), and the kernels that fold in read more than
// those that they replace.  Rounds of one step, us, before / now (in brackets captured, a graph's launch included): 8 workers, one layer of 8 M
// 204.6 / 205.5 (209.3 / 210.0), 4 steps 573 / 557; 2 workers, 30 M 195.6 / 196.3 (200.4 / 201.7), 549 / 531; 64 workers, 1 M 214.2 / 214.9 (218.6 / 220.1),
// 572 / 563; behind another kernel of 28 us ResNet-20 on 4 workers (40.1 / 39.5), and, where a block of 1024 threads took the layers before, 8 workers,
// 12 layers of 12 k (37.0 / 38.6), 32 workers, one layer of 18 k (36.1 / 37.7), 4 workers, 9 k and 58 of 2 k (34.9 / 35.8), 2
// workers, 60 layers of 8.7 k (37.2 / 39.9, four steps 50.9 / 52.2).  A step and the communication captured apart, 8 workers, 8 M 215.8 / 219.9: the
// communication cannot know that nothing is left to fold in.
// The lines.  Beyond 2^17 blocks a step lasts 200 us and more, and the buffers take memory.  Layers: every one is a wave's work for each worker in the step
// and a block in the launch of the weights: 4 workers, 2000 layers of 400 columns, four steps and one 66.5 / 54.5 and 29.1 / 25.7, 4000 layers
// 106 / 97.5 and 38.5 / 39.4, 2 workers, 8000 116 / 104 and 44.6 / 48.3.  Sums: 64 workers, 300 layers 110 / 91 and 39 / 33, 8 workers, 5000
// 177 / 171 and 61.8 / 63.7, 100 workers, 1000 465 / 501 and 190 / 192.  Where some layer is longer than a wave adds, a block for every sum: 8 workers, 600 k columns and
// 127 layers of 700 78.8 / 65.5 and 28.9 / 27.5, 255 84.8 / 79.1 and 30.9 / 34.6, 400 92.2 / 91.6 and 33.9 / 40.8.
#define GRAWA_FOLD_MAX_BLOCKS ((int64_t)1 << 17)
#define GRAWA_FOLD_MAX_LAYERS 2048
#define GRAWA_FOLD_MAX_UNITS 20480     // workers times layers
#define GRAWA_FOLD_MAX_UNITS_LONG 1024 // where some layer is longer than a wave adds
#define GRAWA_FOLD_WAVE_TILES 512      // up to here a wave adds the tiles of a layer, beyond it a block
static inline bool grawa_fold_later(int K, int L, int64_t P, int64_t max_tiles)
{
    if (grawa_step_by_layers(K, L, P, max_tiles) || L > GRAWA_FOLD_MAX_LAYERS) return false;
    const int64_t units = max_tiles > GRAWA_FOLD_WAVE_TILES ? GRAWA_FOLD_MAX_UNITS_LONG : GRAWA_FOLD_MAX_UNITS;
    return (int64_t)K * ((P + 1023) / 1024) <= GRAWA_FOLD_MAX_BLOCKS && (int64_t)K * L <= units;
}

// Where the blocks of a scored step that fold in the sums before stand in its grid (group, K, n_groups): at the head of each row, or as rows ahead of the
// workers', whatever takes fewer blocks.  The length of a row, modulo 8, decides which XCD a column goes to from row to row, and with it what lies in its
// L2, so it stays as it is (64 workers, 256 k columns, a step 28.5 us without such blocks, 33.0 with one at the head of each row, 28.9 so; with the center 28.8,
// 35.3, 28.7; 16 workers, four layers of 64 k, a round of four steps 49.5 -> 41.7).  With the center it becomes a multiple of 8, so that all rows read a
// column of it from one XCD: rounds of four steps, us, as it is / so: 8 workers, 1 M columns 94.3 / 80.1, 3 M 257 / 223, 16 workers, 1 M 171 / 145, 3 M
// 500 / 429, 32 workers, 250 k 83.2 / 79.5, 3 M 967 / 824.  Not for short rows and many workers: 64 workers, 60 k 43.5 / 45.9, 500 k 289 / 298, 24 workers,
// 128 k 37.8 / 39.4.
#define GRAWA_FOLD_ALIGN_GROUP 200
#define GRAWA_FOLD_ALIGN_WORKERS 40
static inline void grawa_fold_blocks(int K, int L, int64_t max_tiles, bool center, int64_t group, int64_t n_groups, unsigned *blocks, unsigned *rows)
{
    const int64_t units = (int64_t)K * L, all = max_tiles <= GRAWA_FOLD_WAVE_TILES ? (units + 3) / 4 : units;
    const bool align = center && group >= GRAWA_FOLD_ALIGN_GROUP && K <= GRAWA_FOLD_ALIGN_WORKERS;
    const int64_t least = (all + K * n_groups - 1) / (K * n_groups), from = align ? group : 0;
    const int64_t head = (from + least + 7) / 8 * 8 - from, ahead = (all + group - 1) / group;
    const bool apart = n_groups == 1 && ahead * group < head * K && !(align && group % 8);
    *blocks = apart ? 0 : (unsigned)head;
    *rows = apart ? (unsigned)ahead : 0;
}

// Whether the launch of the per-layer weights adds what is pending itself.  Layers that a wave adds: as long as its 16 waves do not walk many workers with many
// tiles.  One step and the communication, one layer, us, k_fold before / this: 64 workers, 125 tiles 33.8 / 34.5, 250 61.1 / 63.2, 500 110.9 / 114.4; 48, 125 28.7 /
// 28.6, 250 48.3 / 49.2; 38, 250 40.3 / 40.7; 32, 250 36.2 / 35.9, 500 59.0 / 59.2; 16, 60 14.5 / 12.7.  Longer layers: up to 8 workers, whose parts its 16 waves take at once, and 4096 tiles, 8 of
// them to a lane.  Else k_fold goes before, a launch of 5 us.  One step and the communication, us, k_fold / this: 2 workers, one layer of 600 k
// columns and 250 of 3 k 24.4 / 21.5, of 1.5 M alone 23.6 / 21.4; 8 workers, 600 k alone 26.1 / 24.7, ResNet-18 295.4 / 293.9; beyond, 16 workers
// (twice as many parts): 600 k alone 39.0 / 38.9, three of 2 M 310 / 314.
#define GRAWA_FOLD_LONG_WORKERS 8
#define GRAWA_FOLD_LONG_TILES 4096
#define GRAWA_FOLD_WORKERS 32
#define GRAWA_FOLD_TILES 8000 // of a layer, times workers
static inline bool grawa_fold_in_weights(int K, int64_t max_tiles)
{
    if (max_tiles > GRAWA_FOLD_WAVE_TILES) return K <= GRAWA_FOLD_LONG_WORKERS && max_tiles <= GRAWA_FOLD_LONG_TILES;
    return K <= GRAWA_FOLD_WORKERS || max_tiles * K < GRAWA_FOLD_TILES;
}

// Whether the one block of the model-level weights adds what is pending itself: as long as a thread has one worker and layer, and its 16 waves a
// longer one each.  Else k_fold goes before.  One step and the communication, us, k_fold / this: 4 workers, one layer of 9 k 11.6 / 9.1, and 58 of 2 k
// 13.4 / 12.2; beyond, 8 workers, 12 layers of 12 k (96 longer ones) 16.4 / 17.9, ResNet-20 on 8 (40) 21.2 / 25.1.
#define GRAWA_FOLD_MODEL_UNITS 1024
#define GRAWA_FOLD_MODEL_WAVES 16
static constexpr int64_t grawa_thread_tiles(int lanes) { return lanes < 16 ? lanes : 16; } // whose sum a thread adds in the order of `lanes` lanes
static inline bool grawa_fold_in_model_weights(int K, int L, int64_t max_tiles, int64_t longer)
{
    return (int64_t)K * L <= GRAWA_FOLD_MODEL_UNITS && (int64_t)K * longer <= GRAWA_FOLD_MODEL_WAVES && max_tiles <= GRAWA_FOLD_WAVE_TILES;
}

// Lanes of a wave that share a worker's tiles where the wave takes all K workers of a layer: the largest power of two not above 64 / K.
static inline int grawa_group_lanes(int K)
{
    int group = 64;
    while (group > 1 && group * K > 64) group >>= 1;
    return group;
}

// Communication of such a round: whether every block of the pull works out the weights of its own layers from the estimates, as
// grawa_weights_in_pull has it for tile sums.  Its tiles are a quarter as long.  ResNet-20 on 4 workers, the weights as a launch and the pull 4.8 +
// 5.0 us and the boundary, now 7.7; a round of four steps 31.0 -> 29.1 replayed, one of one step 15.7 -> 13.6.
#define GRAWA_ESTIMATE_IN_PULL_TILES 512 // of a layer, times workers
static inline bool grawa_estimate_in_pull(int K, int64_t n_cells, int64_t max_tiles)
{
    return grawa_weights_in_pull(K, n_cells) && max_tiles * K <= GRAWA_ESTIMATE_IN_PULL_TILES && max_tiles <= GRAWA_FOLD_WAVE_TILES;
}

// Which buffer of tile sums a step takes there, so that it never finds its own pending, whatever is called or replayed after what.
// Calls made one by one take 0 and 1 in turn.  A recorded call is replayed with the buffer that it was recorded with: the first step of a recording
// takes 2 and is followed by a launch that folds it in (the recording may hold no other and be replayed twice), those after it take
// 3 and 4 in turn.
struct GrawaSteps {
    unsigned sent;                // calls made one by one
    unsigned recorded;            // calls recorded after the first one of a recording
    unsigned long long recording; // the last one that a step was recorded in
    bool folded;                  // that step has a launch of its own that folds it in
};
#define GRAWA_SUM_BUFFERS 5
// at_once: the step is to be folded in by a launch of its own.
static inline unsigned grawa_step_buffer(const GrawaSteps &s, bool recorded, unsigned long long id, bool *at_once)
{
    *at_once = recorded && s.recording != id;
    return !recorded ? s.sent & 1u : *at_once ? 2u : 3u + (s.recorded & 1u);
}
static inline void grawa_step_sent(GrawaSteps &s, bool recorded, unsigned long long id)
{
    if (!recorded) {
        s.sent += 1;
        return;
    }
    s.folded = s.recording != id;
    if (!s.folded) s.recorded += 1;
    s.recording = id;
}
// Whether a communication that is being recorded finds nothing pending: it follows a step that is folded in at once, and before that one nothing is
// pending either, since its launch folds in what calls before the replay left.
static inline bool grawa_all_folded(const GrawaSteps &s, bool recorded, unsigned long long id)
{
    return recorded && s.recording == id && s.folded;
}

// Running estimate of one worker and layer there.
struct GrawaEstimate {
    double mvg;      // moving average up to step n, with `left` up to the step before
    double gamma;    // of step n
    uint64_t n;      // scored steps since the plan was made: 64 bits, since the counts of communications below stay behind for good where a program uses only one kind
    uint32_t buffer; // of d_sums that holds the sums of step n
    uint32_t left;   // 1: they are not folded in yet
};
// The step that the last communication took into account: the later one of what launches of the weights and what pulls noted.
static constexpr uint64_t grawa_last_used(uint64_t by_weights, uint64_t by_pull) { return by_weights > by_pull ? by_weights : by_pull; }
static constexpr bool grawa_estimate_pending(const GrawaEstimate &e, uint64_t used) { return e.left && e.n != used; }
// Moving average up to step e.n, which is 0 after a communication; `norm`: of that step, if it is pending.
static constexpr double grawa_estimate_value(const GrawaEstimate &e, uint64_t used, double norm)
{
    if (e.n == used) return 0.0;
    if (!grawa_estimate_pending(e, used)) return e.mvg;
    return e.gamma * (e.n - 1 == used ? 0.0 : e.mvg) + (1.0 - e.gamma) * norm;
}

// 1 - gamma^t for 0 < gamma < 1, by squaring, since pow() is a chain of a microsecond in k_local_weights.  Every product keeps what its
// rounding drops, so that the error stays at the last place however near to 1 gamma is (plain squaring loses t units of it, pow() one, and the
// difference divides both by 1 - gamma^t).  Used on the device too (constexpr).
static constexpr double grawa_one_minus_power(double gamma, int64_t t)
{
    double power = 1.0, power_rest = 0.0, factor = gamma, factor_rest = 0.0; // value and what its rounding dropped
    for (int64_t e = t; e > 0; e >>= 1) {
        if (e & 1) {
            const double p = power * factor;
            power_rest = __builtin_fma(power, factor, -p) + (power * factor_rest + power_rest * factor);
            power = p;
        }
        const double f = factor * factor;
        factor_rest = __builtin_fma(factor, factor, -f) + 2.0 * factor * factor_rest;
        factor = f;
    }
    return (1.0 - power) - power_rest;
}

#endif
