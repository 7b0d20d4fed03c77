// Prints the launch shapes that the host-side rules of paper_2403_04206_amd/csrc/grawa_route.h give (no GPU toolchain).
//   split <n_cells>...   -> per launch: n_cells, first cell, blocks, threads
//   model <L>...         -> per line: L, 1 if the last block of the norms' launch forms the model-level weights
//   counts <K>...        -> per line: K, 1 if the weights-in-the-pull form has a kernel for it
//   offgrid <K>...       -> per line, without and with the fp32 SGD step: K, 0 or 1, form, groups, merge, 1 if that has a kernel
//   offgrid_large <K> <sgd> <MB>... -> per triple: the triple, 1 if a pull of so many bytes takes that form (others from 128 MB on)
//   rowstep              -> bf16, center, scored, MB beyond which loads stream and the L2 merges (-1: at no size)
//   layers <K> <L> <P> <max_tiles>... -> per case: the case, 1 if a block owns a layer in the scored step
//   fold <K> <L> <P> <max_tiles>... -> per case: 1 if a scored step's sums are left to the next launch; there, 1 if the pull forms the weights from
//                           the estimates, 1 if the launch of the per-layer weights adds what is pending itself
//   fold_blocks <K> <L> <max_tiles> <center> <group> <n_groups>... -> per case: the case, blocks at the head of a row, rows ahead
//   fold_model <K> <L> <max_tiles> <longer>... -> per case: 1 if the launch of the model-level weights folds in itself
//   cachedg <K> <P> <elem_bytes>... -> per triple: the triple, columns of g that the norm pass of a fused update reads through the caches
//   power <gamma> <t>... -> per pair, exactly (%a): gamma, 1 - gamma^t
//   plain <K> <n_cells>... -> per pair: the pair, 1 if the one-column-per-lane form serves it
//   tiles <K> <n_cells>... -> per pair: the pair, 1 if the pull forms the per-layer weights
//   estimate <K> <L> <max_tiles> ... -> per triple: the triple, rows, threads
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "grawa_route.h"

int main(int argc, char **argv)
{
    if (argc < 2) return 2;
    if (!std::strcmp(argv[1], "split")) {
        for (int i = 2; i < argc; ++i) {
            const int64_t n = std::atoll(argv[i]);
            for (int64_t at = 0; at < n; at += grawa_split_blocks(n, at))
                std::printf("%lld %lld %lld %d\n", (long long)n, (long long)at, (long long)grawa_split_blocks(n, at), GRAWA_SPLIT_THREADS);
        }
        return 0;
    }
    if (!std::strcmp(argv[1], "model")) {
        for (int i = 2; i < argc; ++i) std::printf("%s %d\n", argv[i], grawa_model_weights_by_last_block(std::atoi(argv[i])));
        return 0;
    }
    if (!std::strcmp(argv[1], "counts")) {
        for (int i = 2; i < argc; ++i) std::printf("%s %d\n", argv[i], grawa_tiles_has_kernel(std::atoi(argv[i])));
        return 0;
    }
    if (!std::strcmp(argv[1], "offgrid")) {
        for (int i = 2; i < argc; ++i)
            for (int f32_sgd = 0; f32_sgd < 2; ++f32_sgd) {
                const GrawaOffGrid f = grawa_off_grid(std::atoi(argv[i]), f32_sgd);
                std::printf("%s %d %d %d %d %d\n", argv[i], f32_sgd, f.form, f.groups, f.merge,
                            grawa_off_grid_has_kernel(std::atoi(argv[i]), f32_sgd));
            }
        return 0;
    }
    if (!std::strcmp(argv[1], "offgrid_large")) {
        for (int i = 2; i + 2 < argc; i += 3)
            std::printf("%s %s %s %d\n", argv[i], argv[i + 1], argv[i + 2],
                        grawa_off_grid_large(std::atoi(argv[i]), std::atoi(argv[i + 1]), (int64_t)std::atoll(argv[i + 2]) << 20, (int64_t)128 << 20));
        return 0;
    }
    if (!std::strcmp(argv[1], "rowstep")) {
        for (int i = 0; i < 8; ++i) {
            const int64_t from = grawa_row_step_merges_from(i & 4, i & 2, i & 1);
            std::printf("%d %d %d %lld\n", i >> 2, i >> 1 & 1, i & 1, from == GRAWA_ROW_STEP_NEVER ? -1LL : (long long)(from >> 20));
        }
        return 0;
    }
    if (!std::strcmp(argv[1], "layers")) {
        for (int i = 2; i + 3 < argc; i += 4)
            std::printf("%s %s %s %s %d\n", argv[i], argv[i + 1], argv[i + 2], argv[i + 3],
                        grawa_step_by_layers(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoll(argv[i + 2]), std::atoll(argv[i + 3])));
        return 0;
    }
    if (!std::strcmp(argv[1], "fold")) {
        for (int i = 2; i + 3 < argc; i += 4) {
            const int K = std::atoi(argv[i]), L = std::atoi(argv[i + 1]);
            const int64_t P = std::atoll(argv[i + 2]), tiles = std::atoll(argv[i + 3]);
            std::printf("%d %d %d\n", grawa_fold_later(K, L, P, tiles), grawa_estimate_in_pull(K, (P + 255) / 256, tiles),
                        grawa_fold_in_weights(K, tiles));
        }
        return 0;
    }
    if (!std::strcmp(argv[1], "fold_blocks")) {
        for (int i = 2; i + 5 < argc; i += 6) {
            unsigned blocks = 0, rows = 0;
            grawa_fold_blocks(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoll(argv[i + 2]), std::atoi(argv[i + 3]), std::atoll(argv[i + 4]),
                              std::atoll(argv[i + 5]), &blocks, &rows);
            std::printf("%s %s %s %s %s %s %u %u\n", argv[i], argv[i + 1], argv[i + 2], argv[i + 3], argv[i + 4], argv[i + 5], blocks, rows);
        }
        return 0;
    }
    if (!std::strcmp(argv[1], "fold_model")) {
        for (int i = 2; i + 3 < argc; i += 4)
            std::printf("%d\n", grawa_fold_in_model_weights(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoll(argv[i + 2]), std::atoll(argv[i + 3])));
        return 0;
    }
    if (!std::strcmp(argv[1], "cachedg")) {
        for (int i = 2; i + 2 < argc; i += 3)
            std::printf("%s %s %s %lld\n", argv[i], argv[i + 1], argv[i + 2],
                        (long long)grawa_cached_grad_cols(std::atoi(argv[i]), std::atoll(argv[i + 1]), std::atoi(argv[i + 2])));
        return 0;
    }
    if (!std::strcmp(argv[1], "power")) {
        for (int i = 2; i + 1 < argc; i += 2)
            std::printf("%a %a\n", std::atof(argv[i]), grawa_one_minus_power(std::atof(argv[i]), std::atoll(argv[i + 1])));
        return 0;
    }
    if (!std::strcmp(argv[1], "plain")) {
        for (int i = 2; i + 1 < argc; i += 2)
            std::printf("%s %s %d\n", argv[i], argv[i + 1], grawa_plain_form(std::atoi(argv[i]), std::atoll(argv[i + 1])));
        return 0;
    }
    if (!std::strcmp(argv[1], "tiles")) {
        for (int i = 2; i + 1 < argc; i += 2)
            std::printf("%s %s %d\n", argv[i], argv[i + 1], grawa_weights_in_pull(std::atoi(argv[i]), std::atoll(argv[i + 1])));
        return 0;
    }
    if (!std::strcmp(argv[1], "estimate")) {
        for (int i = 2; i + 2 < argc; i += 3) {
            int rows = 0, threads = 0, wave_tiles = 0;
            grawa_estimate_shape(std::atoi(argv[i]), std::atoi(argv[i + 1]), std::atoll(argv[i + 2]), &rows, &threads, &wave_tiles);
            std::printf("%s %s %s %d %d %d\n", argv[i], argv[i + 1], argv[i + 2], rows, threads, wave_tiles);
        }
        return 0;
    }
    return 2;
}
