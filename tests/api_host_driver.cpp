// Host side of the ABI (grawa_api.cpp, grawa_maps.cpp) with the HIP runtime and the kernels replaced by stubs, so that
// launches can be made to fail: what a call reports and what state it leaves the plan in.
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "grawa_internal.h"

static int fail_weights, fail_pull, n_pulls, n_one_launch, n_resets;

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = std::malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
}

bool grawa_pull_from_tiles(const grawa_plan *) { return false; }
hipError_t grawa_launch_sumsq(const grawa_plan *, const void *, int64_t, grawa_dtype_t, int64_t, hipStream_t, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t grawa_launch_finalize_layers(const grawa_plan *, int, float *, float *, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_local_weights(const grawa_plan *, double, int, float *, float *, hipStream_t)
{
    return fail_weights ? hipErrorLaunchFailure : hipSuccess;
}
hipError_t grawa_launch_local_pull(const grawa_plan *, float *, int64_t, double, float, float *, float *, float *, hipStream_t, hipEvent_t, hipEvent_t)
{
    if (fail_pull) return hipErrorInvalidConfiguration;
    ++n_one_launch;
    return hipSuccess;
}
hipError_t grawa_launch_zero_estimate(const grawa_plan *, hipStream_t)
{
    ++n_resets;
    return hipSuccess;
}
hipError_t grawa_launch_clear_flags(const grawa_plan *, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_row_step(float *, int64_t, const void *, int64_t, grawa_dtype_t, float, const float *, float, int, int64_t, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_row_step_scored(grawa_plan *, float *, int64_t, const void *, int64_t, grawa_dtype_t, float, const float *, float, double, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_center_pull(const grawa_plan *, float *, int64_t, const float *, int, float, const void *, int64_t, grawa_dtype_t, float, int, float *, float, int, float *, hipStream_t, hipEvent_t, hipEvent_t)
{
    if (fail_pull) return hipErrorInvalidConfiguration;
    ++n_pulls;
    return hipSuccess;
}
hipError_t grawa_launch_nesterov(float *, int64_t, const void *, int64_t, grawa_dtype_t, float *, int64_t, int, int64_t, float, float, float, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_leader_weights(const grawa_plan *, const float *, int *, hipStream_t) { return hipSuccess; }
hipError_t grawa_launch_stream_copy(void *, const void *, int64_t, hipStream_t) { return hipSuccess; }

#define EXPECT(cond)                                                        \
    do {                                                                    \
        if (!(cond)) {                                                      \
            std::printf("line %d: %s\n", __LINE__, #cond);                  \
            return 1;                                                       \
        }                                                                   \
    } while (0)

int main()
{
    alignas(16) static float x[3 * 16];
    const int64_t off[3] = {0, 5, 16};
    grawa_plan_t *p = nullptr;
    EXPECT(grawa_plan_create(&p, 3, 16, 2, off) == GRAWA_OK && p);
    for (int per_layer = 0; per_layer < 2; ++per_layer) {
        const auto update = [&] {
            return per_layer ? grawa_local_lgrawa_update(p, x, 16, 0.5f, nullptr, nullptr, nullptr, nullptr)
                             : grawa_local_mgrawa_update(p, x, 16, 0.5f, nullptr, nullptr, nullptr, nullptr);
        };
        const auto step = [&] { return grawa_local_step_scored(p, x, 16, x, 16, GRAWA_F32, 0.1f, nullptr, 0.f, 1.f, 0.9f, nullptr); };
        EXPECT(update() == GRAWA_ERR_INVALID_ARG); // no step yet
        // The weights were not launched: the estimate is still there and the call may be repeated.
        EXPECT(step() == GRAWA_OK);
        fail_weights = 1;
        EXPECT(update() == GRAWA_ERR_HIP);
        fail_weights = 0;
        n_pulls = 0;
        EXPECT(update() == GRAWA_OK && n_pulls == 1);
        EXPECT(update() == GRAWA_ERR_INVALID_ARG);
        // The weights were launched and have reset the estimate, the pull was not: a repeated call would pull toward the
        // plain average, so it is refused until there is a new step.
        EXPECT(step() == GRAWA_OK);
        fail_pull = 1;
        EXPECT(update() == GRAWA_ERR_HIP);
        fail_pull = 0;
        n_pulls = 0;
        EXPECT(update() == GRAWA_ERR_INVALID_ARG && n_pulls == 0);
        EXPECT(step() == GRAWA_OK && update() == GRAWA_OK && n_pulls == 1);
    }
    EXPECT(grawa_plan_destroy(p) == GRAWA_OK);

    // Weights and pull in one launch (a small model with a layer of more than 7 tiles): where it fails nothing is used up, so the
    // call may be repeated, and nothing else is launched.
    alignas(16) static float y[3 * 9000];
    const int64_t long_off[3] = {0, 8900, 9000};
    EXPECT(grawa_plan_create(&p, 3, 9000, 2, long_off) == GRAWA_OK && p);
    const auto update = [&] { return grawa_local_lgrawa_update(p, y, 9000, 0.5f, nullptr, nullptr, nullptr, nullptr); };
    EXPECT(update() == GRAWA_ERR_INVALID_ARG);
    EXPECT(grawa_local_step_scored(p, y, 9000, y, 9000, GRAWA_F32, 0.1f, nullptr, 0.f, 1.f, 0.9f, nullptr) == GRAWA_OK);
    n_pulls = n_one_launch = n_resets = 0;
    for (fail_pull = 2; fail_pull > 0; --fail_pull) EXPECT(update() == GRAWA_ERR_HIP);
    EXPECT(n_one_launch == 0 && n_resets == 0);
    EXPECT(update() == GRAWA_OK && n_one_launch == 1 && n_pulls == 0);
    EXPECT(update() == GRAWA_ERR_INVALID_ARG);
    EXPECT(grawa_plan_destroy(p) == GRAWA_OK);
    std::puts("ok");
    return 0;
}
