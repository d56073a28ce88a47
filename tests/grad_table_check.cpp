// grad_table_check.cpp -- the gradient-pointer table after a write that failed
// part way: the library's own host code (api.cpp, plan.cpp) over stand-ins of
// the HIP calls and kernel launchers, in host memory.  Every step has to see
// either the new pointers, all of them, or the old ones.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../paper_2609_30342_amd/csrc/adafactor.hpp"
#include "../paper_2609_30342_amd/csrc/kernels.hpp"
#include "../include/rikfad.h"

static int fail_after = -1;              // pointers the next table write gets through, or all
static std::vector<const void *> seen;   // the table as the last step's first pass read it
static size_t ntensors = 0;

static void look(const void *const *table) { seen.assign(table, table + ntensors); }

static hipError_t table_write(const void **dst, const void *const *src, size_t n)
{
    const size_t ok = fail_after < 0 ? n : static_cast<size_t>(fail_after);
    std::memcpy(dst, src, sizeof(void *) * (ok < n ? ok : n));
    fail_after = -1;
    return ok < n ? hipErrorLaunchFailure : hipSuccess;
}

namespace rk {
hipError_t launch_stream(const TensorDesc *, const void *const *grads, const Tile *,
                         const TileGroup *, int, float *, const Coeffs &, int, int *, hipStream_t,
                         hipEvent_t, hipEvent_t)
{
    look(grads);
    return hipSuccess;
}
hipError_t launch_adafm_stats(const TensorDesc *, const void *const *grads, const Tile *,
                              const TileGroup *, int, float *, float *, const AdaCoeffs &, bool,
                              hipStream_t, hipEvent_t, hipEvent_t)
{
    look(grads);
    return hipSuccess;
}
hipError_t launch_set_grads(const void **dst, const void *const *src, int64_t n, hipStream_t)
{
    return table_write(dst, src, static_cast<size_t>(n));
}
hipError_t launch_finalize(const FinItem *, int64_t, int, bool, float *, const Coeffs &, int *, int,
                           hipStream_t, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t launch_apply(const TensorDesc *, const Tile *, const TileGroup *, int, const float *,
                        const Coeffs &, hipStream_t, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t launch_ikfad(const TensorDesc *, const void *const *, const Tile *, int64_t,
                        const Coeffs &, int *, hipStream_t, hipEvent_t, hipEvent_t)
{ return hipSuccess; }
hipError_t launch_adafm_rms(const TensorDesc *, const void *const *, const Tile *,
                            const TileGroup *, int, const float *, float *, int64_t, hipStream_t,
                            hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t launch_adafm_scale(const TensorRange *, int64_t, const float *, float *,
                              const AdaCoeffs &, hipStream_t, hipEvent_t, hipEvent_t)
{ return hipSuccess; }
hipError_t launch_adafm_update(const TensorDesc *, const void *const *, const Tile *,
                               const TileGroup *, int, const float *, const float *,
                               const TensorRange *, bool, const AdaCoeffs &, hipStream_t,
                               hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t launch_probe_stream(const float *, const float *, const float *, float *, float *,
                               int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_probe_mix(void *, const void *, float *, int64_t, int, int, hipStream_t)
{ return hipSuccess; }
hipError_t launch_probe_read(const void *, int64_t, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_probe_write(void *, int64_t, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_probe_copy(const void *, void *, int64_t, hipStream_t) { return hipSuccess; }
}  // namespace rk

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return (*p = std::calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    return table_write(static_cast<const void **>(d), static_cast<const void *const *>(s),
                       n / sizeof(void *));
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
}

static int failures = 0;
static void expect(bool ok, const char *what, int count)
{
    if (ok) return;
    std::printf("FAIL: %s (%d tensors)\n", what, count);
    ++failures;
}

template <typename Step, typename StepGrads>
static void check(int count, const std::vector<const void *> &a, const std::vector<const void *> &b,
                  Step step, StepGrads step_grads)
{
    expect(step() == RIKFAD_OK && seen == a, "first step reads the planned pointers", count);
    for (int part : {count / 2, 0}) {
        // new pointers, written in part: the step is refused ...
        fail_after = part;
        expect(step_grads(b) == RIKFAD_EHIP, "the failed write is reported", count);
        // ... and whatever comes next sees one whole table
        expect(step() == RIKFAD_OK && seen == a, "a step after it reads the old pointers", count);
        fail_after = part;
        expect(step_grads(b) == RIKFAD_EHIP, "the failed write is reported", count);
        expect(step_grads(a) == RIKFAD_OK && seen == a, "the old pointers, given again", count);
        fail_after = part;
        expect(step_grads(b) == RIKFAD_EHIP, "the failed write is reported", count);
        expect(step_grads(b) == RIKFAD_OK && seen == b, "the new pointers, given again", count);
        expect(step() == RIKFAD_OK && seen == b, "a step after them", count);
        expect(step_grads(a) == RIKFAD_OK && seen == a, "back", count);
    }
}

int main()
{
    for (int count : {1, 2, 257, 512, 513}) {
        ntensors = static_cast<size_t>(count);
        const size_t elems = 4 * 8;
        std::vector<float> mem(ntensors * elems * 5 + 4);
        float *base = mem.data();
        while (reinterpret_cast<uintptr_t>(base) % 16) ++base;
        std::vector<rikfad_tensor> t(ntensors);
        std::vector<const void *> a(ntensors), b(ntensors);
        for (size_t i = 0; i < ntensors; ++i) {
            float *q = base + i * elems * 5;
            t[i] = rikfad_tensor{q, q + elems, q + 2 * elems, q + 3 * elems, q + 4 * elems, 4, 8,
                                 RIKFAD_FP32, 0};
            a[i] = q + elems;
            b[i] = q + 3 * elems;       // any other aligned place
        }
        const rikfad_hparams hp{1e-3, 0.0, 0.1, 1.0, 1e-8};
        rikfad_ctx *rc = nullptr;
        if (rikfad_create(t.data(), count, &hp, 0, &rc) != RIKFAD_OK) return 2;
        check(count, a, b, [&] { return rikfad_step(rc, nullptr); },
              [&](const std::vector<const void *> &g) {
                  return rikfad_step_grads(rc, g.data(), nullptr);
              });
        rikfad_destroy(rc);
        adafm_hparams ah{};
        ah.h = 1e-3;
        ah.beta1 = 0.9;
        ah.decay_rate = -0.8;
        ah.eps1 = 1e-30;
        ah.eps2 = 1e-3;
        ah.clip_threshold = 1.0;
        adafm_ctx *ac = nullptr;
        if (adafm_create(t.data(), count, &ah, &ac) != RIKFAD_OK) {
            std::printf("%s\n", rikfad_last_error());
            return 2;
        }
        check(count, a, b, [&] { return adafm_step(ac, nullptr); },
              [&](const std::vector<const void *> &g) {
                  return adafm_step_grads(ac, g.data(), nullptr);
              });
        adafm_destroy(ac);
    }
    std::printf("grad_table_check: %d failures\n", failures);
    return failures == 0 ? 0 : 1;
}
