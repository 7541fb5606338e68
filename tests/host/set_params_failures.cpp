// The library's host code on a stand-in of the HIP runtime (device memory is
// host memory, kernels are only counted), whose fallible calls can be made to
// fail one by one: what dm_set_params leaves behind when the device runs out
// of memory or a copy fails.  Prints one line per finding; exit status 0 if
// there is none.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <vector>

#include "../../include/dnamodes.h"

static std::set<void *> live;      // allocations not yet freed
static long launches = 0;          // kernels launched
static long countdown = -1;        // this many fallible calls succeed, then one fails
static bool failed = false;

static hipError_t maybe(hipError_t e)
{
    if (countdown < 0 || countdown-- > 0) return hipSuccess;
    failed = true;
    return e;
}

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    *p = nullptr;
    const hipError_t e = maybe(hipErrorOutOfMemory);
    if (e == hipSuccess) live.insert(*p = calloc(1, n ? n : 1));
    return e;
}
hipError_t hipFree(void *p)
{
    if (p && !live.erase(p)) {
        printf("free of memory that is not allocated\n");
        exit(1);
    }
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    const hipError_t e = maybe(hipErrorUnknown);
    if (e == hipSuccess) memcpy(d, s, n);
    return e;
}
hipError_t hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h,
                            hipMemcpyKind, hipStream_t)
{
    for (size_t i = 0; i < h; ++i) memcpy((char *)d + i * dp, (const char *)s + i * sp, w);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) { return memset(d, v, n), hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    const hipError_t e = maybe(hipErrorUnknown);
    if (e == hipSuccess) memset(d, v, n);
    return e;
}
hipError_t hipStreamSynchronize(hipStream_t) { return maybe(hipErrorUnknown); }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "made to fail"; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *)
{
    memset(a, 0, sizeof *a);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t)
{
    ++launches;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s)
{
    *g = *b = dim3(1);
    *l = 0;
    *s = nullptr;
    return hipSuccess;
}
void **__hipRegisterFatBinary(const void *) { return nullptr; }
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *,
                           void *, void *, int *)
{
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void **) {}
}

static int findings = 0;
#define EXPECT(x)                                                                     \
    do {                                                                              \
        if (!(x)) ++findings, printf("precision %d, call %ld fails: not %s\n", prec, k, #x); \
    } while (0)

int main()
{
    for (int prec : {DM_FP64, DM_FP32, DM_BF16X3}) {
        // several lengths: plans with lists of buckets and items
        std::vector<int32_t> beads;
        for (int M : {40, 64, 96, 256, 300})
            for (int c = 0; c < 7; ++c) beads.push_back(prec == DM_FP64 ? M + 1 : M);
        const int32_t lengths[] = {40, 41, 64, 65, 96, 97, 256, 257, 300, 301};
        const double dt[] = {10, 10, 10, 10, 10, 10, 10, 10, 10, 10};
        size_t total = 0;
        for (int32_t M : beads) total += 3 * (size_t)M;
        std::vector<double> pos(total);
        for (size_t i = 0; i < total; ++i) pos[i] = (double)i;
        dm_params p;
        memset(&p, 0, sizeof p);
        p.T_star = 0.034;
        p.nu = 0.35;
        p.nonlinear = 1;
        p.n_lengths = 10;
        p.lengths = lengths;
        p.dt = dt;
        p.sample_every = 5;
        p.corr_lags = 3;
        int fails = 0;
        for (long k = 0;; ++k) {
            dm_ctx *ctx = nullptr;
            countdown = -1;
            EXPECT(dm_init_chains(&ctx, (int32_t)beads.size(), beads.data(), pos.data(), 1, prec,
                                  nullptr) == DM_OK);
            EXPECT(dm_set_params(ctx, &p) == DM_OK);
            EXPECT(dm_step_modes(ctx, 7) == DM_OK);
            countdown = k;
            failed = false;
            const int rc = dm_set_params(ctx, &p);
            countdown = -1;
            const bool hit = failed;
            fails += hit;
            if (hit) {
                EXPECT(rc == DM_ENOMEM || rc == DM_EHIP);
                // no step advances part of the ensemble, or all of it under
                // parameters that were not accepted
                const long before = launches;
                int64_t step = 0;
                EXPECT(dm_step_modes(ctx, 7) == DM_ESTATE);
                EXPECT(dm_step_euler(ctx, 7, 0.1) == DM_ESTATE);
                EXPECT(launches == before);
                EXPECT(dm_get_step(ctx, &step) == DM_OK && step == 7);
                // a call that is refused for its arguments changes nothing
                EXPECT(dm_set_params(ctx, &p) == DM_OK);
            } else {
                EXPECT(rc == DM_OK);
            }
            p.corr_lags = 99;
            EXPECT(dm_set_params(ctx, &p) == DM_EINVAL);
            p.corr_lags = 3;
            EXPECT(dm_step_modes(ctx, 7) == DM_OK);
            EXPECT(dm_destroy(ctx) == DM_OK);
            EXPECT(live.empty());
            if (!hit || findings > 40) break;
        }
        printf("precision %d: %d failing calls\n", prec, fails);
        if (fails < 10) ++findings, printf("too few calls were made to fail\n");
    }
    return findings ? 1 : 0;
}
