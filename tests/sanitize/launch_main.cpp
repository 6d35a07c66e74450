// Driver of the launch-error checks (test infrastructure, no GPU): the executable defines
// the HIP calls that the library makes, so they take the place of the runtime's, and
// nothing is launched.  Every entry point is called along each branch of its dispatch;
// with all launches succeeding it must return MOE_OK, and with any one of them failing
// MOE_ERR_DEVICE.  As in the runtime, a launch's error stays until hipGetLastError reads
// and clears it.  Prints "launch errors: OK" when every status is the expected one.
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>

#include <functional>
#include <vector>

#include "moe.h"

static int launches, fail_at = -1, last_error;

struct Dim3 {
    uint32_t x, y, z;
};
static Dim3 grid_, block_;

extern "C" {
// the launch shape between a <<< >>> and its kernel's host stub
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*) {
    grid_ = grid;
    block_ = block;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = grid_;
    *block = block_;
    *lds = 0;
    *stream = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3 grid, Dim3 block, void**, size_t, void*) {
    const bool empty = grid.x == 0 || grid.y == 0 || grid.z == 0 || block.x == 0;
    if (empty || launches++ == fail_at) return last_error = empty ? 9 : 719;
    return 0;
}
int hipGetLastError() {
    const int e = last_error;
    last_error = 0;
    return e;
}
int hipGetDevice(int* d) {
    *d = 0;
    return 0;
}
int hipDeviceGetAttribute(int* v, int, int) {
    *v = 256;
    return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
    *p = (void*)0x100000;
    return 0;
}
}

int main(int argc, char** argv) {
    void* lib = dlopen(argc > 1 ? argv[1] : "", RTLD_NOW);
    if (!lib) {
        fprintf(stderr, "%s\n", dlerror());
        return 1;
    }
#define FN(name) auto name##_ = (decltype(&name))dlsym(lib, #name)
    FN(moe_route_topk);
    FN(moe_expert_histogram);
    FN(moe_permute);
    FN(moe_permute_noalloc);
    FN(moe_route_package);
    FN(moe_grouped_ffn_products);
    FN(moe_grouped_ffn_combine);
    FN(moe_grouped_ffn_rows_shared);
    FN(moe_combine_shared);
    FN(moe_quantize_e4m3);
    FN(moe_route_topk_e4m3);
#undef FN
    void* F = (void*)0x1000;                 // handed to kernels only, and none runs
    float* f = (float*)F;
    int32_t* i32 = (int32_t*)F;
    void* W = (void*)0x100000;
    const size_t big = (size_t)1 << 40;
    const void* w[MOE_MAX_GROUPS];
    for (auto& p : w) p = F;
    std::vector<uint8_t> one(MOE_MAX_E, 1), half(MOE_MAX_E * 2);
    for (int e = 0; e < MOE_MAX_E; ++e) half[e * 2 + (e & 1)] = 1;

    int failures = 0, calls = 0, runs = 0;
    auto check = [&](const char* what, long a, long b, long c, const std::function<int()>& call) {
        launches = last_error = 0;
        fail_at = -1;
        int st = call();
        const int n = launches;
        ++calls;
        if (st != MOE_OK || n == 0) {
            fprintf(stderr, "%s %ld %ld %ld: status %d after %d launches\n", what, a, b, c, st, n);
            ++failures;
        }
        for (int i = 0; i < n; ++i, ++runs) {
            launches = last_error = 0;
            fail_at = i;
            st = call();
            if (st != MOE_ERR_DEVICE) {
                fprintf(stderr, "%s %ld %ld %ld: launch %d of %d failed, status %d\n", what, a, b,
                        c, i, n, st);
                ++failures;
            }
        }
    };

    const int64_t Ts[] = {1, 64, 600, 2048, 9000, 40000};
    const int Es[] = {8, 24, 60, 128, 200};
    for (int64_t T : Ts)
        for (int E : Es)
            for (int d : {64, 2048}) {
                const int k = E <= 8 ? 2 : 6;
                for (int dtype : {MOE_F32, MOE_BF16})
                    for (float* lg : {f, (float*)nullptr})
                        check("route_topk", T, E, d, [&] {
                            return moe_route_topk_(F, dtype, F, f, T, d, E, k, MOE_RENORM, lg, i32, f,
                                                   W, big, nullptr);
                        });
                check("route_topk_e4m3", T, E, d, [&] {
                    return moe_route_topk_e4m3_((uint8_t*)F, f, (uint8_t*)F, f, f, T, d, E, k, 0, f,
                                                i32, f, nullptr);
                });
                for (int32_t* co : {i32, (int32_t*)nullptr}) {
                    check("expert_histogram", T, E, co != nullptr, [&] {
                        return moe_expert_histogram_(i32, T, k, E, i32, co, nullptr);
                    });
                    for (int flags : {0, MOE_LOGITS_IN})
                        check("route_package", T, E, flags, [&] {
                            return moe_route_package_(F, MOE_BF16, F, f, T, d, E, k, flags, f, i32, f,
                                                      W, big, i32, co, half.data(), 2, 0, 0, F, T * k,
                                                      i32, i32, f, i32, i32, W, big, nullptr);
                        });
                }
                const int El = E < MOE_MAX_GROUPS ? E : MOE_MAX_GROUPS;
                check("permute", T, E, d, [&] {
                    return moe_permute_(F, MOE_BF16, i32, f, i32, T, d, k, El, one.data(), 1, 0, 0, F,
                                        T * k, i32, i32, f, i32, i32, W, big, nullptr);
                });
                check("permute_noalloc", T, E, d, [&] {
                    return moe_permute_noalloc_(F, MOE_F32, i32, f, i32, T, d, k, El, one.data(), 1, 0,
                                                0, F, T * k, i32, i32, f, i32, i32, nullptr);
                });
            }
    for (int64_t cap : {40, 500, 5000})
        for (int n : {1, 8, 40})
            for (int dim : {256, 4160})
                for (int hint : {0, MOE_FFN_SMALL_GROUPS, MOE_FFN_LARGE_GROUPS})
                    for (int products : {1, 2, 3}) {
                        for (int dtype : {MOE_F32, MOE_BF16})
                            check("grouped_ffn", cap, n, dim, [&] {
                                return moe_grouped_ffn_products_(F, dtype, i32, n, w, w, dim, 4160, cap,
                                                                 F, W, big, products | hint, nullptr);
                            });
                        check("grouped_ffn_rows_shared", cap, n, dim, [&] {
                            return moe_grouped_ffn_rows_shared_(F, cap, i32, MOE_BF16, i32, n, 2, w, w,
                                                                4160, dim, cap, F, W, big,
                                                                products | hint, nullptr);
                        });
                    }
    for (int64_t T : {1, 60, 256})
        for (int k : {1, 2, 4, 8, 16})
            for (int dim : {256, 4160})
                check("grouped_ffn_combine", T, k, dim, [&] {
                    return moe_grouped_ffn_combine_(F, MOE_BF16, i32, 8, w, w, 256, dim, T * k, i32, f, F,
                                                    T, k, F, W, big, nullptr);
                });
    for (int64_t T : {1, 300, 9000})
        for (int d : {7, 64, 512, 2048})
            for (int k : {1, 3, 8, 16})
                for (int ns : {0, 1, 3})
                    check("combine_shared", T, d, k, [&] {
                        return moe_combine_shared_(F, MOE_BF16, i32, f, F, ns, T, d, k, F, nullptr);
                    });
    for (int64_t rows : {1, 1000, 5000})
        for (int cols : {7, 64, 1024, 4096, 8192})
            for (int dtype : {MOE_F32, MOE_BF16})
                check("quantize_e4m3", rows, cols, dtype, [&] {
                    return moe_quantize_e4m3_(F, dtype, rows, cols, (uint8_t*)F, f, nullptr);
                });
    if (failures) return 1;
    printf("launch errors: OK (%d calls, %d failed launches)\n", calls, runs);
    return 0;
}
