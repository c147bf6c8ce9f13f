// Host-side behaviour at the edges, against the stand-in for the HIP runtime (hip_stub.cpp): calls made while a stream
// captures, and calls of the runtime that fail. The runtime's calls named in test_host_edges.py are wrapped by the linker,
// so that a scenario can make them fail. Each scenario prints its name and what it found; the Python side asserts.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>

#include "mar.h"

extern "C" {
long hip_stub_errors();
long hip_stub_launches();
hipError_t __real_hipStreamSynchronize(hipStream_t s);
static bool fail_sync = false;
hipError_t __wrap_hipStreamSynchronize(hipStream_t s) {
    return fail_sync ? hipErrorUnknown : __real_hipStreamSynchronize(s);
}
}

namespace {

struct Sys {
    int64_t M = 0, nnzH = 0;
    mar_ctx* c = nullptr;
    int32_t *seeds = nullptr, *nu = nullptr;
    double *rho = nullptr, *eb = nullptr, *e = nullptr, *n = nullptr;
};

Sys load(const std::string& path) {
    Sys s;
    FILE* f = fopen(path.c_str(), "rb");
    int64_t h[3];
    auto rd = [&](void* p, size_t n) {
        if (fread(p, 1, n, f) != n) fprintf(stderr, "short read of %s\n", path.c_str());
    };
    rd(h, sizeof h);
    s.M = h[0];
    s.nnzH = h[1];
    std::vector<int64_t> rp[2];
    std::vector<int32_t> col[2];
    std::vector<double> val[2];
    for (int k = 0; k < 2; ++k) {
        rp[k].resize(s.M + 1);
        col[k].resize(h[1 + k]);
        val[k].resize(h[1 + k]);
        rd(rp[k].data(), 8 * rp[k].size());
        rd(col[k].data(), 4 * col[k].size());
        rd(val[k].data(), 8 * val[k].size());
    }
    fclose(f);
    if (mar_create(s.M, rp[0].data(), col[0].data(), val[0].data(), rp[1].data(), col[1].data(), val[1].data(), &s.c) != MAR_OK)
        fprintf(stderr, "mar_create: %s\n", mar_last_error(nullptr));
    std::vector<int32_t> all(s.M);
    for (int64_t j = 0; j < s.M; ++j) all[j] = (int32_t)j;
    (void)hipMalloc((void**)&s.seeds, 4 * s.M);
    (void)hipMemcpy(s.seeds, all.data(), 4 * s.M, hipMemcpyHostToDevice);
    (void)hipMalloc((void**)&s.rho, 8 * s.nnzH);
    (void)hipMalloc((void**)&s.eb, 8);
    (void)hipMalloc((void**)&s.e, 8 * s.M);
    (void)hipMalloc((void**)&s.n, 8 * s.M);
    (void)hipMalloc((void**)&s.nu, 4 * s.M);
    return s;
}

mar_status solve(const Sys& s, int64_t n, int nu, mar_precision prec, hipStream_t st) {
    return mar_solve_async(s.c, s.seeds, n, nu, -0.4, 0.1, prec, MAR_FORM_BATCHED, s.rho, s.eb, s.e, s.n, s.nu, nullptr,
                           nullptr, st);
}

void drop(Sys& s) {
    mar_destroy(s.c);
    (void)hipFree(s.seeds);
    (void)hipFree(s.rho);
    (void)hipFree(s.eb);
    (void)hipFree(s.e);
    (void)hipFree(s.n);
    (void)hipFree(s.nu);
}

}  // namespace

int main(int argc, char** argv) {
    if (argc < 3) return 2;
    const std::string what = argv[1];
    Sys s = load(argv[2]);
    hipStream_t st;
    (void)hipStreamCreate(&st);
    hipGraph_t g;
    if (what == "region_under_capture") {   // the setter is host state: a capture goes on
        (void)hipStreamBeginCapture(st, hipStreamCaptureModeGlobal);
        const mar_status r = mar_set_local_region(s.c, 3);
        (void)hipStreamEndCapture(st, &g);
        printf("status %d hops %d\n", (int)r, mar_local_region(s.c));
        (void)hipGraphDestroy(g);
    } else if (what == "region_sizes_fail") {   // a failure is reported, and forgotten when it has passed
        fail_sync = true;
        const mar_status a = mar_set_local_region(s.c, 3);
        const mar_status b = solve(s, 64, 12, MAR_FP32, st);
        fail_sync = false;
        const mar_status c = solve(s, 64, 12, MAR_FP32, st);
        printf("setter %d, solve %d (%s), again %d\n", (int)a, (int)b, b ? mar_last_error(s.c) : "", (int)c);
        if (b == MAR_OK) return 1;
    } else if (what == "more_seeds_under_capture") {   // past the widest block the workspace need not grow with the seeds
        for (int nu : {12, 60})
            for (mar_precision p : {MAR_FP32, MAR_FP64}) {
                const mar_status a = solve(s, 300, nu, p, st);
                const long before = hip_stub_launches();
                (void)hipStreamBeginCapture(st, hipStreamCaptureModeGlobal);
                const mar_status b = solve(s, s.M, nu, p, st);
                (void)hipStreamEndCapture(st, &g);
                printf("warm %d, captured %d\n", (int)a, (int)b);
                if (a || b || hip_stub_launches() == before) return 1;
                (void)hipGraphDestroy(g);
            }
    } else {
        return 2;
    }
    drop(s);
    (void)hipStreamDestroy(st);
    printf("stub errors %ld\n", hip_stub_errors());
    return 0;
}
