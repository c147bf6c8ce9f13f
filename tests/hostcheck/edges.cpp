// Host-side behaviour at the edges, against the stand-in for the HIP runtime (hip_stub.cpp): calls made while a stream
// captures, and calls of the runtime that fail. The runtime's calls named in test_host_edges.py are wrapped by the linker,
// so that a scenario can make them fail. Each scenario prints its name and what it found; the Python side asserts.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "mar.h"

extern "C" {
long hip_stub_errors();
long hip_stub_launches();
hipError_t __real_hipStreamSynchronize(hipStream_t s);
hipError_t __real_hipMalloc(void** p, size_t n);
hipError_t __real_hipFree(void* p);
static bool fail_sync = false;
static std::map<void*, size_t> live;          // what the device holds
static size_t held = 0, budget = SIZE_MAX;    // bytes, and the device's size
hipError_t __wrap_hipMalloc(void** p, size_t n) {
    if (held + n > budget) return hipErrorOutOfMemory;
    const hipError_t e = __real_hipMalloc(p, n);
    if (e == hipSuccess && *p) held += live[*p] = n;
    return e;
}
hipError_t __wrap_hipFree(void* p) {
    auto it = live.find(p);
    if (it != live.end()) {
        held -= it->second;
        live.erase(it);
    }
    return __real_hipFree(p);
}
hipError_t __wrap_hipMemGetInfo(size_t* f, size_t* t) {
    *t = budget == SIZE_MAX ? 288ull << 30 : budget;
    *f = *t - held;
    return hipSuccess;
}
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

mar_status eigen_state(const Sys& s, int64_t n, int nu, hipStream_t st) {   // (1024 seeds, nu = 24: 201 MB of basis)
    return mar_eigen_state_async(s.c, s.seeds, n, nu, (int)(n / 2), 0.02, MAR_FP64, MAR_FORM_BATCHED, s.e, s.n, nullptr,
                                 st);
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
    } else if (what == "seed_counts_under_capture") {   // argv: seeds of both calls, the form
        const int64_t warm = atoi(argv[3]), cap = atoi(argv[4]);
        const std::string form = argv[5];
        mar_tuning plain, t;
        memset(&plain, 0, sizeof plain);
        t = plain;
        t.upd_q = form == "blocks" || form == "then_blocks" ? 4 : 0;
        t.schedule = form == "textbook" ? MAR_SCHED_TEXTBOOK : MAR_SCHED_AUTO;
        for (mar_precision p : {MAR_FP32, MAR_FP64}) {
            (void)mar_set_tuning(s.c, form == "then_blocks" ? &plain : &t);
            (void)mar_set_local_region(s.c, -1);
            const mar_status a = solve(s, warm, 60, p, st);
            (void)mar_set_tuning(s.c, &t);
            (void)hipStreamBeginCapture(st, hipStreamCaptureModeGlobal);
            if (form == "then_region") (void)mar_set_local_region(s.c, 3);
            const mar_status b = solve(s, cap, 60, p, st);
            (void)hipStreamEndCapture(st, &g);
            printf("warm %d, captured %d\n", (int)a, (int)b);
            (void)hipGraphDestroy(g);
        }
    } else if (what == "kept_basis_gives_way") {   // a later solve gets the memory that an eigen state's basis holds
        const mar_status a = eigen_state(s, s.M, 24, st);
        budget = 500ull << 20;
        mar_tuning t;
        memset(&t, 0, sizeof t);
        t.upd_q = 4;   // seed blocks: 210 MB of basis, 126 MB of subspace matrices
        const mar_status b = mar_set_tuning(s.c, &t), c = solve(s, 128, 200, MAR_FP64, st);
        printf("eigen state %d, tuning %d, solve %d\n", (int)a, (int)b, (int)c);
    } else if (what == "kept_basis_without_room_for_the_pass") {   // the basis alone fits: the state is found without it
        const mar_status a = eigen_state(s, 256, 24, st);
        printf("with the basis %zu KB\n", held >> 10);
        drop(s);
        s = load(argv[2]);
        budget = 70ull << 20;
        const mar_status b = eigen_state(s, 256, 24, st);
        printf("eigen state %d, on less memory %d (%s)\n", (int)a, (int)b, b ? mar_last_error(s.c) : "");
    } else {
        return 2;
    }
    drop(s);
    (void)hipStreamDestroy(st);
    printf("stub errors %ld\n", hip_stub_errors());
    return 0;
}
