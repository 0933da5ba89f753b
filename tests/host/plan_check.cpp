// The host side of the library (plans, workspaces, batches) on a stand-in for the
// HIP runtime: this program defines the runtime's functions itself, so the calls of
// libfmm.so land here.  Device memory is an address range without storage, kernels
// are counted and not run, results are zeros.  What is checked is which calls are
// made and what they return.  Usage: plan_check CASE; prints "ok" or what is wrong.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "fmm.h"

static struct Fake {
    size_t total = (size_t)288 << 30, used = 0;  // bytes of the device
    uintptr_t next = (uintptr_t)1 << 44;
    std::map<uintptr_t, size_t> live;
    long launched = 0, captured = 0, graphs = 0;
    int64_t widest = 0;  // wavefronts of the largest launch
    hipStream_t watched = nullptr;  // launches so far at the first wait of this stream
    long waited_at = -1;
    std::map<hipEvent_t, long> recorded_at;  // launches so far at an event's last record
    long first_wait_for = -1;                // that of the event first waited for
    long allocations_left = -1;  // -1: no limit
    bool capturing = false;
    dim3 grid, block;
    size_t shared = 0;
    hipStream_t stream = nullptr;
} fk;

extern "C" {
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceTotalMem(size_t *b, hipDevice_t) { *b = fk.total; return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = fk.total - fk.used; *t = fk.total; return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t b) {
    *p = nullptr;
    if (fk.capturing) return hipErrorStreamCaptureUnsupported;
    if (b > fk.total - fk.used || fk.allocations_left == 0) return hipErrorOutOfMemory;
    if (fk.allocations_left > 0) --fk.allocations_left;
    fk.used += b;
    fk.live[fk.next] = b;
    *p = (void *)fk.next;
    fk.next += (b + 4095) / 4096 * 4096 + 4096;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = fk.live.find((uintptr_t)p);
    if (it == fk.live.end()) {
        std::printf("free of %p, which is not allocated\n", p);
        std::exit(1);
    }
    fk.used -= it->second;
    fk.live.erase(it);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t b, unsigned) { *p = std::calloc(1, b); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
static hipError_t copy(void *d, const void *s, size_t b, hipMemcpyKind k) {
    auto inside = [&](const void *p) {  // of one live allocation
        auto it = fk.live.upper_bound((uintptr_t)p);
        return it != fk.live.begin() && (--it, (uintptr_t)p + b <= it->first + it->second);
    };
    if ((k != hipMemcpyDeviceToHost && !inside(d)) || (k != hipMemcpyHostToDevice && !inside(s))) {
        std::printf("copy of %zu bytes outside the allocations\n", b);
        std::exit(1);
    }
    if (k == hipMemcpyDeviceToHost) std::memset(d, 0, b);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t b, hipMemcpyKind k) { return copy(d, s, b, k); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t b, hipMemcpyKind k, hipStream_t) { return copy(d, s, b, k); }
hipError_t hipMemcpyToSymbol(const void *, const void *, size_t, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = (void *)((uintptr_t)1 << 43); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)std::malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
    if (fk.first_wait_for < 0) fk.first_wait_for = fk.recorded_at[e];
    if (s == fk.watched && fk.waited_at < 0) fk.waited_at = fk.launched;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { fk.recorded_at[e] = fk.launched; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { fk.capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    fk.capturing = false;
    *g = (hipGraph_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { std::free(g); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *e = (hipGraphExec_t)std::malloc(1);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { std::free(e); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { ++fk.graphs; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
    fk.grid = g;
    fk.block = b;
    fk.shared = sh;
    fk.stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s) {
    *g = fk.grid;
    *b = fk.block;
    *sh = fk.shared;
    *s = fk.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3 g, dim3 b, void **, size_t, hipStream_t) {
    if (g.x == 0 || g.y == 0 || g.z == 0 || b.x * b.y * b.z == 0 || b.x * b.y * b.z > 1024) {
        std::printf("launch of %u x %u x %u blocks of %u threads\n", g.x, g.y, g.z, b.x * b.y * b.z);
        std::exit(1);
    }
    ++(fk.capturing ? fk.captured : fk.launched);
    const int64_t waves = (int64_t)g.x * g.y * g.z * ((b.x * b.y * b.z + 63) / 64);
    if (waves > fk.widest) fk.widest = waves;
    return hipSuccess;
}
}

static int bad = 0;
#define CHECK(c)                                                      \
    do {                                                              \
        if (!(c)) {                                                   \
            std::printf("line %d: %s\n", __LINE__, #c);               \
            ++bad;                                                    \
        }                                                             \
    } while (0)

static double *device(size_t n) {  // an input or output array
    void *p = nullptr;
    if (hipMalloc(&p, sizeof(double) * n) != hipSuccess) std::abort();
    return (double *)p;
}

// The symmetric solute-solvent pass takes the boxes' workspaces as kernel arguments,
// and these move when a larger box comes by: its kernels are launched on every call.
static void batch_replay() {
    const double box[3] = {20.0, 21.0, 22.0};
    const int levels[3] = {2, 3, 1};
    const int64_t a[4] = {0, 300, 700, 900}, b[4] = {0, 3000, 7000, 9000};
    double *pos = device(3 * 9000), *q = device(9000), e[3], u[3];
    const uint8_t *mask = (const uint8_t *)device(9000 / 8);
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan_batch(3, box, nullptr, levels, 4, &plan) == FMM_OK);
    for (int scheme : {(int)FMM_UV_SYMMETRIC, FMM_UV_SYMMETRIC | FMM_UV_SWAP}) {
        CHECK(fmm_plan_options(plan, FMM_BOUNDARY_CONDUCTING, scheme) == FMM_OK);
        CHECK(fmm_energy_forces_batch(plan, a, pos, q, e, nullptr) == FMM_OK);
        CHECK(fmm_solute_solvent_energy_batch(plan, mask, u) == FMM_OK);
        CHECK(fmm_energy_forces_batch(plan, b, pos, q, e, nullptr) == FMM_OK);
        CHECK(fmm_energy_forces_batch(plan, a, pos, q, e, nullptr) == FMM_OK);
        const long before = fk.launched;
        CHECK(fmm_solute_solvent_energy_batch(plan, mask, u) == FMM_OK);
        CHECK(fk.launched - before >= 3 * 8);
    }
    fmm_destroy(plan);
}

// A new plan within the fixed scratch has its operators, whatever they take.
static void plan_then_noalloc() {
    const int sizes[][2] = {{4, 13}, {4, 14}, {4, 15}, {3, 19}, {3, 20}, {2, 20}, {5, 4}};  // levels, p
    double *pos = device(300), *q = device(100), e;
    for (const auto &c : sizes) {
        fmm_plan_t plan = nullptr;
        CHECK(fmm_plan(20.0, c[0], c[1], &plan) == FMM_OK);
        const fmm_status st = fmm_energy_forces_noalloc(plan, 100, pos, q, &e, nullptr, nullptr);
        if (st != FMM_OK) {
            std::printf("levels %d p %d: %s\n", c[0], c[1], fmm_last_error(plan));
            ++bad;
        }
        fmm_destroy(plan);
    }
}

// After a call that found no memory, smaller calls have all their buffers.
static void call_after_no_memory() {
    double *pos = device(3), *q = device(1), e, u;
    uint32_t *keys = (uint32_t *)device(1000);
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan(20.0, 3, 4, &plan) == FMM_OK);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    fk.allocations_left = 0;
    CHECK(fmm_energy_forces(plan, 2000, pos, q, &e, nullptr, nullptr) == FMM_ERR_NOMEM);
    fk.allocations_left = -1;
    CHECK(fmm_bin(plan, 1000, pos, keys, nullptr, nullptr) == FMM_OK);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    fmm_destroy(plan);
    // the list operators, with memory for k of their buffers at first: a call that
    // goes through afterwards has all of them, however many were there before
    size_t want = 0;
    for (int k = 12; k >= 0; --k) {
        CHECK(fmm_plan(20.0, 3, 4, &plan) == FMM_OK);
        CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
        CHECK(fmm_solute_solvent_energy(plan, (const uint8_t *)q, &u) == FMM_OK);
        fk.allocations_left = k;
        (void)fmm_plan_options(plan, FMM_BOUNDARY_CONDUCTING, FMM_UV_SPARSE);
        (void)fmm_solute_solvent_energy(plan, (const uint8_t *)q, &u);
        fk.allocations_left = -1;
        CHECK(fmm_solute_solvent_energy(plan, (const uint8_t *)q, &u) == FMM_OK);
        CHECK(fmm_plan_config(plan, FMM_FP64, 0.0, nullptr) == FMM_OK);  // what was given back for them
        if (k == 12) want = fk.live.size();
        if (fk.live.size() != want) {
            std::printf("%d allocations first: %zu buffers, not %zu\n", k, fk.live.size(), want);
            ++bad;
        }
        fmm_destroy(plan);
    }
}

static int64_t conv_levels(fmm_plan_t plan) {
    int64_t info[FMM_INFO_COUNT];
    CHECK(fmm_plan_info(plan, info, FMM_INFO_COUNT) == FMM_OK);
    return info[11];
}

// Memory of the convolution's operators goes to workspaces that need it.
static void short_of_memory() {
    double *pos = device(3), *q = device(1), e;
    uint32_t *keys = (uint32_t *)device(1000);
    void *others = nullptr;
    CHECK(hipMalloc(&others, fk.total - fk.used - ((size_t)22 << 30)) == hipSuccess);
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan(100.0, 6, 12, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    CHECK(conv_levels(plan) == 6);  // 10 of the 22 GiB
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    CHECK(conv_levels(plan) == 6);
    // 50 million atoms: 12 GiB of workspace beside the 3 of the tree
    CHECK(fmm_energy_forces(plan, 50000000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    CHECK(conv_levels(plan) == 0);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    // more than there is: refused, and smaller calls work again
    CHECK(fmm_energy_forces(plan, 400000000, pos, q, &e, nullptr, nullptr) == FMM_ERR_NOMEM);
    CHECK(fmm_bin(plan, 1000, pos, keys, nullptr, nullptr) == FMM_OK);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    // memory is back: so are the operators, once the plan is configured
    CHECK(hipFree(others) == hipSuccess);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    CHECK(conv_levels(plan) == 6);
    fmm_destroy(plan);

    // a batch: the second box's workspace takes what the first would use
    const double box[2] = {100.0, 100.0};
    const int levels[2] = {6, 5};
    const int64_t off[3] = {0, 1000, 50001000};
    double energies[2];
    CHECK(hipMalloc(&others, fk.total - fk.used - ((size_t)22 << 30)) == hipSuccess);
    CHECK(fmm_plan_batch(2, box, nullptr, levels, 12, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    const int64_t small[3] = {0, 1000, 2000};
    CHECK(fmm_energy_forces_batch(plan, small, pos, q, energies, nullptr) == FMM_OK);
    CHECK(fmm_energy_forces_batch(plan, off, pos, q, energies, nullptr) == FMM_OK);
    fmm_destroy(plan);
    // operators take at most half of what is free
    CHECK(hipFree(others) == hipSuccess);
    CHECK(hipMalloc(&others, fk.total - fk.used - ((size_t)12 << 30)) == hipSuccess);
    CHECK(fmm_plan(100.0, 6, 12, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    CHECK(conv_levels(plan) == 5);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    fmm_destroy(plan);
    CHECK(hipFree(others) == hipSuccess);
    CHECK(fk.used == sizeof(double) * (3 + 1 + 1000));
}

// Operators that fmm_plan_options cannot upload are its failure, not a later call's.
static void options_without_memory() {
    const double box[2] = {20.0, 20.0};
    const int levels[2] = {2, 2};
    double *pos = device(3), *q = device(1), e, u;
    fmm_plan_t single = nullptr, batch = nullptr;
    CHECK(fmm_plan(20.0, 3, 4, &single) == FMM_OK);
    CHECK(fmm_plan_batch(2, box, nullptr, levels, 4, &batch) == FMM_OK);
    for (fmm_plan_t plan : {single, batch}) {
        fk.allocations_left = 0;
        CHECK(fmm_plan_options(plan, FMM_BOUNDARY_VACUUM, FMM_UV_SYMMETRIC) == FMM_OK);
        CHECK(fmm_plan_options(plan, FMM_BOUNDARY_VACUUM, FMM_UV_SPARSE) == FMM_ERR_NOMEM);
        CHECK(std::strlen(fmm_last_error(plan)) > 0);
        fk.allocations_left = -1;
        CHECK(fmm_plan_options(plan, FMM_BOUNDARY_VACUUM, FMM_UV_SPARSE) == FMM_OK);
    }
    CHECK(fmm_energy_forces(single, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    CHECK(fmm_solute_solvent_energy(single, (const uint8_t *)q, &u) == FMM_OK);
    fmm_destroy(single);
    fmm_destroy(batch);
}

// The near field of few crowded leaves is split into a wavefront for every 8 of its
// targets, up to 64 a leaf (the other launches of these calls are smaller).
static void crowded_leaves() {
    const int64_t cases[][3] = {{1, 3000, 8 * 47}, {2, 8000, 64 * 16}, {2, 30000, 64 * 59}, {2, 60000, 64 * 64}};
    double *pos = device(3), *q = device(1), e;
    for (const auto &c : cases)
        for (int prec : {FMM_FP64, FMM_MIXED}) {
            fmm_plan_t plan = nullptr;
            CHECK(fmm_plan(20.0, (int)c[0], 2, &plan) == FMM_OK);
            CHECK(fmm_plan_config(plan, prec, 0.0, nullptr) == FMM_OK);
            fk.widest = 0;
            CHECK(fmm_energy_forces(plan, c[1], pos, q, &e, nullptr, nullptr) == FMM_OK);
            if (fk.widest < c[2]) {
                std::printf("levels %d, %d atoms: %d wavefronts\n", (int)c[0], (int)c[1], (int)fk.widest);
                ++bad;
            }
            fmm_destroy(plan);
        }
}

// Settings timed with other kernels are not taken from the autotuner's cache file.
static void old_cache_line(const char *path) {
    const double box[2] = {20.0, 21.0};
    const int levels[2] = {2, 2};
    const int64_t off[3] = {0, 300, 700};
    double *pos = device(3), *q = device(1);
    FILE *fp = std::fopen(path, "wb");
    CHECK(fp != nullptr);
    std::fprintf(fp, "fmm-autotune-1 arch=gfx950 p=4 prec=0 fp64_levels=3 boxes=20:300,21:400\t3,3\t8,8\n");
    std::fclose(fp);
    int hit = 1;
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan_batch(2, box, nullptr, levels, 4, &plan) == FMM_OK);
    CHECK(fmm_autotune_batch_cached(plan, off, pos, q, nullptr, path, &hit) == FMM_OK);
    CHECK(hit == 0);
    CHECK(fmm_autotune_batch_cached(plan, off, pos, q, nullptr, path, &hit) == FMM_OK);
    CHECK(hit == 1);  // the line that the first call wrote
    fmm_destroy(plan);
}

// The batch's stream waits for the boxes once all of them are enqueued.
static void batch_joins() {
    const double box[3] = {20.0, 21.0, 22.0};
    const int levels[3] = {2, 3, 1};
    const int64_t off[4] = {0, 300, 700, 900};
    double *pos = device(3), *q = device(1), e[3], u[3];
    hipStream_t s = nullptr;
    CHECK(hipStreamCreateWithFlags(&s, 0) == hipSuccess);
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan_batch(3, box, nullptr, levels, 4, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_FP64, 0.0, s) == FMM_OK);
    CHECK(fmm_energy_forces_batch(plan, off, pos, q, e, nullptr) == FMM_OK);  // the operators
    fk.watched = s;
    CHECK(fmm_energy_forces_batch(plan, off, pos, q, e, nullptr) == FMM_OK);
    CHECK(fk.waited_at == fk.launched);
    const long before = fk.launched;
    fk.waited_at = -1;
    CHECK(fmm_solute_solvent_energy_batch(plan, (const uint8_t *)q, u) == FMM_OK);
    CHECK(fk.waited_at - before >= 3 * 8);  // all dense passes; the shared stages follow
    fk.watched = nullptr;
    fmm_destroy(plan);
    CHECK(hipStreamDestroy(s) == hipSuccess);
}

// The near field starts with the P2M beside a convolution, after it beside the lists:
// five launches sort the atoms, the sixth is the P2M.
static void near_field_fork() {
    double *pos = device(3), *q = device(1), e;
    for (int prec : {FMM_FP64, FMM_MIXED, FMM_MIXED_SPLIT16_M2L, FMM_MIXED_BF16_M2L}) {
        fmm_plan_t plan = nullptr;
        CHECK(fmm_plan(20.0, 4, 4, &plan) == FMM_OK);
        CHECK(fmm_plan_config(plan, prec, 0.0, nullptr) == FMM_OK);
        const long before = fk.launched;
        fk.first_wait_for = -1;
        CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
        CHECK(fk.first_wait_for - before == (conv_levels(plan) > 0 ? 5 : 6));
        fmm_destroy(plan);
    }
}

// And so does that of list operators that need it, in a batch for all boxes.
static void lists_short_of_memory() {
    double *pos = device(3), *q = device(1), e, u;
    void *others = nullptr;
    fmm_plan_t plan = nullptr;
    CHECK(fmm_plan(100.0, 6, 12, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    CHECK(fmm_solute_solvent_energy(plan, (const uint8_t *)q, &u) == FMM_OK);
    CHECK(conv_levels(plan) == 6);
    CHECK(hipMalloc(&others, fk.total - fk.used - ((size_t)100 << 20)) == hipSuccess);
    CHECK(fmm_plan_options(plan, FMM_BOUNDARY_CONDUCTING, FMM_UV_SPARSE) == FMM_OK);  // 470 MiB
    CHECK(conv_levels(plan) == 0);
    CHECK(fmm_energy_forces(plan, 1000, pos, q, &e, nullptr, nullptr) == FMM_OK);
    CHECK(fmm_solute_solvent_energy(plan, (const uint8_t *)q, &u) == FMM_OK);
    fmm_destroy(plan);
    CHECK(hipFree(others) == hipSuccess);

    const double box[3] = {100.0, 100.0, 100.0};
    const int levels[3] = {6, 5, 7};
    const int64_t off[4] = {0, 1000, 2000, 3000};
    double energies[3], uv[3];
    CHECK(fmm_plan_batch(3, box, nullptr, levels, 12, &plan) == FMM_OK);
    CHECK(fmm_plan_config(plan, FMM_MIXED, 0.0, nullptr) == FMM_OK);
    CHECK(fmm_energy_forces_batch(plan, off, pos, q, energies, nullptr) == FMM_OK);
    CHECK(fmm_solute_solvent_energy_batch(plan, (const uint8_t *)q, uv) == FMM_OK);
    CHECK(hipMalloc(&others, fk.total - fk.used - ((size_t)100 << 20)) == hipSuccess);
    CHECK(fmm_plan_options(plan, FMM_BOUNDARY_CONDUCTING, FMM_UV_SPARSE) == FMM_OK);
    CHECK(fmm_energy_forces_batch(plan, off, pos, q, energies, nullptr) == FMM_OK);
    CHECK(fmm_solute_solvent_energy_batch(plan, (const uint8_t *)q, uv) == FMM_OK);
    fmm_destroy(plan);
    CHECK(hipFree(others) == hipSuccess);
}

int main(int argc, char **argv) {
    const std::string c = argc > 1 ? argv[1] : "";
    if (c == "batch_replay") batch_replay();
    else if (c == "plan_then_noalloc") plan_then_noalloc();
    else if (c == "call_after_no_memory") call_after_no_memory();
    else if (c == "short_of_memory") short_of_memory();
    else if (c == "options_without_memory") options_without_memory();
    else if (c == "lists_short_of_memory") lists_short_of_memory();
    else if (c == "crowded_leaves") crowded_leaves();
    else if (c == "batch_joins") batch_joins();
    else if (c == "near_field_fork") near_field_fork();
    else if (c == "old_cache_line" && argc > 2) old_cache_line(argv[2]);
    else {
        std::printf("no such case\n");
        return 2;
    }
    if (!bad) std::printf("ok\n");
    return bad != 0;
}
