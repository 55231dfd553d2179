// A device for the library's host code (csrc/*.cpp) that computes nothing and
// records what it is asked to do: the HIP calls and kernel launchers that the
// host code uses, with allocations in host memory (so that uploaded staging
// images can be read back), a limit on device memory, host allocations that
// fail on request, and one record per launch.  Built into a shared library
// together with the host sources by tests/test_host_calls.py.
#include <sys/mman.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <map>
#include <vector>

#include "host.h"

using namespace srp;

namespace {

constexpr size_t NO_LIMIT = (size_t)1 << 60;
std::map<void *, size_t> g_dev;   // device allocations
size_t g_used = 0, g_limit = NO_LIMIT;
int g_fail_host = 0;              // host allocations that fail from now on

enum Kind : int64_t { UPLOAD = 1, ARTICULATE, WINDOW, PRIMARY, TRACE, FANS, ADJOINT, REDUCE };
struct Record {
    int64_t kind, a[7];
};
std::vector<Record> g_log;
int64_t g_faults = 0;             // launches that would have touched memory they must not

void note(int64_t kind, int64_t a = 0, int64_t b = 0, int64_t c = 0, int64_t d = 0, int64_t e = 0, int64_t f = 0) {
    g_log.push_back({kind, {a, b, c, d, e, f, 0}});
}

}  // namespace

extern "C" {

void dev_limit(int64_t bytes) { g_limit = bytes < 0 ? NO_LIMIT : g_used + (size_t)bytes; }
void dev_fail_host(int n) { g_fail_host = n; }
int64_t dev_used() { return (int64_t)g_used; }
int64_t dev_faults() { return g_faults; }
void dev_clear() { g_log.clear(); }
int64_t dev_log(int64_t *out, int64_t cap) {
    const int64_t n = std::min<int64_t>(cap, (int64_t)g_log.size());
    if (n > 0) std::memcpy(out, g_log.data(), (size_t)n * sizeof(Record));
    return (int64_t)g_log.size();
}

// Whether the queues hand out every one of `total` items once, and `blocks` blocks of
// own items do where own_items allows it.
int queue_faults(uint32_t total, uint32_t blocks) {
    int faults = 0;
    std::vector<int> seen(total, 0);
    for (uint32_t r = 0; r < N_QUEUES; ++r)
        for (uint32_t i = 0; i < queue_positions(total, r); ++i) {
            const uint32_t c = queue_item(i, r, total);
            if (c >= total || seen[c]++) ++faults;
        }
    faults += (int)std::count(seen.begin(), seen.end(), 0);
    if (!own_items(total, blocks)) return faults;
    std::fill(seen.begin(), seen.end(), 0);
    for (uint32_t b = 0; b < blocks; ++b)
        for (uint32_t w = 0; w < BLOCK / 64; ++w) {
            const uint32_t c = own_item(b, w, blocks);
            if (c < total && seen[c]++) ++faults;
        }
    return faults + (int)std::count(seen.begin(), seen.end(), 0);
}

uint32_t run_of(uint32_t left, uint32_t blocks, int single) { return queue_run(left, blocks, single != 0); }

hipError_t hipMalloc(void **p, size_t n) {
    *p = nullptr;
    if (g_used + n > g_limit) return hipErrorOutOfMemory;
    void *m = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    g_dev[m] = n;
    g_used += n;
    *p = m;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto f = g_dev.find(p);
    if (f != g_dev.end()) {
        g_used -= f->second;
        munmap(p, f->second);
        g_dev.erase(f);
    }
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = nullptr;
    if (g_fail_host > 0) {
        --g_fail_host;
        return hipErrorOutOfMemory;
    }
    *p = calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;   // compute units
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "recording device"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned int) {
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}

}  // extern "C"

namespace srp {

int launch_upload(char *dst, const char *src, size_t bytes, void *) {
    std::memcpy(dst, src, bytes);
    note(UPLOAD, (int64_t)bytes);
    return 0;
}
int launch_window(const EvalDesc *, int n_evals, int, uint64_t *, uint32_t *, void *) {
    note(WINDOW, n_evals);
    return 0;
}
int launch_articulate(const ArtJob *, int n_jobs, void *) {
    note(ARTICULATE, n_jobs);
    return 0;
}
// Every block of a launch numbered through the batch finds its evaluation.
void check_owners(const uint32_t *base, int n, uint32_t total, uint32_t most) {
    if (base[0] != 0 || base[n] != total) ++g_faults;
    for (int k = 0; k < n; ++k)
        if (base[k + 1] - base[k] > most) ++g_faults;
    for (uint32_t b = 0; b < total; ++b) {
        const BlockOwner own = block_owner(base, n, b, launch_share(most));
        const int e = own.eval;
        if (e < 0 || e >= n || b < base[e] || b >= base[e + 1] || own.first != base[e]) ++g_faults;
    }
}
// PRIMARY: evaluations, of them rasterised, tile, blocks launched
int launch_primary(const EvalDesc *d, int n_evals, const uint64_t *, int tile, const uint32_t *tile_base,
                   uint32_t n_tiles, uint32_t max_tiles, void *) {
    int64_t with = 0;
    for (int k = 0; k < n_evals; ++k) {
        with += d[k].vis != nullptr;
        const uint32_t nt = d[k].vis ? (uint32_t)((16 * d[k].tiles_x + tile - 1) / tile) : 0;   // (the whole patches' tiles)
        if (tile_base[k + 1] - tile_base[k] != nt * nt) ++g_faults;
    }
    check_owners(tile_base, n_evals, n_tiles, max_tiles);
    note(PRIMARY, n_evals, with, tile, n_tiles);
    return 0;
}
// Hit chains of a gradient batch, as the kernels address them: the trace
// marks the first and last word of every patch's chains with the patch's number
// and fills its sums, the adjoint looks for the marks, fills its groups' partials
// and notes them, and the reduction expects every group of every evaluation once
// and the fillings whole.  (Batches of few enough patches to touch their memory.)
constexpr int64_t MARKED_PATCHES = 1000000;
std::map<const double *, int> g_groups;
bool in_device(const void *p, size_t bytes) {
    auto f = g_dev.upper_bound(const_cast<void *>(p));
    if (f == g_dev.begin()) return false;
    --f;
    return (const char *)p + bytes <= (const char *)f->first + f->second;
}
uint32_t *chains_of(const EvalDesc &D, int64_t pt) { return D.chain + pt * (D.bounces + 1) * 64; }
bool filled(const void *p, size_t bytes, unsigned char v) {
    const unsigned char *b = (const unsigned char *)p;
    return std::all_of(b, b + bytes, [v](unsigned char x) { return x == v; });
}
int64_t patches_of(const EvalDesc *d, int n) {
    int64_t np = 0;
    for (int k = 0; k < n; ++k) np += d[k].n_patches - d[k].patch0;
    return np;
}
// TRACE: evaluations, chunks, fans traced inside, fan units listed, chunks taken one at a time
int launch_trace(const EvalDesc *d, const int64_t *chunk_base, int n_evals, const uint64_t *, int64_t total_chunks,
                 uint32_t *, uint32_t *, PatchOut *patches, uint64_t *, bool, int, PatchOut *d_fan_out, uint64_t *,
                 bool fans_inline, bool long_chunks, int4 *d_fan_units, int, const uint32_t *, uint32_t *, void *) {
    int64_t at = 0;
    for (int k = 0; k < n_evals; ++k) {
        if (chunk_base[k] != at) ++g_faults;
        at += (d[k].n_patches - d[k].patch0 + d[k].ppc - 1) / d[k].ppc;
    }
    if (chunk_base[n_evals] != at || total_chunks != at) ++g_faults;
    if (n_evals > 0 && d[0].chain && patches_of(d, n_evals) <= MARKED_PATCHES)
        for (int k = 0; k < n_evals; ++k)
            for (int64_t pt = d[k].patch0; pt < d[k].n_patches; ++pt) {
                uint32_t *c = chains_of(d[k], pt);
                if (!in_device(c, 256 * (size_t)(d[k].bounces + 1))) { ++g_faults; continue; }
                c[0] = c[64 * (d[k].bounces + 1) - 1] = (uint32_t)(d[k].patch_base + pt) + 1u;
                std::memset((void *)&patches[d[k].patch_base + pt], 0xEE, sizeof(PatchOut));
            }
    note(TRACE, n_evals, total_chunks, d_fan_out && fans_inline, d_fan_units != nullptr, long_chunks);
    return 0;
}
// ADJOINT: evaluations, blocks launched, waves per block; every group in a block of its own evaluation
int launch_adjoint(const EvalDesc *d, int n_evals, const uint32_t *block_base, uint32_t n_blocks, uint32_t max_blocks,
                   int block_waves, const PatchOut *, bool, int, void *) {
    for (int k = 0; k < n_evals; ++k) {
        const int64_t nb = block_base[k + 1] - block_base[k], parts = d[k].group / GROUP_PART;
        if (nb * block_waves < d[k].n_groups * parts || (nb - 1) * block_waves >= d[k].n_groups * parts) ++g_faults;
        if (parts < 1 || parts > block_waves) ++g_faults;
        if (d[k].patch0 % d[k].group || d[k].n_groups * d[k].group < d[k].n_patches - d[k].patch0) ++g_faults;
    }
    if (patches_of(d, n_evals) <= MARKED_PATCHES)
        for (int k = 0; k < n_evals; ++k)
            for (int64_t g = 0; g < d[k].n_groups; ++g) {
                ++g_groups[d[k].grad_part + g * d[k].grad_n];
                if (!in_device(d[k].grad_part + g * d[k].grad_n, sizeof(double) * d[k].grad_n)) { ++g_faults; continue; }
                std::memset((void *)(d[k].grad_part + g * d[k].grad_n), 0xDD, sizeof(double) * d[k].grad_n);
                const int64_t p0 = d[k].patch0 + g * d[k].group;
                for (int64_t pt = p0; pt < std::min<int64_t>(p0 + d[k].group, d[k].n_patches); ++pt)
                    for (int w : {0, 64 * (d[k].bounces + 1) - 1})
                        if (chains_of(d[k], pt)[w] != (uint32_t)(d[k].patch_base + pt) + 1u) ++g_faults;
            }
    check_owners(block_base, n_evals, n_blocks, max_blocks);
    note(ADJOINT, n_evals, n_blocks, block_waves);
    return 0;
}
int launch_fans(const EvalDesc *, const uint64_t *, int64_t max_units, uint32_t *, uint32_t *, PatchOut *, uint64_t *,
                const int4 *, bool, int, void *) {
    note(FANS, max_units);
    return 0;
}
// REDUCE: evaluations, range sums; a missing result buffer is a fault
int launch_reduce(const EvalDesc *d, int n_evals, const uint64_t *, const PatchOut *patches, const uint64_t *, const PatchOut *,
                  const uint64_t *, bool, bool grad, const uint32_t *, int64_t total_slices, void *d_out, uint32_t *,
                  const uint32_t *, uint32_t *, void *) {
    note(REDUCE, n_evals, total_slices);
    if (!d_out) ++g_faults;
    if (grad && !g_groups.empty()) {
        int64_t want = 0;
        for (int k = 0; k < n_evals; ++k) {
            want += d[k].n_groups;
            for (int64_t g = 0; g < d[k].n_groups; ++g) {
                const double *part = d[k].grad_part + g * d[k].grad_n;
                if (g_groups[part] != 1 || !filled(part, sizeof(double) * d[k].grad_n, 0xDD)) ++g_faults;
            }
            if (!filled(patches + d[k].patch_base, sizeof(PatchOut) * d[k].n_patches, 0xEE)) ++g_faults;
        }
        if ((int64_t)g_groups.size() != want) ++g_faults;
    }
    g_groups.clear();
    return 0;
}
int trace_blocks_per_cu(bool) { return 4; }
int fan_blocks_per_cu(bool) { return 4; }
int noalloc_scratch_init() { return 0; }
char *noalloc_scratch(int) {
    static char *p = (char *)mmap(nullptr, NOALLOC_SCRATCH_BYTES, PROT_READ | PROT_WRITE,
                                  MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    return p;
}

}  // namespace srp
