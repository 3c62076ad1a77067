// A HIP runtime without a GPU, for tests of the library's host code: memory is host memory, kernels do not run, any call
// can be made to fail, and the pointers that launches are given are checked against what has been freed.  Freed memory is
// never handed out again.  The planner's launch leaves the counts that the test has set where the library reads them.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include "../paper_2407_17437_amd/csrc/kernels.h"

using namespace nerva;

namespace {
std::map<uintptr_t, size_t> live, dead;
std::map<const void *, std::string> kernels;
std::string launched;
PlanCounts counts[2];
unsigned long long strip_counts = 0;   // as BindResult::strip, of plans that have room for strips
int strip_blocks = -1;   // that the last bind asked for
bool capturing = false, pending = false;
int events = 0, waits = 0;
long calls_until_failure = -1;   // of the calls that allocate, fill or wait
int bad_pointers = 0, bad_grids = 0, dirty_tickets = 0, mixed_tickets = 0;
std::map<const int32_t *, int> ticket_ends;   // what each ticket of a shared tile counts up to
size_t live_bytes = 0;
hipError_t last = hipSuccess;

bool fails(hipError_t e)
{
    if (calls_until_failure < 0 || calls_until_failure-- > 0) return false;   // (-1 once it has)
    last = e;
    return true;
}
hipError_t allocate(void **p, size_t n)
{
    *p = malloc(n);
    memset(*p, 0xCB, n < (1 << 20) ? n : 1 << 20);
    live[reinterpret_cast<uintptr_t>(*p)] = n;
    live_bytes += n;
    return hipSuccess;
}
hipError_t release(void *p)
{
    const auto it = live.find(reinterpret_cast<uintptr_t>(p));
    if (!p) return hipSuccess;
    if (it == live.end()) { ++bad_pointers; return hipSuccess; }
    live_bytes -= it->second;
    dead.insert(*it);
    live.erase(it);
    return hipSuccess;
}
bool holds(const void *at, size_t bytes)   // whether one allocation does
{
    const uintptr_t p = reinterpret_cast<uintptr_t>(at);
    auto it = live.upper_bound(p);
    return it != live.begin() && (--it, p + bytes <= it->first + it->second);
}
void check(const void *args, size_t bytes)
{
    for (size_t at = 0; at + 8 <= bytes; at += 8) {
        uintptr_t p;
        memcpy(&p, static_cast<const char *>(args) + at, 8);
        auto it = dead.upper_bound(p);
        if (it != dead.begin() && (--it, p < it->first + it->second)) ++bad_pointers;
    }
}
}  // namespace

extern "C" {
// ---- for the test
void fake_fail_after(long calls) { calls_until_failure = calls; }
long fake_fail_after_left() { return calls_until_failure; }
int fake_bad_pointers() { return bad_pointers; }
int fake_bad_grids() { return bad_grids; }
int fake_dirty_tickets() { return dirty_tickets; }
int fake_mixed_tickets() { return mixed_tickets; }
size_t fake_live_bytes() { return live_bytes; }
int fake_strip_blocks() { return strip_blocks; }
void fake_set_capturing(int on) { capturing = on; }
void fake_set_pending(int on) { pending = on; }   // events that are recorded
int fake_waits() { return waits; }
int fake_events() { return events; }
void fake_set_strips(int chunks, int steps) { strip_counts = static_cast<unsigned>(chunks) | static_cast<unsigned long long>(steps) << 32; }
const char *fake_launched() { static std::string out; out.swap(launched); launched.clear(); return out.c_str(); }
int fake_set(int side, const char *field, int value)
{
#define FIELD(name) if (!strcmp(field, #name)) { counts[side].name = value; return 0; }
    FIELD(n_blocks) FIELD(n_huge_rows) FIELD(n_huge_blocks) FIELD(n_short) FIELD(longest_row) FIELD(n_long_rows) FIELD(hot_nnz) FIELD(hot_lds_nnz) FIELD(n_dense)
    FIELD(dense_nnz) FIELD(staged_ranges) FIELD(staged_rows) FIELD(staged_nnz) FIELD(staged_longest_share)
    return 1;
}

// ---- the runtime
hipError_t hipMalloc(void **p, size_t n) { return fails(hipErrorOutOfMemory) ? hipErrorOutOfMemory : allocate(p, n); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return fails(hipErrorOutOfMemory) ? hipErrorOutOfMemory : allocate(p, n); }
hipError_t hipFree(void *p) { return release(p); }
hipError_t hipHostFree(void *p) { return release(p); }
hipError_t hipMemset(void *p, int v, size_t n)
{
    if (fails(hipErrorUnknown)) return hipErrorUnknown;
    memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipStreamSynchronize(hipStream_t) { return fails(hipErrorUnknown) ? hipErrorUnknown : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char symbol[256]; *p = symbol; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }   // (also of calls before the last one)
const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { if (fails(hipErrorOutOfMemory)) return hipErrorOutOfMemory; *e = reinterpret_cast<hipEvent_t>(&events); ++events; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return pending ? last = hipErrorNotReady : hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++waits; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { events -= e == reinterpret_cast<hipEvent_t>(&events); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host] = name; }

static dim3 config_grid, config_block;
static size_t config_lds;
static hipStream_t config_stream;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    config_grid = grid; config_block = block; config_lds = lds; config_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s)
{
    *grid = config_grid; *block = config_block; *lds = config_lds; *s = config_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3, void **args, size_t, hipStream_t)
{
    const std::string &name = kernels[kernel];
    launched += name + "\n";
    if (grid.x == 0 || grid.x > 0x7FFFFFFFu) ++bad_grids;
    auto takes = [&](const char *type) { return name.find(type) != std::string::npos; };
    // (what a kernel is given beside the arguments that many share)
    if (takes("spmm_strip_kernel")) {
        check(args[2], sizeof(Strips));
        check(args[3], 8);
    } else if (takes("strip_stream_kernel")) {
        check(args[0], sizeof(StripStreams));
    } else if (takes("backward_hot_kernel")) {
        check(args[2], sizeof(HotRows));
        check(args[3], 8);
    } else if (takes("backward_finish_kernel")) {
        check(args[1], 8);
    }
    if (takes("8SpmmArgs")) {
        const SpmmArgs &a = *static_cast<const SpmmArgs *>(args[0]);
        check(&a, sizeof a);
        const int64_t tickets = a.blocks.n_huge_rows > 0 ? (2 * a.blocks.n_huge_rows - 1) * huge_row_tickets(a.scratch_ld) : 0;
        if (tickets > 0) {
            if (!holds(a.scratch, a.blocks.n_huge_blocks * a.scratch_ld * 4) || !holds(a.tickets, tickets * 4))
                ++bad_pointers;
            else
                for (int64_t k = 0; k < tickets; ++k) dirty_tickets += a.tickets[k] != 0;
        }
    } else if (takes("9SddmmArgs")) {
        check(args[0], sizeof(SddmmArgs));
    } else if (takes("12BackwardArgs")) {
        check(args[0], sizeof(BackwardArgs));
    } else if (takes("11SampledArgs")) {
        check(args[0], sizeof(SampledArgs));
    } else if (takes("dense_nn_kernel")) {
        const DenseArgs &a = *static_cast<const DenseArgs *>(args[0]);
        const int slices = *static_cast<const int *>(args[1]);
        check(&a, sizeof a);
        if (slices > 1) {
            const int64_t tiles = (static_cast<int64_t>(a.rows) + 15) / 16 * ((a.batch + 63) / 64);
            if (tiles * slices > grid.x || !holds(a.tickets, tiles * 4) || !holds(a.partial, tiles * slices * 1024 * 4)) ++bad_pointers;
            else
                for (int64_t k = 0; k < tiles; ++k) {
                    dirty_tickets += a.tickets[k] != 0;
                    mixed_tickets += ticket_ends.emplace(a.tickets + k, slices).first->second != slices;
                }
        }
    } else if (takes("plan_kernel")) {
        const PlanArgs &p = *static_cast<const PlanArgs *>(args[0]);
        memset(p.result, 0, sizeof(BindResult));
        memcpy(p.result->plan, counts, sizeof counts);
        strip_blocks = p.side[0].strip_blocks;
        p.result->strip = strip_blocks > 0 ? strip_counts : 0;
    }
    return hipSuccess;
}
}
