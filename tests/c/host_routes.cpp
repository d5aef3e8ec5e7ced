// The library's host code against a stand-in for the HIP runtime, for what one GPU cannot show: memory of two
// devices, runtime calls that report an error, sizes at the end of the 64-bit range.  The executable defines the
// runtime's functions itself and is linked against the built library, whose calls bind to these definitions.
//
// Every stand-in operation runs at once.  "Device" memory is ordinary memory with an owner; a kernel may touch its own
// device's and page-locked memory only, and anything else is counted as a fault.  link_copy_kernel is carried out;
// of the other kernels only the launch is seen.
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "zi.h"
#include "zi_internal.h"

namespace {

struct Alloc { char* base; size_t size; int device; };          // device -1: page-locked host memory
struct Launch { const void* func; };
Alloc allocs[256];
int n_allocs = 0;
const void* kernels[256];                                       // filled while the library is being loaded
const char* kernel_names[256];
int n_kernels = 0;
int current_device = 0;
int n_launches = 0, n_copies = 0, n_faults = 0;
uint64_t bytes_moved = 0;                                       // by the runtime's copies and link_copy_kernel
int n_syncs = 0;                                                // of the stream `watched`
hipStream_t watched = nullptr;
int n_waits = 0;                                                // for events, by the host
int n_link_steps = 0;                                           // launches of the step over the link
uint32_t most_link_tiles = 0;                                   // of one of them
int64_t all_link_tiles = 0;
int n_flat_link_steps = 0;                                      // of them over flat lists
const char* last_kernel = "";                                  // name and workgroups of the launch before
uint32_t last_groups = 0;
const char* last_partial_sum = "";                             // name of the partial-sum kernel launched last
int n_partial_sums = 0, n_waiting = 0, n_final_sums = 0;        // launches of it, of those that make the final sum, of the kernel for that
hipError_t capture_query = hipSuccess;
hipStream_t captured = nullptr;
char streams[64];
int stream_device[64], n_streams = 1;                           // 0 is the null stream
char events[1024];
int n_events = 0;

const Alloc* find(const void* p)
{
    for (int i = 0; i < n_allocs; ++i)
        if ((const char*)p >= allocs[i].base && (const char*)p < allocs[i].base + allocs[i].size) return &allocs[i];
    return nullptr;
}
hipError_t allocate(void** out, size_t bytes, int device)
{
    *out = aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
    allocs[n_allocs++] = {(char*)*out, bytes, device};
    return hipSuccess;
}
hipError_t release(void* p)
{
    for (int i = 0; i < n_allocs; ++i)
        if (allocs[i].base == p) allocs[i] = allocs[--n_allocs];
    free(p);
    return hipSuccess;
}
int device_of(hipStream_t s) { return s ? stream_device[(char*)s - streams] : current_device; }

// What a kernel on `device` may touch.
bool reachable(const void* p, size_t bytes, int device)
{
    const Alloc* a = find(p);
    return a && (a->device == -1 || a->device == device) && bytes <= (size_t)(a->base + a->size - (const char*)p);
}
void run_link_copy(const zi::CopyArgs& a, int device, bool report)
{
    const int64_t block = report ? zi::kCopyBlockElems : zi::kCopyPieceElems;
    for (uint32_t i = 0; i < a.n_segs; ++i) {
        const zi::CopySeg& s = a.t[i];
        if (!reachable(s.src, (size_t)s.elems * 2, device) || !reachable(s.dst, (size_t)s.elems * 2, device)) ++n_faults;
        memcpy(s.dst, s.src, (size_t)s.elems * 2);
        bytes_moved += (size_t)s.elems * 2;
        for (int64_t k = 0; report && k * block < s.elems; ++k) __atomic_store_n(a.flags + s.flag + k, a.serial, __ATOMIC_RELEASE);
    }
}

thread_local struct { dim3 grid, block; size_t shared; hipStream_t stream; } configured;

}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    kernels[n_kernels] = host;
    kernel_names[n_kernels++] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t stream)
{
    configured = {grid, block, shared, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream)
{
    *grid = configured.grid; *block = configured.block; *shared = configured.shared; *stream = configured.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t s)
{
    ++n_launches;
    for (int i = 0; i < n_kernels; ++i) {
        if (kernels[i] != f) continue;
        last_kernel = kernel_names[i];
        last_groups = grid.x;
        if (strstr(kernel_names[i], "sumsq_partial_kernel")) {
            last_partial_sum = kernel_names[i];
            ++n_partial_sums;
            n_waiting += strstr(last_partial_sum, "NormOne")   ? ((const zi::NormOne*)args[0])->out != nullptr
                         : strstr(last_partial_sum, "NormFew") ? ((const zi::NormFew*)args[0])->out != nullptr
                                                               : ((const zi::NormArgs*)args[0])->out != nullptr;
        }
        if (strstr(kernel_names[i], "norm_finalize_kernel")) ++n_final_sums;
        if (strstr(kernel_names[i], "adamw_link_kernel")) ++n_link_steps;
        if (strstr(kernel_names[i], "adamw_link_flat_kernel")) ++n_flat_link_steps;
        if (strstr(kernel_names[i], "adamw_link_")) {
            const uint32_t tiles = strstr(kernel_names[i], "_flat_") ? ((const zi::LinkFlatArgs*)args[0])->n_tiles : ((const zi::LinkArgs*)args[0])->n_tiles;
            if (tiles > most_link_tiles) most_link_tiles = tiles;
            all_link_tiles += tiles;
        }
        if (strstr(kernel_names[i], "link_copy_kernel"))
            run_link_copy(*(const zi::CopyArgs*)args[0], device_of(s), strstr(kernel_names[i], "ILb1E") != nullptr);
    }
    return hipSuccess;
}
hipError_t hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t sh, hipStream_t s, hipEvent_t, hipEvent_t, int)
{
    return hipLaunchKernel(f, g, b, args, sh, s);
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error of the stand-in"; }
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = current_device; return hipSuccess; }
hipError_t hipSetDevice(int d) { current_device = d; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return allocate(p, n, current_device); }
hipError_t hipFree(void* p) { return release(p); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return allocate(p, n, -1); }
hipError_t hipHostFree(void* p) { return release(p); }
hipError_t hipGetSymbolAddress(void** p, const void*)
{
    static void* scratch = nullptr;
    if (!scratch) (void)allocate(&scratch, sizeof(zi::NormPartial) * ZI_NOALLOC_MAX_PARTIALS, 0);
    *p = scratch;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* at, const void* p)
{
    memset(at, 0, sizeof *at);
    const Alloc* a = find(p);
    at->type = !a ? hipMemoryTypeUnregistered : a->device < 0 ? hipMemoryTypeHost : hipMemoryTypeDevice;
    at->device = a && a->device >= 0 ? a->device : 0;
    at->devicePointer = a ? const_cast<void*>(p) : nullptr;
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p)
{
    const Alloc* a = find(p);
    if (!a) return hipErrorNotFound;
    *base = a->base;
    *size = a->size;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t)
{
    ++n_copies;
    bytes_moved += n;
    memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    stream_device[n_streams] = current_device;
    *s = (hipStream_t)(streams + n_streams++);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { n_syncs += s == watched; return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { *d = device_of(s); return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st)
{
    *st = s && s == captured ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return capture_query;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)(events + n_events++); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { ++n_waits; return hipSuccess; }
}

#define CHECK(cond)                                                                                     \
    do {                                                                                                \
        if (!(cond)) {                                                                                  \
            fprintf(stderr, "CHECK failed: %s (line %d; %s)\n", #cond, __LINE__, zi_last_error());      \
            return 1;                                                                                   \
        }                                                                                               \
    } while (0)

static void* on_device(size_t bytes, int device) { void* p; (void)allocate(&p, bytes, device); memset(p, 0, bytes); return p; }
static zi_adamw_config config()
{
    zi_adamw_config c{};
    c.lr = 1e-3f; c.beta1 = 0.9f; c.beta2 = 0.999f; c.eps = 1e-8f; c.weight_decay = 0.01f; c.step = 10; c.loss_scale = 1.0f;
    return c;
}

// Gradients and copies on another device than the engine's: the copies are the runtime's, no kernel touches them.
static int peer()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    CHECK(zi_engine_set_option(e, ZI_OPT_HOST_RING_SLOTS, 3) == ZI_OK);
    for (int owner = 0; owner < 2; ++owner) {
        const size_t bytes = 40000;
        uint16_t* src = (uint16_t*)on_device(bytes, owner);
        for (size_t i = 0; i < bytes / 2; ++i) src[i] = (uint16_t)(i * 7 + 1);
        uint16_t* dst = (uint16_t*)on_device(bytes, -1);
        CHECK(zi_grad_offload(e, src, dst, bytes, nullptr) == ZI_OK);
        CHECK(zi_grad_offload_wait(e) == ZI_OK);
        CHECK(n_faults == 0 && memcmp(src, dst, bytes) == 0);
    }
    const int64_t sizes[] = {70001, 5, 16384, 40003};
    std::vector<std::vector<float>> state[2];
    std::vector<std::vector<uint16_t>> copies[2];
    for (int mixed = 0; mixed < 2; ++mixed) {                  // all on the engine's device, then every other tensor elsewhere
        std::vector<zi_tensor> list;
        for (int i = 0; i < 4; ++i) {
            const size_t n = (size_t)sizes[i];
            zi_tensor t{};
            float* a[3];
            for (int w = 0; w < 3; ++w) {
                state[mixed].emplace_back(n);
                a[w] = state[mixed].back().data();
                for (size_t k = 0; k < n; ++k) a[w][k] = (float)((k * 13 + 5 * (size_t)w) % 997) * 1e-4f;
            }
            uint16_t* g = (uint16_t*)on_device(n * 2, mixed && i % 2 == 0 ? 1 : 0);
            for (size_t k = 0; k < n; ++k) g[k] = (uint16_t)(0x3A00 + k % 200);
            t.p = a[0]; t.m = a[1]; t.v = a[2]; t.g = g;
            t.p_lp = i == 1 ? nullptr : on_device(n * 2, mixed && i >= 2 ? 1 : 0);
            t.numel = sizes[i];
            list.push_back(t);
        }
        const zi_adamw_config c = config();
        for (int twice = 0; twice < 2; ++twice)
            CHECK(zi_adamw_step_cpu(e, list.data(), 4, ZI_BF16, &c, nullptr, 3, nullptr) == ZI_OK);
        CHECK(n_faults == 0);
        zi_stream_stats st{};
        CHECK(zi_engine_last_stats(e, &st) == ZI_OK);
        CHECK(st.bytes_d2h == 2 * (70001 + 5 + 16384 + 40003) && st.bytes_h2d == 2 * (70001 + 16384 + 40003));
        for (int i = 0; i < 4; ++i)
            if (list[(size_t)i].p_lp)
                copies[mixed].emplace_back((uint16_t*)list[(size_t)i].p_lp, (uint16_t*)list[(size_t)i].p_lp + sizes[i]);
    }
    CHECK(state[0] == state[1] && copies[0] == copies[1]);
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// Element counts whose byte counts, or addresses of whose ends, pass the end of the 64-bit range: refused, with nothing
// launched, also behind a tensor that has made the allocations known.
static int sizes()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    CHECK(zi_engine_set_option(e, ZI_OPT_HOST_RING_SLOTS, 3) == ZI_OK);
    const int64_t n = 5000, huge[] = {INT64_MAX, INT64_MAX - 1000, INT64_MAX / 2 + 1, INT64_MAX / 2 + 3, INT64_MAX / 4 + 1};
    const zi_adamw_config c = config();
    char* out = (char*)on_device(64 * 1024 * 8, 0);                // the norm's workspace, and room for its result
    zi_norm_result* norm = (zi_norm_result*)(out + zi_norm_workspace_bytes(0, 0));
    for (int host = 0; host < 2; ++host) {                         // p, m, v; the gradients follow them in the streamed calls
        char* a[4];
        for (char*& x : a) x = (char*)on_device(8 * n, host ? -1 : 0);
        char* g_device = (char*)on_device(8 * n, 0);
        for (int known = 0; known < 2; ++known)
            for (const int64_t bad : huge) {
                zi_tensor t[2]{};
                for (int i = 0; i < 2; ++i) {
                    t[i].p = a[0] + 4 * n * i; t[i].m = a[1] + 4 * n * i; t[i].v = a[2] + 4 * n * i;
                    t[i].g = a[3] + 4 * n * i;
                    t[i].numel = n;
                }
                t[1].numel = bad;
                const zi_tensor* list = known ? t : t + 1;
                const int32_t count = known ? 2 : 1;
                n_launches = n_copies = 0;
                CHECK(zi_grad_norm(list, count, ZI_BF16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), nullptr) < 0);
                CHECK(zi_grad_norm_noalloc(list, count, ZI_BF16, 1.0f, norm, nullptr) < 0);
                CHECK(zi_grad_norm_streamed(e, list, count, ZI_BF16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), nullptr) < 0);
                CHECK(zi_adamw_step(list, count, ZI_BF16, &c, nullptr, nullptr) < 0);
                if (host) {
                    CHECK(zi_adamw_step_streamed(e, list, count, ZI_BF16, &c, nullptr, nullptr) < 0);
                    t[0].g = g_device;
                    t[1].g = g_device + 4 * n;
                    CHECK(zi_adamw_step_streamed(e, list, count, ZI_BF16, &c, nullptr, nullptr) < 0);
                    CHECK(zi_adamw_step_cpu(e, list, count, ZI_BF16, &c, nullptr, 2, nullptr) < 0);
                    CHECK(zi_grad_offload(e, g_device, a[3], (size_t)bad * 2, nullptr) < 0);
                }
                CHECK(n_launches == 0 && n_copies == 0);
            }
    }
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// The query whether a stream is being captured fails for the null stream while another stream is: calls of several
// launches go on as before.
static int capture()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    const zi_adamw_config c = config();
    constexpr int kMost = 700;                                     // three launches each of the step's kernels and the reduction
    const int64_t n = 600;
    char* device = (char*)on_device((size_t)kMost * n * 16, 0);
    char* pinned = (char*)on_device((size_t)kMost * n * 16, -1);
    char* out = (char*)on_device(64 * 1024 * 8, 0);
    zi_norm_result* norm = (zi_norm_result*)(out + zi_norm_workspace_bytes(0, 0));
    for (int32_t count : {60, 200, kMost})
        for (int flat = 0; flat < 2; ++flat)
            for (int host = 0; host < 2; ++host) {
                std::vector<zi_tensor> list((size_t)count);
                for (int32_t i = 0; i < count; ++i) {
                    char* a = host ? pinned : device;
                    const int64_t at = flat ? (int64_t)i * n : (int64_t)((i * 7) % count) * n;
                    zi_tensor& t = list[(size_t)i];
                    t.p = a + 4 * at; t.m = a + 4 * (kMost * n + at); t.v = a + 4 * (2 * kMost * n + at);
                    t.g = device + 2 * (6 * kMost * n + at); t.p_lp = device + 2 * (7 * kMost * n + at);
                    t.numel = n;
                }
                int launches[2][3] = {};
                for (int fails = 0; fails < 2; ++fails) {
                    capture_query = fails ? hipErrorStreamCaptureImplicit : hipSuccess;
                    auto counted = [&](zi_status st, int which) { launches[fails][which] = st == ZI_OK ? n_launches : -1; n_launches = 0; };
                    n_launches = 0;
                    counted(zi_grad_norm(list.data(), count, ZI_BF16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), nullptr), 0);
                    if (host) counted(zi_adamw_step_streamed(e, list.data(), count, ZI_BF16, &c, nullptr, nullptr), 1);
                    else      counted(zi_adamw_step(list.data(), count, ZI_BF16, &c, nullptr, nullptr), 2);
                }
                capture_query = hipSuccess;
                CHECK(launches[0][0] > 0 && launches[0][host ? 1 : 2] > 0);
                CHECK(!memcmp(launches[0], launches[1], sizeof launches[0]));
            }
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// A captured launch is replayed with the same marks, so a partial that came too late for one replay would pass for the next
// one's: under capture no workgroup waits for partials, a kernel of its own makes the final sum.  (A list of one tile is one
// workgroup's, which has no others to wait for.)
static int replays()
{
    char* out = (char*)on_device(64 * 1024 * 8, 0);
    zi_norm_result* norm = (zi_norm_result*)(out + zi_norm_workspace_bytes(0, 0));
    constexpr int kMost = 700;
    const int64_t n = 40'000;
    char* g = (char*)on_device((size_t)kMost * n * 2, 0);
    hipStream_t stream;
    CHECK(hipStreamCreateWithFlags(&stream, 0) == hipSuccess);
    for (int32_t count : {1, 2, 32, 33, 320, 321, kMost})
        for (int64_t numel : {(int64_t)7, n})
            for (int noalloc = 0; noalloc < 2; ++noalloc)
                for (int under = 0; under < 2; ++under) {
                    std::vector<zi_tensor> list((size_t)count);
                    for (int32_t i = 0; i < count; ++i) {
                        list[(size_t)i].g = g + 2 * n * i;
                        list[(size_t)i].numel = numel;
                    }
                    captured = under ? stream : nullptr;
                    n_partial_sums = n_waiting = n_final_sums = 0;
                    CHECK((noalloc ? zi_grad_norm_noalloc(list.data(), count, ZI_BF16, 1.0f, norm, stream)
                                   : zi_grad_norm(list.data(), count, ZI_BF16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), stream)) == ZI_OK);
                    CHECK(n_partial_sums == (count + 319) / 320);
                    const bool separate = under && !(count == 1 && numel == 7);
                    CHECK(n_waiting == (separate ? 0 : 1) && n_final_sums == (separate ? 1 : 0));
                    captured = nullptr;
                }
    return 0;
}

// A skipped step of the CPU placement moves the norm result and nothing else, wherever that and the gradients are, reports no
// traffic, and does not wait for gradients that are still being offloaded.  The step after it is made as if there had been none.
static int skipped()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    CHECK(zi_engine_set_option(e, ZI_OPT_HOST_RING_SLOTS, 6) == ZI_OK);
    const zi_adamw_config c = config();
    uint16_t* parts[2] = {(uint16_t*)on_device(4000, 0), (uint16_t*)on_device(4000, -1)};
    for (int norm_on : {0, 1, -1})
        for (int grads_on : {0, 1, -1})
            for (int offloads = 0; offloads < 2; ++offloads)
                for (int64_t n : {(int64_t)5, (int64_t)16384, (int64_t)9 * 16384 + 3}) {
                    std::vector<float> state[4];
                    for (int w = 0; w < 4; ++w) state[w].assign((size_t)n, 0.25f * (float)(w + 1));
                    zi_tensor t{};
                    t.p = state[0].data(); t.m = state[1].data(); t.v = state[2].data();
                    t.g = on_device((size_t)n * 2, grads_on);
                    t.p_lp = on_device((size_t)n * 2, 0);
                    t.numel = n;
                    zi_norm_result* norm = (zi_norm_result*)on_device(sizeof(zi_norm_result), norm_on);
                    norm->found_inf = 1;
                    if (offloads) CHECK(zi_grad_offload(e, parts[0], parts[1], 4000, nullptr) == ZI_OK);
                    bytes_moved = 0;
                    n_waits = 0;
                    CHECK(zi_adamw_step_cpu(e, &t, 1, ZI_BF16, &c, norm, 3, nullptr) == ZI_SKIPPED_OVERFLOW);
                    CHECK(bytes_moved == sizeof(zi_norm_result));
                    CHECK(n_waits == 0);
                    zi_stream_stats st{};
                    CHECK(zi_engine_last_stats(e, &st) == ZI_OK);
                    CHECK(st.bytes_d2h == 0 && st.bytes_h2d == 0 && st.n_copies == 0 && st.n_slot_uses == 0 && st.seconds == 0.0);
                    for (int w = 0; w < 3; ++w)
                        for (float x : state[w]) CHECK(x == 0.25f * (float)(w + 1));
                    for (int64_t i = 0; i < n; ++i) CHECK(((uint16_t*)t.p_lp)[i] == 0);
                    norm->found_inf = 0;
                    CHECK(zi_adamw_step_cpu(e, &t, 1, ZI_BF16, &c, norm, 3, nullptr) == ZI_OK);
                    CHECK(offloads == 0 || n_waits > 0);
                    CHECK(zi_engine_last_stats(e, &st) == ZI_OK && st.bytes_d2h == (grads_on < 0 ? 0 : 2 * (uint64_t)n) && st.bytes_h2d == 2 * (uint64_t)n);
                    for (float x : state[0]) CHECK(x < 0.25f && x == state[0][0]);
                    for (int64_t i = 0; i < n; ++i) CHECK(((uint16_t*)t.p_lp)[i] == ((uint16_t*)t.p_lp)[0] && ((uint16_t*)t.p_lp)[i] != 0);
                    release(const_cast<void*>(t.g));
                    release(t.p_lp);
                    release(norm);
                }
    CHECK(n_faults == 0);
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// What earlier work on the caller's stream has written to page-locked memory or on another device is certain to be there only
// after the stream has been synchronised: a flag that a later kernel raises is not enough.
static int earlier_work()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    CHECK(zi_engine_set_option(e, ZI_OPT_HOST_RING_SLOTS, 4) == ZI_OK);
    CHECK(hipStreamCreateWithFlags(&watched, 0) == hipSuccess);
    const zi_adamw_config c = config();
    const int64_t n = 20000;
    zi_norm_result* norm = (zi_norm_result*)on_device(sizeof(zi_norm_result), 0);
    std::vector<float> state[3];
    for (auto& x : state) x.assign((size_t)n, 0.5f);
    for (int other = 0; other < 5; ++other)                        // p, m, v, g, p_lp
        for (int on : {-1, 1}) {
            if (other < 3 && on == 1) continue;
            zi_tensor t[2]{};
            for (zi_tensor& x : t) {
                x.p = state[0].data(); x.m = state[1].data(); x.v = state[2].data();
                x.g = on_device((size_t)n * 2, 0); x.p_lp = on_device((size_t)n * 2, 0);
                x.numel = n / 2;
            }
            t[1].p = state[0].data() + n / 2; t[1].m = state[1].data() + n / 2; t[1].v = state[2].data() + n / 2;
            void* there = on_device((size_t)n * 4, on);
            void** const array[5] = {(void**)&t[1].p, (void**)&t[1].m, (void**)&t[1].v, (void**)&t[1].g, (void**)&t[1].p_lp};
            *array[other] = there;
            n_syncs = 0;
            CHECK(zi_adamw_step_cpu(e, t, 2, ZI_BF16, &c, norm, 2, watched) == ZI_OK);
            CHECK(n_syncs > 0);
            release(const_cast<void*>(t[0].g));
            release(t[0].p_lp);
        }
    CHECK(n_faults == 0);
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// How the copies of the CPU placement go up: what one slot use takes, by kernels, except that of a use of one segment of
// at most 64 blocks with more uses behind it.
static int uploads()
{
    const struct { size_t chunk; int64_t numel; int32_t tensors; int copies; } cases[] = {
        {64 << 10, 16384, 1, 0}, {64 << 10, 5 * 16384, 1, 4}, {64 << 10, 5 * 16384 + 1, 1, 5}, {1 << 20, 4 * 262144, 1, 3},
        {64 << 10, 1000, 40, 0}, {4 << 20, 3 << 20, 1, 2}, {8 << 20, 3 << 21, 1, 0}};
    for (const auto& k : cases) {
        zi_engine* e = nullptr;
        CHECK(zi_engine_create(&e, 0, k.chunk, 3) == ZI_OK);
        CHECK(zi_engine_set_option(e, ZI_OPT_HOST_RING_SLOTS, 4) == ZI_OK);
        const size_t all = (size_t)k.numel * (size_t)k.tensors;
        std::vector<float> state(3 * all);
        uint16_t* g = (uint16_t*)on_device(2 * all, 0);
        uint16_t* lp = (uint16_t*)on_device(2 * all, 0);
        for (size_t i = 0; i < all; ++i) state[i] = (float)(i % 1000);
        std::vector<zi_tensor> list((size_t)k.tensors);
        for (size_t i = 0; i < list.size(); ++i) {
            const size_t at = i * (size_t)k.numel;
            list[i] = {state.data() + at, state.data() + all + at, state.data() + 2 * all + at, g + at, lp + at, k.numel};
        }
        zi_adamw_config c = config();
        c.weight_decay = 0.0f;                     // with zero gradients and moments p stays, and the copy is p
        CHECK(zi_adamw_step_cpu(e, list.data(), k.tensors, ZI_BF16, &c, nullptr, 3, nullptr) == ZI_OK);
        zi_stream_stats st{};
        CHECK(zi_engine_last_stats(e, &st) == ZI_OK);
        CHECK(st.n_copies == k.copies && st.bytes_h2d == 2 * all && n_faults == 0);
        for (size_t i = 0; i < all; i += 4096) CHECK(lp[i] == (uint16_t)(__builtin_bit_cast(uint32_t, (float)(i % 1000)) >> 16) || i % 1000 > 255);
        CHECK(zi_engine_destroy(e) == ZI_OK);
        release(g);
        release(lp);
    }
    return 0;
}

// Reductions of up to 176 MiB of gradients in HBM, in one tensor or several, read with ordinary loads; longer ones and
// those over the link with streaming loads.
static int loads()
{
    const int64_t most = (int64_t)11 << 23;
    char* out = (char*)on_device(64 * 1024 * 8, 0);
    zi_norm_result* norm = (zi_norm_result*)(out + zi_norm_workspace_bytes(0, 0));
    void* g;
    (void)allocate(&g, 2 * (size_t)most + 64, 0);
    for (int64_t n : {most, most + 1})
        for (int parts = 1; parts <= 3; parts += 2)
            for (int noalloc = 0; noalloc < 2; ++noalloc) {
                zi_tensor t[3]{};
                for (int i = 0; i < parts; ++i) {
                    t[i].numel = i + 1 < parts ? n / parts : n - (parts - 1) * (n / parts);
                    t[i].g = (uint16_t*)g + i * (n / parts);
                }
                CHECK((noalloc ? zi_grad_norm_noalloc(t, parts, ZI_FP16, 1.0f, norm, nullptr)
                               : zi_grad_norm(t, parts, ZI_FP16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), nullptr)) == ZI_OK);
                CHECK(strstr(last_partial_sum, n <= most ? "ILi1ELb1E" : "ILi1ELb0E"));
            }
    return 0;
}

// Gradients leave without a kernel of the library's, which would take compute units from their producer.
static int offload()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    const size_t most = (size_t)8 << 20;
    char* src = (char*)on_device(most, 0);
    char* dst = (char*)on_device(most, -1);
    for (size_t i = 0; i < most; ++i) src[i] = (char)(i * 31 >> 4);
    for (size_t bytes : {(size_t)2, (size_t)4096, (size_t)100001, (size_t)1 << 20, (size_t)4 << 20, most}) {
        memset(dst, 0, most);
        CHECK(zi_grad_offload(e, src, dst, bytes, nullptr) == ZI_OK && zi_grad_offload_wait(e) == ZI_OK);
        CHECK(n_launches == 0 && !memcmp(src, dst, bytes));
    }
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// Page-locked arrays that span two registrations are for copies only: the chunk pipeline takes them, at the default pacing
// too, and (no kernel being carried out here) brings back what it took.
static int spanning()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 * 1024, 3) == ZI_OK);
    const zi_adamw_config c = config();
    const int64_t n = 100'000;
    char* out = (char*)on_device(64 * 1024 * 8, 0);
    zi_norm_result* norm = (zi_norm_result*)(out + zi_norm_workspace_bytes(0, 0));
    for (int split = 0; split <= 4; ++split) {                     // 0: none, else this array of p, m, v, g
        zi_tensor t{};
        char* a[4];
        for (int w = 0; w < 4; ++w) {
            a[w] = (char*)on_device(4 * n, -1);
            for (int64_t i = 0; i < 4 * n; ++i) a[w][i] = (char)(i * 7 + w);
            if (split != w + 1) continue;
            allocs[n_allocs - 1].size = 40960;
            allocs[n_allocs++] = {a[w] + 40960, 4 * (size_t)n - 40960, -1};
        }
        t.p = a[0]; t.m = a[1]; t.v = a[2]; t.g = a[3];
        t.p_lp = on_device(2 * n, 0);
        t.numel = n;
        n_copies = n_link_steps = 0;
        CHECK(zi_adamw_step_streamed(e, &t, 1, ZI_BF16, &c, nullptr, nullptr) == ZI_OK);
        zi_stream_stats st{};
        CHECK(zi_engine_last_stats(e, &st) == ZI_OK && st.n_copies == n_copies && st.n_slot_uses == 7);
        CHECK(st.bytes_h2d == 14 * (uint64_t)n && st.bytes_d2h == 12 * (uint64_t)n);
        CHECK(split ? n_copies == 7 * 7 && n_link_steps == 0 : n_copies == 0 && n_link_steps == 1);
        n_copies = 0;
        CHECK(zi_grad_norm_streamed(e, &t, 1, ZI_BF16, 1.0f, norm, out, zi_norm_workspace_bytes(0, 0), nullptr) == ZI_OK);
        CHECK(n_copies == (split == 4 ? 7 : 0));
        for (int w = 0; w < 4; ++w)
            for (int64_t i = 0; i < 4 * n; ++i) CHECK(a[w][i] == (char)(i * 7 + w));
    }
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// A launch over the link holds kLinkTilesPerLaunch tiles at most, also where a list that is short on average has long tensors.
static int link_tiles()
{
    zi_engine* e = nullptr;
    CHECK(zi_engine_create(&e, 0, 64 << 20, 3) == ZI_OK);
    const zi_adamw_config c = config();
    const int64_t limit = (int64_t)zi::kLinkTilesPerLaunch * zi::kStepTileElems;
    const struct { int64_t length; int count; bool flat; } long_ones[] = {
        {1000, 0, true}, {limit / 2, 3, true}, {limit - 512, 1, true}, {limit, 1, true}, {limit + 1, 1, false}, {limit + 576, 1, false},
        {limit + limit / 2, 1, false}};
    for (const auto& k : long_ones) {
        std::vector<int64_t> lengths(1400, 700);
        for (int i = 0; i < k.count; ++i) lengths[(size_t)(300 + 2 * i)] = k.length;
        int64_t n = 0;
        for (int64_t x : lengths) n += x;
        void* a[5];
        for (int w = 0; w < 5; ++w) (void)allocate(&a[w], (size_t)n * (w < 3 ? 4 : 2), w < 3 ? -1 : 0);
        std::vector<zi_tensor> list;
        int64_t at = 0, tiles = 0;
        for (int64_t x : lengths) {
            list.push_back({(float*)a[0] + at, (float*)a[1] + at, (float*)a[2] + at, (uint16_t*)a[3] + at, (uint16_t*)a[4] + at, x});
            at += x;
            tiles += (x + 511) / 512;
        }
        n_flat_link_steps = n_link_steps = 0;
        most_link_tiles = 0;
        all_link_tiles = 0;
        CHECK(zi_adamw_step_streamed(e, list.data(), (int32_t)list.size(), ZI_BF16, &c, nullptr, nullptr) == ZI_OK);
        CHECK(most_link_tiles <= zi::kLinkTilesPerLaunch);
        CHECK(all_link_tiles <= tiles + 2 && all_link_tiles >= tiles - 1400);      // (a head of up to 63 elements may save a tile)
        CHECK(k.flat ? n_flat_link_steps >= 6 && n_link_steps == 0 : n_flat_link_steps == 0 && n_link_steps > 6);
        for (void* x : a) release(x);
    }
    CHECK(zi_engine_destroy(e) == ZI_OK);
    return 0;
}

// What one tensor takes by its tiles of 512 elements, and that the workgroups of the launch cover it: fine tiles, two to four
// quads a lane at a pace where all of them are resident at once, and fine tiles again.
static int one_tensor_kernels()
{
    const zi_adamw_config c = config();
    char* base = (char*)on_device(5 * ((size_t)16 << 20), 0);
    const struct { int64_t tiles; const char* kernel; int quads; } rows[] = {
        {1, "adamw_fine_kernel", 1}, {1792, "adamw_fine_kernel", 1}, {1793, "adamw_paced_kernel", 2}, {2047, "adamw_paced_kernel", 2},
        {2048, "adamw_paced_kernel", 2}, {2049, "adamw_paced_kernel", 2}, {4096, "adamw_paced_kernel", 2}, {4097, "adamw_paced_kernel", 3},
        {6144, "adamw_paced_kernel", 3}, {6145, "adamw_paced_kernel", 4}, {7168, "adamw_paced_kernel", 4}, {7169, "adamw_fine_kernel", 1}};
    for (const auto& r : rows)
        for (int64_t less : {0, 505}) {
            zi_tensor t{};
            t.p = base; t.m = base + ((size_t)16 << 20); t.v = base + ((size_t)32 << 20); t.g = base + ((size_t)48 << 20);
            t.p_lp = base + ((size_t)64 << 20);
            t.numel = r.tiles * 512 - less;
            CHECK(zi_adamw_step(&t, 1, ZI_BF16, &c, nullptr, nullptr) == ZI_OK);
            CHECK(strstr(last_kernel, r.kernel));
            char quads[16];
            snprintf(quads, sizeof quads, "Li%dEE", r.quads);
            CHECK(r.quads == 1 || strstr(last_kernel, quads));
            const int64_t per_group = 64 * 4 * r.quads;
            const int64_t groups = (t.numel / 4 * 4 + per_group - 1) / per_group;
            CHECK(last_groups == (groups ? groups : 1));
        }
    // The longest that fine tiles take and the shortest that they do not (in allocations that nobody touches), and whole tiles in a list.
    const size_t at[5] = {(size_t)1 << 44, (size_t)2 << 44, (size_t)3 << 44, (size_t)4 << 44, (size_t)5 << 44};
    for (size_t a : at) allocs[n_allocs++] = {(char*)a, (size_t)1 << 40, 0};
    for (int64_t tiles : {(1 << 25) - 1, 1 << 25, (1 << 25) + 1}) {
        zi_tensor t{};
        t.p = (void*)at[0]; t.m = (void*)at[1]; t.v = (void*)at[2]; t.g = (void*)at[3]; t.p_lp = (void*)at[4];
        t.numel = tiles * 512;
        CHECK(zi_adamw_step(&t, 1, ZI_BF16, &c, nullptr, nullptr) == ZI_OK);
        CHECK(strstr(last_kernel, tiles < 1 << 25 ? "adamw_fine_kernel" : "adamw_wide_kernel"));
        CHECK(last_groups == (tiles < 1 << 25 ? 2 * tiles : tiles));
    }
    std::vector<zi_tensor> list(24);
    for (size_t i = 0; i < list.size(); ++i) {
        const size_t n = 1'000'000, from = i * n;
        list[i] = {(float*)at[0] + from, (float*)at[1] + from, (float*)at[2] + from, (uint16_t*)at[3] + from, nullptr, (int64_t)n};
    }
    CHECK(zi_adamw_step(list.data(), 24, ZI_BF16, &c, nullptr, nullptr) == ZI_OK);
    CHECK(strstr(last_kernel, "adamw_list_kernel") && last_groups == 24 * 1954);
    return 0;
}

int main(int argc, char** argv)
{
    const struct { const char* name; int (*run)(); } all[] = {{"peer", peer}, {"sizes", sizes}, {"capture", capture}, {"replays", replays}, {"skipped", skipped}, {"earlier_work", earlier_work}, {"one_tensor_kernels", one_tensor_kernels}, {"uploads", uploads}, {"loads", loads}, {"offload", offload}, {"spanning", spanning}, {"link_tiles", link_tiles}};
    for (const auto& t : all)
        if (argc == 2 && !strcmp(argv[1], t.name)) return t.run();
    fprintf(stderr, "which check?\n");
    return 2;
}
