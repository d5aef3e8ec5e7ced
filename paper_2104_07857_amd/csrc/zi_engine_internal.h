// The streaming engine's state, shared by the translation units that implement its entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "zi_host.h"
#include "zi_io_pool.h"

namespace zi {
namespace host {

constexpr int kMaxHostSlots = 16;
// A slot holds p, m, v and a fourth array whose first half stages host-resident gradients and whose
// second half stages a host-resident low-precision copy.
constexpr int kSlotArrays = 4;
constexpr int kOffloadEvents = 64;       // events that order gradient offloads after their producers
constexpr uint32_t kEngineMagic = 0x5A49454Eu;

enum { kSrcPinned = 0, kSrcPageable = 1, kSrcFile = 2 };

// Where the fp32 state of one tensor lives for the streamed step.
struct StateSrc {
    int kind;
    char* ptr[3];        // p, m, v (memory kinds)
    int fd[3];           // file kind
    int64_t off[3];
    bool direct[3];      // descriptor was opened with O_DIRECT
    const void* g;       // device, or host when g_host
    void* p_lp;          // device, or host when lp_host; may be null
    bool g_host;         // gradients live in host memory and are staged chunk by chunk
    bool lp_host;        // the low-precision copy is written back to host memory
    bool g_peer, lp_peer;   // device memory, but not the engine's device's: no kernel of this one may touch it
    char* dev[5];        // p, m, v, g, p_lp as the device addresses them, if every host array is mapped (HostRanges)
    int64_t numel;
};

// One block of one segment for the host step's thread pool.
struct CpuBlock {
    float *p, *m, *v;
    const uint16_t* g;
    uint16_t* lp;
    int64_t n;
    const uint32_t* arrived;      // flag of the block's gradients (null: they are in host memory already)
    uint16_t* lp_device;          // where the block of the copy goes (null: it is in its place)
    bool lp_by_copy;              // ... by the runtime's copy, not by a kernel
};

// The norm result's landing place, and a flag that a kernel raises once it is there.
struct HostNorm {
    zi_norm_result result;
    uint32_t arrived;
};

// Page-locked allocations seen during one call: an array that lies in one of them needs no further query,
// and its device address follows from the allocation's.
struct HostRanges {
    struct Range { uintptr_t lo, hi; ptrdiff_t to_device; };
    Range known[8] = {};
    int n_known = 0, next = 0;

    const Range* find(const void* p, size_t bytes) const
    {
        for (int i = 0; i < n_known; ++i)
            if (lies_within(p, bytes, known[i].lo, known[i].hi)) return &known[i];
        return nullptr;
    }

    // Notes the allocation around p if all of [p, p + bytes) lies in it and is mapped for the device.
    // Arrays that span several registrations stay unknown: only a copy engine may touch those.
    void note(const void* p, size_t bytes)
    {
        hipPointerAttribute_t attr{};
        hipDeviceptr_t base = nullptr;
        size_t size = 0;
        if (hipPointerGetAttributes(&attr, p) != hipSuccess || attr.type != hipMemoryTypeHost || !attr.devicePointer ||
            hipMemGetAddressRange(&base, &size, attr.devicePointer) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        const uintptr_t at = reinterpret_cast<uintptr_t>(p), dev = reinterpret_cast<uintptr_t>(attr.devicePointer);
        const uintptr_t lo = reinterpret_cast<uintptr_t>(base);
        if (!lies_within(attr.devicePointer, bytes, lo, lo + size)) return;
        known[next] = {at - (dev - lo), at - (dev - lo) + size, (ptrdiff_t)(dev - at)};
        next = (next + 1) % 8;
        if (n_known < 8) ++n_known;
    }

    // Device address of a page-locked array, null if it is not known to be mapped as a whole.
    char* device_address(const void* p, size_t bytes) const
    {
        const Range* r = find(p, bytes);
        return r ? reinterpret_cast<char*>(reinterpret_cast<uintptr_t>(p) + (uintptr_t)r->to_device) : nullptr;
    }
};

}  // namespace host
}  // namespace zi

struct zi_engine {
    int device = 0;
    size_t chunk_bytes = 0;            // per state array
    int64_t chunk_elems = 0;
    size_t array_bytes = 0;            // chunk_bytes + room for lead-in elements and a rounded-up last block
    uint32_t magic = 0;

    // HBM staging: n_slots slots of kSlotArrays arrays, three streams, events that order slot reuse.
    int n_slots = 0;
    char* staging = nullptr;
    hipStream_t s_h2d = nullptr, s_k = nullptr, s_d2h = nullptr;
    hipEvent_t ev_h2d[8] = {}, ev_k[8] = {}, ev_d2h[8] = {};
    hipEvent_t ev_out_start[8] = {};   // the slot's device-to-host copies are about to start (its update is done)
    hipEvent_t ev_in = nullptr, ev_out = nullptr;
    zi_norm_result* h_norm = nullptr;  // pinned landing place of the norm result: HostNorm's
    uint32_t norm_serial = 0;          // of the last result brought there by a kernel

    // Pinned ring for state that is not page-locked (ordinary memory, files): n_hslots slots shaped
    // like the HBM slots, filled and emptied by two small thread pools, each driven by one parked
    // stage thread.  All of these threads are created with the ring and parked between calls.
    int n_hslots = 0;
    char* hring = nullptr;
    hipEvent_t ev_back[zi::host::kMaxHostSlots] = {};   // the slot's outbound traffic has left / its inbound copy is done
    hipEvent_t ev_fill[zi::host::kMaxHostSlots] = {};   // gradients of another device have landed in the slot
    uint32_t* fill_flags = nullptr;    // page-locked: per ring slot and block of the host-CPU step, see link_copy_kernel
    size_t flags_per_slot = 0;
    uint32_t fill_serial = 0;          // of the last fill; a block's flag equals its fill's serial once it has landed
    int copy_threads = 6;
    zi::host::TaskPool* pool_in = nullptr;
    zi::host::TaskPool* pool_out = nullptr;
    zi::host::StageThread* stage_in = nullptr;
    zi::host::StageThread* stage_out = nullptr;
    zi::host::TaskPool* pool_step = nullptr;            // blocks of the host-CPU step (created on first use)

    // Gradient offload: copies in flight on the device-to-host stream, ordered after their producers.
    hipEvent_t ev_offload[zi::host::kOffloadEvents] = {};
    hipEvent_t ev_offload_done = nullptr;               // recorded behind the offloads when somebody waits for them
    uint64_t n_offloads = 0;
    bool offload_pending = false;

    // Per-call plans.  The vectors keep their capacity between calls, so once a list of a given size
    // has been seen, later calls allocate no host memory either.
    std::vector<zi_tensor> device_list;   // src with addresses as the device sees them
    std::vector<zi::host::StateSrc> src;
    std::vector<int64_t> plan_numel;
    std::vector<zi::host::Segment> segs;
    std::vector<size_t> use_begin;
    std::vector<zi::host::Piece> pieces_in, pieces_out;
    std::vector<int32_t> host_idx;
    std::vector<zi::host::CpuBlock> cpu_blocks;
    std::vector<uint32_t> cpu_done;    // per block of the host-CPU step: stepped in this use

    // options and figures
    int64_t skip_kernel = 0;
    int max_inflight = 0;              // 0: paced by the start of the copy-out two uses back; k: by the end of use - k
    zi_stream_stats stats{};

    float* slot_array(int slot, int which) const
    {
        return reinterpret_cast<float*>(staging + ((size_t)slot * zi::host::kSlotArrays + which) * array_bytes);
    }
    uint16_t* slot_g(int slot) const { return reinterpret_cast<uint16_t*>(slot_array(slot, 3)); }
    uint16_t* slot_lp(int slot) const
    {
        return reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(slot_array(slot, 3)) + array_bytes / 2);
    }
    float* hslot_array(int hslot, int which) const
    {
        return reinterpret_cast<float*>(hring + ((size_t)hslot * zi::host::kSlotArrays + which) * array_bytes);
    }
    uint16_t* hslot_g(int h) const { return reinterpret_cast<uint16_t*>(hslot_array(h, 3)); }
    uint16_t* hslot_lp(int h) const
    {
        return reinterpret_cast<uint16_t*>(reinterpret_cast<char*>(hslot_array(h, 3)) + array_bytes / 2);
    }
};

namespace zi {
namespace host {

inline zi_status check_engine(const zi_engine* e)
{
    if (!e) return fail(ZI_ERR_INVALID_ARG, "engine is NULL");
    if (e->magic != kEngineMagic) return fail(ZI_ERR_INVALID_ARG, "engine is not valid (destroyed?)");
    return ZI_OK;
}

// After a failed call: wait for whatever the engine's streams still hold, dropping the errors.
inline void drain_streams(zi_engine* e)
{
    (void)hipStreamSynchronize(e->s_h2d);
    (void)hipStreamSynchronize(e->s_k);
    (void)hipStreamSynchronize(e->s_d2h);
    (void)hipGetLastError();
}

// First segment of every slot use (segments are sorted by slot use within each planning pass).
inline void index_uses(const std::vector<Segment>& segs, int64_t n_uses, std::vector<size_t>& use_begin)
{
    use_begin.assign((size_t)n_uses + 1, segs.size());
    for (size_t j = segs.size(); j-- > 0;) use_begin[(size_t)segs[j].slot_use] = j;
    for (int64_t u = n_uses - 1; u >= 0; --u)
        if (use_begin[(size_t)u] > use_begin[(size_t)u + 1]) use_begin[(size_t)u] = use_begin[(size_t)u + 1];
}

// Work already enqueued on the device-to-host stream by zi_grad_offload happens before anything a
// streamed call reads from host memory: its copy-in stream waits for the last offload.
// (The event behind the offloads is recorded when somebody waits for them, not with each of them.)
inline hipError_t mark_offloads(zi_engine* e) { return hipEventRecord(e->ev_offload_done, e->s_d2h); }
inline hipError_t order_after_offloads(zi_engine* e, hipStream_t consumer)
{
    if (!e->offload_pending) return hipSuccess;
    const hipError_t he = mark_offloads(e);
    return he != hipSuccess ? he : hipStreamWaitEvent(consumer, e->ev_offload_done, 0);
}
inline hipError_t wait_for_offloads(zi_engine* e)       // blocks the host
{
    if (!e->offload_pending) return hipSuccess;
    const hipError_t he = mark_offloads(e);
    return he != hipSuccess ? he : hipEventSynchronize(e->ev_offload_done);
}

// Maps a C++ exception that reached an entry point to a status (nothing may cross the C ABI).
#define ZI_GUARD_BEGIN try {
#define ZI_GUARD_END                                                                              \
    }                                                                                             \
    catch (const std::bad_alloc&) { return ::zi::host::fail(ZI_ERR_NOMEM, "out of host memory"); } \
    catch (const std::exception& ex_) { return ::zi::host::fail(ZI_ERR_NOMEM, "%s", ex_.what()); }

}  // namespace host
}  // namespace zi
